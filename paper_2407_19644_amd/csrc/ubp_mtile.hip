// Dense-tile kernel of the UBP library (fp16 / bf16): W as zero-filled 16 x 32 operand tiles, both
// operands staged in LDS by wavefronts that do nothing else.
#include "ubp_device.h"

#include <cstdint>
#include <type_traits>

namespace ubp {

namespace {

// Position of the 32-byte unit u (16 pixels) inside row r of a staged X tile is u ^ tile_swizzle(r):
// a transposed read covers 16 consecutive rows of one unit, and LDS has 64 four-byte banks, i.e. 8
// windows of 32 bytes; the swizzle spreads the 16 rows over all 8 (two rows per window, the minimum).
template <int UNITS> __device__ __forceinline__ constexpr int tile_swizzle(int r) {
    return UNITS >= 8 ? (r & 7) : UNITS == 4 ? ((r >> 1) & 3) : UNITS == 2 ? ((r >> 2) & 1) : 0;
}

// Occupancy words (of 32 steps) per stripe that a register of a wavefront with 4 stripes holds: K up to 16384
constexpr int kOccWords = 16;

// 8 16-bit values moved down by n places (0 .. 7)
__device__ __forceinline__ uint4v shift_down(uint4v v, int n) {
    if (n & 4) v = uint4v{v[2], v[3], 0u, 0u};
    if (n & 2) v = uint4v{v[1], v[2], v[3], 0u};
    if (n & 1) v = uint4v{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
    return v;
}

// A workgroup multiplies tiles of 16 WM SM rows x 16 WN PN pixels of Y, one after the other, in stages of 64
// columns of W that pass through a ring of NS slots.  NPW wavefronts do nothing but start the loads of a
// stage NS - 1 stages ahead; WM x WN wavefronts read operands (the next step's while the matrix
// instructions of the last one run) and multiply; one barrier per stage.
// What bounds it: a wavefront starts a load into LDS only every 64 to 85 cycles and stores count in the same
// counter as loads, in order - hence loads in wavefronts of their own, which keep running over a tile's end
// and its stores - and then the way from L2 into LDS, about 100 bytes per ns and CU where one tile needs
// 32 KB per stage: 0.37 us per stage of 128 x 128 (5.7 TFLOP/s and CU; the matrix
// instructions alone could do it in 0.22).  Against the kernels before this one (the multiplying wavefronts
// staged X in chunks, and for full matrices both operands): 256 x 2304 with 6272 pixels 18.5 -> 14.4 us, with
// 12544 20.3 -> 17.2; 1024 x 1024, every tile kept, with 1568 pixels and fp32 results 11.2 -> 8.6.
// SKIP: W has empty 16 x 32 tiles, whose products are left out by a branch per stripe and step; 2 where K is
// above 16384 (in an instantiation of its own: a fetch inside the loop made layers with
// empty tiles 2 % slower, 256 x 2304 with 6272 pixels 14.4 -> 14.75 us).
// RAG: 0 rows of X are 16-byte pieces; 1 any alignment, through registers; 2 the same with 64-bit offsets, for
// rows more than 32 MB apart (64-bit offsets for all odd rows took 2 % longer: 26.5 -> 27.1 us on 256 x 2304 with 6076 pixels).
template <bool BF16, typename TY, int WM, int WN, int SM, int PN, int NS, int NPW, int SKIP, int RAG>
__global__ __launch_bounds__((WM * WN + NPW) * 64, 2) void mtile_kernel(TileArgs a) {
    constexpr int KS = 2;                                   // 32-column steps per stage
    constexpr int NC = WM * WN;                             // multiplying wavefronts; NPW more load
    constexpr int TS = WM * SM, UNITS = WN * PN, TN = 16 * UNITS;
    constexpr int XROWB = 2 * TN, PIECES = XROWB / 16, RPI = 64 / PIECES;
    static_assert(PIECES <= 64 && RPI * PIECES == 64, "a 1 KB load covers whole rows");
    constexpr int WSTAGE = KS * TS * 1024, XSTAGE = KS * 32 * XROWB, STAGE = WSTAGE + XSTAGE;
    constexpr int NWI = KS * TS, NXI = KS * 32 / RPI;       // 1 KB loads per stage
    // RAG: half of the loading wavefronts bring the weights, the other half the rows of X (see there)
    constexpr int NL = RAG ? NPW / 2 : NPW;
    static_assert(NWI % NL == 0 && NXI % NL == 0, "every loading wavefront issues the same number of loads per stage");
    constexpr int PW = NWI / NL, PX = NXI / NL, PER = RAG ? PW : PW + PX;
    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    // Workgroup -> tiles: consecutive workgroup ids go round-robin over the 8 XCDs.  The tiles, row blocks
    // of a pixel block next to each other, are cut into 8 equal runs, one per XCD: X comes from memory
    // about once and from that XCD's L2 for the other row blocks.
    const int xcd = blockIdx.x & 7, wg_step = (int)(gridDim.x >> 3);
    const int all_tiles = a.n_blocks * a.slices;
    const int tile0 = (int)((int64_t)all_tiles * xcd >> 3), my_tiles = (int)((int64_t)all_tiles * (xcd + 1) >> 3) - tile0;
    const int t0 = (int)(blockIdx.x >> 3);
    const int nst = (a.K + 32 * KS - 1) / (32 * KS);
    const int n_tiles = t0 < my_tiles ? (my_tiles - t0 + wg_step - 1) / wg_step : 0;
    const int total = n_tiles * nst;                        // stages this workgroup runs through
    if (total == 0) return;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
    auto next_slot = [&](uint32_t o) { return o + STAGE == (uint32_t)(NS * STAGE) ? 0u : o + STAGE; };

    if (wave >= NC) {
        // ---- loading wavefronts: load q (0 .. PW-1 / PX-1) of this one is number j = me + q NL of the
        // stage's W tiles (step j / TS, stripe j % TS) and of its 1 KB pieces of X (rows j RPI ..)
        const int me = (wave - NC) % NL;
        const bool rows = RAG && wave - NC >= NL;          // RAG: this one brings rows of X
        const int row_in = lane / PIECES, pp = lane % PIECES;
        const uint32_t lane16 = (uint32_t)lane * 16u;
        struct Cursor { int tile = -1, st = 0; } cw, cx;   // the next stage whose W / X is requested
        const uint16_t *wsrc[PW];
        // byte offset of this lane's piece from the stage's first row
        typedef typename std::conditional<RAG == 2, uint64_t, uint32_t>::type off_t;
        off_t xoff[PX];
        int xcol[PX];        // its first pixel
        auto advance = [&](Cursor &c) { // returns whether the tile changed
            if (c.tile >= 0 && ++c.st < nst) return false;
            ++c.tile;
            c.st = 0;
            return true;
        };
        auto load_w = [&](uint32_t slot) { // slot: byte offset of the ring slot
            if (advance(cw)) {
                const int stripe0 = ((tile0 + t0 + cw.tile * wg_step) % a.slices) * TS;
#pragma unroll
                for (int q = 0; q < PW; ++q) {
                    const int j = me + q * NL;
                    wsrc[q] = a.frags + ((int64_t)min(stripe0 + j % TS, a.nstripes - 1) * a.kt_total + j / TS) * 512;
                }
            }
#pragma unroll
            for (int q = 0; q < PW; ++q)
                load16_to_lds(wsrc[q] + (int64_t)cw.st * (KS * 512), lane16, lds0 + slot + (uint32_t)(me + q * NL) * 1024u);
        };
        // Position of X: pieces past column N load the last 8 pixels of the row instead (what they stand
        // for is shifted into place or never used), rows past K load row K - 1 again (W holds zeros there).
        auto next_x = [&]() {
            if (advance(cx)) {
                const int col0 = (tile0 + t0 + cx.tile * wg_step) / a.slices * TN;
#pragma unroll
                for (int q = 0; q < PX; ++q) {
                    const int r = (me + q * NL) * RPI + row_in;
                    xcol[q] = col0 + ((pp >> 1) ^ tile_swizzle<UNITS>(r)) * 16 + (pp & 1) * 8;
                    xoff[q] = (off_t)(((int64_t)r * a.ldx + min(xcol[q], a.N - 8)) * 2);
                }
            }
        };
        auto offset = [&](int q, bool whole) -> off_t {
            if (whole) return xoff[q];
            const int k0 = cx.st * (KS * 32), k = min(k0 + (me + q * NL) * RPI + row_in, a.K - 1);
            return (off_t)(((int64_t)(k - k0) * a.ldx + min(xcol[q], a.N - 8)) * 2);
        };
        uint32_t slot = 0;
        if (!rows) {
            auto load_stage = [&]() {
                load_w(slot);
                if constexpr (!RAG) {
                    next_x();
                    const uint16_t *src = a.X + (int64_t)cx.st * (KS * 32) * a.ldx;
                    const bool whole = (cx.st + 1) * (KS * 32) <= a.K;
                    if (whole) {
#pragma unroll
                        for (int q = 0; q < PX; ++q) load16_to_lds(src, xoff[q], lds0 + slot + (uint32_t)(WSTAGE + (me + q * NL) * 1024));
                    } else {
#pragma unroll
                        for (int q = 0; q < PX; ++q)
                            load16_to_lds(src, offset(q, false), lds0 + slot + (uint32_t)(WSTAGE + (me + q * NL) * 1024));
                    }
                }
                slot = next_slot(slot);
            };
            load_stage();
            if (total > 1) load_stage();
            wait_vmcnt_at_most(min(1, total - 1) * PER);
            lds_barrier(); // stage 0 is there
#pragma unroll
            for (int s = 2; s < NS; ++s)
                if (s < total) load_stage();
            for (int gs = 0; gs + 1 < total; ++gs) {
                if (gs + NS <= total) wait_vmcnt<(NS - 2) * PER>();
                else wait_vmcnt_at_most((total - 2 - gs) * PER);
                lds_barrier(); // stage gs is read, stage gs + 1 is there
                if (gs + NS < total) load_stage();
            }
        } else if constexpr (RAG) {
            // Rows of X at any 2-byte alignment cannot go straight to LDS: they pass through registers, D
            // stages ahead of the slot they go to.  In wavefronts of their own: the compiler, which waits for
            // these loads by their number, does not know of the direct loads of the weights and would wait
            // for the newest rows as soon as both kinds are in flight together (28 us instead of 23 on a
            // 256 x 2304 layer with 6076 pixels).
            constexpr int D = PX >= 8 ? 2 : 4;
            uint4v xr[D][PX];
            int over[D][PX]; // elements by which a piece hangs over the right edge
            int left = total; // stages not yet fetched; behind the last one it is fetched again (a fetch on one path
                              // only would blur the compiler's count of loads in flight)
            auto fetch = [&](uint4v(&v)[PX], int(&ov)[PX]) {
                if (left > 0) next_x();
                --left;
                const char *src = reinterpret_cast<const char *>(a.X + (int64_t)cx.st * (KS * 32) * a.ldx);
                const bool whole = (cx.st + 1) * (KS * 32) <= a.K;
#pragma unroll
                for (int q = 0; q < PX; ++q) {
                    __builtin_memcpy(&v[q], src + offset(q, whole), 16);
                    ov[q] = max(0, xcol[q] - (a.N - 8)) & 7;
                }
            };
            auto put = [&](const uint4v(&v)[PX], const int(&ov)[PX]) {
                bool any = false;
#pragma unroll
                for (int q = 0; q < PX; ++q) any |= ov[q] != 0;
                if (__builtin_amdgcn_ballot_w64(any) == 0) {
#pragma unroll
                    for (int q = 0; q < PX; ++q) *reinterpret_cast<uint4v *>(smem + slot + WSTAGE + (me + q * NL) * 1024 + lane * 16) = v[q];
                } else {
#pragma unroll
                    for (int q = 0; q < PX; ++q)
                        *reinterpret_cast<uint4v *>(smem + slot + WSTAGE + (me + q * NL) * 1024 + lane * 16) = shift_down(v[q], ov[q]);
                }
                slot = next_slot(slot);
            };
            fetch(xr[0], over[0]);
            put(xr[0], over[0]);
#pragma unroll
            for (int d = 0; d < D; ++d)
                fetch(xr[d], over[d]);
            lds_barrier(); // stage 0 is there
            // (stage s goes to its slot one barrier before it is read; NS - 2 slots of X would do)
            for (int gs0 = 0; gs0 + 1 < total; gs0 += D) {
#pragma unroll
                for (int h = 0; h < D; ++h) {
                    const int gs = gs0 + h;
                    if (gs + 1 >= total) break;
                    put(xr[h], over[h]);       // stage gs + 1
                    fetch(xr[h], over[h]);
                    lds_barrier(); // stage gs is read, stage gs + 1 is there
                }
            }
        }
        return;
    }

    // ---- multiplying wavefronts
    const int wm = wave / WN, wn = wave % WN;
    const int g = lane >> 4, n = lane & 15;
    const int e = 4 * g + (n >> 2);   // this lane's part in the transposed reads: rows e and 16 + e of a step
    uint32_t xaddr[PN];
#pragma unroll
    for (int c = 0; c < PN; ++c)
        xaddr[c] = lds0 + (uint32_t)(WSTAGE + e * XROWB + (((wn * PN + c) ^ tile_swizzle<UNITS>(e)) << 5) + (n & 3) * 8);
    const uint32_t waddr = lds0 + (uint32_t)(wm * SM * 1024 + lane * 16);
    typedef __attribute__((address_space(3))) const uint4v *lds_frag_ptr;

    float4v acc[SM][PN];
    uint4v wf[2][SM];
    short8v xf[2][PN];
    short4v xlo[PN];
    constexpr int NM = SM * PN, NR = SM + 2 * PN;
    auto read_one = [&](int b, int r, uint32_t off, int ks) { // operand read r of a step
        if (r < SM) {
            wf[b][r] = *(lds_frag_ptr)(uintptr_t)(waddr + off + (uint32_t)((ks * TS + r) * 1024));
        } else {
            const int c = (r - SM) / 2;
            if (((r - SM) & 1) == 0) {
                xlo[c] = lds_read_tr(xaddr[c] + off + (uint32_t)(ks * 32 * XROWB));
            } else {
                const short4v hi = lds_read_tr(xaddr[c] + off + (uint32_t)(ks * 32 * XROWB + 16 * XROWB));
                xf[b][c] = __builtin_shufflevector(xlo[c], hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
    };
    [[maybe_unused]] const int words = (a.kt_total + 31) >> 5;
    [[maybe_unused]] uint32_t occ[SM];
    // One step: the products of operand set b, the reads of the next step's operands into the other set
    // spread between them.
    auto step = [&](int b, int kt, uint32_t roff, int rks) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (SKIP) {
            // (wave-uniform) a stripe that keeps nothing here is skipped; the reads stay on the one path
#pragma unroll
            for (int i = 0; i < SM; ++i) {
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (r * SM / NR == i) read_one(b ^ 1, r, roff, rks);
                if ((occ[i] >> (kt & 31)) & 1u) {
#pragma unroll
                    for (int c = 0; c < PN; ++c) acc[i][c] = mfma16<BF16>(xf[b][c], __builtin_bit_cast(short8v, wf[b][i]), acc[i][c]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            const int i = m / PN, c = m % PN;
            acc[i][c] = mfma16<BF16>(xf[b][c], __builtin_bit_cast(short8v, wf[b][i]), acc[i][c]);
#pragma unroll
            for (int r = 0; r < NR; ++r)
                if (r * NM / NR == m) read_one(b ^ 1, r, roff, rks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // SKIP: lane ow i + w holds word w (SKIP 2: w0 + w) of the occupancy bits (one per 32-column step) of my
    // stripe i, fetched a tile ahead by a vector load (a scalar one would be waited for together with the LDS
    // reads); SKIP 2: the words behind the first ow are fetched when they are reached
    [[maybe_unused]] const int ow = SKIP == 2 ? kOccWords : words;
    static_assert(kOccWords * SM <= 64, "a wavefront's occupancy words sit in one register");
    [[maybe_unused]] auto load_occ = [&](int t, int w0) -> uint32_t {
        const int i = lane / ow, s = ((tile0 + t0 + t * wg_step) % a.slices) * TS + wm * SM + i;
        if constexpr (SKIP != 2) return i < SM ? a.occupied[(int64_t)min(s, a.nstripes - 1) * words + lane % words] : 0u;
        const int w = w0 + lane % ow;
        return i < SM && w < words ? a.occupied[(int64_t)min(s, a.nstripes - 1) * words + w] : 0u;
    };
    [[maybe_unused]] uint32_t occ_v = 0;
    if constexpr (SKIP) occ_v = load_occ(0, 0);
    lds_barrier(); // stage 0 is there
#pragma unroll
    for (int r = 0; r < NR; ++r) read_one(0, r, 0u, 0);
    uint32_t off = 0; // current slot
    int gs = 0;
    constexpr int YS = (int)sizeof(TY);
    constexpr int RB = 16 * PN * YS;                // bytes of one row of this wavefront's output tile
    constexpr int PR = RB / 16;                     // 16-byte pieces per row
    constexpr int RP = RB >= 256 ? 1 : 256 / RB;    // rows per 256 bytes (one pass over the banks)
    constexpr int NI = (16 * PR) / 64;              // store instructions per stripe
    static_assert(NI >= 1, "a stripe's output tile is at least 1 KB");
    char *scratch = smem + NS * STAGE + wave * (16 * RB);
    TY *Yt = static_cast<TY *>(a.Y);
    for (int t = 0; t < n_tiles; ++t) {
        const int local = tile0 + t0 + t * wg_step;
        const int pcol0 = local / a.slices * TN + wn * PN * 16;
        const int s0 = (local % a.slices) * TS + wm * SM;   // my first stripe
#pragma unroll
        for (int i = 0; i < SM; ++i)
#pragma unroll
            for (int c = 0; c < PN; ++c) acc[i][c] = float4v{0.f, 0.f, 0.f, 0.f};
        [[maybe_unused]] uint32_t occ_next = 0;
        if constexpr (SKIP) occ_next = load_occ(min(t + 1, n_tiles - 1), 0);
        for (int st = 0; st < nst; ++st, ++gs) {
            if constexpr (SKIP) {
                if (((st * KS) & 31) == 0) {
                    const int w = (st * KS) >> 5;
                    if (SKIP == 2 && w != 0 && w % ow == 0) {
                        occ_v = load_occ(t, w); // (used in here too: no other path waits for it)
#pragma unroll
                        for (int i = 0; i < SM; ++i) occ[i] = (uint32_t)__builtin_amdgcn_readlane((int)occ_v, i * ow);
                    } else {
#pragma unroll
                        for (int i = 0; i < SM; ++i) occ[i] = (uint32_t)__builtin_amdgcn_readlane((int)occ_v, i * ow + (SKIP == 2 ? w % ow : w));
                    }
                }
            }
            step(0, st * KS, off, 1);
            if (gs + 1 < total) lds_barrier(); // all of the stage is in registers: its slot is free; the next one is there
            off = next_slot(off);
            step(1, st * KS + 1, off, 0);      // (behind the last stage the reads fetch a dead slot)
        }
        if constexpr (SKIP) occ_v = occ_next;
        // ---- stores: through 16 LDS rows of this wavefront (pieces XOR-swizzled by the row against bank
        // conflicts; one wavefront writes and reads, LDS keeps its order), whole rows out.  Lane (g, n)
        // holds pixels 16 c + 4 g .. + 3 of row n of a stripe's tile c.
#pragma unroll
        for (int i = 0; i < SM; ++i) {
            const int stripe = s0 + i;
            if (a.ep.on) {
                const float b = epilogue_bias(a.ep, stripe * kStripe + n, a.M);
#pragma unroll
                for (int c = 0; c < PN; ++c) epilogue_tile(a.ep, acc[i][c], b);
            }
#pragma unroll
            for (int c = 0; c < PN; ++c) {
                const int byte = (16 * c + 4 * g) * YS;
                const int piece = (byte >> 4) ^ ((n / RP) & (PR - 1) & 7);
                char *dst = scratch + n * RB + piece * 16 + (byte & 15);
                if constexpr (YS == 4) {
                    *reinterpret_cast<float4v *>(dst) = acc[i][c];
                } else {
                    typedef TY ty4 __attribute__((ext_vector_type(4)));
                    ty4 o;
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[v] = from_f32<TY>(acc[i][c][v]);
                    *reinterpret_cast<ty4 *>(dst) = o;
                }
            }
#pragma unroll
            for (int q = 0; q < NI; ++q) {
                const int r = q * (64 / PR) + lane / PR, lp = lane % PR;
                const uint4v o = *reinterpret_cast<const uint4v *>(scratch + r * RB + ((lp ^ ((r / RP) & (PR - 1) & 7)) << 4));
                const int row = stripe * kStripe + r;
                const int px = pcol0 + lp * (16 / YS);
                TY *dst = Yt + (int64_t)row * a.ldy + px;
                if (stripe < a.nstripes && row < a.M) {
                    if (px + 16 / YS <= a.N) {
                        if constexpr (RAG) __builtin_memcpy(dst, &o, 16);
                        else *reinterpret_cast<uint4v *>(dst) = o;
                    } else if constexpr (RAG) {
                        TY p[16 / YS];
                        __builtin_memcpy(p, &o, 16);
#pragma unroll
                        for (int z = 0; z < 16 / YS; ++z)
                            if (px + z < a.N) dst[z] = p[z];
                    }
                }
            }
        }
    }
}

template <bool BF16, typename TY, int WM, int WN, int SM, int PN, int NS, int NPW, int SKIP, int RAG>
ubp_status launch_one(const TileArgs &a, hipStream_t st, bool dry) {
    constexpr int TS = WM * SM, TN = 16 * WN * PN;
    constexpr size_t stage = (size_t)2 * (TS * 1024 + 32 * 2 * TN);
    constexpr size_t lds = NS * stage + (size_t)WM * WN * 16 * 16 * PN * sizeof(TY);
    static_assert(lds <= 160 * 1024, "the stages and the output rows fit LDS");
    static LdsLimit limit;
    const ubp_status rc = limit.raise(reinterpret_cast<const void *>(&mtile_kernel<BF16, TY, WM, WN, SM, PN, NS, NPW, SKIP, RAG>));
    if (rc != UBP_OK || dry) return rc;
    TileArgs b = a;
    b.n_blocks = (a.N + TN - 1) / TN;
    b.slices = (a.nstripes + TS - 1) / TS;
    const unsigned per_cu = lds <= 80 * 1024 ? 2 : 1;
    const unsigned grid = std::min(8u * (unsigned)(((int64_t)b.n_blocks * b.slices + 7) / 8), 256u * per_cu);
    return launch_kernel(&mtile_kernel<BF16, TY, WM, WN, SM, PN, NS, NPW, SKIP, RAG>, dim3(grid), dim3((WM * WN + NPW) * 64), lds, st, b);
}

template <bool BF16, typename TY, int WM, int WN, int SM, int PN, int NPW, int RAG>
ubp_status launch_shape(const TileArgs &a, hipStream_t st, bool dry) {
    if (!a.skip) return launch_one<BF16, TY, WM, WN, SM, PN, 4, NPW, 0, RAG>(a, st, dry);
    return a.kt_total <= 32 * kOccWords ? launch_one<BF16, TY, WM, WN, SM, PN, 4, NPW, 1, RAG>(a, st, dry)
                                        : launch_one<BF16, TY, WM, WN, SM, PN, 4, NPW, 2, RAG>(a, st, dry);
}

// Tiles of 128 x 256 with a ring of three slots, which is all of LDS with a 16-bit Y and more than it with fp32.  For
// K up to 256 and a number of tiles of 128 x 128 that leaves a second round half empty: 256 x 256 with 25088
// pixels, 392 tiles on 256 CUs, 11.3 -> 9.9 us; in the gemm kernel that had this tile before, 10.2.
template <bool BF16, typename TY> ubp_status launch_wide(const TileArgs &a, hipStream_t st, bool dry) {
    if constexpr (sizeof(TY) == 2) {
        if (a.kt_total > 32 * kOccWords) return UBP_ERR_UNSUPPORTED;
        return a.skip ? launch_one<BF16, TY, 2, 4, 4, 4, 3, 4, 1, 0>(a, st, dry) : launch_one<BF16, TY, 2, 4, 4, 4, 3, 4, 0, 0>(a, st, dry);
    } else {
        return UBP_ERR_UNSUPPORTED;
    }
}

template <bool BF16, typename TY>
ubp_status launch_t(const TileArgs &a, int shape, int rows, hipStream_t st, bool dry) {
    // (kMtileShapes)
    if (rows == 2 && shape != 3) return UBP_ERR_UNSUPPORTED;
    switch (shape) {
    case 0: return rows == 1 ? launch_shape<BF16, TY, 2, 4, 4, 2, 8, 1>(a, st, dry) : launch_shape<BF16, TY, 2, 4, 4, 2, 8, 0>(a, st, dry);
    case 1: return rows == 1 ? launch_shape<BF16, TY, 4, 2, 2, 2, 4, 1>(a, st, dry) : launch_shape<BF16, TY, 4, 2, 2, 2, 4, 0>(a, st, dry);
    case 2: return rows == 1 ? UBP_ERR_UNSUPPORTED : launch_shape<BF16, TY, 2, 4, 2, 2, 4, 0>(a, st, dry);
    case 3:
        return rows == 2   ? launch_shape<BF16, TY, 2, 2, 2, 2, 4, 2>(a, st, dry)
               : rows == 1 ? launch_shape<BF16, TY, 2, 2, 2, 2, 4, 1>(a, st, dry)
                           : launch_shape<BF16, TY, 2, 2, 2, 2, 4, 0>(a, st, dry);
    case 4: return rows == 0 ? launch_wide<BF16, TY>(a, st, dry) : UBP_ERR_UNSUPPORTED;
    }
    return UBP_ERR_UNSUPPORTED;
}

} // namespace

ubp_status launch_mtile(const TileArgs &a, bool bf16, bool y_f32, int shape, int rows, void *stream, bool dry) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (bf16) return y_f32 ? launch_t<true, float>(a, shape, rows, st, dry) : launch_t<true, __bf16>(a, shape, rows, st, dry);
    return y_f32 ? launch_t<false, float>(a, shape, rows, st, dry) : launch_t<false, _Float16>(a, shape, rows, st, dry);
}

} // namespace ubp
