// Block kernel of the UBP library (fp16 / bf16, blocks of at most 16 rows): MFMA on aligned
// 16-row stripes with whole blocks as operands.
//
// A block of at most 16 rows has at most one row congruent to n modulo 16.  Stored by that
// residue - the paper's weight rotation (Section 4.2) with period 16 instead of the block
// height - ONE operand fragment serves both stripes an unaligned block reaches into: rows
// n >= o (o = first row modulo 16) belong to the stripe the block starts in, rows n < o to the
// next one, and the accumulator a row lands in is fixed at compile time, as in the paper.  The
// 16 columns of a block are rows of X; they are gathered from an LDS ring, transposed into
// operand order by the read itself.
#include "ubp_device.h"

#include <cstdint>

namespace ubp {

namespace {

constexpr int kBlkCT = 4; // 64-pixel column tiles (as many ring rows as the ring of CT = 4 has)
// A kilobyte of the ring holds 8 rows, the 4 pixel tiles one after the other, 8 x 32 bytes each: the 8 rows that half a
// wavefront reads together are 256 consecutive bytes (no bank conflicts without a swizzle), and the tiles' addresses
// differ by constants.
constexpr int kBlkTile = 256;

// Where a step's products begin (m1: its second metadata word), in dwords from behind the s_getpc in multiply(): 3 of the
// jump itself, 18 for each case before, and 8 of the upper part where that is passed over (bit 13 clear).
template <int G> __device__ __forceinline__ uint32_t multiply_entry(uint32_t m1) {
    return min((m1 >> 8) & 15u, (uint32_t)(G + 1)) * 18u + 11u - ((m1 >> 10) & 8u);
}

// The products of a step, behind one jump.  Case j = 0 .. G, 72 bytes: 4 products of the
// upper part into stripe j (32 bytes, jumped over where the step has none), 4 of the lower part into stripe j - 1, a
// branch to the end; behind the last case an empty step ends.  In assembly because an accumulator is fixed by its
// instruction and the compiler has no cheap way to choose one: a chain of comparisons runs through all G + 1 of them,
// most as taken branches, and with a switch or a tree the register allocator spills.
// Wait states are kept by hand: four scalar instructions lie between what writes the operands and the first product,
// products of one accumulator are at least a step's other half apart, and the caller waits before it reads them.
template <bool BF16, int G>
__device__ __forceinline__ void multiply(float4v (&acc)[G][kBlkCT], const short8v (&x)[kBlkCT], short8v wl, short8v wh, uint32_t entry) {
#define UBP_JUMP "s_getpc_b64 vcc\n\ts_lshl2_add_u32 vcc_lo, %[entry], vcc_lo\n\ts_addc_u32 vcc_hi, vcc_hi, 0\n\ts_setpc_b64 vcc\n\t"
#define UBP_ONE(T, J, C, W) "v_mfma_f32_16x16x32_" T " %[a" #J #C "], %[x" #C "], %[" W "], %[a" #J #C "]\n\t"
#define UBP_FOUR(T, J, W) UBP_ONE(T, J, 0, W) UBP_ONE(T, J, 1, W) UBP_ONE(T, J, 2, W) UBP_ONE(T, J, 3, W)
#define UBP_NONE "s_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0\n\t"
#define UBP_LEAVE "s_branch .Lstep_done%=\n\ts_nop 0\n\t"
#define UBP_CASE(T, J, BELOW) UBP_FOUR(T, J, "wh") UBP_FOUR(T, BELOW, "wl") UBP_LEAVE
#define UBP_FIRST(T) UBP_JUMP UBP_FOUR(T, 0, "wh") UBP_NONE UBP_LEAVE
#define UBP_LAST(T, BELOW) UBP_NONE UBP_FOUR(T, BELOW, "wl") UBP_LEAVE UBP_NONE ".Lstep_done%=:"
#define UBP_ACC(J) [a##J##0] "+v"(acc[J][0]), [a##J##1] "+v"(acc[J][1]), [a##J##2] "+v"(acc[J][2]), [a##J##3] "+v"(acc[J][3])
#define UBP_IN [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [wl] "v"(wl), [wh] "v"(wh), [entry] "s"(entry)
#define UBP_MULTIPLY(T)                                                                                                                 \
    if constexpr (G == 5)                                                                                                               \
        asm(UBP_FIRST(T) UBP_CASE(T, 1, 0) UBP_CASE(T, 2, 1) UBP_CASE(T, 3, 2) UBP_CASE(T, 4, 3) UBP_LAST(T, 4)                          \
            : UBP_ACC(0), UBP_ACC(1), UBP_ACC(2), UBP_ACC(3), UBP_ACC(4) : UBP_IN : "vcc", "scc");                                       \
    else if constexpr (G == 4)                                                                                                          \
        asm(UBP_FIRST(T) UBP_CASE(T, 1, 0) UBP_CASE(T, 2, 1) UBP_CASE(T, 3, 2) UBP_LAST(T, 3)                                            \
            : UBP_ACC(0), UBP_ACC(1), UBP_ACC(2), UBP_ACC(3) : UBP_IN : "vcc", "scc");                                                   \
    else                                                                                                                                \
        asm(UBP_FIRST(T) UBP_CASE(T, 1, 0) UBP_LAST(T, 1) : UBP_ACC(0), UBP_ACC(1) : UBP_IN : "vcc", "scc")
    static_assert(G == 5 || G == 4 || G == 2, "its cases are written out");
    if constexpr (BF16) {
        UBP_MULTIPLY("bf16");
    } else {
        UBP_MULTIPLY("f16");
    }
#undef UBP_MULTIPLY
#undef UBP_IN
#undef UBP_ACC
#undef UBP_LAST
#undef UBP_FIRST
#undef UBP_CASE
#undef UBP_LEAVE
#undef UBP_NONE
#undef UBP_FOUR
#undef UBP_ONE
#undef UBP_JUMP
}

// One workgroup = NP producer wavefronts + up to 16 - NP consumer wavefronts on one tile of 64
// columns of X / Y.
//  * Producers stage X in 64-row chunks into a ring of LDS slots (ring row = X row mod 1024)
//    with direct global->LDS loads, several chunks in flight; each publishes one counter, the
//    number of chunks whose share it has landed.  Every consumer publishes one counter of its
//    own, the number of leading chunks it will not read again; a slot is refilled once all of
//    them have passed the chunk that occupies it.  No workgroup barrier after start-up.
//  * Each consumer owns one row group (a run of at most G aligned 16-row stripes; runs with many
//    blocks are shorter, so that the consumers of a workgroup carry similar loads) and keeps its
//    G x 4 output tiles in fp32 accumulators for the whole K loop (output stationary).  Its steps are a
//    contiguous run of 1 KB operand records, fetched D steps ahead into a register ring, and of
//    8-byte metadata words, fetched 64 steps at a time (one per lane) and handed out with
//    v_readlane: a step costs one vector memory instruction.
//  * A step = two half-blocks (16 columns each) that start in the same stripe: two transposed
//    LDS reads per pixel tile gather their 32 rows of X; two compares and eight selects split the
//    operand into its lower-stripe and upper-stripe part; 4 + 4 MFMAs (16x16x32).  A lane reads
//    the window row congruent to its entry number modulo 16 (the columns of a half are rotated
//    like its rows), so an address is one addition and one and-or away from the window's first row and
//    the four tiles' reads differ by an immediate (with rows of 128 bytes and a swizzle six more vector instructions).
// 4096 x 4096 with 8192 pixels, skewed blocks, in a graph, all in one run: 92 us, with the tiles an immediate apart 88.7,
// the products behind one jump 86.1, the metadata taken apart for 64 steps at once 78.
// What bounds it there: waiting as much as issue.  A SIMD takes 370 cycles per step; the step's own 18 vector and
// 6.7 matrix instructions are 179 of them, and 40 % of the vector instructions belong to no step (polls, start-up, staging,
// stores).  A wavefront spends 40 % of its time waiting for a counter or a load - the first chunks of a workgroup,
// a chunk behind the heaviest row group -, 28 % waiting to issue and 32 % issuing; 12.5 of 16 are there on average.
// Before the last two of those steps (at 86 us) scalar masks in the place of the vector compares took 91.7, and the reads of
// step s + 1 issued behind the products of step s, with masks and addresses worked out while they run, 95.3.
// Every wait is bounded: if one runs out the wavefront raises *err and goes on without waiting
// (wrong numbers, but the kernel always terminates).
template <bool BF16, typename TY, int G, int MAXT>
__global__ __launch_bounds__(MAXT) void blk_kernel(BlkArgs a) {
    constexpr int CT = kBlkCT;
    constexpr int NTW = 16 * CT;
    constexpr int R = ring_slots(CT), KS = kSlotRows, RR = ring_rows(CT);
    constexpr int D = kPrefetchDepth;
    constexpr int PITCH = ring_pitch(CT);
    constexpr int NINST = KS / 8; // direct-to-LDS instructions per chunk (1 KB each: 8 rows)
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    uint32_t *published_p = reinterpret_cast<uint32_t *>(smem + a.ring_bytes); // [4] chunks landed, per producer
    uint32_t *released_p = published_p + 16;                                   // [16] per consumer wavefront

    // workgroup -> (column tile, workgroup row): consecutive workgroup ids go round-robin over the
    // 8 XCDs, so column tiles are dealt by id mod 8; an XCD then walks its tiles workgroup row by
    // workgroup row, so that what it runs at any time mostly shares one row's records in its L2.
    const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
    const int my_tiles = (a.n_coltiles - xcd + 7) >> 3;
    if (local >= my_tiles * a.n_wgrows) return;
    const int ctile = xcd + 8 * (local % my_tiles);
    const int wgrow = local / my_tiles;

    const int NP = a.n_producers;
    const int NC = (int)(blockDim.x >> 6) - NP; // consumer wavefronts; the last NP wavefronts produce
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    // the last tile of a row that is no whole number of tiles begins further left: it overlaps the one before it, whose pixels
    // both compute and store alike
    const int col0 = min(ctile * NTW, a.N - NTW);
    const int active = min(NC, a.nrg - wgrow * NC); // consumers the producers wait for

    // counters start at zero; the slots of producers that do not exist never hold anything back
    if (threadIdx.x < 32) published_p[threadIdx.x] = (threadIdx.x < 4 && (int)threadIdx.x >= NP) ? 0x7fffffffu : 0u;
    __syncthreads();

    // ------------------------------------------------------------------ producer
    if (wave >= NC) {
        const int me = wave - NC; // this producer takes instructions me, me + NP, ... of every chunk
        int published = 0;
        int free_upto = R; // chunks below this may be staged without asking: their slots are free
        bool broken = false;
        auto publish_upto = [&](int upto) {
            // relaxed on purpose: the data is known to have landed (explicit vmcnt wait); a
            // release here would make the compiler drain every load still in flight
            if (upto > published) {
                published = upto;
                if (lane == 0)
                    __hip_atomic_store(published_p + me, (uint32_t)upto, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        };
        // lane w < active looks at consumer w's counter; the other lanes never hold anything back
        auto poll = [&]() -> uint32_t {
            uint32_t v = 0xffffffffu;
            if (lane < active) v = __hip_atomic_load(&released_p[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            asm volatile("" ::: "memory");
            return v;
        };
        __builtin_amdgcn_s_setprio(3); // little work, but everyone else waits for it
        // (Staging through a register ring of ordinary loads instead - 24 loads of 1 KB in flight
        // per producer - was built and measured slower: 113 us against 101 us on the largest layer.)
        const uint32_t ring0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
        // byte offset of this lane's 16-byte piece (row, pixel tile, half of its 32 bytes) for instruction i of a chunk
        // of `rows` rows, from the instruction's first element; rows past K load the chunk's last row again (never
        // read): every chunk then issues the same number of loads, which the in-order vmcnt bookkeeping relies on
        auto piece = [&](int i, int rows) {
            const int r = min((lane >> 1) & 7, rows - 1 - 8 * i);
            return (uint32_t)(((int64_t)max(r, 0) * a.ldx + (lane >> 4) * 16 + (lane & 1) * 8) * 2);
        };
        const uint32_t voff = piece(0, KS);
        const int per = NINST / NP;                    // instructions of a chunk that are mine
        const int lag = max(1, min(48 / per, R / 2));  // chunks kept in flight before they are published
        const int64_t inst_stride = 8 * a.ldx;         // elements between the rows of two instructions
        for (int c = 0; c < a.nch; ++c) {
            const int slot = c % R;
            if (c >= free_upto && !broken) {
                // chunk c replaces chunk c - R: every consumer must have passed that one
                const uint32_t target = (uint32_t)(c - R + 1);
                uint32_t v = poll();
                if (__builtin_amdgcn_ballot_w64(v < target) != 0) {
                    // about to block: first publish every chunk already issued, the consumers
                    // this wait depends on may be waiting for one of them
                    wait_vmcnt<0>();
                    publish_upto(c);
                    int spins = 0;
                    do {
                        if (++spins > kSpinLimit) {
                            broken = true;
                            if (lane == 0) atomicOr(a.err, 1u);
                            break;
                        }
                        __builtin_amdgcn_s_sleep(2);
                        v = poll();
                    } while (__builtin_amdgcn_ballot_w64(v < target) != 0);
                }
                // how far the slowest consumer really is: saves asking again for the next chunks
                int ahead = 1;
                while (ahead < R && __builtin_amdgcn_ballot_w64(v < target + (uint32_t)ahead) == 0) ++ahead;
                free_upto = c + ahead;
            }
            const int k0 = c * KS;
            const int rows = min(KS, a.K - k0);
            const uint32_t dst = ring0 + (uint32_t)(slot * KS * PITCH);
            const uint16_t *base = a.X + (int64_t)k0 * a.ldx + col0; // wave-uniform
            if (rows == KS) {
                for (int i = me; i < NINST; i += NP) load16_to_lds(base + i * inst_stride, voff, dst + (uint32_t)i * 1024u);
            } else {
                for (int i = me; i < NINST; i += NP)
                    load16_to_lds(base + min(8 * i, rows - 1) * a.ldx, piece(i, rows), dst + (uint32_t)i * 1024u);
            }
            if (c + 1 - published > lag) {
                wait_vmcnt_at_most(lag * per); // vector memory completes in order: chunks <= c - lag have landed
                publish_upto(c + 1 - lag);
            }
        }
        // the tail: publish the chunks still in flight one by one as they land
        while (published < a.nch) {
            wait_vmcnt_at_most((a.nch - published - 1) * per);
            publish_upto(published + 1);
        }
        wait_vmcnt<0>();
        publish_upto(a.nch);
        return;
    }
    // Wavefront w runs on SIMD w mod 4 (in some order), and the producers, the last NP wavefronts,
    // take little of theirs: the SIMDs that host a producer have one consumer fewer and get the
    // workgroup's heaviest row groups (rg_order is sorted by decreasing work).
    int pos = wave;
    if (NP == 2 && NC == 14) pos = (wave & 2) ? (wave >> 2) * 2 + (wave & 1) : 6 + (wave >> 2) * 2 + (wave & 1);
    const int q = wgrow * NC + pos;
    if (q >= a.nrg) return; // no row group for this wavefront

    // ------------------------------------------------------------------ consumer
    const int rg = __builtin_amdgcn_readfirstlane(a.rg_order[q]);
    const int stripe0 = __builtin_amdgcn_readfirstlane(a.rg_order[a.nrg + rg]);          // the group's first stripe
    const int stripes = __builtin_amdgcn_readfirstlane(a.rg_order[a.nrg + rg + 1]) - stripe0; // at most G
    const int s_first = __builtin_amdgcn_readfirstlane(a.rg_ptr[rg]);
    const int s_all = __builtin_amdgcn_readfirstlane(a.rg_ptr[rg + 1]);

    float4v acc[G][CT];
#pragma unroll
    for (int j = 0; j < G; ++j)
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[j][c] = float4v{0.f, 0.f, 0.f, 0.f};

    // Records and metadata are fetched through buffer resources: the address of a load is a
    // wave-uniform byte offset in a scalar register plus a fixed per-lane offset, so a refill
    // costs no vector ALU work.  Both arrays carry spare records at their ends: refills simply
    // read on past the row group's last step.
    const __amdgpu_buffer_rsrc_t rsrc_f =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.frags), 0, (int)a.frag_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_m =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.meta), 0, (int)a.meta_bytes, 0x00020000);
    const uint32_t lane8 = (uint32_t)lane * 8u, lane16 = (uint32_t)lane * 16u;
    uint4v wf[D];
    uint32_t rec_next = (uint32_t)s_first * 1024u;
    auto issue = [&](int d) {
        wf[d] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc_f, lane16, rec_next, 0));
        rec_next += 1024u;
    };
    uint32_t meta_next = (uint32_t)s_first * 8u;
    auto load_meta = [&]() {
        const uint2v m = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rsrc_m, lane8, meta_next, 0));
        meta_next += 512u;
        return m;
    };

    // What a step asks of its metadata, worked out for 64 steps at once, one per lane, and laid so that most of it is used as
    // it stands: bits 0-6 multiply_entry, 7-16 ring row of half A's window, 17-27 last chunk read, 28-31 row offset of
    // half A;  7-16 ring row of half B's window, 17-26 chunks handed back, 28-31 row offset of half B.  Taking the words apart
    // step by step: 25 scalar and vector instructions more, 4096 x 4096 with 8192 pixels 86.1 us instead of 78.
    auto derive = [](uint2v m) -> uint2v {
        const uint32_t aA = m[0] & 0xffffu, aB = m[0] >> 16;
        static_assert(RR == 1024 && KS == 64, "10 bits of ring row, 11 of a chunk");
        return uint2v{multiply_entry<G>(m[1]) | (aA & 1023u) << 7 | ((max(aA, aB) + 15u) >> 6) << 17 | m[1] << 28,
                      (aB & 1023u) << 7 | (m[1] >> 22) << 17 | (m[1] >> 4) << 28};
    };

    int ready_upto = 0; // chunks known to be resident
    constexpr int kBroken = 0x7fffffff;
    const uint32_t mine_at = lds_address(reinterpret_cast<char *>(released_p + pos)); // (the producers look at positions 0 .. active - 1)
    auto wait_published = [&](int chunk) {
        if (__builtin_expect(chunk < ready_upto, 1)) return;
        int spins = 0;
        for (;;) {
            const uint32_t seen = flag_load(published_p + (lane & 3)); // unused producer slots were set to "all"
            ready_upto = __builtin_amdgcn_readfirstlane((int)min(min(__builtin_amdgcn_readlane(seen, 0), __builtin_amdgcn_readlane(seen, 1)),
                                                                 min(__builtin_amdgcn_readlane(seen, 2), __builtin_amdgcn_readlane(seen, 3))));
            if (chunk < ready_upto) return;
            if (++spins > kSpinLimit) {
                ready_upto = kBroken; // reported after the step loop (no global atomic inside it)
                return;
            }
            __builtin_amdgcn_s_sleep(1);
        }
    };
    // A counter only says "I will not read chunks below this again", so it can run ahead of the
    // producer (chunks this wavefront never reads) without harm.
    auto release_upto = [&](uint32_t upto) {
        // one lane's store, without a branch and without a wait: LDS executes this wavefront's operations in order, so
        // every read issued before it is served before it becomes visible
        uint64_t all;
        asm volatile("s_and_saveexec_b64 %0, 1\n\tds_write_b32 %1, %2\n\ts_mov_b64 exec, %0" : "=&s"(all) : "v"(mine_at), "v"(upto) : "memory", "scc");
    };

    const uint32_t ring_base = __builtin_amdgcn_readfirstlane(lds_address(smem));
    const int g = lane >> 4, n = lane & 15;
    // this lane's part in a transposed read of a 16-row window that begins at ring row r: window row congruent to e modulo
    // 16, which is 16 ((r + 15 - e) / 16) + e, 8 bytes (4 pixels) number n & 3 of the 32 bytes of pixel tile 0.  The ring
    // begins at LDS address 0 (the kernel has no other LDS, see LdsLimit), so that its wrap is a mask and the parts can be or-ed together.
    const uint32_t e = (uint32_t)(4 * g + (n >> 2));
    const uint32_t up = (15u - e) << 7, at = ring_base + (e >> 3) * 1024u + (e & 7u) * 32u + (uint32_t)(n & 3) * 8u;
    const uint32_t nlast = (uint32_t)n << 28 | 0x0fffffffu;

    if (s_first < s_all) {
        uint2v mcur = load_meta();
        uint2v mnext = load_meta();
#pragma unroll
        for (int d = 0; d < D; ++d) {
            issue(d);
            __builtin_amdgcn_sched_barrier(0); // same issue order as in the loop, slot by slot
        }
        // wait for them here, with a wait the compiler sees (vmcnt(0), other counters untouched):
        // loads it believes pending on registers that the loop body writes would otherwise cost a
        // wait for everything in flight at the first step of every round of the loop
        __builtin_amdgcn_s_waitcnt(0x0f70);
        {
            // nothing below the first step's windows is ever read: say so before the first wait, or
            // a row group whose first block lies beyond the ring would hold the producers back
            const uint32_t first = __builtin_amdgcn_readlane(mcur[0], 0);
            release_upto(min(first & 0xffffu, first >> 16) >> 6);
        }
        mcur = derive(mcur);
        int li = 0; // index of the round's first step within the metadata block
        for (int s = s_first; s < s_all; s += D) {
            if (li == 64) {
                li = 0;
                mcur = derive(mnext);
                mnext = load_meta();
            }
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const uint32_t m0 = __builtin_amdgcn_readlane(mcur[0], li + d);
                const uint32_t m1 = __builtin_amdgcn_readlane(mcur[1], li + d);
                wait_published((int)((m0 >> 17) & 2047u));
                // ---- gather: the 16 + 16 window rows, four pixel tiles
                short8v xf[CT];
                {
                    static_assert(PITCH == 128, "a ring row's bytes are 7 bits");
                    const uint32_t tA = ((m0 + up) & 0x1f800u) | at, tB = ((m1 + up) & 0x1f800u) | at;
#pragma unroll
                    for (int c = 0; c < CT; ++c) {
                        const short4v p0 = lds_read_tr(tA, c * kBlkTile);
                        const short4v p1 = lds_read_tr(tB, c * kBlkTile);
                        xf[c] = __builtin_shufflevector(p0, p1, 0, 1, 2, 3, 4, 5, 6, 7);
                    }
                }
                // hand back the chunks that no later step reads: LDS executes this wavefront's
                // operations in order, so the reads above are served before the counter moves
                release_upto((m1 >> 17) & 1023u);
                // ---- the operand's two parts: rows n >= o stay in the stripe the block starts in
                const uint4v f = wf[d];
                const bool inA = nlast >= m0, inB = nlast >= m1;
                const uint4v wl = {inA ? f[0] : 0u, inA ? f[1] : 0u, inB ? f[2] : 0u, inB ? f[3] : 0u};
                const uint4v wh = {inA ? 0u : f[0], inA ? 0u : f[1], inB ? 0u : f[2], inB ? 0u : f[3]};
                multiply<BF16, G>(acc, xf, __builtin_bit_cast(short8v, wl), __builtin_bit_cast(short8v, wh), m0 & 127u);
                issue(d);
            }
            li += D;
        }
    }
    release_upto((uint32_t)a.nch); // the last step's reads were consumed by its MFMAs
    if (ready_upto == kBroken && lane == 0) atomicOr(a.err, 2u);
    // the last products, which the compiler does not see as such, are in the accumulators behind this, and no read of them
    // is moved ahead of it
    asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
    for (int j = 0; j < G; ++j) asm volatile("" : "+v"(acc[j][0]), "+v"(acc[j][1]), "+v"(acc[j][2]), "+v"(acc[j][3]));

    // ---- store: lane (g = lane/16, n = lane%16) holds pixels col0 + 16*c + 4*g + v of row
    // 16*(stripe0 + j) + n, j < stripes.  Rows no block touches are stored as zeros like any other.
    TY *Yt = static_cast<TY *>(a.Y);
    // the epilogue (bias of the lane's row, clamp) is applied tile by tile on the way out
    const bool fused = a.ep.on != 0;
    if constexpr (sizeof(TY) == 2) {
        if (a.out_bytes != 0) {
            // A 16-bit tile straight from the accumulators is 8 bytes per lane, 32-byte runs per
            // row.  Through 16 LDS rows of this wavefront (16-byte pieces XOR-swizzled by the row
            // against bank conflicts; one wavefront writes and reads, LDS keeps its order) an
            // instruction stores whole rows of the tile, 16 bytes per lane.
            constexpr int RB = 16 * CT * 2;   // bytes per row of the tile
            constexpr int PR = RB / 16;       // 16-byte pieces per row
            constexpr int RP = 256 / RB;      // rows per 256 bytes (one pass over the banks)
            constexpr int NI = PR / 4;        // store instructions per stripe
            char *scratch = smem + a.ring_bytes + 32 * sizeof(uint32_t) + wave * a.out_bytes;
#pragma unroll
            for (int j = 0; j < G; ++j) {
                if (j >= stripes) break;
                const float bj = fused ? epilogue_bias(a.ep, (stripe0 + j) * kStripe + n, a.M) : 0.f;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    typedef TY ty4 __attribute__((ext_vector_type(4)));
                    ty4 o;
                    if (fused) epilogue_tile(a.ep, acc[j][c], bj);
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[v] = from_f32<TY>(acc[j][c][v]);
                    const int piece = (2 * c + (g >> 1)) ^ ((n / RP) & (PR - 1));
                    *reinterpret_cast<ty4 *>(scratch + n * RB + piece * 16 + (g & 1) * 8) = o;
                }
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const int r = i * (64 / PR) + lane / PR, lp = lane % PR;
                    const uint4v o = *reinterpret_cast<const uint4v *>(scratch + r * RB + ((lp ^ ((r / RP) & (PR - 1))) << 4));
                    const int row = (stripe0 + j) * kStripe + r;
                    if (row < a.M) *reinterpret_cast<uint4v *>(Yt + (int64_t)row * a.ldy + col0 + lp * 8) = o;
                }
            }
            return;
        }
    }
#pragma unroll
    for (int j = 0; j < G; ++j) {
        const int row = (stripe0 + j) * kStripe + n;
        if (j >= stripes || row >= a.M) continue;
        const float bj = fused ? epilogue_bias(a.ep, row, a.M) : 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int px = col0 + 16 * c + 4 * g;
            TY *dst = Yt + (int64_t)row * a.ldy + px;
            if (fused) epilogue_tile(a.ep, acc[j][c], bj);
            float v[4] = {acc[j][c][0], acc[j][c][1], acc[j][c][2], acc[j][c][3]};
            store_row<TY, 4>(dst, v);
        }
    }
}

template <bool BF16, typename TY, int G, int MAXT>
ubp_status launch_blk_inst(BlkArgs a, int waves, hipStream_t st, bool dry) {
    if (waves * 64 > MAXT) return UBP_ERR_UNSUPPORTED;
    // ring + the progress counters + (16-bit Y, where it fits) the consumers' output rows
    if (sizeof(TY) == 2) {
        const size_t want = (size_t)16 * 16 * kBlkCT * 2;
        if ((size_t)a.ring_bytes + 32 * sizeof(uint32_t) + (size_t)(waves - a.n_producers) * want <= 160 * 1024) a.out_bytes = (int)want;
    }
    const size_t lds = (size_t)a.ring_bytes + 32 * sizeof(uint32_t) + (size_t)(waves - a.n_producers) * a.out_bytes;
    static LdsLimit limit; // per instantiation
    const ubp_status rc = limit.raise(reinterpret_cast<const void *>(&blk_kernel<BF16, TY, G, MAXT>), true);
    if (rc != UBP_OK || dry) return rc;
    const unsigned grid = 8u * (unsigned)((a.n_coltiles + 7) / 8) * (unsigned)a.n_wgrows;
    return launch_kernel(&blk_kernel<BF16, TY, G, MAXT>, dim3(grid), dim3((unsigned)waves * 64), lds, st, a);
}

template <bool BF16, typename TY>
ubp_status launch_blk_t(const BlkArgs &a, int G, int waves, hipStream_t st, bool dry) {
    if (G == 5) return launch_blk_inst<BF16, TY, 5, 1024>(a, waves, st, dry);
    if (G == 4) return launch_blk_inst<BF16, TY, 4, 1024>(a, waves, st, dry);
    if (G == 2) return launch_blk_inst<BF16, TY, 2, 1024>(a, waves, st, dry);
    return UBP_ERR_UNSUPPORTED;
}

} // namespace

ubp_status launch_blk(const BlkArgs &a, bool bf16, bool y_f32, int G, int waves, void *stream, bool dry) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    // 64 rows of ldx elements must fit the producer's 32-bit lane offsets
    if (a.ldx > (int64_t(1) << 24)) return UBP_ERR_UNSUPPORTED;
    if (bf16) return y_f32 ? launch_blk_t<true, float>(a, G, waves, st, dry) : launch_blk_t<true, __bf16>(a, G, waves, st, dry);
    return y_f32 ? launch_blk_t<false, float>(a, G, waves, st, dry) : launch_blk_t<false, _Float16>(a, G, waves, st, dry);
}

} // namespace ubp
