// fp32 kernel of the UBP library: the paper's WROS dataflow (Section 4.2) on 4 x 4 x 1 matrix instructions,
// X staged in LDS.
#include "ubp_device.h"

#include <cstdint>
#include <utility>

namespace ubp {

namespace {

template <int... I, class F> __device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void each(F &&f) { each_of(std::make_integer_sequence<int, N>{}, f); }

// 4 bytes per lane from global memory straight into LDS at lds_base + 4 * lane (see load16_to_lds)
__device__ __forceinline__ void load4_to_lds(const void *gbase, uint32_t lane_off, uint32_t lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(gbase), "s"(lds_base));
}

// A workgroup = NW wavefronts on PX pixels (64 or 32): all of X for them goes to LDS, then each wavefront walks
// the block columns of one range of output rows, in order of their start rows, as the vector kernel does, and
// begins BH - 1 start rows above its range.
//  * One v_mfma_f32_4x4x1 does 4 rows of a block column: 16 outer products of 4 x 1 by 1 x 4, all with the same 4
//    weights (broadcast out of the 16 sets that a register of 64 lanes holds) and 64 pixels, one lane
//    each; the result is 4 accumulator rows of a pixel in its lane's registers.  Only kept weights are
//    multiplied, and each product is added with one rounding, in the order in which the vector kernel adds: the
//    results are the same bit for bit, Inf and NaN included.
//  * The accumulator of a product is fixed by its instruction, so rotating the weights would ask for a branch per
//    row (4 us more on the layer below); after a row the other accumulator rows move up by one register instead.
//  * The columns come as a stream of records (64 weights in one load, row offsets in another, D records ahead, so that the
//    stream ends with spare records: a buffer's bounds check does not count the scalar offset that the records are reached by), in
//    groups of 4 columns of one start row, the last ones filled up with weights -0 and a row of +0, whose products leave every sum as it is.
//    A group's addresses are formed two groups ahead and its rows of X read one group ahead.
// What bounds it: the matrix instructions' and the LDS reads' issue and the row ends, each about a third of the
// time; an address per vector instruction, which gets in the way of the matrix instructions, took 25 us instead of 21.
// A call among others: 512 x 512 in 4 x 1 blocks at 20 % with 6272 pixels 44.9 -> 20.1 us in a graph (vector kernel: X
// from L2 for every block), 64 x 64 with 196 pixels 9.6 -> 4.7, 512 x 512 with 49 pixels 19.8 -> 7.9, in 16 x 16
// blocks at 10 % with 6272 pixels 72.9 -> 20; 190 layers of up to 1024 x 1024 with 6272 pixels: 2.5 times as fast on
// average, one 3 % slower.
template <int BH, int PX>
__global__ __launch_bounds__(1024) void wros4_kernel(Wros4Args a) {
    constexpr int Q = (BH + 3) / 4;                          // accumulator quads
    constexpr int QP = wros4_quads(BH), COLS = 16 / QP, GROUPS = COLS / 4;
    constexpr int PITCH = 4 * PX;
    constexpr int D = kWros4Depth;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int NW = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    // Workgroup -> (pixel tile, slice of rows): consecutive workgroup ids go round-robin over the 8 XCDs.  The
    // pairs, slices of a tile next to each other, are cut into 8 equal runs, one per XCD: a tile's X comes from
    // memory to about one XCD's L2 only.
    const int pairs = a.n_tiles * a.slices, xcd = blockIdx.x & 7;
    const int pair = (int)((int64_t)pairs * xcd >> 3) + (int)(blockIdx.x >> 3);
    if (pair >= (int)((int64_t)pairs * (xcd + 1) >> 3)) return;
    const int col0 = pair / a.slices * PX;
    const int64_t lo64 = ((int64_t)(pair % a.slices) * NW + wave) * a.rpr;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));

    // ---- X to LDS, rows of PX pixels; pixels beyond N repeat ones inside (and are never stored)
    const int k8 = (a.K + 7) & ~7;
    if (a.vec4) {
        constexpr int LPR = PX / 4, RPI = 64 / LPR;          // lanes per row, rows per load
        const int r_in = lane / LPR, col = min(col0 + 4 * (lane % LPR), a.N - 4);
        for (int r = wave * RPI; r < a.K; r += NW * RPI)
            load16_to_lds(a.X + (int64_t)r * a.ldx, (uint32_t)(((int64_t)min(r_in, a.K - 1 - r) * a.ldx + col) * 4), lds0 + (uint32_t)(r * PITCH));
    } else {
        constexpr int RPI = 64 / PX;
        const int r_in = lane / PX, col = min(col0 + lane % PX, a.N - 1);
        for (int r = wave * RPI; r < a.K; r += NW * RPI)
            load4_to_lds(a.X + (int64_t)r * a.ldx, (uint32_t)(((int64_t)min(r_in, a.K - 1 - r) * a.ldx + col) * 4), lds0 + (uint32_t)(r * PITCH));
    }
    if (threadIdx.x < PX) *reinterpret_cast<float *>(smem + k8 * PITCH + threadIdx.x * 4) = 0.f;

    // ---- the first records of this wavefront's range
    const int lo = (int)min(lo64, (int64_t)a.M), hi = (int)min(lo64 + a.rpr, (int64_t)a.M);
    const int first = min(max(0, lo - BH + 1), a.M - 1);
    const int rec0 = __builtin_amdgcn_readfirstlane(a.rec_of_row[first]);
    const int row0 = __builtin_amdgcn_readfirstlane(a.row_of_rec[rec0]);
    const int rec1 = __builtin_amdgcn_readfirstlane(a.rec_of_end[max(hi, 1) - 1]) + 1;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.weights), 0, (int)a.weight_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.offsets), 0, (int)a.offset_bytes, 0x00020000);
    const uint32_t lane4 = (uint32_t)lane * 4u, olane = (uint32_t)min(lane, 16) * 4u;
    uint32_t w_next = (uint32_t)rec0 * 256u, o_next = (uint32_t)rec0 * 128u;
    float wv[D];
    float ov[D]; // (bit patterns)
    auto fetch = [&](int d) {
        wv[d] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, lane4, w_next, 0));
        ov[d] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(ro, olane, o_next, 0));
        w_next += 256u;
        o_next += 128u;
    };
#pragma unroll
    for (int d = 0; d < D; ++d) fetch(d);
    // (a wait that the compiler sees: it would otherwise wait for all records in flight at the head of the loop)
    __builtin_amdgcn_s_waitcnt(0x0f70);
    asm volatile("" ::: "memory");
    __syncthreads();
    if (lo >= hi) return;

    float4v acc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] = float4v{0.f, 0.f, 0.f, 0.f};
    int i = min(first, row0);                                // the next output row to finish: accumulator row 0
    char *yrow = reinterpret_cast<char *>(a.Y) + (int64_t)i * a.ldy * 4;
    // (a lane without a pixel stores beyond the row's N pixels, which is dropped)
    const uint32_t ycol = PX == 64 || lane < PX ? (uint32_t)(col0 + lane % PX) * 4u : 0xfffffffcu;
    auto finish = [&](int n) {                               // n rows are complete
        for (; n > 0; --n) {
            if ((uint32_t)(i - lo) < (uint32_t)(hi - lo)) {
                float v = acc[0][0];
                if (a.ep.on) {
                    int row = i;
                    asm volatile("" : "+s"(row)); // (no pointer into the bias is carried along where there is none)
                    v = epilogue_value(a.ep, v, a.ep.bias ? a.ep.bias[row] : 0.f);
                }
                const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(yrow, 0, a.N * 4, 0x00020000);
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), ry, ycol, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < BH; ++t) acc[t >> 2][t & 3] = t + 1 < BH ? acc[(t + 1) >> 2][(t + 1) & 3] : 0.f;
#pragma unroll
            for (int q = 0; q < Q; ++q) asm volatile("" : "+v"(acc[q])); // (moved here and not, by the compiler, on every path around)
            ++i;
            yrow += a.ldy * 4;
        }
    };
    finish(row0 - i);
    if (rec0 >= rec1) return;

    // LDS addresses of a group's 4 columns: base + offset, added by one more 4 x 4 x 1 product, offset x 1, on
    // denormal numbers, whose bit patterns are the integers (no rounding: all are below 2^23)
    const float base = __builtin_bit_cast(float, lds0 + (uint32_t)(lane % PX) * 4u), one = PX == 64 ? 1.f : 0.5f;
    const float4v base4 = {base, base, base, base};
    typedef __attribute__((address_space(3))) const float *lds_float_ptr;
    float x[2][4];
    float4v ad[2];
    // group G behind the first one of a round
    auto address = [&](auto G_) {
        constexpr int G = decltype(G_)::value;
        ad[G % 2] = __builtin_amdgcn_mfma_f32_4x4x1f32(ov[G / GROUPS % D], one, base4, 4, G % GROUPS, 0);
    };
    auto read = [&](auto G_) {
        constexpr int G = decltype(G_)::value;
#pragma unroll
        for (int c = 0; c < 4; ++c) x[G % 2][c] = *(lds_float_ptr)(uintptr_t)__builtin_bit_cast(uint32_t, (float)ad[G % 2][c]);
    };
    address(std::integral_constant<int, 0>{});
    read(std::integral_constant<int, 0>{});
    address(std::integral_constant<int, 1>{});
    auto record = [&](auto d_) {
        constexpr int d = decltype(d_)::value;
        const uint32_t ends = (uint32_t)__builtin_amdgcn_readlane(__builtin_bit_cast(int, ov[d]), 16);
        each<GROUPS>([&](auto g_) {
            constexpr int g = decltype(g_)::value, G = d * GROUPS + g;
            read(std::integral_constant<int, G + 1>{});
            address(std::integral_constant<int, G + 2>{});
            each<4>([&](auto c_) {
                constexpr int c = decltype(c_)::value;
                each<Q>([&](auto q_) {
                    constexpr int q = decltype(q_)::value;
                    acc[q] = __builtin_amdgcn_mfma_f32_4x4x1f32(wv[d], x[G % 2][c], acc[q], 4, (4 * g + c) * QP + q, 0);
                });
            });
            finish((int)((ends >> (8 * g)) & 255u));
        });
        fetch(d);
    };
    // (one exit, at the end of a round of D: the records behind the last one are walked for nothing, and nothing is stored)
    for (int r = rec0; r < rec1; r += D) each<D>(record);
}

template <int BH> ubp_status launch_bh(const Wros4Args &a, int PX, int waves, hipStream_t st, bool dry) {
    const size_t lds = (size_t)(((a.K + 7) & ~7) + 1) * 4 * PX;
    static LdsLimit limit64, limit32;
    const ubp_status rc = PX == 64 ? limit64.raise(reinterpret_cast<const void *>(&wros4_kernel<BH, 64>))
                                   : limit32.raise(reinterpret_cast<const void *>(&wros4_kernel<BH, 32>));
    if (rc != UBP_OK || dry) return rc;
    const dim3 grid(8u * (unsigned)(((int64_t)a.n_tiles * a.slices + 7) / 8)), block((unsigned)waves * 64);
    return launch_kernel(PX == 64 ? &wros4_kernel<BH, 64> : &wros4_kernel<BH, 32>, grid, block, lds, st, a);
}

} // namespace

ubp_status launch_wros4(const Wros4Args &a, int bh, int PX, int waves, void *stream, bool dry) {
    hipStream_t st = static_cast<hipStream_t>(stream);
#define UBP_WROS4_CASE(BH) \
    case BH: return launch_bh<BH>(a, PX, waves, st, dry);
    switch (bh) {
        UBP_WROS4_CASE(1) UBP_WROS4_CASE(2) UBP_WROS4_CASE(3) UBP_WROS4_CASE(4) UBP_WROS4_CASE(5) UBP_WROS4_CASE(6)
        UBP_WROS4_CASE(7) UBP_WROS4_CASE(8) UBP_WROS4_CASE(9) UBP_WROS4_CASE(10) UBP_WROS4_CASE(11) UBP_WROS4_CASE(12)
        UBP_WROS4_CASE(13) UBP_WROS4_CASE(14) UBP_WROS4_CASE(15) UBP_WROS4_CASE(16)
    }
#undef UBP_WROS4_CASE
    return UBP_ERR_UNSUPPORTED;
}

} // namespace ubp
