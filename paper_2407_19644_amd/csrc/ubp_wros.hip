// Vector-ALU kernel of the UBP library: the paper's WROS dataflow, literally (Section 4.2).
#include "ubp_device.h"

#include <algorithm>
#include <cstdint>

namespace ubp {

namespace {

// ------------------------------------------------------------------ WROS vector kernel
// Grid: x = tiles of 64 * VEC columns (a multiple of 8 of them, so that all workgroups of a tile
// run on one XCD and share its L2), y = groups of row ranges; each wavefront of a workgroup takes
// one range of `rpr` output rows, and all of them sweep the same columns of X at about the same time.
// A lane owns VEC columns and BH accumulator rows (slots).  With rotated weights a block adds
// element s to slot s wherever it starts, so the walk over the blocks' columns, in order of their
// start rows, is one stream; after start row i is done, output row i is complete (later blocks
// start below it): its slot, i mod BH, is stored and cleared, the others keep accumulating.  A
// range re-walks the BH-1 start rows above it, whose blocks reach into the range, and drops what
// those blocks add to rows it does not own.
//   The stream is taken U columns at a time, and the U rows of X of the next batch are loaded
// before the current one is multiplied, over the ends of start rows too: otherwise every column
// waits for its index and then for its row of X.  fp32, a call among others: 512 x 512 in 4 x 1 blocks at 20 %
// with 6272 pixels 187 -> 53 us, 64 x 64 with 196 pixels 22 -> 10, 512 x 512 with 49 pixels 95 -> 20.  What bounds
// the large ones is reading rows of X again from L2 for every start row (11 TB/s).
// 64 columns of all of X in LDS instead, shared by 16 wavefronts, took longer: 62 us for 6272 pixels,
// 258 for 25088 (161 from L2) - scalar loads of weights and reads of LDS share one counter.
//   indptr: blocks per start row; cols: row of X per column of the stream, followed by
// kWrosBatch spare entries (row 0), which may be loaded and are never multiplied.
//   SHIFT: the dataflow that the weight rotation replaces (Section 3.3), for comparison only.  Accumulator
// row t always belongs to the output row t below the current start row: after a start row, row 0 is stored
// and the others move up by one register row.  Everything else is the same - grid, ranges, loads, batches
// and the order of additions per output element; a weight is read from the rotated array at the slot its row
// has there.  2 x 1, 4 x 1 and 8 x 1 blocks (256 x 256 with 25088 pixels, 512 x 512 with 6272, 1024 x 1024 with
// 1568, f16): 82, 51 and 64 us, with SHIFT 88, 57 and 76.
template <typename TX, typename TY, int BH, int VEC, bool SHIFT>
__device__ __forceinline__ void vector_walk(const int32_t *__restrict__ indptr, const int32_t *__restrict__ cols,
                                            const float *__restrict__ vals, const TX *__restrict__ X, int64_t ldx,
                                            TY *__restrict__ Y, int64_t ldy, int M, int N, int bw, int rpr, Epilogue ep) {
    constexpr int U = BH <= 4 ? 8 : BH <= 8 ? 4 : 2; // (a batch's weights fit the scalar registers)
    static_assert(U <= kWrosBatch, "spare entries of cols");
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t lo64 = ((int64_t)blockIdx.y * (blockDim.x >> 6) + wave) * rpr;
    const uint32_t col = (blockIdx.x * 64u + (threadIdx.x & 63u)) * VEC;
    if (lo64 >= M || col >= (uint32_t)N) return;
    const int lo = (int)lo64;
    const int hi = (int)min(lo64 + rpr, (int64_t)M);
    const int last_start = M - BH; // start rows beyond this hold no block (epilogue rows)
    float acc[BH][VEC];
#pragma unroll
    for (int s = 0; s < BH; ++s)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[s][v] = 0.f;

    auto load_x = [&](int64_t t, float(&x)[U][VEC]) {
#pragma unroll
        for (int u = 0; u < U; ++u) load_row<TX, VEC>(X + (int64_t)cols[t + u] * ldx + col, x[u]);
    };
    const int first = max(0, lo - BH + 1);
    int slot = first % BH; // of the current start row
    auto multiply = [&](const float *__restrict__ w, const float(&x)[VEC]) {
#pragma unroll
        for (int s = 0; s < BH; ++s) {
            const float ws = w[!SHIFT ? s : slot + s >= BH ? slot + s - BH : slot + s];
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[s][v] = fmaf(ws, x[v], acc[s][v]);
        }
    };

    int64_t t = 0;
    float x[U][VEC];
    if (first <= last_start) {
        const int b0 = indptr[first];
        t = (int64_t)b0 * bw;
        if (b0 < indptr[min(hi, last_start + 1)]) load_x(t, x);
    }
    for (int i = first; i < hi; ++i) {
        if (i <= last_start) {
            const int64_t t1 = (int64_t)indptr[i + 1] * bw;
            while (t < t1) {
                const int64_t next = min(t + U, t1);
                float xn[U][VEC];
                load_x(next, xn);
                const float *w = vals + t * BH;
                if (t + U <= t1) {
#pragma unroll
                    for (int u = 0; u < U; ++u) multiply(w + u * BH, x[u]);
                } else {
#pragma unroll
                    for (int u = 0; u < U - 1; ++u)
                        if (t + u < t1) multiply(w + u * BH, x[u]);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) x[u][v] = xn[u][v];
                t = next;
            }
        }
#pragma unroll
        for (int s = 0; s < BH; ++s) {
            if (s != (SHIFT ? 0 : slot)) continue;
            if (i >= lo) {
                if (ep.on) {
                    const float b = ep.bias ? ep.bias[i] : 0.f;
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[s][v] = epilogue_value(ep, acc[s][v], b);
                }
                store_row<TY, VEC>(Y + (int64_t)i * ldy + col, acc[s]);
            }
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[s][v] = 0.f;
        }
        if constexpr (SHIFT) {
#pragma unroll
            for (int s = 0; s + 1 < BH; ++s)
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[s][v] = acc[s + 1][v];
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[BH - 1][v] = 0.f;
        }
        slot = slot + 1 == BH ? 0 : slot + 1;
    }
}

template <typename TX, typename TY, int BH, int VEC>
__global__ __launch_bounds__(256) void wros_kernel(const int32_t *__restrict__ indptr, const int32_t *__restrict__ cols,
                                                  const float *__restrict__ vals, const TX *__restrict__ X, int64_t ldx,
                                                  TY *__restrict__ Y, int64_t ldy, int M, int N, int bw, int rpr, Epilogue ep) {
    vector_walk<TX, TY, BH, VEC, false>(indptr, cols, vals, X, ldx, Y, ldy, M, N, bw, rpr, ep);
}

template <typename TX, typename TY, int BH, int VEC>
__global__ __launch_bounds__(256) void naive_kernel(const int32_t *__restrict__ indptr, const int32_t *__restrict__ cols,
                                                   const float *__restrict__ vals, const TX *__restrict__ X, int64_t ldx,
                                                   TY *__restrict__ Y, int64_t ldy, int M, int N, int bw, int rpr, Epilogue ep) {
    vector_walk<TX, TY, BH, VEC, true>(indptr, cols, vals, X, ldx, Y, ldy, M, N, bw, rpr, ep);
}

template <typename TX, typename TY, int VEC>
ubp_status launch_wros_bh(const ubp_packed *p, const void *X, int64_t ldx, int N, void *Y, int64_t ldy, int rpr,
                          bool naive, const Epilogue &ep, hipStream_t st) {
    const int64_t ranges = ((int64_t)p->M + rpr - 1) / rpr, tiles = ((int64_t)N + 64 * VEC - 1) / (64 * VEC);
    const unsigned waves = tiles > (1 << 22) ? 1u : (unsigned)std::min<int64_t>(4, ranges); // (grid size in threads: 32 bits)
    const dim3 grid((unsigned)((tiles + 7) / 8 * 8), (unsigned)((ranges + waves - 1) / waves));
#define UBP_WROS_CASE(BH)                                                                                              \
    case BH:                                                                                                           \
        hipLaunchKernelGGL((naive ? (naive_kernel<TX, TY, BH, VEC>) : (wros_kernel<TX, TY, BH, VEC>)), grid,            \
                           dim3(waves * 64), 0, st, p->d_indptr, p->d_cols, p->d_values_f32,                           \
                           static_cast<const TX *>(X), ldx, static_cast<TY *>(Y), ldy, p->M, N, p->bw, rpr, ep);       \
        break;
    switch (p->bh) {
        UBP_WROS_CASE(1) UBP_WROS_CASE(2) UBP_WROS_CASE(3) UBP_WROS_CASE(4) UBP_WROS_CASE(5) UBP_WROS_CASE(6)
        UBP_WROS_CASE(7) UBP_WROS_CASE(8) UBP_WROS_CASE(9) UBP_WROS_CASE(10) UBP_WROS_CASE(11) UBP_WROS_CASE(12)
        UBP_WROS_CASE(13) UBP_WROS_CASE(14) UBP_WROS_CASE(15) UBP_WROS_CASE(16)
    default: return UBP_ERR_UNSUPPORTED;
    }
#undef UBP_WROS_CASE
    return hipGetLastError() == hipSuccess ? UBP_OK : UBP_ERR_DEVICE;
}

template <typename TX, typename TY>
ubp_status launch_wros_t(const ubp_packed *p, const void *X, int64_t ldx, int N, void *Y, int64_t ldy, int rpr,
                         bool naive, const Epilogue &ep, hipStream_t st) {
    // 4 columns per lane where every row of X and Y can be accessed as an aligned 4-vector and about a
    // wavefront per SIMD is left (512 x 512 with 6272 pixels: 46 us, with one column 60; 256 x 256 with
    // 784 pixels: 85 us, with one column 25)
    const bool vec_ok = (N % 4 == 0) && (ldx % 4 == 0) && (ldy % 4 == 0) &&
                        (reinterpret_cast<uintptr_t>(X) % (4 * sizeof(TX)) == 0) &&
                        (reinterpret_cast<uintptr_t>(Y) % (4 * sizeof(TY)) == 0);
    const int64_t waves4 = ((int64_t)N + 255) / 256 * (((int64_t)p->M + rpr - 1) / rpr);
    const bool vec = vec_ok && waves4 >= 1000;
    return vec ? launch_wros_bh<TX, TY, 4>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st)
               : launch_wros_bh<TX, TY, 1>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st);
}

} // namespace

ubp_status launch_wros(const ubp_packed *p, const void *X, int64_t ldx, int N, void *Y, int64_t ldy, ubp_dtype y_dtype,
                       int rpr, bool naive, const Epilogue &ep, void *stream, bool dry) {
    if (dry) return p->bh > 16 ? UBP_ERR_UNSUPPORTED : UBP_OK; // static LDS only: nothing to prepare
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (p->bh > 16) return UBP_ERR_UNSUPPORTED;
    switch (p->dtype) {
    case UBP_F32: return launch_wros_t<float, float>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st);
    case UBP_F16:
        return y_dtype == UBP_F32 ? launch_wros_t<_Float16, float>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st)
                                  : launch_wros_t<_Float16, _Float16>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st);
    case UBP_BF16:
        return y_dtype == UBP_F32 ? launch_wros_t<__bf16, float>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st)
                                  : launch_wros_t<__bf16, __bf16>(p, X, ldx, N, Y, ldy, rpr, naive, ep, st);
    }
    return UBP_ERR_INVALID_ARG;
}

// An empty kernel: what a launch costs on this device with nothing to do (measurement only).
__global__ void floor_kernel() {}

ubp_status launch_floor(void *stream) {
    hipLaunchKernelGGL(floor_kernel, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream));
    return hipGetLastError() == hipSuccess ? UBP_OK : UBP_ERR_DEVICE;
}

} // namespace ubp
