// Direct kernel of the UBP library (fp16 / bf16): few pixels or a small layer, any alignment.
//
// Where a product is small, what it takes is a chain of latencies: staging X through LDS, a
// barrier, a ring with counters.  Here a wavefront goes from global memory to the matrix
// instructions with registers only, and the wavefronts of a workgroup split the columns of W.
#include "ubp_device.h"

#include <cstdint>
#include <cstring>

namespace ubp {

namespace {

// CT neighbouring 16-bit pixels of one row of X, as they lie in memory (any 2-byte alignment: the
// target allows unaligned vector access, and the compiler emits one load for the copy)
template <int CT> struct PixelsOf;
template <> struct PixelsOf<1> { typedef uint16_t type; };
template <> struct PixelsOf<2> { typedef uint32_t type; };
template <> struct PixelsOf<4> { typedef uint64_t type; };

// One workgroup = NW wavefronts on one 16-row stripe x 16 * CT pixels; wavefront w takes the
// stripe's steps w, w + NW, ...  A step = 32 columns in which the stripe keeps a weight: 16 bytes
// of weights per lane in operand order and the 8 row numbers of X of the lane's elements.
//  * Lane (g = lane / 16, n = lane mod 16) loads pixels CT n .. CT n + CT - 1 of its 8 rows: 16
//    lanes read 32 CT consecutive bytes of one row.  The operand of pixel tile t (pixels CT n + t,
//    n = 0..15) is element t of those 8 loads: a transposition inside the lane, four byte
//    permutations per tile, no LDS and no shuffles.
//  * The product is formed as weights x pixels: lane (g, n) holds rows 4 g + v of pixels CT n + t,
//    CT neighbouring pixels of a row, stored as one piece.
//  * The partial sums of the wavefronts meet in LDS once, at the end, in wavefront order.
// What bounds it: two dependent memory latencies (row numbers, then rows of X) and the exchange;
// against the gather kernel with its staged X, 11.5 -> 3.3 us on a 960 x 160 layer with 49
// pixels and 79 -> 3.8 us on a 4096 x 4096
// layer with 16 pixels, 24 -> 3.6 us on a 512 x 512 one with 196 (GPU time).
template <bool BF16, typename TY, int CT>
__global__ __launch_bounds__(1024) void direct_kernel(DirectArgs a) {
    typedef typename PixelsOf<CT>::type px_t;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int NW = (int)(blockDim.x >> 6);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, n = lane & 15;
    // Workgroup -> (pixel tile, stripe): consecutive workgroup ids go round-robin over the 8 XCDs.  The
    // pairs, stripes of a pixel tile next to each other, are cut into 8 equal runs, one per XCD, so that a
    // row of X comes from memory to about one XCD's L2 only (208 x 2280 with 2696 pixels: 20.4 -> 14.5 us).
    const int pairs = a.nstripes * a.n_tiles, xcd = blockIdx.x & 7;
    const int pair = (int)((int64_t)pairs * xcd >> 3) + (int)(blockIdx.x >> 3);
    if (pair >= (int)((int64_t)pairs * (xcd + 1) >> 3)) return;
    const int stripe = __builtin_amdgcn_readfirstlane(a.order[pair % a.nstripes]);
    const int px0 = pair / a.nstripes * (16 * CT);
    const int s0 = __builtin_amdgcn_readfirstlane(a.first[stripe]), s1 = __builtin_amdgcn_readfirstlane(a.first[stripe + 1]);

    // A lane whose pixels hang over the right edge loads the last CT pixels of the row and shifts
    // them into place; a lane beyond the edge computes on whatever it loaded and stores nothing.
    const bool edge = px0 + 16 * CT > a.N;
    const int col = px0 + CT * n, lcol = min(col, a.N - CT);
    const uint32_t shift = (uint32_t)min(col - lcol, CT - 1) * 16u;
    const uint32_t lane_off = (uint32_t)lcol * 2u, pitch = (uint32_t)a.ldx * 2u;
    const char *Xb = reinterpret_cast<const char *>(a.X);

    float4v acc[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};

    auto load_ids = [&](int s) { return *reinterpret_cast<const uint4v *>(a.ids + ((int64_t)s * 32 + g * 8)); };
    auto load_w = [&](int s) { return *reinterpret_cast<const uint4v *>(a.frags + ((int64_t)s * 512 + lane * 8)); };
    auto load_x = [&](const uint4v &ids, px_t(&x)[8]) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t id = (e & 1) ? ids[e >> 1] >> 16 : ids[e >> 1] & 0xffffu;
            __builtin_memcpy(&x[e], Xb + (size_t)(id * pitch + lane_off), sizeof(px_t));
        }
    };
    auto multiply = [&](const uint4v &w, px_t(&x)[8]) {
        if (edge) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = (px_t)(x[e] >> shift);
        }
        const short8v wv = __builtin_bit_cast(short8v, w);
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            uint4v f;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                if constexpr (CT == 1) {
                    f[d] = (uint32_t)x[2 * d] | ((uint32_t)x[2 * d + 1] << 16);
                } else {
                    const uint32_t lo = (uint32_t)(x[2 * d] >> (32 * (t >> 1))), hi = (uint32_t)(x[2 * d + 1] >> (32 * (t >> 1)));
                    f[d] = __builtin_amdgcn_perm(hi, lo, (t & 1) ? 0x07060302u : 0x05040100u);
                }
            }
            acc[t] = mfma16<BF16>(wv, __builtin_bit_cast(short8v, f), acc[t]);
        }
    };
    // two steps per round, all their loads issued before the first product; the row numbers of the
    // next round are fetched meanwhile
    int s = s0 + wave;
    if (s < s1) {
        const int last = s1 - 1;
        uint4v i0 = load_ids(s), i1 = load_ids(min(s + NW, last));
        for (; s < s1; s += 2 * NW) {
            px_t x0[8], x1[8];
            const uint4v w0 = load_w(s), w1 = load_w(min(s + NW, last));
            load_x(i0, x0);
            load_x(i1, x1);
            i0 = load_ids(min(s + 2 * NW, last));
            i1 = load_ids(min(s + 3 * NW, last));
            multiply(w0, x0);
            if (s + NW < s1) multiply(w1, x1);
        }
    }

    // ---- sums over the wavefronts, epilogue, store: wavefront v mod NW takes rows 4 g + v
    TY *Yt = static_cast<TY *>(a.Y);
    auto put = [&](int v, float(&o)[CT]) {
        const int row = stripe * kStripe + 4 * g + v;
        if (row >= a.M) return;
        if (a.ep.on) {
            const float b = epilogue_bias(a.ep, row, a.M);
#pragma unroll
            for (int t = 0; t < CT; ++t) o[t] = epilogue_value(a.ep, o[t], b);
        }
        TY r[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) r[t] = from_f32<TY>(o[t]);
        TY *dst = Yt + (int64_t)row * a.ldy + col;
        if (col + CT <= a.N) {
            __builtin_memcpy(dst, r, sizeof r);
        } else {
#pragma unroll
            for (int t = 0; t < CT; ++t)
                if (col + t < a.N) dst[t] = r[t];
        }
    };
    if (NW == 1) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float o[CT];
#pragma unroll
            for (int t = 0; t < CT; ++t) o[t] = acc[t][v];
            put(v, o);
        }
        return;
    }
    float *part = reinterpret_cast<float *>(smem); // [NW][CT][4][64]
#pragma unroll
    for (int t = 0; t < CT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[((wave * CT + t) * 4 + v) * 64 + lane] = acc[t][v];
    __syncthreads();
    for (int v = wave; v < 4; v += NW) {
        float o[CT];
#pragma unroll
        for (int t = 0; t < CT; ++t) o[t] = part[(t * 4 + v) * 64 + lane];
        for (int w = 1; w < NW; ++w)
#pragma unroll
            for (int t = 0; t < CT; ++t) o[t] += part[((w * CT + t) * 4 + v) * 64 + lane];
        put(v, o);
    }
}

template <bool BF16, typename TY, int CT>
ubp_status launch_direct_inst(const DirectArgs &a, int waves, hipStream_t st, bool dry) {
    if (dry) return UBP_OK; // at most 64 KB of LDS: no limit to raise
    const size_t lds = waves > 1 ? (size_t)waves * CT * 1024 : 0;
    DirectArgs b = a;
    b.n_tiles = (a.N + 16 * CT - 1) / (16 * CT);
    const unsigned grid = 8u * (unsigned)(((int64_t)a.nstripes * b.n_tiles + 7) / 8);
    return launch_kernel(&direct_kernel<BF16, TY, CT>, dim3(grid), dim3((unsigned)waves * 64), lds, st, b);
}

template <bool BF16, typename TY>
ubp_status launch_direct_t(const DirectArgs &a, int CT, int waves, hipStream_t st, bool dry) {
    if (CT == 1) return launch_direct_inst<BF16, TY, 1>(a, waves, st, dry);
    if (CT == 2) return launch_direct_inst<BF16, TY, 2>(a, waves, st, dry);
    if (CT == 4) return launch_direct_inst<BF16, TY, 4>(a, waves, st, dry);
    return UBP_ERR_UNSUPPORTED;
}

} // namespace

ubp_status launch_direct(const DirectArgs &a, bool bf16, bool y_f32, int CT, int waves, void *stream, bool dry) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (bf16) return y_f32 ? launch_direct_t<true, float>(a, CT, waves, st, dry) : launch_direct_t<true, __bf16>(a, CT, waves, st, dry);
    return y_f32 ? launch_direct_t<false, float>(a, CT, waves, st, dry) : launch_direct_t<false, _Float16>(a, CT, waves, st, dry);
}

} // namespace ubp
