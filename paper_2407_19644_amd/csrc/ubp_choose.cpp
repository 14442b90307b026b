// Host side of the UBP library: which kernel a call takes, with which launch shape.  No device
// code here: what a call resolves to can be checked without a GPU.
#include <algorithm>
#include <cmath>
#include <new>
#include <stdexcept>

#include "ubp_internal.h"

namespace ubp {

namespace {

// ------------------------------------------------------------------ estimates
// What a 16-bit product would take, in microseconds, by each kernel: linear in the few quantities that
// cost, coefficients fitted (relative least squares, none negative) to layers drawn over the range of layers this
// library is for - 1 x 1 and im2col convolutions at batch 1 to 64, fully connected layers, large layers of 16 x 16
// blocks, aligned and odd rows.  On 3172 layers timed through kernels 2, 8 and the one chosen (up to 4096 x 4096 with 16384
// pixels, densities of 0.4 to 30 %, blocks of 1 x 1 to 16 x 32) the kernel of the smallest estimate took 0.6 % longer than
// the fastest one on average, 3 % at the 95th percentile, 59 % at most.
constexpr double kNever = 1e30;
constexpr double kCUs = 256.0;

int direct_tiles(int N) { return N <= 16 ? 1 : N <= 32 ? 2 : 4; }
// A launch has fewer than 2^32 threads: workgroups (a multiple of 8) of `waves` wavefronts, one per 16 rows x 16 CT pixels.
bool direct_fits(const ubp_packed *p, int N, int CT, int waves) {
    const int64_t pairs = (int64_t)((p->M + 15) / 16) * (((int64_t)N + 16 * CT - 1) / (16 * CT));
    return pairs <= 0x7fffffff && (pairs + 7) / 8 * 8 * waves * 64 < (int64_t(1) << 32);
}
bool direct_able(const ubp_packed *p, int N, int64_t ldx_bytes) { // 16-bit row numbers, 32-bit byte offsets into X
    return p->dtype != UBP_F32 && p->K <= 0x10000 && N >= 1 && ldx_bytes < (int64_t(1) << 24) &&
           (int64_t)p->K * ldx_bytes < (int64_t(1) << 32) && direct_fits(p, N, direct_tiles(N), 1);
}

// Wavefronts per workgroup: enough that a wavefront has one or two steps, as long as the chip is not full.
// waves: in: 0 or pinned; out: what the estimate is for.
double estimate_direct(const ubp_packed *p, int N, int CT, size_t ysz, int &waves) {
    const MaskStats &S = get_mask_stats(p);
    const double stripes = (p->M + 15) / 16, px_tiles = (N + 16 * CT - 1) / (16 * CT), wgs = stripes * px_tiles;
    const double load = S.steps * px_tiles * (1024 + 64 + 1024 * CT) / kCUs * 1e-5; // weights, row numbers, rows of X
    const double fixed = 2.77 + (N % 8 != 0 ? 2.023 : 1.427) * load + 0.594 * 0.2e-6 * p->M * (double)N * ysz +
                         0.352 * 0.4e-6 * p->K * (double)N;
    double best = kNever;
    int best_w = 4;
    for (int w = 1; w <= 16; w *= 2) {
        if (waves != 0 && w != 16) continue;
        const int ww = waves ? waves : w;
        if (w == 16 && CT > 1 && !waves) continue; // (its exchange of partial sums costs more than the steps it saves)
        if (!waves && !direct_fits(p, N, CT, w)) continue;
        const double t = fixed + 0.156 * std::ceil((double)S.steps / stripes / ww) + 0.01404 * wgs * ww * CT / kCUs;
        if (t < best * (ww == 4 ? 1.03 : 1.0)) { // (four where it hardly matters)
            best = t;
            best_w = ww;
        }
    }
    waves = best_w;
    return best;
}

// Dense tiles through LDS, by shape and by whether rows of X take the way through registers
double estimate_mtile(const ubp_packed *p, int N, int shape, bool ragged, size_t ysz) {
    // fixed; per tile and stage of 64 columns (of a CU's tiles one after the other); per tile; per 5 MB of Y;
    // per tile and stage where empty tiles of W are left out; per round of tiles and stage
    static const double kAligned[kNumMtileShapes][6] = {{3.015, 0.370, 0.410, 0.913, 0.039, 0.0},
                                                        {2.606, 0.285, 0.460, 0.788, 0.021, 0.0},
                                                        {2.609, 0.283, 0.430, 0.794, 0.028, 0.0},
                                                        {2.653, 0.129, 0.199, 0.726, 0.012, 0.106},
                                                        {3.356, 0.672, 0.315, 0.908, 0.141, 0.0}}; // (5 % above the fit to 260 layers:
    // of the 16 it takes from the other shapes and kernel 4 none is slower, the mean takes 0.91 of the time)
    static const double kRagged[kNumMtileShapes][6] = {{4.592, 0.695, 0.0, 0.397, 0.020, 0.0},
                                                       {3.788, 0.523, 0.0, 0.297, 0.0, 0.0},
                                                       {kNever, 0.0, 0.0, 0.0, 0.0, 0.0},   // (never the best one there)
                                                       {3.109, 0.0, 0.312, 1.143, 0.0, 0.508},
                                                       {kNever, 0.0, 0.0, 0.0, 0.0, 0.0}};  // (not built)
    const MtileShape &sh = kMtileShapes[shape];
    const MaskStats &S = get_mask_stats(p);
    const double *c = ragged ? kRagged[shape] : kAligned[shape];
    const int64_t tiles = (int64_t)((p->M + sh.rows - 1) / sh.rows) * ((N + sh.pixels - 1) / sh.pixels);
    const double per_cu = (double)(((tiles + 7) / 8 + 31) / 32); // an eighth of the tiles to each XCD, 32 CUs each
    const double stages = (p->K + 63) / 64, rounds = std::ceil(per_cu / sh.per_cu);
    return c[0] + per_cu * (stages * (c[1] + (S.tiles_hit < S.tiles ? c[4] : 0.0)) + c[2]) + rounds * stages * c[5] +
           c[3] * 0.2e-6 * p->M * (double)N * ysz;
}

// Launch shape of the small-K kernel.  64-pixel blocks halve the weight traffic per pixel; 32-pixel blocks
// where those would be few.  Workgroups of 4 wavefronts, about one and a half per CU: two share a CU and the
// one's loading of X overlaps the other's streaming (measured better than one workgroup of 8).  The stripes are
// cut into slices to get there - every slice loads the X block again, so only while a wavefront keeps at least
// 3 stripes.
int xstat_col_tiles(int N) { return N >= 128 * 64 ? 4 : 2; }
int xstat_slices(int nstripes, int n_blocks) {
    return std::max(1, std::min((int)std::lround(384.0 / n_blocks), nstripes / 12));
}

double estimate_xstat(const ubp_packed *p, int N, size_t ysz) {
    const int CT = xstat_col_tiles(N), blocks = (N + 16 * CT - 1) / (16 * CT), stripes = (p->M + 15) / 16;
    const int slices = xstat_slices(stripes, blocks), each = (stripes + slices - 1) / slices;
    const double wgs = (double)blocks * slices, rounds = std::ceil(wgs / (2 * kCUs));
    return 3.13 + 0.795 * 0.2e-6 * p->M * (double)N * ysz + 1.0 * p->K / 256.0 +
           0.01865 * rounds * ((each + 3) / 4) * ((p->K + 31) / 32) * CT + 2.42 * wgs / (2 * kCUs) * p->K * CT / 1024.0;
}

int blk_auto_G(const ubp_packed *p) { // 5 stripes per wavefront where that saves a workgroup row: X is staged once per workgroup row
    auto rows_for = [&](int g) { return ((p->M + 16 * g - 1) / (16 * g) + 13) / 14; };
    return rows_for(5) < rows_for(4) ? 5 : 4;
}

// Whole blocks as operands: per round of workgroups the staging of X and a wavefront's share of the steps (two halves of
// 16 columns each); behind them a launch of the gather kernel for the last columns, where they are left to it.
// Which split - stripes of a wavefront, producers among 16 wavefronts - is a matter of rounds: X is staged once per workgroup
// row, so that 5 stripes and 2 producers do the least work, but as long as more workgroup rows run beside each other and
// not one after the other, each is through sooner with fewer steps per wavefront and with more producers.  4096 x 4096 at 10 %, by
// stripes / producers: 1024 pixels 5/2 34.8, 4/2 31.9, 2/2 27.8, 2/4 25.1 us, 8192 pixels 77, 94, 130, 131; 2048 x 4096 at 5 % with 4096 pixels
// 30.5, 28.5, 45.0 and by 4/4 26.1.
// Coefficients fitted to 600 layers of 512 to 4096 rows, 1152 to 4096 columns and 128 to 8192 pixels at 5 to 20 %, even and skewed: mean
// error 4 to 7 %; on 400 others what is chosen, by this estimate or for another kernel, takes as long as the fastest of the six and the direct kernel
// on average, 5 % longer at the 95th percentile, 17 % at most.
struct BlkSplit {
    int G, NP;
    double fixed, per_stage, per_step, per_y;
};
constexpr BlkSplit kBlkSplits[] = {{2, 2, 5.25, 4.017, 0.2483, 1.272}, {2, 4, 5.27, 3.757, 0.1902, 1.305}, {4, 2, 6.18, 3.543, 0.2561, 0.972},
                                   {4, 4, 6.34, 3.213, 0.2054, 1.011}, {5, 2, 6.64, 3.371, 0.2651, 0.901}, {5, 4, 6.97, 2.961, 0.2171, 0.943}};
double estimate_blk(const ubp_packed *p, int N, size_t ysz, const BlkSplit *&split) {
    const int stripes = (p->M + 15) / 16, tiles = blk_leaves_tail(N) ? N / 64 : (N + 63) / 64;
    const double stage = 1e-3 * p->K, steps = 0.5 * (double)p->nb * ((p->bw + 15) / 16), y = 0.2e-6 * p->M * (double)N * ysz;
    double best = kNever;
    for (const BlkSplit &c : kBlkSplits) {
        const int runs = std::min(stripes, ((stripes + c.G - 1) / c.G + kBlkConsumers - 1) / kBlkConsumers * kBlkConsumers); // (cut_row_groups)
        const int rows = (runs + 15 - c.NP) / (16 - c.NP);                                                                   // of workgroups
        const double rounds = std::ceil((double)((tiles + 7) / 8) * rows / 32);
        const double t = c.fixed + rounds * (c.per_stage * stage + c.per_step * steps / runs) + c.per_y * y;
        if (t < best) {
            best = t;
            split = &c;
        }
    }
    return best + (blk_leaves_tail(N) ? 17.59 + 30.38 * stage : 0.0);
}

int gather_col_tiles(int N) {
    // Column tiles as wide as divides N (a ragged last tile takes the slow staging path), provided that still
    // leaves a few dozen tiles: wide tiles amortise a step's fixed instruction cost over more matrix instructions
    // (from measurements on the benchmark layers).
    for (int ct = 8; ct >= 2; ct /= 2)
        if (N % (16 * ct) == 0 && N / (16 * ct) >= 32) return ct;
    for (int ct = 8; ct >= 2; ct /= 2)
        if ((N + 16 * ct - 1) / (16 * ct) >= 32) return ct;
    return 2;
}

// Launch shape of the gather kernel on row groups of G stripes and tiles of 16 CT pixels.
ubp_status gather_launch(const ubp_packed *p, int N, int G, int CT, const ubp_plan &pl, Shape &s) {
    int waves = pl.waves, NP = pl.producers;
    const int nrg = (p->M + kStripe * G - 1) / (kStripe * G);
    // one wavefront stages about 28 GB/s: a second one as soon as a workgroup's tile is not small
    if (NP == 0) {
        NP = ((int64_t)p->K * 32 * CT >= 64 * 1024) ? 2 : 1;
        if (waves != 0 && waves < NP + 1) NP = 1; // a caller who fixes a tiny workgroup gets one producer
    }
    const int max_waves = stripe_max_waves(G, CT);
    if (max_waves <= NP) return UBP_ERR_UNSUPPORTED;
    // When the ring holds all of K nothing is ever refilled and a consumer may walk several row
    // groups one after the other; the number of workgroup rows is then free.  Otherwise every
    // consumer owns exactly one row group.
    const bool resident = (p->K + kSlotRows - 1) / kSlotRows <= ring_slots(CT);
    int wg_rows = pl.wg_rows;
    if (wg_rows < 0) return UBP_ERR_INVALID_ARG;
    if (!resident) {
        if (waves == 0) {
            // as few workgroup rows as the wavefront limit allows; full workgroups if the last row is
            // then still at least half full (more consumers per CU measured better than even rows),
            // else the consumers spread evenly over the rows
            const int maxc = max_waves - NP;
            const int rows_wg = (nrg + maxc - 1) / maxc;
            const int last = nrg - (rows_wg - 1) * maxc;
            waves = (2 * last >= maxc ? maxc : (nrg + rows_wg - 1) / rows_wg) + NP; // consumers + producers
        }
        if (waves < NP + 1 || waves > max_waves) return UBP_ERR_UNSUPPORTED;
        const int need_rows = (nrg + (waves - NP) - 1) / (waves - NP);
        if (wg_rows != 0 && wg_rows != need_rows) return UBP_ERR_UNSUPPORTED;
        wg_rows = need_rows;
    } else {
        const int64_t ncol = (N + 16 * CT - 1) / (16 * CT);
        if (wg_rows == 0) {
            // about one workgroup per CU in a single round where the column tiles alone do not
            // fill the chip; then as few workgroup rows as give every consumer the same number
            // of row groups (no half-used passes)
            const int target = (int)std::max<int64_t>(1, 256 / std::max<int64_t>(1, ncol));
            const int nc = std::max(1, (waves ? waves : max_waves) - NP);
            const int passes = std::max(1, (nrg + nc * target - 1) / (nc * target));
            wg_rows = (nrg + nc * passes - 1) / (nc * passes);
        }
        wg_rows = std::max(1, std::min(wg_rows, std::max(1, nrg)));
        if (waves == 0) waves = std::min(max_waves - NP, (nrg + wg_rows - 1) / wg_rows) + NP;
        if (waves < NP + 1 || waves > max_waves) return UBP_ERR_UNSUPPORTED;
    }
    s.G = G;
    s.CT = CT;
    s.NP = NP;
    s.waves = waves;
    s.wg_rows = wg_rows;
    s.resident = resident;
    return UBP_OK;
}

// The gather kernel, aligned rows only (on odd rows it was never the fastest, on none of 298 layers): per round of
// workgroups (an XCD's workgroups on its 32 CUs) the staging of X, the workgroup's steps and the longest wavefront's; a
// ragged last tile is a launch of its own behind the others, whose X passes through registers.
double estimate_gather(const ubp_packed *p, int N, size_t ysz) {
    Shape s;
    const int G = gather_stripes(p), CT = gather_col_tiles(N);
    if (gather_launch(p, N, G, CT, ubp_plan{}, s) != UBP_OK) return kNever;
    const double steps = (double)get_mask_stats(p).gather_steps, nrg = (p->M + kStripe * G - 1) / (kStripe * G);
    if (steps * (512 + 1024 * G) >= (double)(int64_t(1) << 31)) return kNever; // (its records have 32-bit byte offsets)
    const double walks = s.resident ? std::ceil(nrg / ((double)s.wg_rows * (s.waves - s.NP))) : 1; // row groups of a wavefront
    const double stage = 1e-3 * p->K * CT / s.NP;
    const int tiles = N / (16 * CT);
    const double rounds = std::ceil((tiles + 7) / 8 * (double)s.wg_rows / 32);
    return 2.445 + rounds * (1.756 * stage + (0.777e-3 * CT * G + 4.846e-3) * steps / s.wg_rows +
                             (0.1542 + 2.15e-3 * CT * G) * walks * steps / nrg + 1.361) +
           1.433 * 0.2e-6 * p->M * (double)N * ysz + (N % (16 * CT) != 0 ? 12.82 + 15.17 * stage : 0.0);
}

int tile_layout_words(const ubp_packed *p) { return (tile_kt_pad(p->M, p->K) + 31) / 32; } // occupancy words per stripe; 0: no dense tiles
bool all_tiles_kept(const ubp_packed *p) {
    const TileLayout &T = get_tile_layout(p);
    return T.kt_pad != 0 && T.tiles_nonzero == (int64_t)T.nstripes * ((p->K + kStep - 1) / kStep);
}
bool mtile_able(const ubp_packed *p, int N) { // a piece of 8 pixels fits a row
    return p->dtype != UBP_F32 && N >= 8 && tile_layout_words(p) > 0;
}
// The way rows of X take: 0 straight into LDS, 1 through registers (rows that are no 16-byte pieces), 2 through
// registers with 64-bit offsets (rows more than 32 MB apart, of which 64 have no 32-bit offsets; tiles of 64 x 64 only).
int mtile_rows(int N, int64_t ldx_bytes, bool vec_ok) { return ldx_bytes > (int64_t(1) << 25) ? 2 : !vec_ok || N % 8 != 0 ? 1 : 0; }
// Shapes built for them; 128 x 256 for a 16-bit Y and K up to 256, where a tile is short and it saves a round.
bool mtile_has(const ubp_packed *p, int rows, int shape, size_t ysz) {
    if (shape == 4) return rows == 0 && ysz == 2 && p->K <= kTileMaxK;
    return rows == 0 || (rows == 1 && shape != 2) || shape == 3;
}
// Tiles a plan may name, 0 for any size: kernel 5 in units of 32 rows x 32 pixels, 7 and 9 of 16 x 16.
bool mtile_named(int kernel, int sub_stripes, int col_tiles) {
    static const int kSeven[][2] = {{16, 16}, {8, 16}, {8, 8}, {16, 4}, {4, 8}, {4, 4}};
    auto in = [](int v, int a, int b, int c) { return v == 0 || v == a || v == b || v == c; };
    if (kernel == 5) return in(sub_stripes, 2, 4, 4) && in(col_tiles, 2, 4, 4);
    if (kernel == 9) return in(sub_stripes, 4, 8, 16) && in(col_tiles, 4, 8, 16);
    for (const int(&t)[2] : kSeven)
        if ((sub_stripes == 0 || sub_stripes == t[0]) && (col_tiles == 0 || col_tiles == t[1])) return true;
    return false;
}

// Whether a gather layout exists: not for a stripe whose columns lie too far apart for the ring, nor beyond 2 GB.
bool gather_usable(const ubp_packed *p, int CT) {
    for (int G = gather_stripes(p); G >= 1; G >>= 1)
        if (get_stripe_layout(p, G, CT).G != 0) return true;
    return false;
}

// The kernel for a 16-bit product by the smallest estimate among those whose weights suit it: dense tiles
// only where blocks reach into at least half of the 16 x 32 tiles (W would grow and most products be by
// zeros otherwise), whole blocks as operands only where a block fills an operand and K is beyond what the
// ring holds at once.  aligned: 16-byte pieces of rows of X and Y lie inside or outside the matrix.
void choose(const ubp_packed *p, int N, int64_t ldx_bytes, bool vec_ok, size_t ysz, Shape &s) {
    const MaskStats &S = get_mask_stats(p);
    const bool aligned = vec_ok && N % 8 == 0;
    const bool mostly = 2 * S.tiles_hit >= S.tiles;
    double best = kNever;
    s.kernel = 2;
    if (direct_able(p, N, ldx_bytes)) {
        int waves = 0;
        best = estimate_direct(p, N, direct_tiles(N), ysz, waves);
        s.kernel = 8;
        s.waves = waves;
    }
    if (mostly && mtile_able(p, N)) {
        const int rows = mtile_rows(N, ldx_bytes, vec_ok);
        for (int sh = 0; sh < kNumMtileShapes; ++sh) {
            if (!mtile_has(p, rows, sh, ysz)) continue;
            const double t = estimate_mtile(p, N, sh, rows != 0, ysz);
            if (t < best) {
                best = t;
                // (7 is for matrices whose every tile holds a weight that is not zero: blocks that reach into every
                // tile do not make one)
                s.kernel = !aligned ? 9 : (p->K <= kTileMaxK || N <= 4096) && all_tiles_kept(p) ? 7 : p->K > kTileMaxK ? 5 : 9;
                s.shape = sh;
            }
        }
    }
    if (mostly && aligned && p->K <= kTileMaxK && tile_layout_words(p) > 0 && estimate_xstat(p, N, ysz) < best) {
        best = estimate_xstat(p, N, ysz);
        s = Shape();
        s.kernel = 4;
    }
    if (blk_eligible(p) && p->bh == kStripe && p->bw >= 16 && p->K > ring_rows(4) && vec_ok && N >= 64) {
        // (A margin in the range of its mean error against the dense tiles, whose estimate is the finer one: it decides 16 of 1998 drawn
        // layers, which by the dense tiles take 0.89 to 1.10 of this kernel's time, 1.02 on average.  None against the direct kernel, whose estimate
        // knows nothing of stripes that hold more than the others: it would decide 31 of 3000 layers, which the direct kernel takes 1.05 of this
        // one's time for on average, 0.91 to 1.20; 1024 x 2864 at 5 %, skewed, with 6144 pixels takes 42.3 us there and 21.5 here.)
        const BlkSplit *split = nullptr;
        const double t = estimate_blk(p, N, ysz, split);
        if ((s.kernel == 8 ? t : 1.06 * t) < best) {
            best = 1.06 * t;
            s = Shape();
            s.kernel = 6;
        }
    }
    // (a margin of twice this estimate's mean error, since it is the coarsest: of the 56 layers that it gives to kernel 2
    // one took more than 5 % longer than before, most half to three quarters of the time - 2928 x 1744 in 8 x 1 blocks
    // with 13120 pixels 429 -> 183 us, 3336 x 2288 in 4 x 4 with 2048 133 -> 59)
    if (best != kNever && aligned && ldx_bytes <= (int64_t(1) << 25) && 1.2 * estimate_gather(p, N, ysz) < best &&
        gather_usable(p, gather_col_tiles(N))) {
        s = Shape();
        s.kernel = 2;
    }
}

int kernel_by_matrix(const ubp_packed *p, int N, int64_t ldx_bytes, bool vec_ok) {
    if (blk_eligible(p) && p->bh == kStripe && p->bw >= 16 && p->K > ring_rows(4) && vec_ok && N >= 64) return 6;
    if (!vec_ok || N % 8 != 0 || tile_layout_words(p) == 0) return 2;
    if (all_tiles_kept(p) && (p->K <= kTileMaxK || N <= 4096) && (int64_t)p->K * ldx_bytes < (int64_t(1) << 31)) return 7;
    const TileLayout &T = get_tile_layout(p);
    if (2 * T.tiles_nonzero < (int64_t)T.nstripes * ((p->K + kStep - 1) / kStep)) return 2;
    return p->K <= kTileMaxK ? 4 : 5;
}

// ------------------------------------------------------------------ fp32 matrix kernel
// Where blocks are few the vector kernel, which reads the rows of X that they need and no others, is the faster one:
// 512 x 512 in 4 x 1 blocks with 6272 pixels at 0.26, 0.64, 1.3 and 2.6 columns per start row 8.6, 10.6, 12.9 and 14.5 us
// against 10.6, 10.5, 11.4 and 11.1; lower blocks fill less of a matrix instruction: 128 x 128 in 1 x 1 blocks with 12544 pixels at
// 2.6, 6.4 and 26 columns 6.1, 7.6 and 12.4 us against 6.8, 7.6 and 10.9, 700 x 700 in 2 x 1 blocks with 5 pixels at 3.5 and 7 columns 6.1 and 7.6
// against 6.7 and 5.6.
// (Rows of X at most 64 MB apart: 32-bit byte offsets within 8 of them.)
bool wros4_able(const ubp_packed *p, int64_t ldx_bytes) {
    return p->dtype == UBP_F32 && p->bh <= 16 && p->K <= wros4_max_K(32) && p->nb * p->bw >= (p->bh > 2 ? 2 : 6) * (int64_t)p->M &&
           ldx_bytes <= (int64_t(1) << 26) && get_wros4_layout(p).usable;
}

// What it would take, in microseconds: per round of workgroups (an XCD's on its 32 CUs, as many to a CU as LDS and
// wavefronts allow) the staging of X and a wavefront's groups and rows, each of them either a chain of latencies or the
// SIMD's share.  Coefficients fitted to 190 layers of the range the benchmark draws from, each timed in 20 to 40 shapes:
// mean error 7 %, and the shape of the smallest estimate took 1.7 % longer than the fastest on average, 21 % at most.
double estimate_wros4(const ubp_packed *p, int N, int px, int waves, int rpr) {
    const Wros4Layout &L = get_wros4_layout(p);
    const double M = p->M, per_row = (double)L.n_records * (4 / wros4_quads(p->bh)) / M; // groups
    const int lds = (((p->K + 7) & ~7) + 1) * 4 * px;
    const int64_t wgs = ((int64_t)N + px - 1) / px * (((int64_t)p->M + (int64_t)rpr * waves - 1) / ((int64_t)rpr * waves));
    const double a_cu = (double)(((wgs + 7) / 8 + 31) / 32), held = std::min({160 * 1024 / lds, 32 / waves, 16});
    const double rounds = std::ceil(a_cu / held), together = std::min(a_cu, held), simd = std::max(1.0, together * waves / 4);
    const double rows = std::min((double)rpr, M) + std::min<double>(p->bh - 1, std::max(0.0, M - rpr));
    const int quads = (p->bh + 3) / 4;
    return 3.55 + rounds * (together * lds * 1.176e-5 + 0.0197 * lds / 1024 / waves * (N % 4 == 0 ? 1 : 4) +
                            rows * per_row * std::max(0.0232 + 0.0218 * quads, simd * (0.0035 + 0.016 * quads)) +
                            rows * std::max(0.0311, simd * 0.0472)) +
           0.504 * 0.8e-6 * M * N;
}

// Pixels and wavefronts of a workgroup and, unless it is pinned, rows of a wavefront by the smallest estimate; px = 0: none.
void wros4_shape(const ubp_packed *p, int N, int rpr, Shape &s) {
    double best = kNever;
    for (int px : {64, 32}) {
        if (p->K > wros4_max_K(px)) continue;
        for (int r : {rpr, p->bh, 2 * p->bh, 4 * p->bh, 16, 32, 64}) {
            if (rpr != 0 ? r != rpr : r < p->bh) continue;
            for (int waves : {4, 8, 16}) {
                const int w = (int)std::min<int64_t>(waves, ((int64_t)p->M + r - 1) / r);
                const int64_t slices = ((int64_t)p->M + (int64_t)r * w - 1) / ((int64_t)r * w);
                // (a launch has fewer than 2^32 threads: workgroups, which come in eights, times up to 1024)
                if ((((int64_t)N + px - 1) / px * slices + 7) / 8 * 8 >= (int64_t(1) << 22)) continue;
                const double t = estimate_wros4(p, N, px, w, r);
                if (t < best) {
                    best = t;
                    s.px = px;
                    s.px_waves = w;
                    s.rpr = r;
                }
            }
        }
    }
}

ubp_status decide(const ubp_packed *p, int N, int64_t ldx_bytes, bool vec_ok, size_t ysz, const ubp_plan &pl, Shape &s) {
    int kernel = pl.kernel;
    // the dense-tile kernels 4, 5 and 7 need 16-byte pieces of X rows that lie entirely inside or outside the matrix
    const bool tile_able = p->dtype != UBP_F32 && vec_ok && N % 8 == 0;
    if (kernel < 0 || kernel > 9) return UBP_ERR_INVALID_ARG;
    if (kernel > 1 && kernel != 3 && p->dtype == UBP_F32) return UBP_ERR_UNSUPPORTED;
    if (kernel == 0 && p->dtype == UBP_F32) kernel = 1;
    if (kernel == 0) {
        choose(p, N, ldx_bytes, vec_ok, ysz, s);
        if (pl.sub_stripes || pl.col_tiles || pl.waves || pl.rows_per_range || pl.producers || pl.wg_rows) {
            // Part of a shape is fixed: the automatic choice's kernel where it takes these fields, else the one
            // that goes by the matrix alone, whose fields do not come and go with the number of pixels.
            ubp_plan named = pl;
            ubp_status rc = UBP_ERR_UNSUPPORTED;
            for (int k : {s.kernel, kernel_by_matrix(p, N, ldx_bytes, vec_ok)}) {
                named.kernel = k;
                s = Shape();
                rc = decide(p, N, ldx_bytes, vec_ok, ysz, named, s);
                if (rc == UBP_OK) break;
            }
            return rc;
        }
        kernel = s.kernel;
    }
    s.kernel = kernel;
    if (kernel == 1 || kernel == 3) {
        if (p->bh > 16) return UBP_ERR_UNSUPPORTED;
        int rpr = pl.rows_per_range;
        if (kernel == 1 && rpr >= 0 && wros4_able(p, ldx_bytes)) {
            wros4_shape(p, N, rpr, s);
            if (s.px != 0) return UBP_OK;
        }
        if (rpr == 0) {
            // Row ranges of one block height (re-walking bh - 1 rows nearly doubles the work, but a small
            // layer is a chain of latencies: 64 x 64 with 196 pixels 10.1 us, against 22.5 with ranges of
            // four) up to 8192 wavefronts of 64 columns, taller beyond (512 x 512 with 25088 pixels
            // 153 us, 158 with ranges of at least four block heights, 180 and more with half the wavefronts).
            const int64_t ranges = std::max<int64_t>(1, 8192 / (((int64_t)N + 63) / 64));
            const int64_t rows = std::max<int64_t>(p->bh, (p->M + ranges - 1) / ranges);
            rpr = (int)std::min<int64_t>((rows + p->bh - 1) / p->bh * p->bh, 0x7fffffff);
        }
        if (rpr < 1) return UBP_ERR_INVALID_ARG;
        if ((p->M + rpr - 1) / rpr > 65535) rpr = (p->M + 65534) / 65535; // grid.y limit
        s.rpr = rpr;
        return UBP_OK;
    }
    if (kernel == 8) {
        if (!direct_able(p, N, ldx_bytes)) return UBP_ERR_UNSUPPORTED;
        s.CT = pl.col_tiles ? pl.col_tiles : direct_tiles(N);
        if ((s.CT != 1 && s.CT != 2 && s.CT != 4) || N < s.CT) return UBP_ERR_UNSUPPORTED;
        s.waves = pl.waves;
        estimate_direct(p, N, s.CT, ysz, s.waves);
        if (s.waves < 1 || s.waves > 16 || !direct_fits(p, N, s.CT, s.waves)) return UBP_ERR_UNSUPPORTED;
        const DirectLayout &L = get_direct_layout(p);
        s.wg_rows = L.nstripes;
        return UBP_OK;
    }
    if (kernel == 5 || kernel == 7 || kernel == 9) {
        if (kernel != 9 && !tile_able) return UBP_ERR_UNSUPPORTED;
        const TileLayout &T = get_tile_layout(p);
        if (T.kt_pad == 0) return UBP_ERR_UNSUPPORTED;
        if (!mtile_named(kernel, pl.sub_stripes, pl.col_tiles)) return UBP_ERR_UNSUPPORTED;
        if (kernel == 5 && (T.kt_pad % 4 != 0 || pl.waves != 0)) return UBP_ERR_UNSUPPORTED;
        if (kernel == 5 && pl.wg_rows < 0) return UBP_ERR_INVALID_ARG;
        // kernel 7 multiplies every tile: only for matrices whose every tile keeps a weight
        if (kernel == 7 && !all_tiles_kept(p)) return UBP_ERR_UNSUPPORTED;
        if (!mtile_able(p, N)) return UBP_ERR_UNSUPPORTED;
        // Of the shapes no larger than what the plan names (kernel 5: in units of 32 rows and 32 pixels,
        // else of 16; all of them where it names nothing) the one with the smallest estimate.  Kernels 5 and 7,
        // which are for aligned rows and have all shapes there, serve rows more than 32 MB apart with the one that is left.
        const int unit = kernel == 5 ? 32 : 16;
        const bool pinned = kernel == 9 || mtile_rows(N, ldx_bytes, vec_ok) == 0;
        s.rows = mtile_rows(N, ldx_bytes, vec_ok);
        const bool wide = kernel != 5 && pl.sub_stripes != 4 && mtile_has(p, s.rows, 4, ysz);
        double best = kNever;
        for (int sh = 0; sh < kNumMtileShapes; ++sh) {
            if (!mtile_has(p, s.rows, sh, ysz) || (sh == 4 && kernel == 5)) continue; // (no name for that one in units of 32)
            const int want_r = pinned ? pl.sub_stripes * unit : 0, want_p = pinned ? pl.col_tiles * unit : 0;
            if (want_r != 0 && kMtileShapes[sh].rows != std::min(want_r, 128)) continue;
            if (want_p != 0 && kMtileShapes[sh].pixels != std::min(want_p, wide ? 256 : 128)) continue;
            const double t = estimate_mtile(p, N, sh, s.rows != 0, ysz);
            if (t < best) {
                best = t;
                s.shape = sh;
            }
        }
        if (best == kNever) return UBP_ERR_UNSUPPORTED;
        const MtileShape &sh = kMtileShapes[s.shape];
        s.G = sh.rows / unit;
        s.CT = sh.pixels / unit;
        s.waves = 0; // (fixed)
        s.wg_rows = (p->M + sh.rows - 1) / sh.rows;
        return UBP_OK;
    }
    if (kernel == 4) {
        if (!tile_able || p->K > kTileMaxK) return UBP_ERR_UNSUPPORTED;
        const TileLayout &T = get_tile_layout(p);
        if (T.kt_pad == 0) return UBP_ERR_UNSUPPORTED;
        int CT = pl.col_tiles;
        if (CT == 0) CT = xstat_col_tiles(N);
        if (CT != 2 && CT != 4) return UBP_ERR_UNSUPPORTED;
        s.CT = CT;
        const int n_blocks = (N + 16 * CT - 1) / (16 * CT);
        int slices = pl.wg_rows;
        if (slices < 0) return UBP_ERR_INVALID_ARG;
        if (slices == 0) slices = xstat_slices(T.nstripes, n_blocks);
        slices = std::min(slices, T.nstripes);
        const int sps = (T.nstripes + slices - 1) / slices;
        slices = (T.nstripes + sps - 1) / sps;
        if ((int64_t)n_blocks * slices > 0x7fffffff) return UBP_ERR_UNSUPPORTED;
        s.wg_rows = slices;
        s.waves = pl.waves ? pl.waves : std::min(4, sps);
        if (s.waves < 1 || s.waves > 8) return UBP_ERR_UNSUPPORTED;
        return UBP_OK;
    }
    if (kernel == 6) {
        if (!blk_eligible(p) || !vec_ok || N < 64) return UBP_ERR_UNSUPPORTED;
        if (pl.col_tiles != 0 && pl.col_tiles != 4) return UBP_ERR_UNSUPPORTED;
        int G = pl.sub_stripes ? pl.sub_stripes : blk_auto_G(p), NP = pl.producers;
        if (G != 2 && G != 4 && G != 5) return UBP_ERR_UNSUPPORTED;
        if (pl.sub_stripes == 0 && pl.producers == 0 && pl.waves == 0 && pl.wg_rows == 0) { // (the rest of a plan goes with what it pins)
            const BlkSplit *split = nullptr;
            estimate_blk(p, N, ysz, split);
            G = split->G;
            NP = split->NP;
        }
        const BlkLayout &L = get_blk_layout(p, G);
        if (L.G == 0) return UBP_ERR_UNSUPPORTED;
        if (NP != 0 && NP != 1 && NP != 2 && NP != 4) return UBP_ERR_UNSUPPORTED;
        int waves = pl.waves;
        // one wavefront stages about 28 GB/s: a second one as soon as a workgroup's tile is not small
        if (NP == 0) {
            NP = ((int64_t)p->K * 32 * 4 >= 64 * 1024) ? 2 : 1;
            if (waves != 0 && waves < NP + 1) NP = 1;
        }
        const int max_waves = blk_max_waves(G);
        if (waves == 0) {
            // as few workgroup rows as the wavefront limit allows; full workgroups if the last row is
            // then still at least half full, else the consumers spread evenly over the rows
            const int maxc = max_waves - NP;
            const int rows_wg = (L.nrg + maxc - 1) / maxc;
            const int last = L.nrg - (rows_wg - 1) * maxc;
            waves = (2 * last >= maxc ? maxc : (L.nrg + rows_wg - 1) / rows_wg) + NP;
        }
        if (waves < NP + 1 || waves > max_waves) return UBP_ERR_UNSUPPORTED;
        const int need_rows = (L.nrg + (waves - NP) - 1) / (waves - NP);
        if (pl.wg_rows != 0 && pl.wg_rows != need_rows) return UBP_ERR_UNSUPPORTED;
        s.G = G;
        s.CT = 4;
        s.NP = NP;
        s.waves = waves;
        s.wg_rows = need_rows;
        return UBP_OK;
    }

    // ---- gather kernel
    int CT = pl.col_tiles, G = pl.sub_stripes;
    if (pl.producers != 0 && pl.producers != 1 && pl.producers != 2 && pl.producers != 4) return UBP_ERR_UNSUPPORTED;
    if ((G != 0 && G != 1 && G != 2 && G != 4) || (CT != 0 && CT != 2 && CT != 4 && CT != 8)) return UBP_ERR_UNSUPPORTED;
    if (CT == 0) CT = gather_col_tiles(N);
    if (G == 0) {
        G = gather_stripes(p);
        while (G > 1 && get_stripe_layout(p, G, CT).G == 0) G >>= 1;
    }
    const StripeLayout &L = get_stripe_layout(p, G, CT);
    if (L.G == 0) return UBP_ERR_UNSUPPORTED; // layout cannot be built for this matrix
    return gather_launch(p, N, G, CT, pl, s);
}

} // namespace

// Decides kernel and shape for (handle, N, alignment) and the caller's pins; builds the host image
// of the layout that shape needs (under the handle's lock).  No device work; a layout that does not
// fit the host's memory is an error, not an exception that would pass the C boundary.
ubp_status resolve(const ubp_packed *p, int N, int64_t ldx_bytes, bool vec_ok, size_t ysz, const ubp_plan &pl, Shape &s) {
    try {
        return decide(p, N, ldx_bytes, vec_ok, ysz, pl, s);
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    } catch (const std::length_error &) {
        return UBP_ERR_ALLOC;
    }
}

} // namespace ubp
