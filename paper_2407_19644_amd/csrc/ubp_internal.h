// Internal definitions shared by the host-side packer, the layout builders and the HIP
// launch code of the UBP library.
#pragma once

#include <cstdint>
#include <mutex>
#include <vector>

#include "ubp.h"

namespace ubp {

constexpr int kStripe = 16;    // rows of one MFMA output tile (aligned row stripe)
constexpr int kStep = 32;      // gathered X rows consumed by one 16x16x32 MFMA
constexpr int kSlotRows = 64;  // X rows per slot of the LDS ring (the unit the producer stages)
constexpr int kPrefetchDepth = 4; // step records a wavefront keeps in flight; row groups hold a multiple of it
constexpr int kNumG = 3;       // stripes per wavefront: 1, 2, 4
constexpr int kNumCT = 3;      // 16-column tiles per wavefront: 2, 4, 8
constexpr int kNumLayouts = kNumG * kNumCT;

// A gather layout exists per (G, CT) the gather kernel is instantiated for; CT fixes the byte
// addresses inside the LDS ring that the records carry.
inline int layout_slot(int G, int CT) {
    const int gi = G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : -1;
    const int ci = CT == 2 ? 0 : CT == 4 ? 1 : CT == 8 ? 2 : -1;
    return (gi < 0 || ci < 0) ? -1 : gi * kNumCT + ci;
}
inline int slot_G(int slot) { return 1 << (slot / kNumCT); }
inline int slot_CT(int slot) { return 2 << (slot % kNumCT); }

// LDS ring geometry for a column-tile width: rows of 32*CT bytes, 128 KB in all, always a
// power-of-two number of rows so that ring row = X row mod rows.
constexpr int ring_pitch(int CT) { return 32 * CT; }
constexpr int ring_rows(int CT) { return 131072 / ring_pitch(CT); }
constexpr int ring_slots(int CT) { return ring_rows(CT) / kSlotRows; }
// Entries are grouped by stripe set inside windows of this many X rows (a quarter of the ring:
// a step may straddle two windows, and the rest of the ring is left to the drift between
// wavefronts and to the chunks the producer has in flight).
constexpr int ring_window(int CT) { return ring_rows(CT) / 4; }

// Position of the 32-byte unit u (16 pixels) inside ring row r is u ^ ring_swizzle(r): LDS
// has 64 four-byte banks, and this spreads 16 consecutive rows of one unit over all of them.
constexpr int ring_swizzle(int CT, int r) { return CT == 2 ? ((r >> 2) & 1) : CT == 4 ? ((r >> 1) & 3) : (r & 7); }

// Gather kernel: the gather of step s+1 is issued before the MFMAs of step s (two operand buffers) except
// for the largest tile, where the second buffer would halve the wavefronts per SIMD.
constexpr bool stripe_pipelined(int G, int CT) { return G * CT < 32; }

// Threads of a workgroup of that kernel.
constexpr int stripe_max_threads(int G, int CT) {
    // accumulators + operand buffer(s) + prefetched step records + addressing, in VGPRs
    // per lane; 512 per SIMD lane are shared by the wavefronts resident on the SIMD
    const int regs = 4 * G * CT + (stripe_pipelined(G, CT) ? 8 : 4) * CT + kPrefetchDepth * (2 + 4 * G) + (G == 1 ? 8 : 20);
    return regs <= 128 ? 1024 : regs <= 256 ? 512 : 256;
}
constexpr int stripe_max_waves(int G, int CT) { return stripe_max_threads(G, CT) / 64; }
// Wavefronts of a workgroup of the block kernel.
constexpr int kBlkConsumers = 14; // of them multiplying, at most
// Whether the last N % 64 pixels go to the gather kernel.  Not where N is a multiple of 8: the last tile then overlaps the one
// before it, its pieces of rows still aligned, for at most a tile's work (16 x 16 blocks, wavefronts of 5 stripes and 2 producers: 4096 x 4096 at 10 %
// with 1000 pixels 196.7 -> 35.1 us, 2048 x 4096 at 5 % with 4040 191 -> 30.1; with the splits that are chosen there now 26.1 and 27.5, by the
// direct kernel 43.1 and 42.4).
constexpr bool blk_leaves_tail(int N) { return N % 8 != 0; }
constexpr int blk_max_waves(int G) { return (G == 2 || G == 4 || G == 5) ? 16 : 0; }

// Host image of the gather kernel's private re-layout of the packed weights, for one (G, CT).
//
// Rows are cut into row groups of 16*G aligned rows.  For a row group the columns of W
// that hold at least one kept weight in it are its "entries"; an entry is one row of X
// to gather plus the 16*G weights of that column (zero where no block covers the row).
// Entries are ordered by window of ring_window(CT) X rows, inside a window by the set of stripes
// they touch and then by column, and grouped 32 at a time into "steps" whose rows fit the
// LDS ring together.
struct StripeLayout {
    int G = 0, CT = 0; // G == 0: not usable for this matrix
    bool built = false;
    int nrg = 0;     // row groups
    int nch = 0;     // slots (chunks of kSlotRows X rows) the producer stages: ceil(K / 64)
    std::vector<int32_t> rg_ptr;     // [nrg + 1] first step of each row group (step counts are multiples of kPrefetchDepth)
    std::vector<int32_t> rg_order;   // row groups, heaviest (most MFMAs) first
    // One fixed-size record per step, (128 + 256*G) dwords, so that the address of any later
    // step is known without reading metadata:
    //   dwords 0..127 : per lane a pair {addr, ctl}
    //       addr bits 0-13 / 14-27 : LDS byte address >> 3 of the lane's two transposed reads
    //                                (ring row, swizzle and the lane's 8-byte column included;
    //                                column tile c is then reached by XOR with c << 5)
    //       addr bits 28-31        : stripes with nonzero weights in this step
    //       ctl (same in all lanes): bits 0-15 highest chunk the step reads, bits 16-31 number
    //                                of leading chunks that no step from here on reads
    //   then G x 256 dwords: weight fragment of stripe j in MFMA operand order (lane-major,
    //                        8 16-bit values per lane), all zero when the step has no weight there
    // A row group's last steps may be empty (no stripes, nothing read): they pad its step count
    // to a multiple of kPrefetchDepth so that the kernel's unrolled loop has a single exit.
    std::vector<uint32_t> stream;
    int64_t nsteps = 0;
    int64_t total_mfma = 0; // MFMA issues per 16-column tile (steps x stripes with weights)
};

// Host image of the block kernel's layout (blocks of at most 16 rows; column tiles of 64 pixels,
// i.e. the ring geometry of CT = 4), for G stripes per wavefront.
//
// Row groups are consecutive runs of at most G aligned 16-row stripes, cut so that runs with many
// blocks are short (a workgroup lasts as long as its heaviest row group).
// A block is cut into "halves" of 16 consecutive columns (a block at most 16 wide is one half).
// For a row group every half of every block that has a row in the group is an incidence.  The X rows of a half are the window [a, a + 16), a = its first column
// (moved left where the window would pass the last row of X).  A step = two halves (A, B) whose
// blocks start in the same stripe of the row group, or one half and nothing.
//   meta : 2 dwords per step
//       m0 : a_A | a_B << 16
//       m1 : bits 0-3 / 4-7  row offset o = (block's first row) mod 16 of half A / B
//            bits 8-11       jj = 1 + index of the stripe (of the row group) the blocks start in,
//                            0 when they start in the stripe above the group, 15 for an empty step
//            bit 12 / 13     some half has rows in stripe jj - 1 ("lower part", rows n >= o) /
//                            in stripe jj ("upper part", rows n < o)
//            bits 22-31      number of leading 64-row chunks of X that no later step reads
//                            (handed back as soon as this step's reads are issued)
//   frags: 256 dwords per step, the MFMA operand of both halves: lane 16 g + n holds, as 16-bit
//          element e (0..3: half A, 4..7: half B), the weight that row-slot n of the block
//          (the block row congruent to n modulo 16: the paper's rotation, Section 4.2, with
//          period 16) has in window row a + ((4 g + e - a) mod 16) - columns are rotated the same
//          way, so that the LDS row a lane reads is congruent to its entry number modulo 16.
// Steps of a row group are contiguous, ordered by the first window row, padded with empty steps
// to a multiple of kPrefetchDepth; kPrefetchDepth spare records end both arrays.
struct BlkLayout {
    int G = 0;
    bool built = false;
    int nrg = 0, nch = 0;
    std::vector<int32_t> rg_ptr;    // [nrg + 1] first step of each row group
    std::vector<int32_t> rg_order;  // [nrg] row groups, heaviest first, then [nrg + 1] the first stripe of each row group
    std::vector<int32_t> rg_first;  // the second part of rg_order while the layout is built
    std::vector<uint32_t> meta, frags;
    int64_t nsteps = 0;
    int64_t total_mfma = 0;   // MFMA issues per 16-column tile
    int64_t halves = 0, paired = 0; // incidences, and how many of them share a step with another
};

// Host image of the dense-tile kernels' layout: W as 16-row x 32-column operand tiles in MFMA
// operand order, zeros where nothing is kept, for every (stripe, 32-column tile) pair.
// kt_pad = 32-column tiles per stripe: for K <= kTileMaxK rounded up to 2, 4, 6 or 8 (such a
// stripe's tiles and a pixel block's X fit a wavefront's registers at once); for larger K
// rounded up to a multiple of 8 (chunks of 256 rows), built only while the zero-filled matrix
// stays below kTileMaxBytes.  occupied holds one bit per tile (bit kt % 32 of word
// stripe * ceil(kt_pad / 32) + kt / 32): the tile has a kept weight.
constexpr int kTileMaxK = 256;
constexpr int64_t kTileMaxBytes = 8 << 20;
// Tiles per stripe of the dense tiles; 0 where they are not built (larger than kTileMaxBytes).
inline int tile_kt_pad(int M, int K) {
    const int kt = (K + kStep - 1) / kStep;
    const int kt_pad = K <= kTileMaxK ? (kt < 2 ? 2 : (kt + 1) / 2 * 2) : (kt + 7) / 8 * 8;
    return (int64_t)((M + kStripe - 1) / kStripe) * kt_pad * 1024 <= kTileMaxBytes ? kt_pad : 0;
}
struct TileLayout {
    bool built = false;
    int kt_pad = 0;                  // 0: not usable for this matrix
    int nstripes = 0;
    std::vector<uint16_t> frags;     // [nstripes][kt_pad][64 lanes][8]
    std::vector<uint32_t> occupied;
    int64_t tiles_nonzero = 0;
};

// Columns of blocks whose rows of X the vector kernel loads together, at most.
constexpr int kWrosBatch = 8;

// Where blocks lie, counted once per handle (16-bit handles): what the estimates of the kernels need.
struct MaskStats {
    bool built = false;
    int64_t steps = 0;      // steps of the direct layout: sum over stripes of ceil(columns with a kept weight / 32)
    int64_t gather_steps = 0; // the same over row groups of gather_stripes(p) stripes, each a multiple of kPrefetchDepth
    int64_t tiles_hit = 0;  // 16 x 32 tiles a block reaches into
    int64_t tiles = 0;      // all of them
};

// Host image of the direct kernel's layout: for every aligned 16-row stripe the columns of W in which
// it keeps a weight, ascending, 32 to a step.
//   first : [nstripes + 1] first step of each stripe
//   order : [nstripes] stripes, most steps first
//   ids   : 32 16-bit row numbers of X per step; entry 8 g + e is element e of lane group g.  A
//           stripe's last step repeats its first row number (with zero weights) to fill up.
//   frags : 512 16-bit weights per step in MFMA operand order: lane 16 g + n holds, as element e, the
//           weight of row n of the stripe in column ids[8 g + e]
struct DirectLayout {
    bool built = false;
    int nstripes = 0;                // 0: not usable for this matrix
    std::vector<int32_t> first, order;
    std::vector<uint16_t> ids, frags;
    int64_t nsteps = 0;
};

// Accumulator quads per block column of the fp32 matrix kernel, as a power of two (it has 4 slots each).
constexpr int wros4_quads(int bh) { return bh <= 4 ? 1 : bh <= 8 ? 2 : 4; }
// Records in flight per wavefront, and records to a round of its loop: it loads, and walks for nothing, up to 2 x kWros4Depth - 1
// records behind the last one.
constexpr int kWros4Depth = 4;
constexpr int kWros4Spare = 2 * kWros4Depth - 1;
// Rows of X that its LDS holds at PX pixels: all of K rounded up to 8, and a row of zeros, of 4 PX bytes each.
constexpr int wros4_max_K(int PX) { return (160 * 1024 / (4 * PX) - 1) / 8 * 8; }

// Host image of the fp32 matrix kernel's layout: the blocks' columns in canonical order (start rows, then column
// origins, then columns), 4 of one start row to a group (filled up with weights -0), 4 / wros4_quads(bh) groups to a record.
//   weights : 64 floats per record: per column 4 wros4_quads(bh) slots, the block's weights from its first row on, then -0
//   offsets : 32 words per record, a cache line.  Word c < 16 / wros4_quads(bh): 256 x the row of X of column c, or
//             256 x (K rounded up to 8), where the kernel keeps zeros, for a column that fills up.  Word 16, byte g: output rows that
//             are complete after group g.  (Where more than 255 rows end behind one group, groups without columns follow.)
//             The other words are not used.
//   (Both end with kWros4Spare records that hold nothing: weights -0, the row of zeros, no row complete.)
//   rec_of_row : [M] the record with the first group of this or a later start row
//   rec_of_end : [M] the record with the group behind which the output row is complete, -1 before the first group
//   row_of_rec : [n_records + 1] the output row that is next to be complete when the record begins, M at the end
struct Wros4Layout {
    bool built = false;
    int n_records = 0;       // without the spare ones (0 also where nothing is kept)
    bool usable = false;     // (the weights take less than 2 GB)
    std::vector<float> weights;
    std::vector<uint32_t> offsets;
    std::vector<int32_t> rec_of_row, rec_of_end, row_of_rec;
};

struct StripeLayoutDev {
    int32_t *rg_ptr = nullptr;
    int32_t *rg_order = nullptr;
    uint32_t *stream = nullptr;
    bool uploaded = false;
};
struct BlkLayoutDev {
    int32_t *rg_ptr = nullptr;
    int32_t *rg_order = nullptr;
    uint32_t *meta = nullptr;
    uint32_t *frags = nullptr;
    bool uploaded = false;
};
struct DirectLayoutDev {
    int32_t *first = nullptr;
    int32_t *order = nullptr;
    uint16_t *ids = nullptr;
    uint16_t *frags = nullptr;
    bool uploaded = false;
};
struct Wros4LayoutDev {
    float *weights = nullptr; // (the allocation; the others lie behind them)
    const uint32_t *offsets = nullptr;
    const int32_t *rec_of_row = nullptr, *rec_of_end = nullptr, *row_of_rec = nullptr;
};
struct TileLayoutDev {
    uint16_t *frags = nullptr;
    uint32_t *occupied = nullptr;
    bool uploaded = false;
};

// ------------------------------------------------------------------ kernel arguments
// What happens to an output value between the accumulator and the store: Y = act(acc + bias[row]),
// in fp32, before the one rounding to Y's type.  on == 0: nothing.  The activation is a clamp to
// [lo, hi] (ReLU: lo = 0, hi = +inf), taken with maxNum / minNum, so that a NaN becomes lo.
struct Epilogue {
    const float *bias; // device, M floats, or null
    int on;
    float lo, hi;
};

struct StripeArgs {
    const int32_t *rg_ptr;
    const int32_t *rg_order;
    const uint32_t *stream;
    uint32_t stream_bytes;   // size of the record stream (buffer-addressed: below 4 GB)
    const uint16_t *X;
    void *Y;
    int64_t ldx, ldy;
    int M, K, N, bh;
    int nrg, nch;            // row groups, 64-row chunks of X
    int ring_bytes;          // bytes of the LDS ring actually used (all of K when K is shorter than the ring)
    int ctile0, n_coltiles;  // first column tile of this launch, number of tiles in it
    int n_wgrows;
    int n_producers;         // producer wavefronts per workgroup: 1, 2 or 4 (the last wavefronts)
    int resident;            // the ring holds all of K: slots are never refilled, a consumer may walk several row groups
    int vec_ok;              // X and Y allow 16-byte vector access on every row
    uint32_t *err;           // set to nonzero when a bounded wait runs out
    Epilogue ep;
};

struct BlkArgs {
    const int32_t *rg_ptr;
    const int32_t *rg_order;
    const uint32_t *meta;
    const uint32_t *frags;
    uint32_t meta_bytes, frag_bytes;
    const uint16_t *X;
    void *Y;
    int64_t ldx, ldy;
    int M, K, N;
    int nrg, nch;
    // of the LDS ring that are used, all of K where K is shorter than the ring: a CU then holds several workgroups (plans that
    // name this kernel: 4096 x 512 with 8192 pixels in workgroups of 8 wavefronts, one producer, 28.1 us, 37.0 with the whole ring)
    int ring_bytes;
    int n_coltiles;          // 64-pixel column tiles this launch covers (from pixel 0; the last one may overlap the one before)
    int n_wgrows;
    int n_producers;
    int out_bytes;           // LDS bytes per consumer for leaving 16-bit tiles as whole rows; 0: none
    uint32_t *err;
    Epilogue ep;
};

struct DirectArgs {
    const int32_t *first, *order;
    const uint16_t *ids, *frags;
    const uint16_t *X;
    void *Y;
    int64_t ldx, ldy;        // (ldx below 2^23, K rows of X below 4 GB: 32-bit byte offsets)
    int M, N, nstripes, n_tiles;
    Epilogue ep;
};

struct Wros4Args {
    const float *weights;
    const uint32_t *offsets;
    const int32_t *rec_of_row, *rec_of_end, *row_of_rec;
    uint32_t weight_bytes, offset_bytes; // (buffer-addressed: below 2 GB)
    const float *X;
    float *Y;
    int64_t ldx, ldy;        // (ldx at most 2^24: 32-bit byte offsets within 8 rows)
    int M, K, N;
    int n_tiles, slices;     // pixel tiles, workgroups that share one
    int rpr;                 // output rows per wavefront
    int vec4;                // rows of X consist of 16-byte pieces
    Epilogue ep;
};

struct TileArgs {
    const uint16_t *frags;   // [nstripes][KT][64][8]
    const uint32_t *occupied; // one bit per tile, ceil(kt_total / 32) words per stripe
    const uint16_t *X;
    void *Y;
    int64_t ldx, ldy;
    int M, K, N;
    int nstripes, sps;       // stripes in all, stripes per workgroup slice
    int n_blocks;            // pixel blocks
    int slices;              // slices the stripes are cut into
    int kt_total;            // 32-column tiles per stripe in frags
    int skip;                // some tile keeps no weight: run the instantiation that tests the occupancy bits
    uint32_t *err;           // the handle's error flags (bounded waits that ran out)
    Epilogue ep;
};

// What a call resolves to: the kernel and its launch shape, every field set.
struct Shape {
    int kernel = 0;   // 1 vector, 2 gather, 4 small-K dense tiles, 5 / 7 / 9 dense tiles through LDS, 6 block, 8 direct
    int shape = 0;    // kernels 5, 7, 9: index into kMtileShapes
    int G = 0, CT = 0, waves = 0, NP = 0, wg_rows = 0, rpr = 0;
    int px = 0;       // kernel 1: pixels of a workgroup of the fp32 matrix kernel; 0: the vector kernel
    int px_waves = 0; // its wavefronts
    bool resident = false;
    int rows = 0;        // kernels 5, 7, 9: the way rows of X take (mtile_rows)
};

// The last few calls without a plan that a handle chose a kernel for: the choice follows from the
// handle and these four alone, and working it out again costs a call bound by the host about 0.2 us (7.43 -> 7.23).
constexpr int kChoices = 4;
struct Choice {
    int32_t N = 0; // 0: unused (a product of no pixels chooses nothing)
    int64_t ldx = 0;
    bool vec_ok = false;
    size_t ysz = 0;
    Shape shape;
};

} // namespace ubp

struct ubp_packed {
    int32_t M = 0, K = 0, bh = 0, bw = 0;
    int64_t nb = 0;
    ubp_dtype dtype = UBP_F32;
    int32_t device = UBP_HOST_ONLY;
    // canonical arrays (Section 4.2 of the paper)
    std::vector<int32_t> indptr, indices;
    std::vector<uint8_t> values; // nb*bw*bh elements of dtype, rotated
    // Private layouts, built on first use (host image) and uploaded on first use on the device;
    // guarded by `lock` because a handle is passed around as a pointer to const.
    mutable std::mutex lock;
    mutable ubp::StripeLayout sg[ubp::kNumLayouts];
    mutable ubp::BlkLayout blk[3];           // G = 2, 4, 5
    mutable ubp::TileLayout tiles;
    mutable ubp::DirectLayout direct;
    mutable ubp::Wros4Layout wros4;
    mutable ubp::MaskStats stats;
    mutable ubp::Choice choices[ubp::kChoices];
    mutable int next_choice = 0;
    // device side
    int32_t *d_indptr = nullptr;
    int32_t *d_indices = nullptr;
    mutable float *d_values_f32 = nullptr; // rotated values widened to fp32 (exact), for the vector kernel
    mutable const int32_t *d_cols = nullptr; // (part of d_values_f32) row of X of every block column, in block order, and kWrosBatch zeros, for the vector kernel
    mutable ubp::StripeLayoutDev d_sg[ubp::kNumLayouts];
    mutable ubp::BlkLayoutDev d_blk[3];
    mutable ubp::TileLayoutDev d_tiles;
    mutable ubp::DirectLayoutDev d_direct;
    mutable ubp::Wros4LayoutDev d_wros4;
    uint32_t *d_error = nullptr;   // set by a kernel whose bounded wait ran out
    mutable int64_t device_bytes = 0;
};

namespace ubp {

inline int64_t dtype_size(ubp_dtype d) { return d == UBP_F32 ? 4 : 2; }
constexpr int kNumBlkLayouts = 3;
inline int blk_slot(int G) { return G == 2 ? 0 : G == 4 ? 1 : G == 5 ? 2 : -1; }

// ---- host: layout builders (ubp_layouts.cpp).  Each builds the host image once; the caller
// holds p->lock.  A layout that cannot be built for this matrix is left marked unusable.
const StripeLayout &get_stripe_layout(const ubp_packed *p, int G, int CT);
const BlkLayout &get_blk_layout(const ubp_packed *p, int G);
const TileLayout &get_tile_layout(const ubp_packed *p);
const DirectLayout &get_direct_layout(const ubp_packed *p);
const Wros4Layout &get_wros4_layout(const ubp_packed *p);
const MaskStats &get_mask_stats(const ubp_packed *p);
// Stripes per wavefront of the gather kernel.  They follow the block height: a 16-row block touches two stripes
// anyway, so tall row groups cost little extra zero fill and divide the staging of X by the rows a workgroup
// covers; for short blocks one stripe keeps the operands dense.
inline int gather_stripes(const ubp_packed *p) { return p->bh >= 16 ? 4 : p->bh >= 8 ? 2 : 1; }
bool blk_eligible(const ubp_packed *p);

// ---- host: choice of kernel and launch shape (ubp_choose.cpp).  Builds the host image of the layout the
// shape needs (the caller holds p->lock); no device work.  vec_ok: rows of X and Y start at multiples of 16
// bytes; ysz: bytes of an element of Y.
ubp_status resolve(const ubp_packed *p, int N, int64_t ldx_bytes, bool vec_ok, size_t ysz, const ubp_plan &pl, Shape &s);

// ---- device (HIP translation units)
ubp_status upload(ubp_packed *p);                 // canonical arrays, at pack time
void release_device(ubp_packed *p);
// upload of one private layout, on first use (caller holds p->lock); UBP_ERR_ALLOC on failure
ubp_status upload_stripe_layout(const ubp_packed *p, int slot);
ubp_status upload_blk_layout(const ubp_packed *p, int slot);
ubp_status upload_tile_layout(const ubp_packed *p);
ubp_status upload_direct_layout(const ubp_packed *p);
ubp_status upload_wros4_layout(const ubp_packed *p);

// Launchers.  `dry` only raises the kernels' dynamic LDS limit on the current device (what a
// first launch of a shape would do), so that a later launch is nothing but a launch.
ubp_status launch_wros(const ubp_packed *p, const void *X, int64_t ldx, int N, void *Y, int64_t ldy, ubp_dtype y_dtype,
                       int rpr, bool naive, const Epilogue &ep, void *stream, bool dry);
ubp_status launch_wros4(const Wros4Args &a, int bh, int PX, int waves, void *stream, bool dry);
ubp_status launch_stripe(const StripeArgs &a, bool bf16, bool y_f32, int G, int CT, int waves, void *stream, bool dry);
ubp_status launch_blk(const BlkArgs &a, bool bf16, bool y_f32, int G, int waves, void *stream, bool dry);
ubp_status launch_xstat(const TileArgs &a, bool bf16, bool y_f32, int CT, int KT, int waves, void *stream, bool dry);
ubp_status launch_direct(const DirectArgs &a, bool bf16, bool y_f32, int CT, int waves, void *stream, bool dry);
// shapes of kernel 5 / 7 / 9: rows x pixels of a workgroup's tile, workgroups a CU holds
struct MtileShape { int rows, pixels, per_cu; };
constexpr int kNumMtileShapes = 5;
constexpr MtileShape kMtileShapes[kNumMtileShapes] = {{128, 128, 1}, {128, 64, 1}, {64, 128, 1}, {64, 64, 2}, {128, 256, 1}};
ubp_status launch_mtile(const TileArgs &a, bool bf16, bool y_f32, int shape, int rows, void *stream, bool dry);
ubp_status launch_floor(void *stream);

} // namespace ubp
