// Device-facing entry points of the UBP library: upload of the packed weights and of the
// kernels' private layouts, launches, the C ABI around them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <stdexcept>
#include <vector>

#include "ubp_internal.h"

namespace ubp {

struct DeviceGuard {
    int prev = -1;
    bool ok = true, changed = false; // (setting the device that is set already costs a call bound by the host, too)
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) ok = false;
        else if (prev != dev) ok = changed = hipSetDevice(dev) == hipSuccess;
        if (!ok) (void)hipGetLastError(); // do not leave a sticky error for the caller's next HIP call
    }
    ~DeviceGuard() {
        if (changed) (void)hipSetDevice(prev);
    }
};

namespace {

template <class T>
bool dev_copy(T **dst, const T *src, size_t n, int64_t *bytes) {
    const size_t sz = std::max<size_t>(n, 1) * sizeof(T);
    if (hipMalloc(reinterpret_cast<void **>(dst), sz) != hipSuccess) { *dst = nullptr; return false; }
    *bytes += (int64_t)sz;
    if (n && hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) return false;
    return true;
}

template <class T>
bool dev_copy_vec(T **dst, const std::vector<T> &v, int64_t *bytes) { return dev_copy(dst, v.data(), v.size(), bytes); }

} // namespace

// ------------------------------------------------------------------ upload / release
ubp_status upload(ubp_packed *p) {
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || p->device >= count) {
        (void)hipGetLastError();
        p->device = UBP_HOST_ONLY; // nothing was allocated; nothing to release
        return UBP_ERR_DEVICE;
    }
    DeviceGuard guard(p->device);
    if (!guard.ok) {
        p->device = UBP_HOST_ONLY;
        return UBP_ERR_DEVICE;
    }
    bool ok = true;
    ok = ok && dev_copy(&p->d_indptr, p->indptr.data(), p->indptr.size(), &p->device_bytes);
    ok = ok && dev_copy(&p->d_indices, p->indices.data(), p->indices.size(), &p->device_bytes);
    {
        const uint32_t zero = 0;
        ok = ok && dev_copy(&p->d_error, &zero, 1, &p->device_bytes);
    }
    if (!ok) {
        (void)hipGetLastError();
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

// (the functions below run with p->lock held and the handle's device current)
ubp_status upload_values_f32(const ubp_packed *p) {
    if (p->d_values_f32) return UBP_OK;
    // rotated values widened to fp32 (exact for fp16 and bf16) for the vector kernel
    const int64_t n = p->nb * p->bw * p->bh;
    std::vector<float> f((size_t)n);
    if (p->dtype == UBP_F32) {
        if (n) std::memcpy(f.data(), p->values.data(), (size_t)n * 4);
    } else {
        const uint16_t *h = reinterpret_cast<const uint16_t *>(p->values.data());
        for (int64_t t = 0; t < n; ++t) {
            if (p->dtype == UBP_BF16) {
                const uint32_t u = (uint32_t)h[t] << 16;
                std::memcpy(&f[(size_t)t], &u, 4);
            } else {
                _Float16 hv;
                std::memcpy(&hv, &h[t], 2);
                f[(size_t)t] = (float)hv;
            }
        }
    }
    // behind them the rows of X of the blocks' columns, one after the other (what the kernel loads ahead
    // may reach kWrosBatch past the end); one allocation and one copy
    const size_t cols = (size_t)(p->nb * p->bw) + kWrosBatch;
    f.resize((size_t)n + cols);
    for (size_t t = 0; t < cols; ++t) {
        const int32_t row = t < cols - kWrosBatch ? p->indices[t / (size_t)p->bw] + (int32_t)(t % (size_t)p->bw) : 0;
        std::memcpy(&f[(size_t)n + t], &row, 4);
    }
    if (!dev_copy(&p->d_values_f32, f.data(), f.size(), &p->device_bytes)) {
        (void)hipGetLastError();
        if (p->d_values_f32) (void)hipFree(p->d_values_f32);
        p->d_values_f32 = nullptr;
        return UBP_ERR_ALLOC;
    }
    p->d_cols = reinterpret_cast<const int32_t *>(p->d_values_f32 + n);
    return UBP_OK;
}

ubp_status upload_stripe_layout(const ubp_packed *p, int slot) {
    StripeLayoutDev &D = p->d_sg[slot];
    if (D.uploaded) return UBP_OK;
    const StripeLayout &L = p->sg[slot];
    bool ok = dev_copy_vec(&D.rg_ptr, L.rg_ptr, &p->device_bytes) && dev_copy_vec(&D.rg_order, L.rg_order, &p->device_bytes) &&
              dev_copy_vec(&D.stream, L.stream, &p->device_bytes);
    if (!ok) {
        (void)hipGetLastError();
        return UBP_ERR_ALLOC;
    }
    D.uploaded = true;
    return UBP_OK;
}

ubp_status upload_blk_layout(const ubp_packed *p, int slot) {
    BlkLayoutDev &D = p->d_blk[slot];
    if (D.uploaded) return UBP_OK;
    const BlkLayout &L = p->blk[slot];
    bool ok = dev_copy_vec(&D.rg_ptr, L.rg_ptr, &p->device_bytes) && dev_copy_vec(&D.rg_order, L.rg_order, &p->device_bytes) &&
              dev_copy_vec(&D.meta, L.meta, &p->device_bytes) && dev_copy_vec(&D.frags, L.frags, &p->device_bytes);
    if (!ok) {
        (void)hipGetLastError();
        return UBP_ERR_ALLOC;
    }
    D.uploaded = true;
    return UBP_OK;
}

ubp_status upload_tile_layout(const ubp_packed *p) {
    TileLayoutDev &D = p->d_tiles;
    if (D.uploaded) return UBP_OK;
    const TileLayout &T = p->tiles;
    bool ok = dev_copy_vec(&D.frags, T.frags, &p->device_bytes) && dev_copy_vec(&D.occupied, T.occupied, &p->device_bytes);
    if (!ok) {
        (void)hipGetLastError();
        return UBP_ERR_ALLOC;
    }
    D.uploaded = true;
    return UBP_OK;
}

ubp_status upload_direct_layout(const ubp_packed *p) {
    DirectLayoutDev &D = p->d_direct;
    if (D.uploaded) return UBP_OK;
    const DirectLayout &L = p->direct;
    bool ok = dev_copy_vec(&D.first, L.first, &p->device_bytes) && dev_copy_vec(&D.order, L.order, &p->device_bytes) &&
              dev_copy_vec(&D.ids, L.ids, &p->device_bytes) && dev_copy_vec(&D.frags, L.frags, &p->device_bytes);
    if (!ok) {
        (void)hipGetLastError();
        return UBP_ERR_ALLOC;
    }
    D.uploaded = true;
    return UBP_OK;
}

ubp_status upload_wros4_layout(const ubp_packed *p) {
    Wros4LayoutDev &D = p->d_wros4;
    if (D.weights) return UBP_OK;
    // one allocation and one copy: weights, offsets, rec_of_row, rec_of_end, row_of_rec
    const Wros4Layout &L = p->wros4;
    std::vector<uint32_t> all(L.weights.size() + L.offsets.size() + L.rec_of_row.size() + L.rec_of_end.size() + L.row_of_rec.size());
    size_t at[6] = {0};
    int n = 0;
    auto add = [&](const auto &v) {
        if (!v.empty()) std::memcpy(&all[at[n]], v.data(), v.size() * 4);
        at[n + 1] = at[n] + v.size();
        ++n;
    };
    add(L.weights);
    add(L.offsets);
    add(L.rec_of_row);
    add(L.rec_of_end);
    add(L.row_of_rec);
    uint32_t *d = nullptr;
    if (!dev_copy_vec(&d, all, &p->device_bytes)) {
        (void)hipGetLastError();
        if (d) (void)hipFree(d);
        return UBP_ERR_ALLOC;
    }
    D.offsets = d + at[1];
    D.rec_of_row = reinterpret_cast<const int32_t *>(d + at[2]);
    D.rec_of_end = reinterpret_cast<const int32_t *>(d + at[3]);
    D.row_of_rec = reinterpret_cast<const int32_t *>(d + at[4]);
    D.weights = reinterpret_cast<float *>(d);
    return UBP_OK;
}

void release_device(ubp_packed *p) {
    if (!p || p->device == UBP_HOST_ONLY) return;
    DeviceGuard guard(p->device);
    if (!guard.ok) return;
    auto rel = [](auto *&ptr) {
        if (ptr) (void)hipFree(ptr);
        ptr = nullptr;
    };
    rel(p->d_indptr);
    rel(p->d_indices);
    rel(p->d_values_f32);
    rel(p->d_error);
    rel(p->d_tiles.frags);
    rel(p->d_tiles.occupied);
    rel(p->d_direct.first);
    rel(p->d_direct.order);
    rel(p->d_direct.ids);
    rel(p->d_direct.frags);
    rel(p->d_wros4.weights);
    for (int s = 0; s < kNumLayouts; ++s) {
        rel(p->d_sg[s].rg_ptr);
        rel(p->d_sg[s].rg_order);
        rel(p->d_sg[s].stream);
    }
    for (int s = 0; s < kNumBlkLayouts; ++s) {
        rel(p->d_blk[s].rg_ptr);
        rel(p->d_blk[s].rg_order);
        rel(p->d_blk[s].meta);
        rel(p->d_blk[s].frags);
    }
}


namespace {

StripeArgs stripe_args(const ubp_packed *p, const Shape &s, const void *X, int64_t ldx, int N, void *Y, int64_t ldy, bool vec_ok,
                       int ctile0, const Epilogue &ep) {
    const int slot = layout_slot(s.G, s.CT);
    const StripeLayout &L = p->sg[slot];
    const StripeLayoutDev &LD = p->d_sg[slot];
    StripeArgs a;
    a.rg_ptr = LD.rg_ptr;
    a.rg_order = LD.rg_order;
    a.stream = LD.stream;
    a.stream_bytes = (uint32_t)(L.stream.size() * sizeof(uint32_t));
    a.X = static_cast<const uint16_t *>(X);
    a.Y = Y;
    a.ldx = ldx;
    a.ldy = ldy;
    a.M = p->M;
    a.K = p->K;
    a.bh = p->bh;
    a.N = N;
    a.nrg = L.nrg;
    a.nch = L.nch;
    a.ring_bytes = std::min(ring_rows(s.CT), L.nch * kSlotRows) * ring_pitch(s.CT);
    a.err = p->d_error;
    a.ctile0 = ctile0;
    a.n_coltiles = 0;
    a.n_wgrows = s.wg_rows;
    a.n_producers = s.NP;
    a.resident = s.resident ? 1 : 0;
    a.vec_ok = vec_ok;
    a.ep = ep;
    return a;
}

// The whole of ubp_spmm_plan / ubp_spmm_prepare.  dry: everything but the launch.
ubp_status execute(const ubp_packed *p, const void *X_dev, int64_t ldx, int32_t N, void *Y_dev, int64_t ldy, ubp_dtype y_dtype,
                   void *stream, const ubp_plan *plan, bool dry, ubp_plan *chosen, const ubp_epilogue *fused) try {
    if (!p || N < 0) return UBP_ERR_INVALID_ARG;
    Epilogue ep = {nullptr, 0, 0.f, 0.f};
    if (fused) {
        if (fused->activation < 0 || fused->activation > 2) return UBP_ERR_INVALID_ARG;
        if (fused->activation == 2 && !(fused->lo <= fused->hi)) return UBP_ERR_INVALID_ARG; // (also refuses NaN bounds)
        ep.bias = fused->bias_dev;
        ep.on = (fused->bias_dev != nullptr || fused->activation != 0) ? 1 : 0;
        ep.lo = fused->activation == 1 ? 0.f : fused->activation == 2 ? fused->lo : -INFINITY;
        ep.hi = fused->activation == 2 ? fused->hi : INFINITY;
    }
    if (p->device == UBP_HOST_ONLY) return UBP_ERR_INVALID_ARG;
    if (y_dtype != UBP_F32 && y_dtype != p->dtype) return UBP_ERR_INVALID_ARG;
    if (N == 0) return UBP_OK;
    if (!X_dev || !Y_dev || ldx < N || ldy < N) return UBP_ERR_INVALID_ARG;
    ubp_plan pl;
    std::memset(&pl, 0, sizeof pl);
    if (plan) pl = *plan;
    DeviceGuard guard(p->device);
    if (!guard.ok) return UBP_ERR_DEVICE;
    const size_t ysz = (y_dtype == UBP_F32) ? 4 : 2;
    const bool vec_ok = (ldx % 8 == 0) && (reinterpret_cast<uintptr_t>(X_dev) % 16 == 0) && ((ldy * ysz) % 16 == 0) &&
                        (reinterpret_cast<uintptr_t>(Y_dev) % 16 == 0);
    const int64_t ldx_bytes = std::min(ldx, int64_t(1) << 60) * dtype_size(p->dtype); // (a single row may claim any pitch)
    const bool bf16 = p->dtype == UBP_BF16, y_f32 = y_dtype == UBP_F32;

    Shape s;
    Shape tail;          // block kernel: the gather kernel's shape for a last column tile that it leaves
    bool has_tail = false;
    {
        // Layouts are built and uploaded on first use, under the handle's lock.  A repeated call
        // finds everything in place and allocates nothing.
        std::lock_guard<std::mutex> hold(p->lock);
        ubp_status rc = UBP_OK;
        const Choice *known = nullptr;
        if (!plan)
            for (const Choice &c : p->choices)
                if (c.N == N && c.ldx == ldx && c.vec_ok == vec_ok && c.ysz == ysz) known = &c;
        if (known) {
            s = known->shape;
        } else {
            rc = resolve(p, N, ldx_bytes, vec_ok, ysz, pl, s);
            if (rc != UBP_OK) return rc;
            if (!plan) {
                p->choices[p->next_choice] = Choice{N, ldx, vec_ok, ysz, s};
                p->next_choice = (p->next_choice + 1) % kChoices;
            }
        }
        switch (s.kernel) {
        case 1:
        case 3: rc = s.px ? upload_wros4_layout(p) : upload_values_f32(p); break;
        case 2: rc = upload_stripe_layout(p, layout_slot(s.G, s.CT)); break;
        case 4:
        case 5:
        case 9:
        case 7: rc = upload_tile_layout(p); break;
        case 8: rc = upload_direct_layout(p); break;
        case 6:
            rc = upload_blk_layout(p, blk_slot(s.G));
            if (rc == UBP_OK && blk_leaves_tail(N)) {
                ubp_plan tp;
                std::memset(&tp, 0, sizeof tp);
                tp.kernel = 2;
                tp.col_tiles = 4;
                rc = resolve(p, N, ldx_bytes, vec_ok, ysz, tp, tail);
                if (rc == UBP_OK) rc = upload_stripe_layout(p, layout_slot(tail.G, tail.CT));
                has_tail = true;
            }
            break;
        }
        if (rc != UBP_OK) return rc;
    }
    if (chosen) {
        std::memset(chosen, 0, sizeof *chosen);
        chosen->kernel = s.kernel;
        chosen->sub_stripes = s.G;
        chosen->col_tiles = s.CT;
        chosen->waves = s.waves;
        chosen->rows_per_range = s.rpr;
        chosen->producers = s.NP;
        chosen->wg_rows = s.wg_rows;
    }

    switch (s.kernel) {
    case 1:
        if (s.px) {
            const Wros4Layout &L = p->wros4;
            Wros4Args a = {};
            a.weights = p->d_wros4.weights;
            a.offsets = p->d_wros4.offsets;
            a.rec_of_row = p->d_wros4.rec_of_row;
            a.rec_of_end = p->d_wros4.rec_of_end;
            a.row_of_rec = p->d_wros4.row_of_rec;
            a.weight_bytes = (uint32_t)(L.weights.size() * sizeof(float));
            a.offset_bytes = (uint32_t)(L.offsets.size() * sizeof(uint32_t));
            a.X = static_cast<const float *>(X_dev);
            a.Y = static_cast<float *>(Y_dev);
            a.ldx = ldx;
            a.ldy = ldy;
            a.M = p->M;
            a.K = p->K;
            a.N = N;
            a.n_tiles = (N + s.px - 1) / s.px;
            a.rpr = s.rpr;
            a.slices = (int)(((int64_t)p->M + (int64_t)s.rpr * s.px_waves - 1) / ((int64_t)s.rpr * s.px_waves));
            a.vec4 = (N % 4 == 0) && (ldx % 4 == 0) && (reinterpret_cast<uintptr_t>(X_dev) % 16 == 0);
            a.ep = ep;
            return launch_wros4(a, p->bh, s.px, s.px_waves, stream, dry);
        }
        [[fallthrough]];
    case 3: return launch_wros(p, X_dev, ldx, N, Y_dev, ldy, y_dtype, s.rpr, s.kernel == 3, ep, stream, dry);
    case 2: return launch_stripe(stripe_args(p, s, X_dev, ldx, N, Y_dev, ldy, vec_ok, 0, ep), bf16, y_f32, s.G, s.CT, s.waves, stream, dry);
    case 4:
    case 5:
    case 9:
    case 7: {
        const TileLayout &T = p->tiles;
        TileArgs a = {};
        a.frags = p->d_tiles.frags;
        a.occupied = p->d_tiles.occupied;
        a.X = static_cast<const uint16_t *>(X_dev);
        a.Y = Y_dev;
        a.ldx = ldx;
        a.ldy = ldy;
        a.M = p->M;
        a.K = p->K;
        a.N = N;
        a.nstripes = T.nstripes;
        a.err = p->d_error;
        a.ep = ep;
        a.kt_total = T.kt_pad;
        a.skip = T.tiles_nonzero != (int64_t)T.nstripes * ((p->K + kStep - 1) / kStep) ? 1 : 0; // (padding tiles aside)
        a.n_blocks = (N + 16 * s.CT - 1) / (16 * s.CT); // (kernel 4; the others count their own tiles)
        a.slices = s.wg_rows;
        a.sps = (T.nstripes + s.wg_rows - 1) / s.wg_rows;
        if (s.kernel == 4) return launch_xstat(a, bf16, y_f32, s.CT, T.kt_pad, s.waves, stream, dry);
        return launch_mtile(a, bf16, y_f32, s.shape, s.rows, stream, dry);
    }
    case 8: {
        DirectArgs a = {};
        a.first = p->d_direct.first;
        a.order = p->d_direct.order;
        a.ids = p->d_direct.ids;
        a.frags = p->d_direct.frags;
        a.X = static_cast<const uint16_t *>(X_dev);
        a.Y = Y_dev;
        a.ldx = ldx;
        a.ldy = ldy;
        a.M = p->M;
        a.N = N;
        a.nstripes = p->direct.nstripes;
        a.ep = ep;
        return launch_direct(a, bf16, y_f32, s.CT, s.waves, stream, dry);
    }
    case 6: {
        const int slot = blk_slot(s.G);
        const BlkLayout &L = p->blk[slot];
        const BlkLayoutDev &LD = p->d_blk[slot];
        BlkArgs a = {};
        a.rg_ptr = LD.rg_ptr;
        a.rg_order = LD.rg_order;
        a.meta = LD.meta;
        a.frags = LD.frags;
        a.meta_bytes = (uint32_t)(L.meta.size() * sizeof(uint32_t));
        a.frag_bytes = (uint32_t)(L.frags.size() * sizeof(uint32_t));
        a.X = static_cast<const uint16_t *>(X_dev);
        a.Y = Y_dev;
        a.ldx = ldx;
        a.ldy = ldy;
        a.M = p->M;
        a.K = p->K;
        a.N = N;
        a.nrg = L.nrg;
        a.nch = L.nch;
        a.ring_bytes = std::min(ring_rows(4), L.nch * kSlotRows) * ring_pitch(4);
        a.n_coltiles = blk_leaves_tail(N) ? N / 64 : (N + 63) / 64;
        a.n_wgrows = s.wg_rows;
        a.n_producers = s.NP;
        a.out_bytes = 0; // set per launch
        a.err = p->d_error;
        a.ep = ep;
        ubp_status rc = launch_blk(a, bf16, y_f32, s.G, s.waves, stream, dry);
        if (rc == UBP_OK && has_tail)
            rc = launch_stripe(stripe_args(p, tail, X_dev, ldx, N, Y_dev, ldy, vec_ok, N / 64, ep), bf16, y_f32, tail.G, tail.CT,
                               tail.waves, stream, dry);
        return rc;
    }
    }
    return UBP_ERR_INVALID_ARG;
} catch (const std::bad_alloc &) { // (the widened weights of kernels 1 and 3, on the host)
    return UBP_ERR_ALLOC;
} catch (const std::length_error &) {
    return UBP_ERR_ALLOC;
}

} // namespace

} // namespace ubp

// ------------------------------------------------------------------ C ABI
extern "C" {

ubp_status ubp_spmm_plan(const ubp_packed *p, const void *X_dev, int64_t ldx, int32_t N, void *Y_dev, int64_t ldy,
                         ubp_dtype y_dtype, void *hip_stream, const ubp_plan *plan) {
    return ubp::execute(p, X_dev, ldx, N, Y_dev, ldy, y_dtype, hip_stream, plan, false, nullptr, nullptr);
}

ubp_status ubp_spmm(const ubp_packed *p, const void *X_dev, int64_t ldx, int32_t N, void *Y_dev, int64_t ldy,
                    ubp_dtype y_dtype, void *hip_stream) {
    return ubp::execute(p, X_dev, ldx, N, Y_dev, ldy, y_dtype, hip_stream, nullptr, false, nullptr, nullptr);
}

ubp_status ubp_spmm_fused(const ubp_packed *p, const void *X_dev, int64_t ldx, int32_t N, void *Y_dev, int64_t ldy,
                          ubp_dtype y_dtype, const ubp_epilogue *epilogue, void *hip_stream, const ubp_plan *plan) {
    return ubp::execute(p, X_dev, ldx, N, Y_dev, ldy, y_dtype, hip_stream, plan, false, nullptr, epilogue);
}

ubp_status ubp_spmm_prepare(const ubp_packed *p, const void *X_dev, int64_t ldx, int32_t N, void *Y_dev, int64_t ldy,
                            ubp_dtype y_dtype, const ubp_plan *plan, ubp_plan *chosen) {
    return ubp::execute(p, X_dev, ldx, N, Y_dev, ldy, y_dtype, nullptr, plan, true, chosen, nullptr);
}

ubp_status ubp_packed_device_error(const ubp_packed *p, uint32_t *flags) {
    if (!p || !flags || p->device == UBP_HOST_ONLY) return UBP_ERR_INVALID_ARG;
    ubp::DeviceGuard guard(p->device);
    if (!guard.ok) return UBP_ERR_DEVICE;
    if (hipMemcpy(flags, p->d_error, sizeof(uint32_t), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return UBP_ERR_DEVICE;
    }
    return UBP_OK;
}

ubp_status ubp_launch_floor(void *hip_stream) { return ubp::launch_floor(hip_stream); }

} // extern "C"
