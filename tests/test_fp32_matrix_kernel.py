"""The fp32 matrix kernel (kernel 1 on fp32 handles): its stream of block columns, walked on the CPU, and its products on the GPU;
the fp32 layers that the vector kernel keeps."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2407_19644_amd as ubp
from synthetic import make_activations, make_weights, select_blocks

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_19644_amd", "csrc")

DRIVER = r"""
#include "ubp_internal.h"
namespace ubp { // the device half of the library
ubp_status upload(ubp_packed *) { return UBP_ERR_DEVICE; }
void release_device(ubp_packed *) {}
}
extern "C" int stream_of(const ubp_packed *p, int64_t *sizes, const void **arrays) {
    std::lock_guard<std::mutex> hold(p->lock);
    const ubp::Wros4Layout &L = ubp::get_wros4_layout(p);
    const int64_t n[5] = {(int64_t)L.weights.size(), (int64_t)L.offsets.size(), (int64_t)L.rec_of_row.size(), (int64_t)L.rec_of_end.size(), (int64_t)L.row_of_rec.size()};
    const void *a[5] = {L.weights.data(), L.offsets.data(), L.rec_of_row.data(), L.rec_of_end.data(), L.row_of_rec.data()};
    for (int i = 0; i < 5; ++i) { sizes[i] = n[i]; arrays[i] = a[i]; }
    return L.usable ? L.n_records : -1;
}
extern "C" int shape_of(const ubp_packed *p, int N, int64_t ldx, int rpr, int *out) {
    std::lock_guard<std::mutex> hold(p->lock);
    ubp::Shape s;
    ubp_plan pl = {};
    pl.kernel = 1;
    pl.rows_per_range = rpr;
    const int rc = ubp::resolve(p, N, 4 * ldx, true, 4, pl, s);
    const int f[4] = {s.kernel, s.px, s.px_waves, s.rpr};
    for (int i = 0; i < 4; ++i) out[i] = f[i];
    return rc;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("stream")
    (d / "driver.cpp").write_text(DRIVER)
    so = d / "libstream.so"
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(d / "driver.cpp")] +
                          [os.path.join(CSRC, f) for f in ("ubp_host.cpp", "ubp_layouts.cpp", "ubp_choose.cpp")] +
                          ["-o", str(so), "-pthread", "-Wl,-Bsymbolic"])
    return ctypes.CDLL(str(so))


def _pack(lib, W, bh, bw, blocks):
    h = ctypes.c_void_p()
    b = np.ascontiguousarray(blocks, dtype=np.int32).reshape(-1, 2)
    rc = lib.ubp_pack(W.ctypes.data_as(ctypes.c_void_p), 0, W.shape[0], W.shape[1], ctypes.c_int64(W.shape[1]), bh, bw,
                      b.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(len(b)), -1, ctypes.byref(h))
    assert rc == 0
    return h


# M, K, bh, bw, blocks (a density, or the list itself): one start row with a remainder of every size, empty start rows,
# more than 255 rows that end behind one group, nothing kept, a single block at the first and at the last start row
LAYERS = [(64, 64, 4, 4, 0.5), (33, 45, 5, 3, 0.5), (50, 630, 16, 1, 0.05), (257, 31, 1, 1, 0.3), (90, 60, 3, 2, 0.004), (130, 600, 16, 16, 0.15),
          (48, 520, 2, 6, 0.35), (100, 100, 8, 8, 0.3), (40, 60, 9, 2, 0.3), (40, 60, 13, 5, 0.4), (1400, 8, 4, 4, [(700, 0)]),
          (1400, 8, 4, 4, [(0, 0), (1396, 4)]), (30, 8, 4, 4, []), (700, 20, 2, 1, [(0, 3), (0, 4), (0, 5), (300, 7), (698, 0)])]


@pytest.mark.parametrize("case", LAYERS, ids=lambda c: "x".join(map(str, c[:4])) + "-" + str(c[4])[:8])
def test_the_stream_walked_as_the_kernel_walks_it(lib, case):
    """Every range of rows, from its first record: each output row is complete exactly once, in order, and accumulator row 0 then
    holds the row's weights, added in the order of start rows and columns; fill-up columns point to the row of zeros."""
    M, K, bh, bw, blocks = case
    W = make_weights(M, K, 5, "f32")
    blocks = select_blocks(M, K, bh, bw, blocks, 3, "uniform", 1.1) if isinstance(blocks, float) else blocks
    h = _pack(lib, W, bh, bw, blocks)
    sizes, arrays = (ctypes.c_int64 * 5)(), (ctypes.c_void_p * 5)()
    records = lib.stream_of(h, sizes, arrays)
    assert records >= 0

    def view(i, dt):
        return np.frombuffer((ctypes.c_char * (sizes[i] * 4)).from_address(arrays[i]), dt).copy() if sizes[i] else np.zeros(0, dt)
    weights, offsets = view(0, np.float32).reshape(-1, 64), view(1, np.uint32).reshape(-1, 32)
    assert len(weights) == len(offsets)
    rec_of_row, rec_of_end, row_of_rec = (view(i, np.int32) for i in (2, 3, 4))
    lib.ubp_packed_free(h)
    slots = 4 if bh <= 4 else 8 if bh <= 8 else 16
    cols = 64 // slots
    assert len(rec_of_row) == len(rec_of_end) == M and len(row_of_rec) == records + 1
    zero = -(-K // 8) * 8
    want = [[] for _ in range(M)]                                   # (column, weight) of every output row, in the order of addition
    for r, c in sorted((int(r), int(c)) for r, c in blocks):
        for q in range(bw):
            for t in range(bh):
                want[r + t].append((c + q, W[r + t, c + q]))
    for rpr in sorted({bh, 3 * bh, 16, M}):
        for lo in range(0, M, rpr):
            hi = min(lo + rpr, M)
            first = min(max(0, lo - bh + 1), M - 1)
            rec0, rec1 = rec_of_row[first], rec_of_end[hi - 1] + 1
            i = min(first, row_of_rec[rec0])
            acc, done = [[] for _ in range(slots)], []

            def finish(n):
                nonlocal i
                for _ in range(n):
                    if lo <= i < hi:
                        assert acc[0] == want[i], (rpr, lo, i)
                        done.append(i)
                    acc[:bh] = acc[1:bh] + [[]]
                    i += 1
            finish(row_of_rec[rec0] - i)
            rec = rec0
            loaded = rec0 + 4                                       # records of which the first 4 are under way before the loop
            while rec < rec1:
                for _ in range(4):                                  # a round of the kernel; each record walked is replaced by one more
                    for c in range(cols):
                        row = int(offsets[rec, c])
                        assert row % 256 == 0 and (row // 256 < K or row // 256 == zero)
                        w = weights[rec, c * slots:(c + 1) * slots]
                        # (-0 x +0 leaves every sum as it is; +0 x +0 would turn one of -0, left by products that underflow, into +0)
                        assert row // 256 < K or (not w.any() and np.signbit(w).all())
                        assert not w[bh:].any()
                        assert rec < records or (row // 256 == zero and offsets[rec, 16] == 0)
                        for s in range(bh if row // 256 < K else 0):
                            acc[s].append((row // 256, w[s]))
                        if c % 4 == 3:
                            finish((int(offsets[rec, 16]) >> (8 * (c // 4))) & 255)
                    rec += 1
                    loaded += 1
            assert loaded <= len(weights), "records are loaded past the stream's end"
            assert done == list(range(lo, hi)), (rpr, lo, done)


def test_where_it_is_used(lib):
    """64 pixels while all of X for them fits LDS, 32 beyond, the vector kernel where K is too large for that or blocks are few;
    a pinned range is kept, and the range that comes back gives the same shape."""
    for K, blocks, want in ((632, 0.2, (64, 32)), (633, 0.2, (32,)), (1272, 0.2, (32,)), (1273, 0.2, (0,)), (632, 0.002, (0,))):
        W = make_weights(96, K, 5, "f32")
        h = _pack(lib, W, 4, 4, select_blocks(96, K, 4, 4, blocks, 3, "uniform", 1.1))
        out, again = (ctypes.c_int * 4)(), (ctypes.c_int * 4)()
        for N in (1, 49, 6272):
            for rpr in (0, 4, 7, 96, 5000):
                assert lib.shape_of(h, N, ctypes.c_int64(N), rpr, out) == 0 and out[0] == 1 and out[1] in want, (K, N, rpr, list(out))
                assert rpr == 0 or out[3] == rpr
                assert lib.shape_of(h, N, ctypes.c_int64(N), out[3], again) == 0 and list(again) == list(out)
            assert lib.shape_of(h, N, ctypes.c_int64(1 << 24), 0, out) == 0 and out[1] in want   # 64 MB
            assert lib.shape_of(h, N, ctypes.c_int64((1 << 24) + 8), 0, out) == 0 and out[1] == 0
        assert lib.shape_of(h, 64, ctypes.c_int64(64), -1, out) == 1
        lib.ubp_packed_free(h)


# M, K, N, bh, bw, density: layers of the vector kernel, K too large or too few blocks for the other.  Around its batches of 8 (blocks of
# up to 4 rows), 4 (up to 8) and 2 columns: start rows with no, one and several batches and every remainder, ends of the matrix and
# of a pixel tile, one column and four columns a lane.
VECTOR = [(40, 1273, 63, 4, 1, 0.02), (24, 1300, 65, 1, 1, 0.13), (33, 1275, 65, 5, 3, 0.05), (50, 1280, 130, 16, 1, 0.02), (60, 1290, 64, 8, 2, 0.1),
          (90, 2000, 31, 3, 2, 0.002), (70, 1301, 129, 9, 4, 0.1), (30, 1273, 1, 12, 1, 0.1), (800, 1280, 1536, 4, 1, 0.02), (1040, 1288, 1028, 8, 8, 0.05),
          (1600, 1300, 1028, 16, 2, 0.02), (90, 60, 257, 3, 2, 0.004), (512, 512, 100, 4, 1, 0.01), (300, 100, 40, 1, 1, 0.03)]


@pytest.mark.parametrize("shape", VECTOR, ids=lambda s: "x".join(map(str, s)))
def test_layers_of_the_vector_kernel(lib, shape):
    M, K, N, bh, bw, d = shape
    h = _pack(lib, make_weights(M, K, 5, "f32"), bh, bw, select_blocks(M, K, bh, bw, d, M + 1, "uniform", 1.1))
    out = (ctypes.c_int * 4)()
    for rpr in (0, bh, 5 * bh):
        assert lib.shape_of(h, N, ctypes.c_int64(N), rpr, out) == 0 and list(out[:3]) == [1, 0, 0]
    lib.ubp_packed_free(h)


def test_launches_have_fewer_than_2_to_the_32_threads(lib):
    """Workgroups come in eights: 64-pixel tiles times slices of rows up to 2^22 - 1 would be a launch of 2^22 workgroups of 1024."""
    M, K = 23 * 64, 16                                              # 23 slices of 16 wavefronts of 4 rows
    W = make_weights(M, K, 5, "f32")
    h = _pack(lib, W, 4, 4, select_blocks(M, K, 4, 4, 0.5, 3, "uniform", 1.1))
    out = (ctypes.c_int * 4)()
    for tiles in (1000, 182360, 182361, 182362):                    # 23 x 182361 = 2^22 - 1
        for rpr in (0, 4):
            assert lib.shape_of(h, 64 * tiles, ctypes.c_int64(64 * tiles), rpr, out) == 0
            _, px, waves, rows = out
            assert px == 0 or -(-(-(-64 * tiles // px) * -(-M // (rows * waves))) // 8) * 8 * waves * 64 < 2 ** 32, (tiles, rpr, list(out))
            assert rpr == 0 or (px != 0) == (tiles < 182361), (tiles, list(out))
    lib.ubp_packed_free(h)


# ------------------------------------------------------------------ on the device
# M, K, N, bh, bw, density: every block height; K around the limits of 64 and 32 pixels and of the kernel, K mod 8; N around a tile
PRODUCTS = [(60 + bh, 40 + bh, 61 + bh, bh, 1 + bh % 3, 0.45) for bh in range(1, 17)] + [
    (40, 632, 65, 4, 1, 0.2), (40, 633, 64, 4, 1, 0.2), (70, 1272, 33, 8, 2, 0.2), (70, 1273, 32, 8, 2, 0.2), (64, 64, 1, 4, 4, 0.5),
    (1, 64, 196, 1, 1, 0.9), (16, 16, 3, 16, 16, 1.0), (1000, 24, 130, 4, 4, 0.4)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", PRODUCTS, ids=lambda s: "x".join(map(str, s)))
def test_product(shape):
    """Against the oracle, and bit for bit the vector kernel's sums (kernel 3, never this one): whole and odd rows, a pitch and a
    start that 16-byte loads cannot take, bias and clamp, weights and X among the denormal numbers, Inf and NaN in X."""
    import torch
    import oracle
    from gpu_util import check
    from synthetic import decode_f64
    M, K, N, bh, bw, d = shape
    blocks = select_blocks(M, K, bh, bw, d, M, "uniform", 1.1)
    W, X = make_weights(M, K, K, "f32"), make_activations(K, N, N, "f32", "normal")
    p = ubp.pack(W, "f32", bh, bw, blocks, device=torch.cuda.current_device())
    stream = torch.cuda.current_stream().cuda_stream
    bias = torch.randn(M, device="cuda")

    def run(Xh, plan, pad=0, at=0, fused=False):
        buf = torch.zeros(K * (N + pad) + 8, device="cuda")
        Xd = buf[at:at + K * (N + pad)].view(K, N + pad)
        Xd[:, :N] = torch.from_numpy(Xh).cuda()
        Yd = torch.full((M, N + pad), 7.0, device="cuda")
        if fused:
            ubp.spmm_fused(p, Xd.data_ptr(), N + pad, N, Yd.data_ptr(), N + pad, "f32", bias.data_ptr(), "clamp", -0.25, 0.5, stream, plan)
        else:
            ubp.spmm(p, Xd.data_ptr(), N + pad, N, Yd.data_ptr(), N + pad, "f32", stream, plan)
        assert (Yd[:, N:] == 7.0).all()
        return Yd[:, :N].cpu().numpy()

    def same_bits(a, b):
        return np.array_equal(a.view(np.uint32), b.view(np.uint32))
    vector = ubp.Plan(kernel=3)
    want = run(X, vector)
    Yref, Yabs = oracle.spmm(decode_f64(W, "f32"), bh, bw, blocks, decode_f64(X, "f32"), want_abs=True)
    check(want.astype(np.float64), Yref, Yabs, "f32")
    for plan in (None, ubp.Plan(kernel=1, rows_per_range=bh), ubp.Plan(kernel=1, rows_per_range=3 * bh + 1)):
        for pad, at in ((0, 0), (4, 0), (3, 1)):
            assert same_bits(run(X, plan, pad, at), want), (plan, pad, at)
    assert same_bits(run(X, None, fused=True), run(X, vector, fused=True))
    for scale in (1e-38, 1e-44):                      # products and sums among the denormal numbers; products that underflow to zeros of either sign
        Xs = X * np.float32(scale)
        assert same_bits(run(Xs, None), run(Xs, vector)), scale
    Xn = X.copy()
    Xn[K // 2, N // 2], Xn[K // 3, 0], Xn[0, N - 1] = np.inf, np.nan, -np.inf
    got, want = run(Xn, None), run(Xn, vector)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and same_bits(got[~np.isnan(want)], want[~np.isnan(want)])
    p.free()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", VECTOR, ids=lambda s: "x".join(map(str, s)))
def test_vector_kernel(shape):
    """The layers above against the oracle and bit for bit the shifting dataflow (kernel 3)."""
    import oracle
    from gpu_util import check, run_spmm
    from synthetic import decode_f64
    M, K, N, bh, bw, d = shape
    blocks = select_blocks(M, K, bh, bw, d, M + 1, "uniform", 1.1)
    W, X = make_weights(M, K, K, "f32"), make_activations(K, N, N, "f32", "normal")
    Yref, Yabs = oracle.spmm(decode_f64(W, "f32"), bh, bw, blocks, decode_f64(X, "f32"), want_abs=True)
    want = run_spmm(W, "f32", bh, bw, blocks, X, "f32", ubp.Plan(kernel=3, rows_per_range=bh))
    for plan, pad in ((None, 0), (ubp.Plan(kernel=1, rows_per_range=bh), 0), (ubp.Plan(kernel=1, rows_per_range=5 * bh), 3)):
        Y = run_spmm(W, "f32", bh, bw, blocks, X, "f32", plan, ldx=N + pad, ldy=N + pad)
        check(Y, Yref, Yabs, "f32", "f32")
        assert np.array_equal(Y.view(np.uint64), want.view(np.uint64)), plan
