"""Which kernel a 16-bit product takes, with which launch shape: ubp_choose.cpp, compiled with the host
compiler and called without a device."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2407_19644_amd as ubp
from synthetic import make_weights, select_blocks

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_19644_amd", "csrc")
OK, INVALID, UNSUPPORTED = 0, 1, 4

DRIVER = r"""
#include <cstdlib>
#include <new>
#include "ubp_internal.h"

// allocations left until one fails (< 0: none does), the bytes in use and their peak
static long left_ = -1, now_ = 0, peak_ = 0;
void *operator new(std::size_t n, const std::nothrow_t &) noexcept {
    if (left_ == 0) return nullptr;
    if (left_ > 0) --left_;
    char *q = static_cast<char *>(std::malloc(n + 16));
    if (!q) return nullptr;
    *reinterpret_cast<std::size_t *>(q) = n;
    now_ += (long)n;
    if (now_ > peak_) peak_ = now_;
    return q + 16;
}
void *operator new(std::size_t n) {
    void *q = operator new(n, std::nothrow);
    if (!q) throw std::bad_alloc();
    return q;
}
void operator delete(void *q) noexcept {
    if (!q) return;
    char *b = static_cast<char *>(q) - 16;
    now_ -= (long)*reinterpret_cast<std::size_t *>(b);
    std::free(b);
}
void operator delete(void *q, std::size_t) noexcept { operator delete(q); }
void operator delete(void *q, const std::nothrow_t &) noexcept { operator delete(q); }
extern "C" void fail_after(long n) { left_ = n; }
extern "C" long peak_bytes() { // since the last call
    const long v = peak_ - now_;
    peak_ = now_;
    return v;
}

namespace ubp { // the device half of the library
ubp_status upload(ubp_packed *) { return UBP_ERR_DEVICE; }
void release_device(ubp_packed *) {}
}

extern "C" int choice(const ubp_packed *p, int N, int64_t ldx_bytes, int aligned, int ysz, const ubp_plan *pl, int *out) {
    ubp::Shape s;
    std::lock_guard<std::mutex> hold(p->lock);
    const int rc = ubp::resolve(p, N, ldx_bytes, aligned != 0, (size_t)ysz, *pl, s);
    const int f[8] = {s.kernel, s.shape, s.G, s.CT, s.waves, s.NP, s.wg_rows, s.rpr};
    for (int i = 0; i < 8; ++i) out[i] = f[i];
    return rc;
}

// the direct kernel's layout: sizes, then the four arrays
extern "C" int direct_layout(const ubp_packed *p, int64_t *sizes, const void **arrays) {
    std::lock_guard<std::mutex> hold(p->lock);
    const ubp::DirectLayout &L = ubp::get_direct_layout(p);
    const int64_t n[5] = {L.nsteps, (int64_t)L.first.size(), (int64_t)L.order.size(), (int64_t)L.ids.size(), (int64_t)L.frags.size()};
    const void *a[4] = {L.first.data(), L.order.data(), L.ids.data(), L.frags.data()};
    for (int i = 0; i < 5; ++i) sizes[i] = n[i];
    for (int i = 0; i < 4; ++i) arrays[i] = a[i];
    return L.nstripes;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("choice")
    (d / "driver.cpp").write_text(DRIVER)
    so = d / "libchoice.so"
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                           str(d / "driver.cpp")] + [os.path.join(CSRC, f) for f in ("ubp_host.cpp", "ubp_layouts.cpp", "ubp_choose.cpp")] +
                          ["-o", str(so), "-pthread", "-Wl,-Bsymbolic"])
    lib = ctypes.CDLL(str(so))
    lib.fail_after.argtypes, lib.peak_bytes.restype = [ctypes.c_long], ctypes.c_long
    lib.ubp_packed_info.restype = ctypes.c_int64
    return lib


class Layer:
    """A packed host-only handle of the driver's own copy of the host code."""

    def __init__(self, lib, M, K, bh, bw, density, W=None, dtype="bf16", blocks=None):
        self.lib, self.handle, self.esz = lib, ctypes.c_void_p(), 4 if dtype == "f32" else 2
        W = make_weights(M, K, 4, dtype) if W is None else W
        b = np.ascontiguousarray(select_blocks(M, K, bh, bw, density, 3, "uniform", 1.1) if blocks is None else blocks, dtype=np.int32)
        rc = lib.ubp_pack(W.ctypes.data_as(ctypes.c_void_p), {"f32": 0, "f16": 1, "bf16": 2}[dtype], M, K, ctypes.c_int64(K), bh, bw,
                          b.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(len(b)), -1, ctypes.byref(self.handle))
        assert rc == OK

    def choice(self, N, aligned=None, ysz=2, ldx=None, **plan):
        """(status, {field: value}) of a call on N pixels; plan fields by name."""
        ldx = N if ldx is None else ldx
        aligned = ldx % 8 == 0 if aligned is None else aligned
        pl = ubp.Plan()
        for k, v in plan.items():
            setattr(pl, k, v)
        out = (ctypes.c_int * 8)()
        rc = self.lib.choice(self.handle, N, ctypes.c_int64(self.esz * ldx), int(aligned), ysz, ctypes.byref(pl), out)
        return rc, dict(zip(("kernel", "shape", "G", "CT", "waves", "NP", "wg_rows", "rpr"), out))

    def __del__(self):
        self.lib.ubp_packed_free(self.handle)


@pytest.mark.parametrize("M,K,N,bh,bw,density", [(960, 160, 3136, 4, 4, 0.3), (1024, 1024, 1568, 8, 1, 0.1), (64, 64, 4096, 4, 4, 0.6),
                                                 (256, 2304, 12544, 4, 4, 0.25)])
def test_kept_weights_that_are_all_zero_are_no_reason_to_refuse(lib, M, K, N, bh, bw, density):
    """Blocks reach every 16 x 32 tile; the weights of one tile (or all weights) are zero: the automatic choice takes
    the call, and not with the kernel that wants a weight in every tile."""
    for zero in ((slice(0, 16), slice(0, 32)), (slice(None), slice(None)), (slice(M - 16, M), slice(K - 32, K))):
        W = make_weights(M, K, 4, "bf16")
        W[zero] = 0
        layer = Layer(lib, M, K, bh, bw, density, W)
        for n in (16, 200, N, N + 1):
            for ysz in (2, 4):
                rc, c = layer.choice(n, ysz=ysz)
                assert rc == OK and c["kernel"] != 7, (n, ysz, c)


@pytest.mark.parametrize("M,N", [(4096, 1 << 20), (65536, 1 << 17), (65536, 1 << 19), (65536, 1 << 21), (1 << 20, 1 << 14), (1 << 20, 1 << 17)])
def test_direct_launches_have_fewer_than_2_to_the_32_threads(lib, M, N):
    """Whatever kernel 8 is chosen or pinned with, its workgroups times their threads fit a launch; beyond that the automatic
    choice takes another kernel and a pin is refused."""
    layer = Layer(lib, M, 32, 4, 4, 0.002)

    def threads(CT, waves):
        pairs = -(-M // 16) * -(-N // (16 * CT))
        return -(-pairs // 8) * 8 * waves * 64
    rc, c = layer.choice(N)
    assert rc == OK and c["kernel"] == (8 if threads(4, 1) < 2 ** 32 else 2)
    assert c["kernel"] == 2 or threads(c["CT"], c["waves"]) < 2 ** 32
    for CT in (0, 1, 2, 4):
        for waves in (0, 1, 4, 16):
            rc, c = layer.choice(N, kernel=8, col_tiles=CT, waves=waves)
            able = threads(4, 1) < 2 ** 32      # (what kernel 8 takes at all, whatever is pinned)
            fits = able and threads(CT or 4, waves or 1) < 2 ** 32
            assert rc == (OK if fits else UNSUPPORTED), (CT, waves, c)
            assert not fits or threads(c["CT"], c["waves"]) < 2 ** 32


def test_dense_tiles_at_any_k_and_pitch(lib):
    """Pinned kernel 5 is kernel 5 wherever its tiles exist: a K of more occupancy words than a register holds, rows of X too
    far apart for 32-bit offsets."""
    layer = Layer(lib, 16, 20000, 4, 4, 0.05)
    for ldx in (64, (1 << 24) + 8, 1 << 26):
        for pins in ({}, dict(sub_stripes=2, col_tiles=4), dict(sub_stripes=4, wg_rows=3)):
            rc, c = layer.choice(64, ldx=ldx, kernel=5, **pins)
            assert rc == OK and c["kernel"] == 5, (ldx, pins, c)


def test_a_stream_too_large_for_the_fp32_matrix_kernel_is_not_built(lib):
    """140 million columns, 16 bytes each in that kernel's stream: the vector kernel takes the layer, and nothing is laid out for the other."""
    M, K = 200000, 700
    layer = Layer(lib, M, K, 1, K, None, W=np.zeros((M, K), np.float32), dtype="f32", blocks=np.stack([np.arange(M), np.zeros(M)], axis=1))
    lib.peak_bytes()
    rc, c = layer.choice(64)
    assert rc == OK and c["kernel"] == 1 and lib.peak_bytes() < 1 << 20


def test_a_pinned_kernel_is_the_kernel_that_runs(lib):
    """Kernels 2, 6 and 7 named without a shape, on layers where the automatic choice is another kernel."""
    for M, K, bh, bw, d, N in ((160, 1100, 4, 4, 0.25, 256), (64, 64, 4, 4, 0.6, 128), (90, 1280, 16, 16, 0.15, 1280)):
        layer = Layer(lib, M, K, bh, bw, d)
        for kernel in (2, 6, 7, 8, 9):
            rc, c = layer.choice(N, kernel=kernel)
            assert rc == UNSUPPORTED and kernel == 7 and bh == 16 or rc == OK and c["kernel"] == kernel, (M, kernel, rc, c)


FIELDS = ("sub_stripes", "col_tiles", "waves", "producers", "wg_rows")
# what a call resolves to, as a plan: layers and calls that reach every kernel
ROUND_TRIP = [(160, 1100, 4, 4, 0.25, (256, 4608, 4603)), (1024, 1024, 4, 4, 0.45, (1568, 16)), (256, 256, 8, 8, 0.12, (12544, 64)),
              (90, 1280, 16, 16, 0.15, (1280,)), (40, 2100, 4, 4, 0.02, (64, 4096)), (256, 256, 2, 1, 0.3, (25088,))]


@pytest.mark.parametrize("case", ROUND_TRIP, ids=lambda c: "x".join(map(str, c[:4])))
def test_the_chosen_plan_is_taken_back(lib, case):
    """What a call resolves to, automatically or with a named kernel, given as the plan of the same call: the same kernel and shape."""
    M, K, bh, bw, d, pixels = case
    layer = Layer(lib, M, K, bh, bw, d)
    for N in pixels:
        for kernel in (0, 1, 2, 4, 5, 6, 7, 8, 9):
            rc, c = layer.choice(N, kernel=kernel)
            if rc != OK:
                continue
            back = dict(kernel=c["kernel"], sub_stripes=c["G"], col_tiles=c["CT"], waves=c["waves"], rows_per_range=c["rpr"],
                        producers=c["NP"], wg_rows=c["wg_rows"])
            assert layer.choice(N, **back) == (OK, c), (N, kernel, back)


def test_tiles_that_kernels_5_7_and_9_take(lib):
    """Kernel 7 takes the workgroup tiles it has always taken, kernel 5 stripes and tiles of 2 or 4, kernel 9 whole 64s up to 256;
    a negative number of slices is an invalid argument; no size is too large to be refused."""
    layer = Layer(lib, 160, 1100, 4, 4, 0.45)
    sizes = (0, 1, 2, 3, 4, 5, 8, 12, 16, 17, 32, 100, 2 ** 27 + 8, 2 ** 31 - 1, -1, -8)
    seven = {(16, 16), (8, 16), (8, 8), (16, 4), (4, 8), (4, 4)}
    for G in sizes:
        for CT in sizes:
            want = {5: G in (0, 2, 4) and CT in (0, 2, 4), 9: G in (0, 4, 8, 16) and CT in (0, 4, 8, 16),
                    7: any(G in (0, a) and CT in (0, b) for a, b in seven)}
            for kernel, ok in want.items():
                rc, c = layer.choice(512, kernel=kernel, sub_stripes=G, col_tiles=CT)
                assert rc == (OK if ok else UNSUPPORTED), (kernel, G, CT, rc)
                unit = 32 if kernel == 5 else 16
                assert not ok or G == 0 or c["G"] == min(G, 128 // unit)
                assert not ok or CT == 0 or c["CT"] == min(CT, 128 // unit)
    assert layer.choice(512, kernel=5, wg_rows=-1)[0] == INVALID
    assert layer.choice(512, kernel=5, wg_rows=3)[0] == OK and layer.choice(512, kernel=5, waves=4)[0] == UNSUPPORTED


def _kernel_by_matrix(layer, M, K, bh, bw, N, aligned, ldx):
    """The kernel a plan of fields without a name has always meant: by the matrix and the alignment alone."""
    tiles_kept, tiles = (layer.lib.ubp_packed_info(layer.handle, w) for w in (10, 11))
    if bh == 16 and bw >= 16 and K > 1024 and aligned and N >= 64:
        return 6
    if not (aligned and N % 8 == 0) or tiles < 0:
        return 2
    if tiles_kept == tiles and (K <= 256 or N <= 4096) and K * ldx * 2 < 2 ** 31:
        return 7
    return 2 if 2 * tiles_kept < tiles else 4 if K <= 256 else 5


@pytest.mark.parametrize("case", ROUND_TRIP + [(96, 200, 4, 4, 0.5, (392, 49)), (300, 300, 16, 16, 0.05, (8,))],
                         ids=lambda c: "x".join(map(str, c[:4])))
def test_fields_without_a_kernel(lib, case):
    """A plan may fix part of a shape and leave the kernel open: what the automatic choice's kernel takes is taken by it, and
    what the kernel that goes by the matrix alone takes stays accepted; nothing else is."""
    M, K, bh, bw, d, pixels = case
    layer = Layer(lib, M, K, bh, bw, d)
    plans = [{f: v} for f in FIELDS for v in (-1, 1, 2, 3, 4, 5, 8, 12, 17)] + [dict(rows_per_range=8), dict(sub_stripes=2, col_tiles=8),
             dict(sub_stripes=4, waves=6, producers=2), dict(col_tiles=2, waves=3, wg_rows=2), dict(col_tiles=4, waves=8)]
    for N in pixels:
        automatic = layer.choice(N)[1]["kernel"]
        by_matrix = _kernel_by_matrix(layer, M, K, bh, bw, N, N % 8 == 0, N)
        for plan in plans:
            named = [layer.choice(N, kernel=k, **plan) for k in (automatic, by_matrix)]
            rc, c = layer.choice(N, **plan)
            taken = [n for n in named if n[0] == OK]
            assert (rc, c) == taken[0] if taken else rc == named[1][0], (N, plan, rc, c, named)


ALLOC = 6


@pytest.mark.parametrize("M,K,bh,bw,density,N", [(160, 1100, 4, 4, 0.25, 256), (256, 256, 8, 8, 0.12, 12544), (90, 1280, 16, 16, 0.15, 1280),
                                                 (40, 70000, 4, 4, 0.02, 64)])
def test_an_allocation_that_fails_is_an_error_and_leaves_the_handle_whole(lib, M, K, bh, bw, density, N):
    """One of the host allocations of a choice and of the layouts behind it fails, the first few and then every sixth or so: the call reports it, nothing is thrown, and the
    same call afterwards resolves to what a fresh handle resolves to, with the same layouts."""
    for kernel in (0, 2, 5, 6, 8):
        fresh = Layer(lib, M, K, bh, bw, density)
        want = fresh.choice(N, kernel=kernel)
        n = 0
        while True:
            layer = Layer(lib, M, K, bh, bw, density)
            lib.fail_after(n)
            rc, _ = layer.choice(N, kernel=kernel)
            lib.fail_after(-1)
            assert rc in (want[0], ALLOC), (kernel, n, rc)
            assert layer.choice(N, kernel=kernel) == want, (kernel, n)
            if kernel == 2 and rc == ALLOC:
                for what in (10, 11) + tuple(range(100, 109)) + tuple(range(200, 209)):
                    assert lib.ubp_packed_info(layer.handle, what) == lib.ubp_packed_info(fresh.handle, what)
            if rc == want[0]:
                break
            n += 1 + n // 6
    layer = Layer(lib, M, K, bh, bw, density)
    for what in (10, 100, 300):
        lib.fail_after(0)
        assert lib.ubp_packed_info(layer.handle, what) == -1
        lib.fail_after(-1)
        assert lib.ubp_packed_info(layer.handle, what) == lib.ubp_packed_info(fresh.handle, what)


def test_a_choice_takes_no_memory_by_rows_times_columns(lib):
    """A large sparse layer: choosing a kernel counts its blocks without a bitmap of the matrix (8 MB here, one bit a stripe and column)."""
    M, K = 1 << 15, 1 << 15
    W = np.zeros((M, K), np.uint16)     # (never touched: no memory behind it)
    layer = Layer(lib, M, K, 4, 4, 0, W, blocks=[(8 * i, 4 * (i % 1000)) for i in range(1000)])
    lib.peak_bytes()
    rc, c = layer.choice(8, kernel=8)
    assert rc == OK and c["kernel"] == 8
    assert lib.peak_bytes() < 4 << 20


def test_the_two_vector_dataflows_walk_the_same_ranges(lib):
    """Kernel 3 is there to be timed beside kernel 1: the same row ranges, whatever the layer and the pixels."""
    for M, K, bh, bw, d in ((512, 512, 4, 1, 0.2), (64, 64, 4, 4, 0.5), (1024, 1024, 8, 1, 0.1), (257, 31, 1, 1, 0.3)):
        layer = Layer(lib, M, K, bh, bw, d, dtype="f16")
        for N in (1, 49, 196, 1568, 6272, 25088):
            (rc1, a), (rc3, b) = layer.choice(N, kernel=1), layer.choice(N, kernel=3)
            assert rc1 == rc3 == OK and a["rpr"] == b["rpr"] > 0, (M, N, a, b)


# layers of many pixels whose zero-filled W passes 8 MB or whose tiles are mostly empty: M, K, bh, bw, density, {pixels: kernel}
WEIGHED = [(3336, 2288, 4, 4, 0.27, {2048: 2, 64: 8, 2049: 8}), (2928, 1744, 8, 1, 0.28, {13120: 2, 100: 8, 13117: 8}),
           (1784, 3608, 2, 1, 0.07, {14592: 2, 49: 8}), (1656, 2080, 16, 16, 0.06, {800: 8, 64: 8}),
           (4096, 4096, 16, 16, 0.1, {8192: 6, 16: 8}), (256, 256, 8, 8, 0.12, {64: 8, 784: 8}), (1024, 256, 8, 8, 0.12, {12544: 4})]


@pytest.mark.parametrize("case", WEIGHED, ids=lambda c: "x".join(map(str, c[:4])))
def test_every_kernel_is_weighed(lib, case):
    """The gather kernel where it was measured to be the fastest and not beside it; whole blocks as operands only where there
    are workgroups enough and no launch for a last ragged tile behind them; the direct kernel on few pixels whatever the tiles."""
    M, K, bh, bw, d, want = case
    layer = Layer(lib, M, K, bh, bw, d)
    for N, kernel in want.items():
        rc, c = layer.choice(N)
        assert rc == OK and c["kernel"] == kernel, (N, c)


@pytest.mark.parametrize("M,K,bh,bw,density", [(64, 64, 4, 4, 0.5), (33, 70, 4, 4, 0.3), (17, 31, 5, 3, 0.4), (130, 600, 16, 16, 0.1), (257, 31, 1, 1, 0.3),
                                               (90, 130, 20, 3, 0.2), (16, 2100, 4, 1, 0.02), (200, 100, 8, 8, 0.01)])
def test_the_direct_layout_is_the_matrix(lib, M, K, bh, bw, density):
    """Decoded: every weight once, in the order of the kernel's operands, padding and all; columns ascending within a stripe, and each
    step's padding a row of X that the stripe reads anyway."""
    W, blocks = make_weights(M, K, 4, "bf16"), select_blocks(M, K, bh, bw, density, 3, "uniform", 1.1)
    layer = Layer(lib, M, K, bh, bw, density, W, blocks=blocks)
    want, kept = np.zeros((-(-M // 16) * 16, K), np.uint16), np.zeros((-(-M // 16) * 16, K), bool)
    for r, c in blocks:
        want[r:r + bh, c:c + bw] = W[r:r + bh, c:c + bw]
        kept[r:r + bh, c:c + bw] = True
    sizes, arrays = (ctypes.c_int64 * 5)(), (ctypes.c_void_p * 4)()
    nstripes = lib.direct_layout(layer.handle, sizes, arrays)
    assert nstripes == -(-M // 16) and sizes[1] == nstripes + 1 and sizes[2] == nstripes
    nsteps = sizes[0]
    assert sizes[3] == 32 * nsteps and sizes[4] == 512 * nsteps

    def view(i, n, dt):
        return np.frombuffer((ctypes.c_char * (n * np.dtype(dt).itemsize)).from_address(arrays[i]), dt).copy() if n else np.zeros(0, dt)
    first, order = view(0, nstripes + 1, np.int32), view(1, nstripes, np.int32)
    ids, frags = view(2, 32 * nsteps, np.uint16).reshape(-1, 32), view(3, 512 * nsteps, np.uint16).reshape(-1, 4, 16, 8)
    assert first[0] == 0 and first[-1] == nsteps and sorted(order) == list(range(nstripes))
    assert (np.diff(np.diff(first)[order]) <= 0).all()                          # most steps first
    for st in range(nstripes):
        cols = np.flatnonzero(kept[16 * st:16 * st + 16].any(axis=0))
        assert first[st + 1] - first[st] == -(-len(cols) // 32)
        got = ids[first[st]:first[st + 1]].reshape(-1).astype(np.int64)
        assert np.array_equal(got[:len(cols)], cols) and np.isin(got[len(cols):], cols).all()
        # lane 16 g + n, element e: row n of the stripe in column 8 g + e of the step
        w = frags[first[st]:first[st + 1]].transpose(2, 0, 1, 3).reshape(16, -1)
        assert np.array_equal(w[:, :len(cols)], want[16 * st:16 * st + 16][:, cols]) and not w[:, len(cols):].any()


def test_tiles_of_128_by_256(lib):
    """For a 16-bit Y, K up to 256 and aligned rows: by the estimate where they save a round, or named with kernel 7 or 9."""
    layer = Layer(lib, 256, 256, 2, 1, 0.3, dtype="f16")
    assert layer.choice(25088)[1]["shape"] == 4 and layer.choice(25088)[1]["CT"] == 16
    for N, kw in ((25088, dict(ysz=4)), (25083, {}), (12544, {}), (25088, dict(kernel=5, sub_stripes=4, col_tiles=4)), (25088, dict(kernel=9, sub_stripes=4, col_tiles=16))):
        rc, c = layer.choice(N, **kw)
        assert rc == OK and c["shape"] != 4, (N, kw, c)
    for kernel in (7, 9):
        rc, c = layer.choice(512, kernel=kernel, sub_stripes=8, col_tiles=16)
        assert rc == OK and (c["shape"], c["G"], c["CT"]) == (4, 8, 16)
    rc, c = Layer(lib, 256, 260, 4, 4, 0.5).choice(25088, kernel=9, sub_stripes=8, col_tiles=16)
    assert rc == OK and c["shape"] == 0 and c["CT"] == 8


@pytest.mark.parametrize("M,K,N,want", [(4096, 4096, 1024, (2, 4)), (2048, 4096, 4096, (4, 4)), (4096, 4096, 8192, (5, 2)), (512, 1152, 64, (2, 4)), (16, 1152, 64, (2, 4))])
def test_split_of_the_block_kernel(lib, M, K, N, want):
    """Kernel 6 by itself: light wavefronts and four producers while the workgroups run beside each other, few workgroup rows where they
    come in rounds; what a plan pins goes with the rest as it always did, and the plan that comes out is taken back."""
    layer = Layer(lib, M, K, 16, 16, 0.1)
    rc, c = layer.choice(N, kernel=6)
    assert rc == OK and (c["G"], c["NP"]) == want
    assert c["waves"] - c["NP"] >= 1 and c["wg_rows"] * (c["waves"] - c["NP"]) * c["G"] * 16 >= M
    rc, back = layer.choice(N, kernel=6, sub_stripes=c["G"], col_tiles=c["CT"], waves=c["waves"], producers=c["NP"], wg_rows=c["wg_rows"])
    assert rc == OK and back == c
    for pins, G, NP in ((dict(waves=16), None, 2), (dict(producers=4), None, 4), (dict(sub_stripes=2), 2, 2)):
        rc, c = layer.choice(N, kernel=6, **pins)
        rows = lambda g: -(-(-(-M // (16 * g))) // 14)
        assert rc == OK and (c["G"], c["NP"]) == (G or (5 if rows(5) < rows(4) else 4), NP), pins
