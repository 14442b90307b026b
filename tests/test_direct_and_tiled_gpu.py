"""GPU parity of kernel 1 on fp32 layers, of the direct kernel (8) and of the LDS-staged dense tiles at any alignment (9), at the
edges of their tiles, against the CPU oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle                                    # noqa: E402
import paper_2407_19644_amd as ubp               # noqa: E402
from synthetic import decode_f64, make_activations, make_weights, select_blocks   # noqa: E402
from gpu_util import check, run_spmm, to_device  # noqa: E402

pytestmark = pytest.mark.gpu


def _plan(**kw):
    p = ubp.Plan()
    for k, v in kw.items():
        setattr(p, k, v)
    return p


def _case(M, K, N, bh, bw, density, dtype, seed):
    blocks = select_blocks(M, K, bh, bw, density, seed, "uniform", 1.1)
    W = make_weights(M, K, seed + 1, dtype)
    X = make_activations(K, N, seed + 2, dtype, "normal")
    return blocks, W, X, oracle.spmm(decode_f64(W, dtype), bh, bw, blocks, decode_f64(X, dtype), want_abs=True)


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 8, 15, 16, 17, 31, 32, 33, 49, 63, 64, 65, 130])
@pytest.mark.parametrize("shape", [(33, 70, 4, 4, 0.3), (130, 600, 16, 16, 0.1), (17, 31, 5, 3, 0.4), (16, 2100, 4, 1, 0.02)],
                         ids=lambda s: "x".join(map(str, s)))
def test_direct_kernel(shape, N):
    """Pixel tiles that hang over the right edge, rows of 2-byte alignment, more wavefronts than
    steps, stripes without any step, a last stripe beyond M."""
    M, K, bh, bw, d = shape
    for dtype in ("f16", "bf16"):
        blocks, W, X, (Yref, Yabs) = _case(M, K, N, bh, bw, d, dtype, seed=M + N)
        for CT, waves, pad in [(0, 0, 0), (1, 1, 1), (1, 16, 0), (2, 3, 3), (4, 2, 1), (4, 16, 8)]:
            if N < CT:
                with pytest.raises(ubp.UBPError):
                    run_spmm(W, dtype, bh, bw, blocks, X, "f32", _plan(kernel=8, col_tiles=CT))
                continue
            for y_dtype in (dtype, "f32"):
                Y = run_spmm(W, dtype, bh, bw, blocks, X, y_dtype, _plan(kernel=8, col_tiles=CT, waves=waves),
                             ldx=N + pad, ldy=N + pad)
                check(Y, Yref, Yabs, dtype, y_dtype)


@pytest.mark.parametrize("N", [8, 9, 15, 16, 63, 65, 127, 136, 200, 385])
@pytest.mark.parametrize("shape", [(64, 64, 4, 4, 0.6), (130, 65, 4, 4, 0.5), (17, 300, 8, 8, 0.3), (300, 129, 16, 16, 0.2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_staged_tiles_at_any_alignment(shape, N):
    """Every tile size, rows of X with and without 16-byte alignment, pieces of 8 pixels over the right
    edge, a last stage of fewer than 64 columns, one stage only, rows beyond M; matrices with and
    without empty operand tiles."""
    M, K, bh, bw, d = shape
    for dtype in ("f16", "bf16"):
        blocks, W, X, (Yref, Yabs) = _case(M, K, N, bh, bw, d, dtype, seed=M + N + 1)
        for G, CT, pad in [(0, 0, 0), (8, 8, 1), (8, 4, 3), (4, 8, -N % 8), (4, 4, 0), (8, 8, -N % 8), (4, 4, 5),
                           (8, 16, -N % 8)]:
            if (G, CT) == (4, 8) and N % 8:
                continue        # (that shape is for aligned rows)
            for y_dtype in (dtype, "f32"):
                Y = run_spmm(W, dtype, bh, bw, blocks, X, y_dtype, _plan(kernel=9, sub_stripes=G, col_tiles=CT),
                             ldx=N + pad, ldy=N + pad)
                check(Y, Yref, Yabs, dtype, y_dtype)
    with pytest.raises(ubp.UBPError):
        run_spmm(W, dtype, bh, bw, blocks, X[:, :7], dtype, _plan(kernel=9))


@pytest.mark.parametrize("shape", [(16, 20000, 64, 0.05, 5), (64, 36000, 200, 0.02, 5), (16, 17000, 64, 0.45, 7)],
                         ids=lambda s: "x".join(map(str, s)))
def test_kernels_5_and_7_where_the_occupancy_words_pass_a_register(shape):
    """K beyond 16384: a stripe has more than 16 words of occupancy bits.  The pinned kernel is the one that runs."""
    M, K, N, d, kernel = shape
    dtype = "bf16"
    blocks, W, X, (Yref, Yabs) = _case(M, K, N, 4, 4, d, dtype, seed=5)
    Xd = torch.empty(K, N, dtype=torch.bfloat16, device="cuda")
    p = ubp.pack(W, dtype, 4, 4, blocks, device=torch.cuda.current_device())
    for k in (kernel, 9):
        plan = _plan(kernel=k, sub_stripes=4, col_tiles=4)
        assert ubp.spmm_prepare(p, Xd.data_ptr(), N, N, Xd.data_ptr(), N, dtype, plan).kernel == k
        check(run_spmm(W, dtype, 4, 4, blocks, X, "f32", plan, packed=p), Yref, Yabs, dtype, "f32")
    p.free()


def test_rows_of_x_more_than_32_mb_apart():
    """64 rows have no 32-bit offsets then: kernels 5, 7 and 9 and the automatic choice, a last stage of fewer than 64 rows."""
    M, K, N, dtype = 70, 100, 200, "bf16"
    ldx = (1 << 24) + 8
    blocks, W, X, (Yref, Yabs) = _case(M, K, N, 4, 4, 0.6, dtype, seed=21)
    Xd = torch.empty(K * ldx, dtype=torch.bfloat16, device="cuda").view(K, ldx)
    Xd[:, :N] = to_device(X, dtype)
    p = ubp.pack(W, dtype, 4, 4, blocks, device=torch.cuda.current_device())
    for plan in (_plan(kernel=7, sub_stripes=4, col_tiles=8), _plan(kernel=9), _plan(kernel=9, sub_stripes=4, col_tiles=4), None):
        Yd = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        ubp.spmm(p, Xd.data_ptr(), ldx, N, Yd.data_ptr(), N, "f32", torch.cuda.current_stream().cuda_stream, plan)
        check(Yd.cpu().numpy().astype(np.float64), Yref, Yabs, dtype, "f32")
    p.free()


VECTOR = [
    # M, K, N, bh, bw, density: blocks per start row around the vector kernel's batches of 8, 4 and 2 columns.  (The fp32 matrix kernel
    # takes the layers with several columns per row; test_fp32_matrix_kernel.py has ones that stay with the vector kernel.)
    (40, 36, 63, 4, 1, 0.5),
    (64, 64, 64, 1, 1, 0.13),
    (33, 45, 65, 5, 3, 0.5),
    (50, 640, 130, 16, 1, 0.05),
    (300, 100, 1028, 8, 8, 0.3),
    (90, 60, 257, 3, 2, 0.004),     # most start rows empty
    (20, 8, 1, 4, 4, 0.3),
]


@pytest.mark.parametrize("shape", VECTOR, ids=lambda s: "x".join(map(str, s)))
def test_vector_kernel_batches(shape):
    M, K, N, bh, bw, d = shape
    blocks, W, X, (Yref, Yabs) = _case(M, K, N, bh, bw, d, "f32", seed=M + K + N)
    want = run_spmm(W, "f32", bh, bw, blocks, X, "f32", _plan(kernel=3, rows_per_range=bh))
    for plan in (None, _plan(kernel=1), _plan(kernel=1, rows_per_range=bh), _plan(kernel=1, rows_per_range=5 * bh)):
        Y = run_spmm(W, "f32", bh, bw, blocks, X, "f32", plan)
        check(Y, Yref, Yabs, "f32", "f32")
        assert np.array_equal(Y, want)  # the same additions in the same order


@pytest.mark.parametrize("shape", [(960, 160, 1568, 4, 4, 0.3), (1024, 1024, 1568, 8, 1, 0.1)], ids=lambda s: "x".join(map(str, s)))
def test_blocks_in_every_tile_and_one_tile_of_zeros(shape):
    """Kept weights may all be zero: the automatic choice computes the layer, prepared, plain and fused."""
    M, K, N, bh, bw, d = shape
    blocks = select_blocks(M, K, bh, bw, d, 8, "uniform", 1.1)
    W = make_weights(M, K, 9, "f16")
    W[:16, :32] = 0
    X = make_activations(K, N, 10, "f16", "normal")
    Yref, Yabs = oracle.spmm(decode_f64(W, "f16"), bh, bw, blocks, decode_f64(X, "f16"), want_abs=True)
    p = ubp.pack(W, "f16", bh, bw, blocks, device=torch.cuda.current_device())
    Xd = torch.from_numpy(X).cuda()
    for tdt, y_dtype in ((torch.float16, "f16"), (torch.float32, "f32")):
        Yd = torch.full((M, N), float("nan"), dtype=tdt, device="cuda")
        assert ubp.spmm_prepare(p, Xd.data_ptr(), N, N, Yd.data_ptr(), N, y_dtype).kernel in (4, 5, 9)
        check(run_spmm(W, "f16", bh, bw, blocks, X, y_dtype, packed=p), Yref, Yabs, "f16", y_dtype)
        ubp.spmm_fused(p, Xd.data_ptr(), N, N, Yd.data_ptr(), N, y_dtype, None, "relu", 0.0, 0.0,
                       torch.cuda.current_stream().cuda_stream)
        check(Yd.cpu().numpy().astype(np.float64), np.maximum(Yref, 0), Yabs, "f16", y_dtype)
    p.free()
