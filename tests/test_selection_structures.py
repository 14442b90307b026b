"""Where the selectors' tree of maxima (8 children to a node) and their set of remaining entries (64 to a word) can go wrong:
sizes around a power of either, blocks longer than a node, a word or the list, ties, entries that may not be kept."""
import numpy as np
import pytest

import oracle.selection as sel
import paper_2407_19644_amd as ubp


@pytest.mark.parametrize("b", [1, 2, 7, 8, 9, 63, 64, 65, 127, 129, 511, 512, 513, 4095, 4096, 4097])
def test_sizes_around_a_node_and_a_word(b):
    rng = np.random.default_rng(b)
    for N in sorted({1, 2, 5, 9, 70, b, 2 * b} if b < 1000 else {3, 70}):
        for kind in range(3):
            S = rng.integers(0, 4, size=b).astype(np.float64) if kind == 0 else rng.standard_normal(b)     # many ties; negative scores
            if kind == 2:
                S[rng.random(b) < 0.7] = -np.inf
            for m in sorted({1, b // (2 * N) + 1, b}) if b < 1000 else (b // 6,):
                assert ubp.select_greedy(S, N, m).tolist() == sel.select_greedy(S, N, m), (N, kind, m)
                assert ubp.select_bed(S, N, m).tolist() == sel.select_bed(S, N, m), (N, kind, m)


def test_one_end_to_the_other():
    """Best entries from the front, from the back, and outwards from the middle: runs of removed entries over many words."""
    b, N = 3000, 2
    ramp = np.arange(b, dtype=np.float64)
    for S in (ramp, -ramp, -np.abs(ramp - b // 2)):
        assert ubp.select_bed(S, N, b).tolist() == sel.select_bed(S, N, b)
        assert ubp.select_greedy(S, N, b).tolist() == sel.select_greedy(S, N, b)


def test_scores_whose_sums_pass_the_largest_double():
    """A power of two times other scores: the same choice."""
    S = np.abs(np.random.default_rng(3).standard_normal(300)) + 0.5
    S *= 0.49 / S.max()
    for N, m in ((2, 100), (4, 60)):
        assert ubp.select_bed(S * 2.0 ** 1000 * 2.0 ** 24, N, m).tolist() == ubp.select_bed(S, N, m).tolist()
        assert ubp.select_bed(np.ldexp(S, 1024), N, m).tolist() == ubp.select_bed(S, N, m).tolist()


def test_the_smallest_scores_beside_the_largest():
    """Scores keep all their bits beside ones whose sums pass the largest double."""
    tiny = 2.0 ** -1074
    for top in (2.0 ** 1000, 2.0 ** 1016, 1.7e308):
        S = np.array([3 * tiny, top, 5 * tiny, 4 * tiny, 6 * tiny, -tiny])
        for m in range(1, 7):
            assert ubp.select_bed(S, 1, m).tolist() == sel.select_bed(S, 1, m), (top, m)
    S = np.array([top, -np.inf, 3 * tiny, -np.inf, 5 * tiny, -np.inf, 4 * tiny, -np.inf, top, 0.75 * top, 0.5 * top, -np.inf])
    assert [ubp.select_bed(S, 2, m).tolist() for m in (1, 2, 3, 4, 5)] == [[0], [0, 8], [0, 8, 10], [0, 4, 8, 10], [0, 4, 6, 8, 10]]


@pytest.mark.parametrize("M,K,bh,bw", [(1, 1, 1, 1), (7, 130, 7, 1), (9, 65, 3, 1), (64, 64, 4, 2), (129, 200, 16, 3), (3000, 3, 5, 1), (140000, 2, 2, 1)])
def test_scores_of_odd_shapes(M, K, bh, bw):
    """Pieces of 8 rows by 64 column groups, and single columns where M is large; every fp16 and bf16 bit pattern that is a number."""
    rng = np.random.default_rng(M)
    for dtype in ("f32", "f16", "bf16"):
        bits = rng.integers(0, 1 << 16, size=(M, K)).astype(np.uint16)
        top = 0x7c00 if dtype == "f16" else 0x7f80
        bits[(bits & top) == top] &= ~np.uint16(top)          # (no Inf, no NaN)
        W = rng.standard_normal((M, K)).astype(np.float32) if dtype == "f32" else bits.view(np.float16) if dtype == "f16" else bits
        V = W.astype(np.float64) if dtype != "bf16" else (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        norm = np.zeros((M, K // bw))
        for q in range(bw):
            norm += np.abs(V[:, q:K // bw * bw:bw])
        for aligned in (False, True):
            want = np.full((M, K // bw), -np.inf)
            for i in range(0, M - bh + 1, bh if aligned else 1):
                s = np.zeros(K // bw)
                for t in range(bh):
                    s = s + norm[i + t]
                want[i] = s
            assert np.array_equal(ubp.block_scores(W, dtype, bh, bw, aligned), want.T.reshape(-1)), (dtype, aligned)


def test_every_half():
    """All fp16 bit patterns; an Inf or a NaN among the weights is refused by the selection."""
    bits = np.arange(1 << 16, dtype=np.uint16).reshape(256, 256)
    W = bits.view(np.float16)
    S = ubp.block_scores(W, "f16", 1, 1)
    want = np.abs(W.astype(np.float64)).T.reshape(-1)
    assert np.array_equal(S, want, equal_nan=True)
    with pytest.raises(ubp.UBPError) as e:
        ubp.select_blocks(W, "f16", 1, 1, 0.1)
    assert e.value.code == 1
