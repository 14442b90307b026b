"""Where the selectors go through the runs of candidates that no round reaches out of one by one: 4096 rounds or more, 16 runs
or more.  Runs of odd and even lengths, many equal scores, scores that differ by run (a sample of the runs then says little
of the others), more rounds than there are candidates for, zeros of either sign."""
import heapq

import numpy as np
import pytest

import oracle.selection as sel
import paper_2407_19644_amd as ubp

NEG = -np.inf


def greedy(S, N, m):
    """The definition with a heap for the arg max (the oracle's loop over all scores at each of these many rounds takes minutes)."""
    free, heap, I = np.isfinite(S), [(-s, k) for k, s in enumerate(S) if np.isfinite(s)], []
    heapq.heapify(heap)
    while heap and len(I) < m:
        _, k = heapq.heappop(heap)
        if free[k]:
            I.append(k)
            free[max(0, k - N + 1):k + N] = False
    return I


def bed(S, N, m):
    """Algorithms 1 and 2 over links between what is left, a heap for the arg max (entries whose score has changed are passed over)."""
    S, b = S.copy(), len(S)
    after, before = list(range(1, b + 1)), list(range(-1, b - 1))
    heap = [(-s, k) for k, s in enumerate(S) if np.isfinite(s)]
    heapq.heapify(heap)
    I = []
    while heap and len(I) < m:
        s, k = heapq.heappop(heap)
        if -s != S[k]:
            continue
        right = [k]
        while len(right) < N + 1 and right[-1] < b:
            right.append(after[right[-1]])
        gone = [r for r in right[:N] if r < b]
        left, top = k, S[k]
        for n in range(1, N):
            left = before[left]
            if left < 0:
                break
            j = right[N - n] if N - n < len(right) and right[N - n] < b else -1
            S[left] = S[left] + (S[j] if j >= 0 else NEG) - top
            if np.isfinite(S[left]):
                heapq.heappush(heap, (-S[left], left))
        end, start = after[gone[-1]], before[k]
        if start >= 0:
            after[start] = end
        if end < b:
            before[end] = start
        S[gone] = NEG
        I.append(k)
    I.sort()
    nxt = 0
    for t, k in enumerate(I):
        if nxt > k:
            I[t], nxt = nxt, nxt + N
        else:
            nxt = k + N
    return I


def scores(kind, columns, rows, N, rng):
    S = rng.random((columns, rows)) + 0.5
    if kind == "ties":
        S = rng.integers(1, 5, size=(columns, rows)).astype(np.float64)
    elif kind == "by run":
        S *= np.exp(3.0 * rng.standard_normal((columns, 1)))
    elif kind == "last runs":                                       # all that is taken lies in a few runs
        S[columns - 6:] += 100.0
    elif kind == "zeros":
        S = np.where(rng.random((columns, rows)) < 0.5, 0.0, -0.0) - (rng.random((columns, rows)) < 0.3)
    elif kind == "holes":
        S[rng.random((columns, rows)) < 0.2] = NEG
    if N > 1:
        S[:, rows - N + 1:] = NEG
    return S.reshape(-1)


def test_the_definitions_here_are_the_oracles():
    rng = np.random.default_rng(5)
    for kind in ("plain", "ties", "holes"):
        for N in (1, 2, 4):
            S = scores(kind, 7, 20, N, rng)
            for m in (1, 10, 140):
                assert greedy(S, N, m) == sel.select_greedy(S, N, m) and bed(S, N, m) == sel.select_bed(S, N, m), (kind, N, m)


@pytest.mark.parametrize("kind", ["plain", "ties", "by run", "last runs", "zeros", "holes"])
@pytest.mark.parametrize("columns,rows,N,m", [(64, 517, 4, 5000), (16, 1031, 2, 4096), (300, 129, 3, 6000), (40, 400, 2, 20000), (15, 1200, 2, 4500), (33, 700, 1, 8000)])
def test_runs(kind, columns, rows, N, m):
    S = scores(kind, columns, rows, N, np.random.default_rng(columns))
    assert ubp.select_greedy(S, N, m).tolist() == greedy(S, N, m)
    assert ubp.select_bed(S, N, m).tolist() == bed(S, N, m)


@pytest.mark.parametrize("aligned", [False, True])
def test_layers_by_columns(aligned):
    rng = np.random.default_rng(9)
    for M, K, bh, bw, d in ((515, 260, 4, 1, 0.4), (256, 640, 8, 2, 0.9), (130, 1100, 2, 1, 0.1)):
        W = (rng.standard_normal((M, K)) * np.exp(rng.standard_normal((M, 1)))).astype(np.float16)
        S, m = ubp.block_scores(W, "f16", bh, bw, aligned), ubp.target_block_count(M, K, bh, bw, d)
        for method, f in (("greedy", greedy), ("bed", bed)):
            I = np.array(f(S, bh, m))
            assert ubp.select_blocks(W, "f16", bh, bw, d, method, aligned).tolist() == np.stack([I % M, I // M * bw], axis=1).tolist()
