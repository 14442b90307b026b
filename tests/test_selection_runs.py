"""Where the selectors go through parts of the candidates that no round reaches out of side by side: 4096 rounds or more, four cores
or more.  Columns of odd and even lengths, many equal scores, scores that differ by column (a few columns then say little
of the others), more rounds than there are candidates for, zeros of either sign; the number of rounds made, and the threads under sanitizers."""
import heapq
import os
import shutil
import subprocess
import textwrap

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


def test_columns_of_different_size():
    """Input channels of different importance, most of them dead, and a layer without a weight."""
    rng = np.random.default_rng(17)
    for M, K, bh, d in ((256, 300, 2, 0.12), (515, 128, 4, 0.3)):
        N = rng.standard_normal((M, K))
        for scale in (np.exp(rng.standard_normal((1, K))), np.exp(2.0 * rng.standard_normal((1, K))), rng.random((1, K)) > 0.8, np.zeros((1, K))):
            W = (N * scale).astype(np.float32)
            S, m = ubp.block_scores(W, "f32", bh, 1), ubp.target_block_count(M, K, bh, 1, d)
            assert m >= 4096
            assert ubp.select_greedy(S, bh, m).tolist() == greedy(S, bh, m)
            assert ubp.select_bed(S, bh, m).tolist() == bed(S, bh, m)


# By parts against one tree over all candidates, with teams of eight threads whatever cores there are, in two callers at once.
DRIVER = r"""
#include "ubp_select.cpp"
#include <cstdio>
#include <random>

extern "C" int64_t ubp_target_block_count(int32_t, int32_t, int32_t, int32_t, double) { return 0; }

static std::atomic<int64_t> counter[2];
template <Rounds R, int C> bool counted(Part &part, int32_t N, double above, int64_t most) {
    const size_t before = part.taken.size();
    const bool end = R(part, N, above, most);
    counter[C] += (int64_t)(part.taken.size() - before);
    return end;
}

static int64_t caller(int c, int64_t m_shift, int kinds) {
    std::mt19937_64 rng(11 + c);
    std::normal_distribution<double> normal;
    int64_t bad = 0, by_parts = 0;
    struct Layer { int64_t rows, columns; int32_t N; int64_t m; };
    const Layer layers[] = {{512, 128, 4, 6553}, {1024, 64, 2, 4200}, {700, 61, 3, 9000}, {257, 300, 1, 5000}, {4099, 20, 8, 4096}};
    for (const Layer &l : layers)
        for (int kind = 0; kind < kinds; ++kind) {
            const int64_t b = l.rows * l.columns;
            std::vector<double> S((size_t)b);
            for (int64_t j = 0; j < l.columns; ++j) {
                const double spread = kind == 1 ? 1.0 : kind == 2 ? 2.0 : 0.0, size = std::exp(spread * normal(rng)), dead = rng() % 5 != 0;
                for (int64_t i = 0; i < l.rows; ++i) {
                    double s = size * (1.0 + 0.3 * std::fabs(normal(rng)));
                    if (kind == 3 && dead) s = 0.0;                          // columns without a weight
                    if (kind == 4) s = (double)(1 + rng() % 5);              // many equal scores
                    if (kind == 5) s = 0.0;                                  // nothing but equal ones
                    if (kind == 6) s = j + 3 < l.columns ? s : 1e3 * s;      // all that is taken in a few columns
                    if (kind == 7 && rng() % 3 == 0) s = i % 2 ? kNegInf : -0.0;
                    S[(size_t)(j * l.rows + i)] = i + l.N > l.rows ? kNegInf : s;
                }
            }
            for (int method = 0; method < 2; ++method)
                for (int64_t m : {l.m, l.m + b / 3, std::numeric_limits<int64_t>::max() >> m_shift}) {
                    Team alone(1, 1), team(8, 8);
                    std::vector<int64_t> one((size_t)b), parts((size_t)b);
                    const auto select = method == 0 ? greedy_in_order : expand_and_divide;
                    const int64_t n = select(S.data(), b, l.N, m, one.data(), nullptr, alone);
                    if (select(S.data(), b, l.N, m, parts.data(), nullptr, team) != n || !std::equal(one.begin(), one.begin() + n, parts.begin())) {
                        std::printf("differs: %lld x %lld, N %d, kind %d, method %d, m %lld\n", (long long)l.columns, (long long)l.rows, l.N, kind, method, (long long)m);
                        ++bad;
                    }
                    counter[c] = 0;
                    const Rounds rounds = method == 0 ? (c ? counted<greedy, 1> : counted<greedy, 0>) : (c ? counted<expand, 1> : counted<expand, 0>);
                    by_parts += pick(rounds, S.data(), b, l.N, m, nullptr, team).size() > 1;
                    // a fifth more than are asked for and a started piece of 32 for each thread; half as many again where a few columns are unlike the others
                    if (counter[c] > n + n / (kind == 6 ? 2 : 5) + 8 * 32) {
                        std::printf("%lld rounds for %lld: %lld x %lld, N %d, kind %d, method %d\n", (long long)counter[c], (long long)n, (long long)l.columns, (long long)l.rows, l.N, kind, method);
                        ++bad;
                    }
                }
        }
    // what a part's thread throws, and the next call of the same team
    Team team(8, 8);
    bool caught = false;
    try {
        team.share(64, [](size_t p, size_t) { if (p == 33) throw std::length_error("33"); });
    } catch (const std::length_error &) {
        caught = true;
    }
    std::atomic<int> sum{0};
    for (int i = 0; i < 50; ++i) team.share(100, [&](size_t p, size_t) { sum += (int)p; });
    if (!caught || sum != 50 * 4950) ++bad;
    std::printf("caller %d: %lld by parts\n", c, (long long)by_parts);
    return bad + (by_parts == 0);
}

// As many threads as there are cores to run on, and one tree where those are few.
static int cores() {
    cpu_set_t had, set;
    if (sched_getaffinity(0, sizeof had, &had) != 0) return 1;
    const std::vector<double> S(100000, 1.0);
    int bad = 0;
    for (int few = 1; few <= 3; ++few) {
        CPU_ZERO(&set);
        for (int c = 0, n = 0; c < CPU_SETSIZE && n < few; ++c)
            if (CPU_ISSET(c, &had)) CPU_SET(c, &set), ++n;
        const size_t n = (size_t)CPU_COUNT(&set);
        if (sched_setaffinity(0, sizeof set, &set) != 0) return 1;
        Team team(8);
        bad += team.size() != n || threads_for_rounds(50000) != 1 || pick(greedy, S.data(), 100000, 1, 50000, nullptr, team).size() != 1;
    }
    bad += threads_for_scores(888, 124, 4) != 1 || threads_for_scores(512, 512, 1) != 8; // pieces of 64 columns
    return bad + (sched_setaffinity(0, sizeof had, &had) != 0);
}

int main(int argc, char **) { // (any argument: fewer scores)
    if (cores() != 0) {
        std::printf("threads for cores that there are not\n");
        return 1;
    }
    const int kinds = argc > 1 ? 4 : 8;
    int64_t bad[2] = {0, 0};
    std::thread second([&] { bad[1] = caller(1, 1, kinds); });
    bad[0] = caller(0, 0, kinds);
    second.join();
    std::printf(bad[0] + bad[1] ? "FAILED\n" : "parts ok\n");
    return bad[0] + bad[1] != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("sanitize", ["", "address,undefined,float-cast-overflow", "thread"])
def test_parts_take_what_one_tree_takes(tmp_path, sanitize):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    (tmp_path / "driver.cpp").write_text(textwrap.dedent(DRIVER))
    flags = ["-fsanitize=" + sanitize, "-fno-sanitize-recover=all", "-g", "-static-lib" + ("tsan" if sanitize == "thread" else "asan")] if sanitize else []
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-function", "-I", os.path.join(root, "include"), "-I", os.path.join(root, "paper_2407_19644_amd", "csrc"),
                           str(tmp_path / "driver.cpp"), "-o", str(tmp_path / "driver"), "-pthread"] + flags)
    res = subprocess.run([str(tmp_path / "driver")] + ([sanitize] if sanitize else []), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=600)
    assert res.returncode == 0 and "parts ok" in res.stdout, res.stdout[-4000:]
