// Block selection on the host: which m of a layer's b candidate blocks are kept (Sections 3.1,
// 3.2 and 4.1).  Scores (Eq. 1), the greedy selector (Eq. 3), the optimal selector (Eq. 4),
// block expansion and division (Algorithms 1 and 2) and the efficacy figure (Eq. 5).
//
// The selectors return what the paper's step-by-step descriptions return, but not by those
// steps where a faster route gives the same indices:
//   greedy   : the arg max comes from a tree of maxima (leftmost leaf wins a tie), so one of the m
//              rounds costs O(N + log b) instead of O(b), and where -inf separates columns from each other they are gone
//              through one by one, by several threads, and what they give is merged;
//   expansion: the shrinking score list is a set of the original indices, its arg max from the same tree, by columns as well;
//   optimal  : Eq. 4's table row by row with one decision bit per cell and a walk back from
//              (b, m) instead of carrying index sets, cells that cannot lie on a path to (b, m)
//              left out: O(b m) time, b m bits.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <exception>
#include <limits>
#include <mutex>
#include <new>
#include <numeric>
#include <stdexcept>
#include <system_error>
#include <thread>
#include <utility>
#include <vector>

#if defined(__SSE2__)
#include <emmintrin.h>
#endif

#include "ubp.h"

namespace {

constexpr double kNegInf = -std::numeric_limits<double>::infinity();

inline double from_bits(uint64_t u) {
    double d;
    std::memcpy(&d, &u, 8);
    return d;
}

// |value| of fp16 bits, without branches: the exponent re-biased in place, zero and subnormal numbers as 10 bits times 2^-24
inline double half_magnitude(uint16_t h) {
    const uint64_t m = h & 0x7fff;
    const double normal = from_bits((m << 42) + ((m >= 0x7c00 ? uint64_t(2047 - 31) : uint64_t(1023 - 15)) << 52));
    return m < 0x400 ? (double)(int32_t)m * 0x1p-24 : normal;
}

inline double bf16_bits_to_double(uint16_t h) {
    const uint32_t u = (uint32_t)h << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return (double)f;
}

inline double magnitude(float w) { return std::fabs((double)w); }
inline double magnitude_f16(uint16_t w) { return half_magnitude(w); }
inline double magnitude_bf16(uint16_t w) { return std::fabs(bf16_bits_to_double(w)); }

inline double element_magnitude(const void *W, ubp_dtype dtype, int64_t at) {
    switch (dtype) {
    case UBP_F32: return magnitude(static_cast<const float *>(W)[at]);
    case UBP_F16: return magnitude_f16(static_cast<const uint16_t *>(W)[at]);
    default: return magnitude_bf16(static_cast<const uint16_t *>(W)[at]);
    }
}

bool layer_ok(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t K, int32_t bh, int32_t bw) {
    return W && (dtype == UBP_F32 || dtype == UBP_F16 || dtype == UBP_BF16) && M >= 1 && K >= 1 && bh >= 1 && bw >= 1 &&
           bh <= M && bw <= K && ldw >= K;
}

// scores may be finite or -inf; anything else (NaN, +inf) has no order the selectors could use
bool scores_ok(const double *S, int64_t b) {
    bool ok = true; // (no early exit: the loop is done by vector instructions)
    for (int64_t k = 0; k < b; ++k) ok &= S[k] <= std::numeric_limits<double>::max();
    return ok;
}

bool selector_args_ok(const double *S, int64_t b, int32_t N, int64_t m, const int64_t *I, const int64_t *count) {
    return b >= 0 && (b == 0 || S) && N >= 1 && m >= 0 && (m == 0 || I) && count;
}

// f(state, part) for parts 0 .. parts - 1, each once, by up to `threads` threads (the caller among them) with a State each; what
// one of them throws is thrown here, after all have ended.  A thread that cannot be had is done without.
template <class State, class F> void share_out(size_t parts, size_t threads, F &&f) {
    constexpr size_t kMost = 8; // (a thread takes some 15 us to start)
    threads = std::min({threads, parts, kMost});
    if (threads > 1) threads = std::min(threads, (size_t)std::thread::hardware_concurrency()); // (which asks the system: some 2 us)
    std::atomic<size_t> next{0};
    std::mutex lock;
    std::exception_ptr thrown;
    const auto work = [&]() {
        try {
            State state;
            for (size_t p; (p = next.fetch_add(1)) < parts;) f(state, p);
        } catch (...) {
            std::lock_guard<std::mutex> hold(lock);
            thrown = std::current_exception();
            next = parts;
        }
    };
    struct Pool {
        std::thread thread[kMost];
        ~Pool() {
            for (std::thread &t : thread)
                if (t.joinable()) t.join();
        }
    };
    {
        Pool pool;
        try {
            for (size_t t = 1; t < threads; ++t) pool.thread[t] = std::thread(work);
        } catch (const std::system_error &) {
        } catch (const std::bad_alloc &) {
        }
        work();
    }
    if (thrown) std::rethrow_exception(thrown);
}

// Tree of maxima over the scores of n candidates, 8 children to a node: a node's children fill a cache line, n = 2^18 has 6
// levels, and the neighbouring candidates that a round changes share almost all of their nodes.  best() is the leftmost
// candidate with the largest score.  Scores are never NaN.
struct MaxTree {
    static constexpr int kWidth = 8;
    std::vector<std::vector<double>> level; // [0]: the scores; [l + 1][i] = the largest of [l][8 i .. 8 i + 7]
    size_t levels = 0;                      // of them in use (a tree is filled again and again, see pick)
    void reset(const double *S, int64_t n) {
        if (level.empty()) level.emplace_back();
        level[0].resize(padded(n));
        std::copy_n(S, n, level[0].data());
        std::fill(level[0].begin() + n, level[0].end(), kNegInf);
        build();
    }
    void take(std::vector<double> &&scores) { // (with room for the fill at their end)
        if (level.empty()) level.emplace_back();
        scores.resize(padded((int64_t)scores.size()), kNegInf);
        level[0] = std::move(scores);
        build();
    }
    void build() {
        levels = 1;
        while (level[levels - 1].size() > kWidth) {
            const size_t below = level[levels - 1].size() / kWidth;
            if (level.size() == levels) level.emplace_back();
            std::vector<double> &up = level[levels];
            const std::vector<double> &down = level[levels - 1];
            up.resize(padded((int64_t)below));
            for (size_t i = 0; i < below; ++i) up[i] = largest(&down[i * kWidth]);
            std::fill(up.begin() + (std::ptrdiff_t)below, up.end(), kNegInf);
            ++levels;
        }
    }
    static size_t padded(int64_t n) { return (size_t)((n + kWidth - 1) / kWidth * kWidth); }
#if defined(__SSE2__)
    static double largest(const double *v) {
        const __m128d a = _mm_max_pd(_mm_max_pd(_mm_loadu_pd(v), _mm_loadu_pd(v + 2)), _mm_max_pd(_mm_loadu_pd(v + 4), _mm_loadu_pd(v + 6)));
        return _mm_cvtsd_f64(_mm_max_sd(a, _mm_unpackhi_pd(a, a)));
    }
    static int first_equal(const double *v, double x) {
        const __m128d t = _mm_set1_pd(x);
        auto pair = [&](int i) { return (unsigned)_mm_movemask_pd(_mm_cmpeq_pd(_mm_loadu_pd(v + i), t)) << i; };
        return __builtin_ctz(pair(0) | pair(2) | pair(4) | pair(6) | 1u << (kWidth - 1));
    }
#else
    static double largest(const double *v) { return *std::max_element(v, v + kWidth); }
    static int first_equal(const double *v, double x) { return (int)std::min<std::ptrdiff_t>(std::find(v, v + kWidth, x) - v, kWidth - 1); }
#endif
    double &score(int64_t k) { return level[0][(size_t)k]; }
    double most() const { return largest(level[levels - 1].data()); }
    int64_t best(double x) const { // x = most()
        int64_t at = 0;
        for (size_t l = levels; l-- > 0;) at = at * kWidth + first_equal(&level[l][(size_t)at * kWidth], x);
        return at;
    }
    // The scores of candidates in the nodes lo .. hi of the lowest level (candidate / 8) have changed.
    void refresh(int64_t lo, int64_t hi) {
        for (size_t l = 0; l + 1 < levels; ++l) {
            bool changed = false;
            for (int64_t i = lo; i <= hi; ++i) {
                const double x = largest(&level[l][(size_t)i * kWidth]);
                double &old = level[l + 1][(size_t)i];
                changed |= !(x == old);
                old = x;
            }
            if (!changed) return;
            lo /= kWidth;
            hi /= kWidth;
        }
    }
};

// A round's changes, candidate by candidate: nodes next to each other are refreshed together.
struct Changes {
    MaxTree &tree;
    int64_t lo = 0, hi = -1;
    void add(int64_t k) {
        const int64_t i = k / MaxTree::kWidth;
        if (hi < lo) lo = hi = i;
        else if (i >= lo - 2 && i <= hi + 2) { lo = std::min(lo, i); hi = std::max(hi, i); }
        else { flush(); lo = hi = i; }
    }
    void flush() {
        if (hi >= lo) tree.refresh(lo, hi);
        lo = 0;
        hi = -1;
    }
};

// l1 norms of groups of bw weights of columns j0 .. j1 - 1 (of groups) of one row
template <class T, class Mag> void row_norms(const T *w, int32_t bw, int32_t n, double *out, Mag mag) {
    if (bw == 1) {
        for (int32_t j = 0; j < n; ++j) out[j] = mag(w[j]);
        return;
    }
    for (int32_t j = 0; j < n; ++j) {
        double s = 0.0;
        for (int32_t q = 0; q < bw; ++q) s += mag(w[(int64_t)j * bw + q]);
        out[j] = s;
    }
}

// The shrinking list of Algorithm 1: which of b entries are left, a bit each, with a bit per word above that says whether any
// is (32 KB in the first cache level for b = 2^18, where links between neighbours were 2 to 4 MB).
struct Remaining {
    std::vector<std::vector<uint64_t>> level;
    size_t levels = 0; // of them in use
    void reset(int64_t b) {
        levels = 0;
        do {
            if (level.size() == levels) level.emplace_back();
            std::vector<uint64_t> &words = level[levels++];
            words.assign((size_t)((b + 63) / 64), ~uint64_t(0));
            if (b % 64) words.back() = (uint64_t(1) << (b % 64)) - 1;
            b = (b + 63) / 64;
        } while (b > 1);
    }
    void remove(int64_t k) {
        for (size_t l = 0; l < levels; ++l) {
            uint64_t &w = level[l][(size_t)(k / 64)];
            w &= ~(uint64_t(1) << (k % 64));
            if (w) return;
            k /= 64;
        }
    }
    int64_t after(int64_t k) const { // -1: none
        for (size_t l = 0; l < levels; ++l, k /= 64) {
            if (k % 64 == 63) continue;
            const uint64_t w = level[l][(size_t)(k / 64)] & (~uint64_t(1) << (k % 64));
            if (!w) continue;
            k = k / 64 * 64 + __builtin_ctzll(w);
            while (l-- > 0) k = k * 64 + __builtin_ctzll(level[l][(size_t)k]);
            return k;
        }
        return -1;
    }
    int64_t before(int64_t k) const {
        for (size_t l = 0; l < levels; ++l, k /= 64) {
            const uint64_t w = level[l][(size_t)(k / 64)] & ((uint64_t(1) << (k % 64)) - 1);
            if (!w) continue;
            k = k / 64 * 64 + 63 - __builtin_clzll(w);
            while (l-- > 0) k = k * 64 + 63 - __builtin_clzll(level[l][(size_t)k]);
            return k;
        }
        return -1;
    }
};

// A round takes the candidate with the largest score, the leftmost of equal ones.
struct Taken {
    double score;
    int64_t k;
};

struct Workspace {
    MaxTree tree;
    Remaining list;
    std::vector<int64_t> right;
    std::vector<double> *own = nullptr; // the scores, where they are all of them and the caller has no more use for them: not copied (16 us of 160 for 49600)
    void fill(const double *S, int64_t n) {
        if (own) tree.take(std::move(*own));
        else tree.reset(S, n);
    }
};

// Rounds over the candidates first .. first + n - 1, appended to `out`: at most `most`, and none whose score lies below `bound`.
typedef void (*Rounds)(Workspace &w, const double *S, int64_t first, int64_t n, int32_t N, double bound, int64_t most, std::vector<Taken> &out);

// Expansion (Algorithm 1).
void expand(Workspace &w, const double *S, int64_t first, int64_t n, int32_t N, double bound, int64_t most, std::vector<Taken> &out) {
    MaxTree &tree = w.tree;
    Remaining &list = w.list;
    w.fill(S + first, n);
    list.reset(n);
    std::vector<int64_t> &right = w.right;
    right.resize((size_t)std::min<int64_t>(N, n));
    Changes changes{tree};
    for (int64_t got = 0; got < most; ++got) {
        const double top = tree.most();
        if (top == kNegInf || top < bound) break;
        const int64_t k = tree.best(top);
        // right[t] = the t-th entry after k in the list as it stands, for t < n_right
        int32_t n_right = 0;
        for (int64_t at = k; n_right < N && at >= 0; at = list.after(at)) right[(size_t)n_right++] = at;
        // the entry n places before k becomes the block made of the n weights before k's block
        // and the N-n weights after it
        int64_t left = k;
        for (int32_t t = 1; t < N; ++t) {
            left = list.before(left);
            if (left < 0) break;
            const double joined = N - t < n_right ? tree.score(right[(size_t)(N - t)]) : kNegInf;
            double &s = tree.score(left);
            // (Where two scores pass the largest double their difference to top does not: s, joined <= top.  An infinity would
            // make differences that have no order.)
            const double sum = s + joined;
            s = sum <= std::numeric_limits<double>::max() ? sum - top : ((0.25 * s + 0.25 * joined) - 0.25 * top) * 4.0;
            changes.add(left);
        }
        // k and the N-1 entries after it leave the list
        for (int32_t t = 0; t < n_right; ++t) {
            tree.score(right[(size_t)t]) = kNegInf;
            changes.add(right[(size_t)t]);
            list.remove(right[(size_t)t]);
        }
        changes.flush();
        out.push_back(Taken{top, first + k});
    }
}

void greedy(Workspace &w, const double *S, int64_t first, int64_t n, int32_t N, double bound, int64_t most, std::vector<Taken> &out) {
    MaxTree &tree = w.tree;
    w.fill(S + first, n);
    for (int64_t got = 0; got < most; ++got) {
        const double top = tree.most();
        if (top == kNegInf || top < bound) break;
        const int64_t k = tree.best(top);
        out.push_back(Taken{top, first + k});
        const int64_t lo = std::max<int64_t>(0, k - N + 1), hi = std::min<int64_t>(n - 1, k + N - 1);
        std::fill(&tree.score(lo), &tree.score(hi) + 1, kNegInf);
        tree.refresh(lo / MaxTree::kWidth, hi / MaxTree::kWidth);
    }
}

// Where each run of candidates that no round reaches out of begins, and b at the end.  N - 1 or more scores of -inf one
// after the other separate what lies before them from what lies behind:
//  * greedy shuts out N - 1 candidates to either side;
//  * in expansion a candidate with fewer than N - 1 others left between it and the end of its run has -inf: from the
//    beginning, and when a round brings one there, since what it is joined with has as few behind it.  So a block that is
//    taken leaves with entries of its own run, and those before the run that it would be joined with have -inf and keep it.
// (At least kLeast candidates to a run: aligned blocks would make one each.)
std::vector<int64_t> find_runs(const double *S, int64_t b, int32_t N) {
    constexpr int64_t kLeast = 128;
    std::vector<int64_t> first(1, 0);
    for (int64_t k = kLeast; k < b;) { // k: could begin a run
        int64_t at = k - 1;            // ... if the N - 1 scores before it are -inf
        while (at >= 0 && k - 1 - at < N - 1 && S[at] == kNegInf) --at;
        if (k - 1 - at >= N - 1) {
            first.push_back(k);
            k += kLeast;
        } else {
            k = at + N; // (behind the first score from there that is not -inf)
        }
    }
    first.push_back(b);
    return first;
}

// The m rounds over all candidates, in order.
//
// One run after the other, by several threads - its scores, its tree and its list then stay in the first cache level, where
// those of 2^18 candidates ask for lines of the second and third at every step - as far as its scores are at least a
// bound, which a sample of the runs gives with some to spare.  A round gives no candidate more than the score it takes, so
// that a run's scores never rise, and the m largest of all, in the order of the runs where they are equal, are what
// the rounds over all candidates take.
// A selection of 13107 blocks (512 x 512 in 4 x 1 blocks at 20 %, expansion, on 16 cores): 1.74 ms by one tree over all, 1.35 by
// runs in one thread (50 ns a round instead of 100), 1.02 in eight, scores in eight as well; one of 2048 x 512, 2 x 1, 50 %: 30 -> 11.6.
std::vector<Taken> pick(Rounds rounds, const double *S, int64_t b, int32_t N, int64_t m, std::vector<double> *own) {
    m = std::min(m, b); // (a share of any other would be out of range)
    std::vector<Taken> out;
    constexpr size_t kRuns = 16; // (fewer have no sample)
    constexpr int64_t kRounds = 4096; // (with fewer the sample and the threads cost what they save: 2900 rounds 485 us, by runs 567)
    const std::vector<int64_t> first = N >= 2 && m >= kRounds ? find_runs(S, b, N) : std::vector<int64_t>{0, b};
    const size_t runs = first.size() - 1;
    if (runs < kRuns) {
        Workspace w;
        w.own = own;
        out.reserve((size_t)std::min(m, b));
        rounds(w, S, 0, b, N, kNegInf, m, out);
        return out;
    }
    const size_t threads = (size_t)std::min<int64_t>(m / 1024, 64); // (a round: 50 ns)
    // the sample: a quarter of few runs, some 48 of many, spread so that nothing that comes back every so many runs is all there is
    // of it, each as far as twice its share of m
    const size_t samples = std::min<size_t>((runs + 3) / 4, 48);
    double share = 0.0;
    std::vector<double> sample;
    {
        std::vector<std::vector<Taken>> part(samples);
        std::vector<size_t> run(samples);
        for (size_t i = 0; i < samples; ++i) {
            run[i] = std::min(runs - 1, (size_t)((double)runs * std::fmod((double)(i + 1) * 0.6180339887498949, 1.0)));
            share += (double)m * (double)(first[run[i] + 1] - first[run[i]]) / (double)b;
        }
        share_out<Workspace>(samples, threads / 2, [&](Workspace &w, size_t i) {
            const int64_t n = first[run[i] + 1] - first[run[i]];
            rounds(w, S, first[run[i]], n, N, kNegInf, (int64_t)(2.0 * (double)m * (double)n / (double)b) + 8, part[i]);
        });
        for (const std::vector<Taken> &p : part)
            for (const Taken &t : p) sample.push_back(t.score);
    }
    const size_t parts = std::min<size_t>(runs, 64);
    std::vector<std::vector<Taken>> part(parts);
    for (double spare = 1.1;; spare *= 1.5) {
        const size_t at = (size_t)(spare * share) + 4;
        double bound = kNegInf;
        if (at < sample.size()) {
            std::nth_element(sample.begin(), sample.begin() + (std::ptrdiff_t)at, sample.end(), std::greater<double>());
            bound = sample[at];
        }
        share_out<Workspace>(parts, threads, [&](Workspace &w, size_t p) {
            part[p].clear();
            for (size_t r = runs * p / parts; r < runs * (p + 1) / parts; ++r) rounds(w, S, first[r], first[r + 1] - first[r], N, bound, m, part[p]);
        });
        size_t all = 0;
        for (const std::vector<Taken> &p : part) all += p.size();
        if ((int64_t)all < m && bound != kNegInf) continue;
        out.reserve(all);
        for (const std::vector<Taken> &p : part) out.insert(out.end(), p.begin(), p.end());
        break;
    }
    if ((int64_t)out.size() > m) { // the m largest, the first ones of equal scores
        std::vector<double> score(out.size());
        for (size_t t = 0; t < out.size(); ++t) score[t] = out[t].score;
        std::nth_element(score.begin(), score.begin() + (std::ptrdiff_t)(m - 1), score.end(), std::greater<double>());
        const double least = score[(size_t)(m - 1)];
        int64_t equal = m;
        for (const Taken &t : out) equal -= t.score > least;
        const auto out_of = [&](const Taken &t) { return t.score < least || (t.score == least && equal-- <= 0); };
        size_t n = 0;
        for (const Taken &t : out)
            if (!out_of(t)) out[n++] = t;
        out.resize(n);
    }
    return out;
}

// Expansion, then division (Algorithm 2).
int64_t expand_and_divide(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, std::vector<double> *own = nullptr) {
    if (b == 0 || m == 0) return 0;
    std::vector<uint64_t> kept((size_t)(b + 63) / 64, 0);
    for (const Taken &t : pick(expand, S, b, N, m, own)) kept[(size_t)t.k / 64] |= uint64_t(1) << (t.k % 64);
    int64_t got = 0;
    for (size_t w = 0; w < kept.size(); ++w)
        for (uint64_t bits = kept[w]; bits; bits &= bits - 1) I[got++] = (int64_t)(64 * w) + __builtin_ctzll(bits);
    int64_t next_idx = 0;
    for (int64_t at = 0; at < got; ++at) {
        const int64_t k = I[at];
        if (next_idx > k) { I[at] = next_idx; next_idx += N; }
        else { next_idx = k + N; }
    }
    return got;
}

int64_t greedy_in_order(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, std::vector<double> *own = nullptr) {
    if (b == 0 || m == 0) return 0;
    std::vector<Taken> all = pick(greedy, S, b, N, m, own);
    if (all.empty()) return 0;
    // (in order already where there was one run; else 8 bits of the scores at a time, from the lowest, keeps equal ones in the order of the runs)
    const auto key = [](double x) { // larger ones first; the same for zeros of either sign
        uint64_t u;
        x += 0.0;
        std::memcpy(&u, &x, 8);
        return u >> 63 ? u : ~u & ~(uint64_t(1) << 63);
    };
    const auto before = [](const Taken &x, const Taken &y) { return x.score > y.score; };
    if (!std::is_sorted(all.begin(), all.end(), before)) {
        std::vector<Taken> other(all.size());
        for (int shift = 0; shift < 64; shift += 8) {
            size_t count[256] = {0};
            for (const Taken &t : all) ++count[(key(t.score) >> shift) & 255];
            if (count[(key(all[0].score) >> shift) & 255] == all.size()) continue;
            size_t at = 0;
            for (size_t &c : count) at += std::exchange(c, at);
            for (const Taken &t : all) other[count[(key(t.score) >> shift) & 255]++] = t;
            all.swap(other);
        }
    }
    for (size_t t = 0; t < all.size(); ++t) I[t] = all[t].k;
    return (int64_t)all.size();
}

}  // namespace

extern "C" {

ubp_status ubp_block_scores(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t K, int32_t bh, int32_t bw,
                            int32_t aligned, double *S, int64_t b) {
    if (!layer_ok(W, dtype, ldw, M, K, bh, bw) || !S || b != (int64_t)M * (K / bw)) return UBP_ERR_INVALID_ARG;
    // Rows of W are read as they lie, kCols groups at a time, and the scores, which lie column by column, leave in pieces of
    // kRows (walking W down its columns took 2.9 ms for 512 x 512 in fp16, this 0.6).
    constexpr int32_t kCols = 64, kRows = 8;
    const int32_t groups = K / bw;
    struct Buffers {
        std::vector<double> norm; // of the rows' weights in some columns
        double part[kRows][kCols];
    };
    try {
        const int32_t cols = std::max(1, std::min(kCols, (1 << 17) / M)); // (at most 1 MB, or one column)
        const size_t threads = (size_t)std::min<int64_t>((int64_t)M * K / 32768, 64); // (a weight: about 1 ns)
        share_out<Buffers>((size_t)((groups + cols - 1) / cols), threads, [&](Buffers &buffers, size_t piece) {
            std::vector<double> &norm = buffers.norm;
            double(&part)[kRows][kCols] = buffers.part;
            norm.resize((size_t)M * (size_t)cols);
            const int32_t j0 = (int32_t)piece * cols;
            const int32_t n = std::min(cols, groups - j0);
            for (int32_t i = 0; i < M; ++i) {
                const int64_t at = (int64_t)i * ldw + (int64_t)j0 * bw;
                double *out = &norm[(size_t)i * (size_t)cols];
                switch (dtype) {
                case UBP_F32: row_norms(static_cast<const float *>(W) + at, bw, n, out, magnitude); break;
                case UBP_F16: row_norms(static_cast<const uint16_t *>(W) + at, bw, n, out, magnitude_f16); break;
                default: row_norms(static_cast<const uint16_t *>(W) + at, bw, n, out, magnitude_bf16); break;
                }
            }
            for (int32_t i0 = 0; i0 < M; i0 += kRows) {
                const int32_t rows = std::min(kRows, M - i0);
                for (int32_t r = 0; r < rows; ++r) {
                    const int32_t i = i0 + r;
                    if (i + bh > M || (aligned && i % bh)) {
                        std::fill_n(part[r], n, kNegInf);
                        continue;
                    }
                    const double *from = &norm[(size_t)i * (size_t)cols];
                    std::copy_n(from, n, part[r]);
                    for (int32_t t = 1; t < bh; ++t)
                        for (int32_t j = 0; j < n; ++j) part[r][j] += from[(size_t)t * (size_t)cols + (size_t)j];
                }
                for (int32_t j = 0; j < n; ++j)
                    for (int32_t r = 0; r < rows; ++r) S[(int64_t)(j0 + j) * M + i0 + r] = part[r][j];
            }
        });
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    } catch (const std::length_error &) {
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

ubp_status ubp_select_greedy(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, int64_t *count) {
    if (!selector_args_ok(S, b, N, m, I, count)) return UBP_ERR_INVALID_ARG;
    *count = 0;
    if (!scores_ok(S, b)) return UBP_ERR_INVALID_ARG;
    try {
        *count = greedy_in_order(S, b, N, m, I);
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    } catch (const std::length_error &) {
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

ubp_status ubp_select_bed(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, int64_t *count) {
    if (!selector_args_ok(S, b, N, m, I, count)) return UBP_ERR_INVALID_ARG;
    *count = 0;
    if (!scores_ok(S, b)) return UBP_ERR_INVALID_ARG;
    try {
        *count = expand_and_divide(S, b, N, m, I);
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    } catch (const std::length_error &) {
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

ubp_status ubp_select_optimal(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, int64_t *count) {
    if (!selector_args_ok(S, b, N, m, I, count)) return UBP_ERR_INVALID_ARG;
    *count = 0;
    if (!scores_ok(S, b)) return UBP_ERR_INVALID_ARG;
    if (m == 0) return UBP_OK;
    if (m > (b + N - 1) / N) return UBP_ERR_INFEASIBLE;
    const int64_t words = (m + 63) / 64;
    if ((long double)b * (long double)words * 8.0L > 2147483648.0L) return UBP_ERR_UNSUPPORTED;   // decision bits above 2 GiB
    try {
        std::vector<uint64_t> took((size_t)(b * words), 0);
        // rows k-N .. k of T, row k at slot k mod (N+1); T[k][0] = 0, T[<=0][n>0] = -inf
        const int64_t ring = (int64_t)N + 1;
        std::vector<double> T((size_t)(ring * (m + 1)), kNegInf);
        for (int64_t r = 0; r < ring; ++r) T[(size_t)(r * (m + 1))] = 0.0;
        for (int64_t k = 1; k <= b; ++k) {
            double *cur = &T[(size_t)((k % ring) * (m + 1))];
            const double *skip_row = &T[(size_t)(((k - 1) % ring) * (m + 1))];
            const double *take_row = k - N >= 1 ? &T[(size_t)(((k - N) % ring) * (m + 1))] : nullptr;
            // cells that can lie on a path to (b, m): n <= ceil(k / N) blocks fit before k, and the
            // m - n still missing must fit into the b - k candidates after it
            const int64_t n_hi = std::min<int64_t>(m, (k + N - 1) / N);
            const int64_t n_lo = std::max<int64_t>(1, m - (b - k + N - 1) / N);
            const double s = S[k - 1];
            uint64_t *bits = &took[(size_t)((k - 1) * words)];
            for (int64_t n = n_lo; n <= n_hi; ++n) {
                const double before = take_row ? take_row[n - 1] : (n == 1 ? 0.0 : kNegInf);
                const double take = before + s, skip = k > 1 ? skip_row[n] : kNegInf;
                if (take > skip) { cur[n] = take; bits[(n - 1) >> 6] |= 1ull << ((n - 1) & 63); }
                else cur[n] = skip;
            }
            if (n_hi < m) cur[n_hi + 1] = kNegInf;      // the one cell above the band that row k+1 reads
        }
        if (T[(size_t)((b % ring) * (m + 1) + m)] == kNegInf) return UBP_ERR_INFEASIBLE;
        int64_t k = b, n = m;
        while (n > 0 && k > 0) {
            if (took[(size_t)((k - 1) * words + ((n - 1) >> 6))] >> ((n - 1) & 63) & 1) { I[--n] = k - 1; k -= N; }
            else --k;
        }
        if (n != 0) return UBP_ERR_INFEASIBLE;
        *count = m;
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

ubp_status ubp_selection_to_blocks(const int64_t *I, int64_t count, int32_t M, int32_t bw, ubp_block *blocks) {
    if (count < 0 || (count > 0 && (!I || !blocks)) || M < 1 || bw < 1) return UBP_ERR_INVALID_ARG;
    for (int64_t at = 0; at < count; ++at) {
        if (I[at] < 0) return UBP_ERR_INVALID_ARG;
        const int64_t group = I[at] <= 0xffffffff ? (uint32_t)I[at] / (uint32_t)M : I[at] / M; // (a third of the time in 32 bits)
        if (group > std::numeric_limits<int32_t>::max() / bw) return UBP_ERR_INVALID_ARG;
        blocks[at].r = (int32_t)(I[at] - group * M);
        blocks[at].c = (int32_t)group * bw;
    }
    return UBP_OK;
}

ubp_status ubp_select_blocks(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t K, int32_t bh, int32_t bw,
                             double density, int32_t method, int32_t aligned, ubp_block *out, int64_t capacity,
                             int64_t *out_nb) {
    if (!layer_ok(W, dtype, ldw, M, K, bh, bw) || !out_nb || method < 0 || method > 2) return UBP_ERR_INVALID_ARG;
    *out_nb = 0;
    const int64_t m = ubp_target_block_count(M, K, bh, bw, density);
    if (m < 0) return UBP_ERR_INVALID_ARG;
    if (capacity < m || (m > 0 && !out)) { *out_nb = m; return UBP_ERR_INVALID_ARG; }
    try {
        const int64_t b = (int64_t)M * (K / bw);
        std::vector<double> S;
        S.reserve(MaxTree::padded(b));
        S.resize((size_t)b);
        std::vector<int64_t> I((size_t)std::max<int64_t>(m, 1));
        ubp_status rc = ubp_block_scores(W, dtype, ldw, M, K, bh, bw, aligned, S.data(), b);
        if (rc != UBP_OK) return rc;
        int64_t got = 0;
        if (method == 2) {
            rc = ubp_select_optimal(S.data(), b, bh, m, I.data(), &got);
            if (rc != UBP_OK) return rc;
        } else {
            if (!scores_ok(S.data(), b)) return UBP_ERR_INVALID_ARG;
            got = method == 0 ? greedy_in_order(S.data(), b, bh, m, I.data(), &S)
                              : expand_and_divide(S.data(), b, bh, m, I.data(), &S);
        }
        rc = ubp_selection_to_blocks(I.data(), got, M, bw, out);
        if (rc != UBP_OK) return rc;
        *out_nb = got;
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    } catch (const std::length_error &) {
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

ubp_status ubp_selection_efficacy(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t K, int32_t bh, int32_t bw,
                                  const ubp_block *ubp_blocks, int64_t nb, const ubp_block *abp_blocks, int64_t nb_abp,
                                  double *l1, double *efficacy) {
    if (!layer_ok(W, dtype, ldw, M, K, bh, bw) || nb < 0 || nb_abp < 0 || (nb && !ubp_blocks) || (nb_abp && !abp_blocks) ||
        !efficacy)
        return UBP_ERR_INVALID_ARG;
    try {
        auto kept = [&](const ubp_block *blocks, int64_t count, double *sum) -> ubp_status {
            std::vector<unsigned char> mark((size_t)M * (size_t)K, 0);
            for (int64_t at = 0; at < count; ++at) {
                const ubp_block o = blocks[at];
                if (o.r < 0 || o.c < 0 || o.r + bh > M || o.c + bw > K) return UBP_ERR_OUT_OF_BOUNDS;
                for (int32_t t = 0; t < bh; ++t)
                    std::memset(&mark[(size_t)(o.r + t) * K + o.c], 1, (size_t)bw);
            }
            double s = 0.0;
            for (int32_t i = 0; i < M; ++i)
                for (int32_t c = 0; c < K; ++c)
                    if (mark[(size_t)i * K + c]) s += element_magnitude(W, dtype, (int64_t)i * ldw + c);
            *sum = s;
            return UBP_OK;
        };
        double ubp = 0.0, abp = 0.0, ep = 0.0;
        ubp_status rc = kept(ubp_blocks, nb, &ubp);
        if (rc != UBP_OK) return rc;
        rc = kept(abp_blocks, nb_abp, &abp);
        if (rc != UBP_OK) return rc;
        // element-wise pruning keeps as many weights as the unaligned selection, the largest ones
        std::vector<double> mags((size_t)M * (size_t)K);
        for (int32_t i = 0; i < M; ++i)
            for (int32_t c = 0; c < K; ++c) mags[(size_t)i * K + c] = element_magnitude(W, dtype, (int64_t)i * ldw + c);
        const size_t keep = (size_t)std::min<int64_t>((int64_t)mags.size(), nb * bh * bw);
        std::partial_sort(mags.begin(), mags.begin() + (std::ptrdiff_t)keep, mags.end(), std::greater<double>());
        for (size_t at = 0; at < keep; ++at) ep += mags[at];
        if (l1) { l1[0] = ubp; l1[1] = abp; l1[2] = ep; }
        *efficacy = (ubp - abp) / (ep - abp);
    } catch (const std::bad_alloc &) {
        return UBP_ERR_ALLOC;
    }
    return UBP_OK;
}

}  // extern "C"
