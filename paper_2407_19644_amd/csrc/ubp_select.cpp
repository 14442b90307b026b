// Block selection on the host: which m of a layer's b candidate blocks are kept (Sections 3.1,
// 3.2 and 4.1).  Scores (Eq. 1), the greedy selector (Eq. 3), the optimal selector (Eq. 4),
// block expansion and division (Algorithms 1 and 2) and the efficacy figure (Eq. 5).
//
// The selectors return what the paper's step-by-step descriptions return, but not by those
// steps where a faster route gives the same indices:
//   greedy   : the arg max comes from a tree of maxima (leftmost leaf wins a tie), so one of the m
//              rounds costs O(N + log b) instead of O(b), and where -inf separates columns from each other several threads go
//              through parts of them side by side, and what they give is merged;
//   expansion: the shrinking score list is a set of the original indices, its arg max from the same tree, by parts as well;
//   optimal  : Eq. 4's table row by row with one decision bit per cell and a walk back from
//              (b, m) instead of carrying index sets, cells that cannot lie on a path to (b, m)
//              left out: O(b m) time, b m bits.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <exception>
#include <limits>
#include <mutex>
#include <new>
#include <numeric>
#include <stdexcept>
#include <system_error>
#include <thread>
#include <type_traits>
#include <utility>
#include <vector>

#if defined(__linux__)
#include <sched.h>
#endif
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

// Waits for `done`, but not longer than a few times what a thread that sleeps takes to wake up.
template <class F> void spin(int us, F &&done) {
    const auto end = std::chrono::steady_clock::now() + std::chrono::microseconds(us);
    do {
        for (int i = 0; i < 16; ++i) {
            if (done()) return;
#if defined(__SSE2__)
            _mm_pause();
#endif
        }
    } while (std::chrono::steady_clock::now() < end);
}

// Those that this process may run on (std::thread::hardware_concurrency counts all of the machine's).
inline size_t usable_cores() {
#if defined(__linux__)
    cpu_set_t set;
    if (sched_getaffinity(0, sizeof set, &set) == 0) return (size_t)CPU_COUNT(&set);
#endif
    return std::thread::hardware_concurrency();
}

// Up to kMost threads for the length of one call, the caller among them.  A thread that cannot be had is done without.
class Team {
  public:
    explicit Team(size_t want, size_t cores = 0) { // (0: as many as there are)
        want = std::min(want, kMost);
        if (want > 1) threads = std::max<size_t>(1, std::min(want, cores ? cores : usable_cores()));
        start(1);
    }
    ~Team() { end(); }
    void end() { // the caller goes on alone
        {
            std::lock_guard<std::mutex> hold(lock);
            over = true;
            ++turn;
        }
        wake.notify_all();
        for (std::thread &t : thread) // (the ones that start others come before those)
            if (t.joinable()) t.join();
        threads = 1;
    }
    Team(const Team &) = delete;
    Team &operator=(const Team &) = delete;
    size_t size() const { return threads; }

    // f(part, member) for parts 0 .. parts - 1, each once, by the same thread as the last time where that one is not late: what a part
    // reads and writes is then in that core's caches (a line out of another core's takes 100 to 200 ns).  What one of them
    // throws is thrown here, after all have ended.  Behind the last ones the threads end by themselves (to be told costs 10 us).
    template <class F> void share(size_t parts, F &&f, bool last = false) {
        if (threads == 1 || parts < 2) {
            for (size_t p = 0; p < parts; ++p) f(p, 0);
            return;
        }
        typedef typename std::remove_reference<F>::type Body;
        {
            std::lock_guard<std::mutex> hold(lock);
            body = [](void *what, size_t p, size_t me) { (*static_cast<Body *>(what))(p, me); };
            with = const_cast<void *>(static_cast<const void *>(&f));
            for (size_t t = 0; t < size(); ++t) {
                share_of[t].next = parts * t / size();
                share_of[t].end = parts * (t + 1) / size();
            }
            open = true;
            over = last;
            ++turn;
        }
        wake.notify_all();
        work(0);
        spin(200, [this] { return inside == 0; });
        std::unique_lock<std::mutex> hold(lock);
        open = false; // (who wakes up only now has nothing left to do)
        done.wait(hold, [this] { return inside == 0; });
        if (thrown) std::rethrow_exception(std::exchange(thrown, nullptr));
    }

  private:
    static constexpr size_t kMost = 8;
    // A thread takes some 15 us to start, so that it starts the next ones by itself: 1 those from 2 on, 2 and 3 two each.
    void start(size_t t) {
        if (t >= threads) return;
        try {
            thread[t] = std::thread([this, t] { member(t); });
        } catch (const std::system_error &) {
        } catch (const std::bad_alloc &) {
        }
    }
    void member(size_t me) {
        start(2 * me);
        start(2 * me + 1);
        for (uint64_t seen = 0;;) {
            spin(50, [&] { return turn != seen; });
            std::unique_lock<std::mutex> hold(lock);
            wake.wait(hold, [&] { return turn != seen; });
            seen = turn;
            if (open) {
                ++inside;
                hold.unlock();
                work(me);
                hold.lock();
                if (--inside == 0) done.notify_one();
            }
            if (over) return;
        }
    }
    void work(size_t me) {
        try {
            for (size_t t = 0; t < size(); ++t) { // its own share, then what is left of the others'
                Share &s = share_of[(me + t) % size()];
                for (size_t p; (p = s.next.fetch_add(1)) < s.end;) body(with, p, me);
            }
        } catch (...) {
            std::lock_guard<std::mutex> hold(lock);
            thrown = std::current_exception();
            for (size_t t = 0; t < size(); ++t) share_of[t].next = share_of[t].end;
        }
    }
    struct alignas(64) Share {
        std::atomic<size_t> next{0};
        size_t end = 0;
    };
    Share share_of[kMost];
    std::mutex lock; // of what follows, but for reads while spinning
    std::condition_variable wake, done;
    std::atomic<uint64_t> turn{0}; // goes up with every share(), and at the end
    std::atomic<size_t> inside{0};
    size_t threads = 1;
    bool open = false, over = false;
    void (*body)(void *, size_t, size_t) = nullptr;
    void *with = nullptr;
    std::exception_ptr thrown;
    std::thread thread[kMost];
};

// Tree of maxima over the scores of n candidates, 8 children to a node: a node's children fill a cache line, n = 2^18 has 6
// levels, and the neighbouring candidates that a round changes share almost all of their nodes.  best() is the leftmost
// candidate with the largest score.  Scores are never NaN.
struct MaxTree {
    static constexpr int kWidth = 8;
    std::vector<std::vector<double>> level; // [0]: the scores; [l + 1][i] = the largest of [l][8 i .. 8 i + 7]
    void fill(std::vector<double> &&scores) { // (with room for the fill at their end)
        scores.resize(padded((int64_t)scores.size()), kNegInf);
        level.push_back(std::move(scores));
        while (level.back().size() > kWidth) level.emplace_back(padded((int64_t)(level.back().size() / kWidth)), kNegInf);
        for (size_t l = 0; l + 1 < level.size(); ++l)
            for (size_t i = 0; i < level[l].size() / kWidth; ++i) level[l + 1][i] = largest(&level[l][i * kWidth]);
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
    double most() const { return largest(level.back().data()); }
    int64_t best(double x) const { // x = most()
        int64_t at = 0;
        for (size_t l = level.size(); l-- > 0;) at = at * kWidth + first_equal(&level[l][(size_t)at * kWidth], x);
        return at;
    }
    // The scores of candidates in the nodes lo .. hi of the lowest level (candidate / 8) have changed.
    void refresh(int64_t lo, int64_t hi) {
        for (size_t l = 0; l + 1 < level.size(); ++l) {
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
    void fill(int64_t b) {
        do {
            level.emplace_back((size_t)((b + 63) / 64), ~uint64_t(0));
            if (b % 64) level.back().back() = (uint64_t(1) << (b % 64)) - 1;
            b = (b + 63) / 64;
        } while (b > 1);
    }
    void remove(int64_t k) {
        for (std::vector<uint64_t> &words : level) {
            uint64_t &w = words[(size_t)(k / 64)];
            w &= ~(uint64_t(1) << (k % 64));
            if (w) return;
            k /= 64;
        }
    }
    int64_t after(int64_t k) const { // -1: none
        for (size_t l = 0; l < level.size(); ++l, k /= 64) {
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
        for (size_t l = 0; l < level.size(); ++l, k /= 64) {
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

// Neighbouring candidates, which rounds go through: what is left of them and what has been taken, in order.
struct Part {
    MaxTree tree;
    Remaining list;
    std::vector<int64_t> right;
    int64_t first = 0, n = 0;
    std::vector<Taken> taken;
    void fill(std::vector<double> &&scores) { // (with room for the fill at their end)
        n = (int64_t)scores.size();
        tree.fill(std::move(scores));
    }
};

// Up to `most` rounds whose scores lie above `above`.  False: there may be more.
typedef bool (*Rounds)(Part &part, int32_t N, double above, int64_t most);

// Expansion (Algorithm 1).
bool expand(Part &part, int32_t N, double above, int64_t most) {
    MaxTree &tree = part.tree;
    Remaining &list = part.list;
    std::vector<int64_t> &right = part.right;
    if (list.level.empty()) {
        list.fill(part.n);
        right.resize((size_t)std::min<int64_t>(N, part.n));
    }
    Changes changes{tree};
    for (int64_t got = 0; got < most; ++got) {
        const double top = tree.most();
        if (!(top > above)) return true;
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
        part.taken.push_back(Taken{top, part.first + k});
    }
    return false;
}

bool greedy(Part &part, int32_t N, double above, int64_t most) {
    MaxTree &tree = part.tree;
    for (int64_t got = 0; got < most; ++got) {
        const double top = tree.most();
        if (!(top > above)) return true;
        const int64_t k = tree.best(top);
        part.taken.push_back(Taken{top, part.first + k});
        const int64_t lo = std::max<int64_t>(0, k - N + 1), hi = std::min<int64_t>(part.n - 1, k + N - 1);
        std::fill(&tree.score(lo), &tree.score(hi) + 1, kNegInf);
        tree.refresh(lo / MaxTree::kWidth, hi / MaxTree::kWidth);
    }
    return false;
}

// Threads that go through parts side by side: where there are fewer, or fewer rounds, one goes through all candidates.
constexpr size_t kLeastTeam = 4;
constexpr int64_t kLeastRounds = 4096;
size_t threads_for_rounds(int64_t m) {
    if (m < kLeastRounds || usable_cores() < kLeastTeam) return 1;
    return (size_t)std::min<int64_t>(m / 1024, 64);
}

// Where to cut b candidates into up to `most` parts that no round reaches out of, some b / most each.  N - 1 or more scores of
// -inf one after the other separate what lies before them from what lies behind:
//  * greedy shuts out N - 1 candidates to either side;
//  * in expansion a candidate with fewer than N - 1 others left between it and the end of its part has -inf: from the
//    beginning, and when a round brings one there, since what it is joined with has as few behind it.  So a block that is
//    taken leaves with entries of its own part, and those before the part that it would be joined with have -inf and keep it.
std::vector<int64_t> cuts(const double *S, int64_t b, int32_t N, int64_t most) {
    std::vector<int64_t> first(1, 0);
    for (int64_t p = 1; p < most; ++p) {
        const int64_t from = b / most * p, to = from + b / most;
        int64_t at = from, gone = 0; // scores of -inf right before at
        while (gone < N - 1 && gone < from && S[from - 1 - gone] == kNegInf) ++gone;
        for (; gone < N - 1 && at < to; ++at) gone = S[at] == kNegInf ? gone + 1 : 0;
        if (gone >= N - 1 && at < to) first.push_back(at);
    }
    first.push_back(b);
    return first;
}

// The scores that part p has taken lie above x before this one.
inline std::vector<Taken>::const_iterator above(const Part &p, double x) {
    return std::partition_point(p.taken.begin(), p.taken.end(), [x](const Taken &t) { return t.score > x; });
}

inline double below(double x) { return std::nextafter(x, kNegInf); }

// The m rounds over all candidates: what they take, part by part, in order within each.
//
// The rounds over a part take what those over all candidates take of it, in the same order, and a round gives no candidate
// more than the score it takes, so that the scores that are taken never rise: what all rounds take is the m largest of what the
// parts give, those of earlier parts where they are equal.  So parts are gone through side by side, all down to the same
// score, then to a lower one, until m are taken.  The scores to stop at are those of a sample of the candidates: a block has a
// candidate's score or less, so that there are at most as many blocks above a score as candidates, and how many there
// have been so far says where m will be reached.  Equal scores at the last of them are taken in order.
// When m / 8 more than m have been made the bound was too low for parts that came first, and the m-th score so far takes its
// place.  Whatever the scores are there are 2.2 m rounds at most; 1.0 to 1.1 m where columns differ by any smooth law or many have no
// weight, up to 1.4 m where a few of them are a hundred times the others.
//
// 512 x 512 in 4 x 1 blocks at 20 % (13107 rounds) with scores, by one tree -> by parts on 16 cores: rows of different size, greedy 1.56 -> 0.8,
// expansion 1.74 -> 0.7 ms; columns of different size (log-normal, sigma 2) 1.45 -> 0.75 and 1.65 -> 0.7; four columns in five zero 1.25
// -> 0.8 and 1.6 -> 0.7; all zero 0.82 -> 0.8.  1024 x 512, 2 x 1, 2 %, sigma 2: 1.1 -> 0.9, 1.15 -> 0.85.  On 4 cores the first two 1.57 -> 0.87, 1.73
// -> 0.74; on 3, with 4259 rounds, up to 1.3 times one tree's time, which is why kLeastTeam is 4.  Slower are small layers without a
// weight, whose rounds are made in order all the same: 1024 x 64, 9830 rounds, 0.34 -> 0.5.
std::vector<Part> pick(Rounds rounds, const double *S, int64_t b, int32_t N, int64_t m, std::vector<double> *own, Team &team) {
    constexpr int64_t kParts = 64;
    constexpr double kSamples = 128.0; // among the m best candidates
    constexpr std::ptrdiff_t kEqual = 3; // (2 % of m)
    m = std::min(m, b);
    std::vector<int64_t> first(1, 0);
    if (team.size() >= kLeastTeam && m >= kLeastRounds) first = cuts(S, b, N, std::min<int64_t>(kParts, b / 1024));
    else first.push_back(b);
    const size_t parts = first.size() - 1;
    std::vector<Part> part(parts);
    if (parts < 2) {
        std::vector<double> copy;
        if (!own) {
            copy.reserve(MaxTree::padded(b));
            copy.assign(S, S + b);
        }
        part[0].taken.reserve((size_t)m);
        part[0].fill(std::move(own ? *own : copy));
        rounds(part[0], N, kNegInf, m);
        return part;
    }
    const double per_sample = std::max(1.0, (double)m / kSamples); // candidates
    std::vector<size_t> from(parts + 1, 0);
    for (size_t p = 0; p < parts; ++p) from[p + 1] = from[p] + (size_t)((double)(first[p + 1] - first[p]) / per_sample);
    std::vector<double> sample(from[parts]);
    team.share(parts, [&](size_t p, size_t) {
        Part &here = part[p];
        const double *scores = S + first[p];
        const int64_t n = first[p + 1] - first[p];
        double at = 0.5;
        for (size_t i = from[p]; i < from[p + 1]; ++i) { // spread so that nothing that comes back every so many candidates is all there is of it
            at += 0.6180339887498949;
            at -= at >= 1.0;
            sample[i] = scores[std::min(n - 1, (int64_t)(at * (double)n))];
        }
        std::vector<double> copy;
        copy.reserve(MaxTree::padded(n));
        copy.assign(scores, scores + n);
        here.first = first[p];
        here.fill(std::move(copy));
    });
    const auto taken = [&] {
        int64_t all = 0;
        for (const Part &p : part) all += (int64_t)p.taken.size();
        return all;
    };
    // every part down to `bound`; false: `most` rounds have been made before
    const auto walk = [&](double bound, int64_t most) {
        constexpr int64_t kChunk = 32;
        std::atomic<int64_t> left{most};
        std::atomic<bool> all{true};
        team.share(parts, [&](size_t p, size_t) {
            for (;;) {
                if (left.fetch_sub(kChunk) <= 0) {
                    if (part[p].tree.most() > bound) all = false;
                    return;
                }
                const size_t before = part[p].taken.size();
                const bool end = rounds(part[p], N, bound, kChunk);
                left += kChunk - (int64_t)(part[p].taken.size() - before);
                if (end) return;
            }
        });
        return all.load();
    };
    // the m-th largest of the scores taken, of which fewer than m lie above `sure`
    const auto mth = [&](double sure) {
        std::vector<double> rest;
        int64_t nth = m;
        for (const Part &p : part) {
            auto t = above(p, sure);
            nth -= t - p.taken.begin();
            for (; t != p.taken.end(); ++t) rest.push_back(t->score);
        }
        std::nth_element(rest.begin(), rest.begin() + (std::ptrdiff_t)(nth - 1), rest.end(), std::greater<double>());
        return rest[(size_t)(nth - 1)];
    };
    // All above `score` are taken: those equal to it, as far as m asks for them.  True: m are taken.
    const auto take_equal = [&](double score) {
        int64_t want = m;
        for (const Part &p : part) want -= above(p, score) - p.taken.begin();
        for (size_t p = 0; p < parts && want > 0; ++p) {
            want -= above(part[p], below(score)) - above(part[p], score);
            if (want <= 0) break;
            const size_t before = part[p].taken.size();
            rounds(part[p], N, below(score), want);
            want -= (int64_t)(part[p].taken.size() - before);
        }
        return want <= 0;
    };
    double bound = std::numeric_limits<double>::infinity(); // all above it are taken, `have` of them
    size_t rank = 0, step = (size_t)kSamples;               // of the bound among the sample, and how much lower the next one is
    double slope = 0.0;                                     // blocks that a sample further down has brought
    for (int64_t have = 0;;) {
        double next = kNegInf;
        if (rank + step < sample.size()) {
            const auto begin = sample.begin() + (std::ptrdiff_t)rank, at = begin + (std::ptrdiff_t)step;
            std::nth_element(begin, at, sample.end(), std::greater<double>());
            next = *at;
        }
        if (next == bound || std::count(sample.begin() + (std::ptrdiff_t)rank, sample.end(), bound) > kEqual) {
            if (take_equal(bound)) break;
            have = taken();
            sample.erase(std::remove(sample.begin() + (std::ptrdiff_t)rank, sample.end(), bound), sample.end());
        } else {
            bool end = walk(next, m - have + m / 8);
            while (!end && taken() < m) end = walk(next, m / 8);
            const int64_t now = taken();
            if (!end) {
                next = mth(bound);
                walk(next, std::numeric_limits<int64_t>::max() / 2);
                take_equal(next);
                break;
            }
            if (now >= m || next == kNegInf) break;
            rank += step;
            slope = (double)(now - have) / (double)step;
            have = now;
            bound = next;
        }
        // a little short of m while that is far, then a little beyond; and while it is far as if a sample brought half of what it has on
        // the whole, since what comes may be unlike what came last (a few heavy columns, all taken)
        const double still = (double)(m - have);
        const bool far = 4 * still > (double)m;
        const double least = far ? 0.5 * (double)have / (double)std::max<size_t>(rank, 1) : 0.0;
        step = (size_t)std::max(1.0, std::min(4.0 * (double)(rank + kEqual), (far ? 0.9 * still : still + (double)m / 64) / std::max({slope, least, 1e-3})));
    }
    if (taken() > m) {
        const double least = mth(bound);
        int64_t equal = m;
        for (const Part &p : part) equal -= above(p, least) - p.taken.begin();
        for (Part &p : part) {
            const int64_t more = above(p, least) - p.taken.begin(), all = above(p, below(least)) - p.taken.begin();
            const int64_t kept = std::min(all - more, equal);
            equal -= kept;
            p.taken.resize((size_t)(more + kept));
        }
    }
    return part;
}

// Expansion, then division (Algorithm 2).
int64_t expand_and_divide(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, std::vector<double> *own, Team &team) {
    if (b == 0 || m == 0) return 0;
    std::vector<uint64_t> kept((size_t)(b + 63) / 64, 0);
    for (const Part &p : pick(expand, S, b, N, m, own, team))
        for (const Taken &t : p.taken) kept[(size_t)t.k / 64] |= uint64_t(1) << (t.k % 64);
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

int64_t greedy_in_order(const double *S, int64_t b, int32_t N, int64_t m, int64_t *I, std::vector<double> *own, Team &team) {
    if (b == 0 || m == 0) return 0;
    const std::vector<Part> part = pick(greedy, S, b, N, m, own, team);
    if (part.size() == 1) {
        for (size_t t = 0; t < part[0].taken.size(); ++t) I[t] = part[0].taken[t].k;
        return (int64_t)part[0].taken.size();
    }
    // The parts' are in order: a range of scores at a time, cut at scores that are taken about as often.
    constexpr size_t kRanges = 32, kFromEach = 16;
    std::vector<double> edge;
    for (const Part &p : part)
        for (size_t i = 0; i < kFromEach && !p.taken.empty(); ++i) edge.push_back(p.taken[p.taken.size() * i / kFromEach].score);
    if (edge.empty()) return 0;
    std::sort(edge.begin(), edge.end(), std::greater<double>());
    team.share(kRanges, [&](size_t r, size_t) {
        const double from = r == 0 ? std::numeric_limits<double>::infinity() : edge[edge.size() * r / kRanges];
        const double to = r + 1 == kRanges ? kNegInf : edge[edge.size() * (r + 1) / kRanges];
        std::vector<Taken> here;
        int64_t *out = I;
        for (const Part &p : part) {
            const auto begin = above(p, from), end = above(p, to);
            out += begin - p.taken.begin();
            here.insert(here.end(), begin, end);
        }
        const auto before = [](const Taken &x, const Taken &y) { return x.score > y.score || (x.score == y.score && x.k < y.k); };
        if (!std::is_sorted(here.begin(), here.end(), before)) std::sort(here.begin(), here.end(), before);
        for (size_t t = 0; t < here.size(); ++t) out[t] = here[t].k;
    });
    int64_t got = 0;
    for (const Part &p : part) got += (int64_t)p.taken.size();
    return got;
}

// The scores of n groups of columns from j0 on.  Rows of W are read as they lie, and the scores, which lie column by column,
// leave in pieces of kRows (walking W down its columns took 2.9 ms for 512 x 512 in fp16, this 0.6).
constexpr int32_t kScoreCols = 64;
void scores_of(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t bh, int32_t bw, int32_t aligned, int32_t j0, int32_t n,
               std::vector<double> &norm, double *S) {
    constexpr int32_t kRows = 8;
    double part[kRows][kScoreCols];
    norm.resize((size_t)M * (size_t)n); // of the rows' weights in these columns
    for (int32_t i = 0; i < M; ++i) {
        const int64_t at = (int64_t)i * ldw + (int64_t)j0 * bw;
        double *out = &norm[(size_t)i * (size_t)n];
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
            const double *from = &norm[(size_t)i * (size_t)n];
            std::copy_n(from, n, part[r]);
            for (int32_t t = 1; t < bh; ++t)
                for (int32_t j = 0; j < n; ++j) part[r][j] += from[(size_t)t * (size_t)n + (size_t)j];
        }
        for (int32_t j = 0; j < n; ++j)
            for (int32_t r = 0; r < rows; ++r) S[(int64_t)(j0 + j) * M + i0 + r] = part[r][j];
    }
}

int32_t score_cols(int32_t M) { return std::max(1, std::min(kScoreCols, (1 << 17) / M)); } // (at most 1 MB of norms, or one column)
size_t score_pieces(int32_t M, int32_t K, int32_t bw) { return ((size_t)(K / bw) + (size_t)score_cols(M) - 1) / (size_t)score_cols(M); }
size_t threads_for_scores(int32_t M, int32_t K, int32_t bw) { // (a weight: about 1 ns)
    return std::min((size_t)std::min<int64_t>((int64_t)M * K / 32768, 64), score_pieces(M, K, bw));
}

void block_scores(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t K, int32_t bh, int32_t bw, int32_t aligned, double *S,
                  Team &team, bool last) {
    const int32_t groups = K / bw, cols = score_cols(M);
    std::vector<std::vector<double>> norms(team.size());
    const auto score = [&](size_t piece, size_t member) {
        const int32_t j0 = (int32_t)piece * cols;
        scores_of(W, dtype, ldw, M, bh, bw, aligned, j0, std::min(cols, groups - j0), norms[member], S);
    };
    team.share(score_pieces(M, K, bw), score, last);
}

}  // namespace

extern "C" {

ubp_status ubp_block_scores(const void *W, ubp_dtype dtype, int64_t ldw, int32_t M, int32_t K, int32_t bh, int32_t bw,
                            int32_t aligned, double *S, int64_t b) {
    if (!layer_ok(W, dtype, ldw, M, K, bh, bw) || !S || b != (int64_t)M * (K / bw)) return UBP_ERR_INVALID_ARG;
    try {
        Team team(threads_for_scores(M, K, bw));
        block_scores(W, dtype, ldw, M, K, bh, bw, aligned, S, team, true);
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
        Team team(threads_for_rounds(m));
        *count = greedy_in_order(S, b, N, m, I, nullptr, team);
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
        Team team(threads_for_rounds(m));
        *count = expand_and_divide(S, b, N, m, I, nullptr, team);
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
        const size_t for_rounds = method == 2 ? 1 : threads_for_rounds(m);
        Team team(std::max(threads_for_scores(M, K, bw), for_rounds));
        block_scores(W, dtype, ldw, M, K, bh, bw, aligned, S.data(), team, for_rounds == 1);
        if (for_rounds == 1) team.end();
        ubp_status rc = UBP_OK;
        int64_t got = 0;
        if (method == 2) {
            rc = ubp_select_optimal(S.data(), b, bh, m, I.data(), &got);
            if (rc != UBP_OK) return rc;
        } else {
            if (!scores_ok(S.data(), b)) return UBP_ERR_INVALID_ARG;
            got = method == 0 ? greedy_in_order(S.data(), b, bh, m, I.data(), &S, team)
                              : expand_and_divide(S.data(), b, bh, m, I.data(), &S, team);
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
