// Block selection on the host: which m of a layer's b candidate blocks are kept (Sections 3.1,
// 3.2 and 4.1).  Scores (Eq. 1), the greedy selector (Eq. 3), the optimal selector (Eq. 4),
// block expansion and division (Algorithms 1 and 2) and the efficacy figure (Eq. 5).
//
// The selectors return what the paper's step-by-step descriptions return, but not by those
// steps where a faster route gives the same indices:
//   greedy   : the arg max comes from a tree of maxima (leftmost leaf wins a tie), so one of the m
//              rounds costs O(N + log b) instead of O(b);
//   expansion: the shrinking score list is a set of the original indices, its arg max from the same tree;
//   optimal  : Eq. 4's table row by row with one decision bit per cell and a walk back from
//              (b, m) instead of carrying index sets, cells that cannot lie on a path to (b, m)
//              left out: O(b m) time, b m bits.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <new>
#include <numeric>
#include <stdexcept>
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

// Tree of maxima over the scores of b candidates, 8 children to a node: a node's children fill a cache line, b = 2^18 has 6
// levels, and the neighbouring candidates that a round changes share almost all of their nodes (the binary tournament
// before, each leaf refreshed up 18 levels by itself, took 24 ms where this takes 5: expansion on 512 x 512 in 4 x 1
// blocks at 20 %).  best() is the leftmost leaf with the largest score.  Scores are never NaN.
struct MaxTree {
    static constexpr int kWidth = 8;
    std::vector<std::vector<double>> level; // [0]: the scores; [l + 1][i] = the largest of [l][8 i .. 8 i + 7]
    explicit MaxTree(std::vector<double> &&scores) {
        scores.resize(padded((int64_t)scores.size()), kNegInf); // (room for that: see copy_of)
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
    // -1 where only -inf is left
    int64_t best() const {
        const double x = most();
        if (x == kNegInf) return -1;
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
    explicit Remaining(int64_t b) {
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

// Expansion (Algorithm 1): the indices, ascending in I, and their number.
int64_t expand(std::vector<double> &&S, int32_t N, int64_t m, int64_t *I) {
    const int64_t b = (int64_t)S.size();
    Remaining list(b);
    std::vector<int64_t> right((size_t)std::min<int64_t>(N, b));
    std::vector<uint64_t> kept((size_t)(b + 63) / 64, 0);
    MaxTree tree(std::move(S));
    Changes changes{tree};
    int64_t got = 0;
    while (got < m) {
        const int64_t k = tree.best();
        if (k < 0) break;
        const double top = tree.score(k);
        // right[t] = the t-th entry after k in the list as it stands, for t < n_right
        int32_t n_right = 0;
        for (int64_t at = k; n_right < N && at >= 0; at = list.after(at)) right[(size_t)n_right++] = at;
        // the entry n places before k becomes the block made of the n weights before k's block
        // and the N-n weights after it
        int64_t left = k;
        for (int32_t n = 1; n < N; ++n) {
            left = list.before(left);
            if (left < 0) break;
            const double joined = N - n < n_right ? tree.score(right[(size_t)(N - n)]) : kNegInf;
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
        kept[(size_t)k / 64] |= uint64_t(1) << (k % 64);
        ++got;
    }
    int64_t at = 0;
    for (size_t w = 0; w < kept.size(); ++w)
        for (uint64_t bits = kept[w]; bits; bits &= bits - 1) I[at++] = (int64_t)(64 * w) + __builtin_ctzll(bits);
    return got;
}

// Expansion, then division (Algorithm 2).
int64_t expand_and_divide(std::vector<double> &&S, int32_t N, int64_t m, int64_t *I) {
    if (S.empty() || m == 0) return 0;
    const int64_t got = expand(std::move(S), N, m, I);
    int64_t next_idx = 0;
    for (int64_t at = 0; at < got; ++at) {
        const int64_t k = I[at];
        if (next_idx > k) { I[at] = next_idx; next_idx += N; }
        else { next_idx = k + N; }
    }
    return got;
}

int64_t greedy(std::vector<double> &&S, int32_t N, int64_t m, int64_t *I) {
    if (S.empty() || m == 0) return 0;
    const int64_t b = (int64_t)S.size();
    MaxTree tree(std::move(S));
    int64_t got = 0;
    while (got < m) {
        const int64_t k = tree.best();
        if (k < 0) break;
        I[got++] = k;
        const int64_t lo = std::max<int64_t>(0, k - N + 1), hi = std::min<int64_t>(b - 1, k + N - 1);
        std::fill(&tree.score(lo), &tree.score(hi) + 1, kNegInf);
        tree.refresh(lo / MaxTree::kWidth, hi / MaxTree::kWidth);
    }
    return got;
}

// Scores with room for the tree's fill at their end
std::vector<double> copy_of(const double *S, int64_t b) {
    std::vector<double> copy;
    copy.reserve(MaxTree::padded(b));
    copy.assign(S, S + b);
    return copy;
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
    try {
        const int32_t cols = std::max(1, std::min(kCols, (1 << 17) / M)); // (at most 1 MB, or one column)
        std::vector<double> norm((size_t)M * (size_t)cols); // of the rows' weights in these columns
        double part[kRows][kCols];
        for (int32_t j0 = 0; j0 < groups; j0 += cols) {
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
        }
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
        *count = greedy(copy_of(S, b), N, m, I);
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
        *count = expand_and_divide(copy_of(S, b), N, m, I);
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
        if (I[at] < 0 || I[at] / M > std::numeric_limits<int32_t>::max() / bw) return UBP_ERR_INVALID_ARG;
        blocks[at].r = (int32_t)(I[at] % M);
        blocks[at].c = (int32_t)(I[at] / M) * bw;
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
            got = method == 0 ? greedy(std::move(S), bh, m, I.data()) : expand_and_divide(std::move(S), bh, m, I.data());
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
