// Selection metrics and baselines over problems (section "Selection Regret
// (The Target Metric)"; baselines of section "Final Fit and Test Protocol").
//
// Per-problem passes read each segment once (one workgroup per problem);
// the aggregates are exact order statistics and fixed-order binary64 sums
// over at most a few hundred thousand problems.
#include <limits.h>

#include <mutex>

#include "internal.hpp"

namespace hwsel {
namespace {

constexpr int kEvalThreads = 512;

// Strictly faster runtime; NaN is slower than everything, +inf included.
__device__ __forceinline__ bool faster(float a, float b)
{
    const bool na = a != a, nb = b != b;
    if (na || nb) return !na && nb;
    return a < b;
}

// y = t_best / t: 1 for equal runtimes (inf included), 0 for NaN.
__device__ __forceinline__ double y_of(float t_best, float t)
{
    if (t == t_best) return 1.0;
    if (t != t) return 0.0;
    return (double)t_best / (double)t;
}

// Runtimes in flight per thread: a pass over a problem is bound by the latency
// of its loads.  600 problems of 8,192 rows on average: 26 us with 256 threads
// and one in flight, 17 us with 512 and eight.
constexpr int kEvalLoads = 8;

// Runtimes of rows j, j + blockDim.x, ... < n (NaN past the end), a step's
// loads all requested before the first is used.
template <class F>
__device__ __forceinline__ void each_runtime(const float *__restrict__ rt, int64_t base, int64_t n, F &&visit)
{
    for (int64_t j0 = threadIdx.x; j0 < n; j0 += kEvalLoads * kEvalThreads) {
        float t[kEvalLoads];
#pragma unroll
        for (int i = 0; i < kEvalLoads; ++i) {
            const int64_t j = j0 + i * kEvalThreads;
            t[i] = rt[base + (j < n ? j : n - 1)];
        }
#pragma unroll
        for (int i = 0; i < kEvalLoads; ++i)
            if (j0 + i * kEvalThreads < n) visit(t[i]);
    }
}

// Fastest runtime of rows [base, base + n) for a whole workgroup.
__device__ float block_fastest(const float *__restrict__ rt, int64_t base, int64_t n, float *red)
{
    float best = __builtin_nanf("");
    each_runtime(rt, base, n, [&](float t) {
        if (faster(t, best)) best = t;
    });
    for (int off = 32; off > 0; off >>= 1) {
        const float o = __shfl_xor(best, off);
        if (faster(o, best)) best = o;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = best;
    __syncthreads();
    best = red[0];
    for (int w = 1; w < kEvalThreads / 64; ++w)
        if (faster(red[w], best)) best = red[w];
    return best;
}

__global__ __launch_bounds__(kEvalThreads) void k_eval_groups(const float *__restrict__ rt,
                                                              const int64_t *__restrict__ seg, int32_t P,
                                                              const int32_t *__restrict__ idx, int32_t k,
                                                              double *__restrict__ regret, int32_t *__restrict__ rank,
                                                              double *__restrict__ ybar)
{
    __shared__ float red[kEvalThreads / 64];
    __shared__ double wave_y[kEvalThreads / 64];
    __shared__ int64_t wave_n[kEvalThreads / 64];
    const int32_t p = blockIdx.x;
    if (p >= P) return;                                   // one workgroup per problem
    const int64_t base = seg[p], n = seg[p + 1] - seg[p];
    if (n <= 0) {
        if (threadIdx.x == 0) {
            regret[p] = __builtin_nan("");
            rank[p] = 0;
            ybar[p] = __builtin_nan("");
        }
        return;
    }
    const float t_best = block_fastest(rt, base, n, red);
    const int32_t sel = idx[(int64_t)p * k];
    const bool counted = sel >= 0 && sel < n;
    const float t_sel = counted ? rt[base + sel] : 0.0f;
    double ys = 0.0;
    int64_t nb = 0;
    each_runtime(rt, base, n, [&](float t) {
        ys += y_of(t_best, t);
        nb += faster(t, t_sel) ? 1 : 0;
    });
    // a fixed tree within the waves, then the waves in order
    for (int off = 32; off > 0; off >>= 1) {
        ys += __shfl_xor(ys, off);
        nb += __shfl_xor(nb, off);
    }
    if ((threadIdx.x & 63) == 0) {
        wave_y[threadIdx.x >> 6] = ys;
        wave_n[threadIdx.x >> 6] = nb;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kEvalThreads / 64; ++w) {
            ys += wave_y[w];
            nb += wave_n[w];
        }
    if (threadIdx.x == 0) {
        ybar[p] = ys / (double)n;
        regret[p] = counted ? 1.0 - y_of(t_best, t_sel) : __builtin_nan("");
        rank[p] = counted ? (int32_t)(1 + nb) : 0;
    }
}

// Order statistics of the counted regrets by radix selection: for each
// requested rank, eight passes over the 64-bit keys (an order-preserving map
// of the binary64 values), one byte per pass from the top, each counting the
// candidates that still match the prefix.  Linear in P per pass; the counts
// are integers, so the result is exact and independent of scheduling.
// stats[i] = the value of rank ranks[i] (0-based) among the counted regrets,
// for the ranks of the median and the 95th percentile.
__device__ __forceinline__ uint64_t order_key(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}

__device__ __forceinline__ double key_value(uint64_t k)
{
    return __builtin_bit_cast(double, (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k);
}

constexpr int kSelectThreads = 1024;

__global__ __launch_bounds__(kSelectThreads) void k_eval_select(const double *__restrict__ regret,
                                                                const int32_t *__restrict__ rank, int32_t P,
                                                                double *__restrict__ stats)
{
    __shared__ int64_t hist[256];
    __shared__ int64_t cnt_s;
    __shared__ uint64_t prefix_s;
    __shared__ int64_t k_s;
    // number of counted problems
    if (threadIdx.x == 0) cnt_s = 0;
    __syncthreads();
    int64_t local = 0;
    for (int32_t i = threadIdx.x; i < P; i += kSelectThreads) local += rank[i] != 0;
    atomicAdd(reinterpret_cast<unsigned long long *>(&cnt_s), (unsigned long long)local);
    __syncthreads();
    const int64_t n = cnt_s;
    if (n == 0) return;
    // ranks: floor and ceil positions of q (n - 1) for q = 0.5, 0.95
    int64_t want[4];
    {
        const double p50 = 0.5 * (double)(n - 1), p95 = 0.95 * (double)(n - 1);
        const int64_t l50 = (int64_t)__builtin_floor(p50), l95 = (int64_t)__builtin_floor(p95);
        want[0] = l50;
        want[1] = l50 + 1 < n ? l50 + 1 : n - 1;
        want[2] = l95;
        want[3] = l95 + 1 < n ? l95 + 1 : n - 1;
    }
    for (int t = 0; t < 4; ++t) {
        uint64_t prefix = 0, mask = 0;
        int64_t k = want[t];
        for (int shift = 56; shift >= 0; shift -= 8) {
            for (int b = threadIdx.x; b < 256; b += kSelectThreads) hist[b] = 0;
            __syncthreads();
            for (int32_t i = threadIdx.x; i < P; i += kSelectThreads) {
                if (rank[i] == 0) continue;
                const uint64_t key = order_key(regret[i]);
                if ((key & mask) == prefix)
                    atomicAdd(reinterpret_cast<unsigned long long *>(&hist[(key >> shift) & 255u]), 1ull);
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                int64_t acc = 0;
                int d = 0;
                for (; d < 255; ++d) {
                    if (acc + hist[d] > k) break;
                    acc += hist[d];
                }
                k_s = k - acc;
                prefix_s = prefix | ((uint64_t)d << shift);
            }
            __syncthreads();
            prefix = prefix_s;
            k = k_s;
            mask |= 0xffull << shift;
            __syncthreads();
        }
        if (threadIdx.x == 0) stats[t] = key_value(prefix);
    }
}

// value at position q (n - 1) by linear interpolation between its two
// neighbouring order statistics
__device__ double interpolate(double lo_v, double hi_v, int64_t n, double q)
{
    const double pos = q * (double)(n - 1);
    const double lo = __builtin_floor(pos);
    return lo_v + (pos - lo) * (hi_v - lo_v);
}

__global__ void k_eval_aggregate(const double *__restrict__ regret, const int32_t *__restrict__ rank,
                                 const double *__restrict__ ybar, const double *__restrict__ stats, int32_t P,
                                 double *__restrict__ out, double *__restrict__ regret_out,
                                 int32_t *__restrict__ rank_out, double *__restrict__ ybar_out)
{
    if (threadIdx.x == 0) {
        int64_t cnt = 0, top1 = 0, top5 = 0, w5 = 0;
        double sum = 0.0, rsum = 0.0, mx = -__builtin_inf();
        for (int32_t p = 0; p < P; ++p) {
            if (rank[p] == 0) continue;
            const double r = regret[p];
            ++cnt;
            sum += r;
            rsum += 1.0 - ybar[p];
            mx = r > mx ? r : mx;
            top1 += rank[p] == 1;
            top5 += rank[p] <= 5;
            w5 += r <= 0.05;
        }
        if (cnt == 0) {
            for (int i = 0; i < 8; ++i) out[i] = __builtin_nan("");
            out[8] = 0.0;
        } else {
            out[0] = sum / (double)cnt;
            out[1] = interpolate(stats[0], stats[1], cnt, 0.5);
            out[2] = interpolate(stats[2], stats[3], cnt, 0.95);
            out[3] = mx;
            out[4] = (double)top1 / (double)cnt;
            out[5] = (double)top5 / (double)cnt;
            out[6] = (double)w5 / (double)cnt;
            out[7] = rsum / (double)cnt;
            out[8] = (double)cnt;
        }
    }
    for (int32_t p = threadIdx.x; p < P; p += blockDim.x) {
        if (regret_out) regret_out[p] = regret[p];
        if (rank_out) rank_out[p] = rank[p];
        if (ybar_out) ybar_out[p] = ybar[p];
    }
}

// Up to kSmallP problems: one workgroup stages the per-problem values in LDS,
// then its waves work side by side: waves 0 and 1 each select the two order
// statistics around one quantile, wave 2 takes the two sums in problem order,
// both before the outputs.  The same outputs as k_eval_select +
// k_eval_aggregate.  Bound by latency; P = 600: 15 us (46 us with a bitonic
// sort of the regrets and the sums taken from broadcast lanes).
constexpr int kSmallP = 4096;
constexpr int kSmallT = 1024, kSmallM = kSmallP / kSmallT;

__device__ __forceinline__ uint64_t wave_min(uint64_t v)
{
    for (int off = 32; off > 0; off >>= 1) {
        const uint64_t o = __shfl_xor((unsigned long long)v, off);
        v = o < v ? o : v;
    }
    return v;
}

// The values of ranks k and k + 1 (k + 1 < n, or k twice) among the n keys
// below ~0 of key[0, m), m a multiple of 256, by one wave: the k-th key is the
// largest v that at most k keys lie below, found bit by bit from the top; a
// count is a ballot per 64 keys.  The search ends as soon as exactly k keys
// lie below v (the k-th is then the smallest at or above it), and looks every
// eight bits whether one value alone is left, as when many regrets are 0.
__device__ void order_pair(const uint64_t *key, int32_t m, int64_t k, int64_t n, int lane, double *lo_v, double *hi_v)
{
    constexpr int kHeld = 16;                        // up to 1,024 keys stay in registers
    uint64_t held[kHeld];
#pragma unroll
    for (int i = 0; i < kHeld; ++i) held[i] = 64 * i < m ? key[64 * i + lane] : ~0ull;
    auto below = [&](uint64_t v) {                   // keys < v
        int32_t c = 0;
#pragma unroll
        for (int i = 0; i < kHeld; i += 4)
            if (64 * i < m)
                c += __popcll(__ballot(held[i] < v)) + __popcll(__ballot(held[i + 1] < v)) +
                     __popcll(__ballot(held[i + 2] < v)) + __popcll(__ballot(held[i + 3] < v));
        for (int32_t i = 64 * kHeld + lane; i < m; i += 256) {
            const uint64_t x0 = key[i], x1 = key[i + 64], x2 = key[i + 128], x3 = key[i + 192];
            c += __popcll(__ballot(x0 < v)) + __popcll(__ballot(x1 < v)) + __popcll(__ballot(x2 < v)) +
                 __popcll(__ballot(x3 < v));
        }
        return c;
    };
    auto smallest = [&](uint64_t v) {                // smallest key >= v
        uint64_t s = ~0ull;
#pragma unroll 4
        for (int32_t i = lane; i < m; i += 64) {
            const uint64_t x = key[i];
            s = x >= v && x < s ? x : s;
        }
        return wave_min(s);
    };
    uint64_t v = 0;
    for (int bit = 63; bit >= 0; --bit) {
        const uint64_t next = v | (1ull << bit);
        const int32_t c = below(next);
        if (c <= k) v = next;
        if (c == k) break;
        if ((bit & 7) == 0) {                        // [v, v + 2^bit) holds the k-th key
            const uint64_t s = smallest(v);
            if (below(s + 1) > k) { v = s; break; }
        }
    }
    const uint64_t at = smallest(v);
    const uint64_t up = below(at + 1) > k + 1 || k + 1 >= n ? at : smallest(at + 1);
    *lo_v = key_value(at);
    *hi_v = key_value(up);
}

__global__ __launch_bounds__(kSmallT) void k_eval_small(const double *__restrict__ regret,
                                                        const int32_t *__restrict__ rank,
                                                        const double *__restrict__ ybar, int32_t P,
                                                        double *__restrict__ out, double *__restrict__ regret_out,
                                                        int32_t *__restrict__ rank_out, double *__restrict__ ybar_out)
{
    __shared__ uint64_t key_s[kSmallP];              // counted regrets, ~0 elsewhere
    __shared__ double term_s[2][kSmallP];            // regret and 1 - ybar of counted problems, 0 elsewhere
    __shared__ double sum_s[2], stat_s[2][2], wmax[kSmallT / 64];
    __shared__ int32_t wcnt[4][kSmallT / 64];
    const int32_t tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t m = (P + 255) & ~255;
    int32_t cnt = 0, top1 = 0, top5 = 0, w5 = 0;
    double mx = -__builtin_inf();
#pragma unroll
    for (int s = 0; s < kSmallM; ++s) {
        const int32_t i = tid + kSmallT * s;
        if (i >= m) continue;
        const bool in = i < P;
        const double r = in ? regret[i] : 0.0, y = in ? ybar[i] : 0.0;
        const int32_t rk = in ? rank[i] : 0;
        if (in && regret_out) regret_out[i] = r;
        if (in && rank_out) rank_out[i] = rk;
        if (in && ybar_out) ybar_out[i] = y;
        const bool c = rk != 0;
        key_s[i] = c ? order_key(r) : ~0ull;
        term_s[0][i] = c ? r : 0.0;
        term_s[1][i] = c ? 1.0 - y : 0.0;
        cnt += c;
        top1 += c && rk == 1;
        top5 += c && rk <= 5;
        w5 += c && r <= 0.05;
        mx = (c && r > mx) ? r : mx;
    }
    // counts and the maximum: wave totals, then the waves in order (integer
    // sums and a maximum do not depend on the order)
    for (int off = 32; off > 0; off >>= 1) {
        cnt += __shfl_xor(cnt, off);
        top1 += __shfl_xor(top1, off);
        top5 += __shfl_xor(top5, off);
        w5 += __shfl_xor(w5, off);
        const double o = __shfl_xor(mx, off);
        mx = o > mx ? o : mx;
    }
    if (lane == 0) {
        wcnt[0][wave] = cnt; wcnt[1][wave] = top1; wcnt[2][wave] = top5; wcnt[3][wave] = w5;
        wmax[wave] = mx;
    }
    __syncthreads();
    cnt = 0;
    for (int w = 0; w < kSmallT / 64; ++w) cnt += wcnt[0][w];
    if (cnt > 0 && wave < 2) {
        const double q = wave == 0 ? 0.5 : 0.95;
        const int64_t k = (int64_t)__builtin_floor(q * (double)(cnt - 1));
        double lo_v, hi_v;
        order_pair(key_s, m, k, cnt, lane, &lo_v, &hi_v);
        if (lane == 0) {
            stat_s[wave][0] = lo_v;
            stat_s[wave][1] = hi_v;
        }
    }
    if (wave == 2) {
        // in problem order, one sum in even and one in odd lanes (adding +0.0
        // for an uncounted problem leaves a sum that starts at +0.0 unchanged)
        const double *t = term_s[lane & 1];
        double sum = 0.0;
#pragma unroll 1
        for (int32_t p = 0; p < P; p += 16) {
            double v[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = t[p + i];
#pragma unroll
            for (int i = 0; i < 16; ++i) sum += v[i];
        }
        if (lane < 2) sum_s[lane] = sum;
    }
    __syncthreads();
    if (tid == 0) {
        top1 = top5 = w5 = 0;
        mx = -__builtin_inf();
        for (int w = 0; w < kSmallT / 64; ++w) {
            top1 += wcnt[1][w]; top5 += wcnt[2][w]; w5 += wcnt[3][w];
            mx = wmax[w] > mx ? wmax[w] : mx;
        }
        if (cnt == 0) {
            for (int i = 0; i < 8; ++i) out[i] = __builtin_nan("");
            out[8] = 0.0;
        } else {
            out[0] = sum_s[0] / (double)cnt;
            out[1] = interpolate(stat_s[0][0], stat_s[0][1], cnt, 0.5);
            out[2] = interpolate(stat_s[1][0], stat_s[1][1], cnt, 0.95);
            out[3] = mx;
            out[4] = (double)top1 / (double)cnt;
            out[5] = (double)top5 / (double)cnt;
            out[6] = (double)w5 / (double)cnt;
            out[7] = sum_s[1] / (double)cnt;
            out[8] = (double)cnt;
        }
    }
}

// ---------------------------------------------------------------------------
// Best static configuration
// ---------------------------------------------------------------------------
// A problem's rows are grouped by ranges of kRangeIds consecutive ids, so that
// one workgroup can then take a range through all problems with an id per
// lane.  The workspace's P x n_cfg words hold either
//   * the grouped rows, where they fit: first row of every range per problem
//     [P][ranges + 1], then for every row (local index << 6 | id within the
//     range, runtime), problems packed one after another, or
//   * a table [P][n_cfg] of each id's first local index (INT_MAX: absent),
//     where there are about half as many rows as P x n_cfg, or more.
// Grouped rows cost 16 bytes a row to write and read; the table costs 8 bytes
// an id and an atomic a row.  600 problems of 8,192 rows on average and 65,536
// ids: 90 us (33 grouping, 55 summing), 270 us through the table.
constexpr int kRangeIds = 64;
constexpr int32_t kMaxRanges = 10240;          // a counter each in LDS

__host__ __device__ constexpr int32_t id_ranges(int32_t n_cfg) { return (int32_t)(((int64_t)n_cfg + kRangeIds - 1) / kRangeIds); }

// Where problem p's rows are, read alike by both kernels.
struct StaticRows {
    bool grouped;                              // the same for every problem
    int64_t base, n;                           // rows [base, base + n)
    const int32_t *first;                      // grouped: [ranges + 1], places in all problems' rows
    const int2 *row;                           // grouped: [n]
};

__device__ __forceinline__ StaticRows static_rows(const int64_t *__restrict__ seg, int32_t P, int32_t p, int32_t n_cfg,
                                                  const int32_t *table)
{
    const int64_t ranges = id_ranges(n_cfg), lo = seg[0], total = seg[P] - lo;
    const int64_t head = (P * (ranges + 1) + 1) & ~(int64_t)1;       // words before the rows
    StaticRows r;
    r.grouped = ranges <= kMaxRanges && total >= 0 && total < (1 << 25) && head + 2 * total <= (int64_t)P * n_cfg;
    r.base = seg[p];
    r.n = seg[p + 1] - r.base;
    // offsets that do not ascend leave no room for a problem's rows
    if (r.n < 0 || (r.grouped && (r.base < lo || r.base - lo + r.n > total))) r.n = 0;
    r.first = table + p * (ranges + 1);
    r.row = reinterpret_cast<const int2 *>(table + head) + (r.grouped ? r.base - lo : 0);
    return r;
}

constexpr int kGroupThreads = 512;
constexpr int kGroupLoads = 8;                 // rows in flight per thread

// One workgroup per problem: its fastest runtime and its grouped rows (or its
// table).  Lists are usually ordered by id, so neighbouring lanes hold rows of
// one range: the first lane of each such run takes the places of the whole
// run with one LDS atomic (a lane each would queue on one counter).
__global__ __launch_bounds__(kGroupThreads) void k_static_group(const float *__restrict__ rt,
                                                                const int64_t *__restrict__ seg, int32_t P,
                                                                int32_t p0, const int32_t *__restrict__ cfg,
                                                                int32_t n_cfg, int32_t *__restrict__ table,
                                                                float *__restrict__ t_best)
{
    extern __shared__ int32_t place[];         // [ranges]
    __shared__ float red[kGroupThreads / 64];
    __shared__ int32_t wave_sum[kGroupThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t p = p0 + (int32_t)blockIdx.x;
    const StaticRows my = static_rows(seg, P, p, n_cfg, table);
    const int64_t base = my.base, n = my.n;
    const bool grouped = my.grouped;
    const int32_t ranges = id_ranges(n_cfg);
    int32_t *mine = table + (int64_t)p * n_cfg, *range_first = const_cast<int32_t *>(my.first);
    int2 *row = const_cast<int2 *>(my.row);
    const int2 *rows0 = row - (grouped ? base - seg[0] : 0);
    if (grouped)
        for (int32_t i = tid; i < ranges; i += kGroupThreads) place[i] = 0;
    else
        for (int32_t i = tid; i < n_cfg; i += kGroupThreads) mine[i] = INT_MAX;
    __syncthreads();

    // Visits the rows in steps of kGroupLoads per thread, loads first; a row
    // past the end or of no valid id comes with id -1.
    auto rows = [&](auto &&visit) {
        for (int64_t j0 = tid; j0 - lane < n; j0 += kGroupLoads * kGroupThreads) {
            int32_t id[kGroupLoads];
            float t[kGroupLoads];
#pragma unroll
            for (int i = 0; i < kGroupLoads; ++i) {
                const int64_t j = j0 + i * kGroupThreads;
                id[i] = j < n ? cfg[base + j] : -1;
                t[i] = j < n ? rt[base + j] : __builtin_nanf("");
            }
#pragma unroll
            for (int i = 0; i < kGroupLoads; ++i)
                visit((int32_t)(j0 + i * kGroupThreads), id[i] >= 0 && id[i] < n_cfg ? id[i] : -1, t[i]);
        }
    };
    // The run of equal ranges the lane is in: its first lane and length.
    auto run_of = [&](int32_t range, int &first, int &length) {
        const int32_t left = __shfl_up(range, 1);
        const uint64_t heads = __ballot(lane == 0 || left != range);
        const uint64_t upto = heads & (~0ull >> (63 - lane));
        first = 63 - __builtin_clzll(upto);
        const uint64_t after = lane < 63 ? heads >> (lane + 1) : 0ull;
        length = (after ? lane + 1 + __builtin_ctzll(after) : 64) - first;
    };

    float best = __builtin_nanf("");
    rows([&](int32_t j, int32_t id, float t) {
        if (faster(t, best)) best = t;
        if (!grouped) {
            if (id >= 0) atomicMin(&mine[id], j);
            return;
        }
        const int32_t range = id >> 6;         // -1 for no id
        int first, length;
        run_of(range, first, length);
        if (lane == first && range >= 0) atomicAdd(&place[range], length);
    });
    for (int off = 32; off > 0; off >>= 1) {
        const float o = __shfl_xor(best, off);
        if (faster(o, best)) best = o;
    }
    if (lane == 0) red[wave] = best;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kGroupThreads / 64; ++w)
            if (faster(red[w], best)) best = red[w];
        t_best[p] = best;
    }
    if (!grouped) return;

    // counts to first places, a run of counters per thread
    const int32_t per = (ranges + kGroupThreads - 1) / kGroupThreads;
    const int32_t lo = tid * per < ranges ? tid * per : ranges, hi = lo + per < ranges ? lo + per : ranges;
    int32_t sum = 0;
    for (int32_t i = lo; i < hi; ++i) sum += place[i];
    int32_t scan = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t o = __shfl_up(scan, off);
        scan += lane >= off ? o : 0;
    }
    if (lane == 63) wave_sum[wave] = scan;
    __syncthreads();
    int32_t at = scan - sum;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    for (int32_t i = lo; i < hi; ++i) {
        const int32_t c = place[i];
        place[i] = at;
        range_first[i] = (int32_t)(row - rows0) + at;
        at += c;
    }
    if (tid == kGroupThreads - 1) range_first[ranges] = (int32_t)(row - rows0) + at;
    __syncthreads();
    rows([&](int32_t j, int32_t id, float t) {
        const int32_t range = id >> 6;
        int first, length;
        run_of(range, first, length);
        int32_t to = 0;
        if (lane == first && range >= 0) to = atomicAdd(&place[range], length);
        to = __shfl(to, first) + lane - first;
        if (range >= 0) row[to] = make_int2((j << 6) | (id & 63), __float_as_int(t));
    });
}

constexpr int kSumWaves = 8;                        // at most
constexpr int kSumProblems = 8;                     // problems per wave and step

struct StaticBest {
    double mean;
    int32_t id, count;                               // id -1: none qualifies
};

// The better of two: higher mean, then lower id.
__device__ __forceinline__ StaticBest better(StaticBest a, StaticBest b)
{
    const bool first = b.id < 0 || (a.id >= 0 && (a.mean > b.mean || (a.mean == b.mean && a.id < b.id)));
    return StaticBest{first ? a.mean : b.mean, first ? a.id : b.id, first ? a.count : b.count};
}

__device__ __forceinline__ StaticBest wave_better(StaticBest v)
{
    for (int off = 32; off > 0; off >>= 1)
        v = better(v, StaticBest{__shfl_xor(v.mean, off), __shfl_xor(v.id, off), __shfl_xor(v.count, off)});
    return v;
}

// One workgroup per range of ids.  A step takes eight problems a wave (64 with
// eight waves; few problems get few waves): each wave finds the first row of
// every id in eight of them (the smallest local index, by LDS atomics on index
// and runtime together), which leaves its y there, 0 for an absent id (a y for
// every row, not every id: the quotients bound this kernel); the first
// wave then adds the y in problem order, an id per lane (adding +0 leaves a sum
// that starts at +0 as it is).  Where a step's rows lie is read a step ahead.
// Neighbouring ranges share cache lines, so the workgroups of one XCD (b % 8)
// take neighbouring ranges.
__global__ __launch_bounds__(64 * kSumWaves, 8) void k_static_sum(const float *__restrict__ rt,
                                                               const int64_t *__restrict__ seg, int32_t P,
                                                               int32_t n_cfg, const int32_t *__restrict__ table,
                                                               const float *__restrict__ t_best,
                                                               double *__restrict__ best_mean,
                                                               int32_t *__restrict__ best_id,
                                                               int32_t *__restrict__ best_count)
{
    const int step = (int)(blockDim.x >> 6) * kSumProblems;
    constexpr uint64_t kAbsent = ~0ull;
    extern __shared__ uint64_t slot[][kRangeIds];    // [step]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t ranges = id_ranges(n_cfg);
    const int32_t per_xcd = (ranges + 7) / 8;
    const int32_t range = (int32_t)(blockIdx.x % 8) * per_xcd + (int32_t)(blockIdx.x / 8);
    if (range >= ranges) return;
    const int32_t id0 = range * kRangeIds;
    // eight lanes per problem
    const int sub = lane >> 3, part = lane & 7;
    const StaticRows any = static_rows(seg, P, 0, n_cfg, table);     // its `grouped` holds for all
    const int2 *rows = any.row - (any.grouped ? any.base - seg[0] : 0);
    struct Place {
        int32_t e0, e1;                              // grouped rows [e0, e1)
        float best;                                  // fastest runtime
    };
    // plain loads, so that nothing waits for them before their step
    auto place_of = [&](int32_t p0) {
        const int32_t p = p0 + wave * kSumProblems + sub;
        Place c{0, 0, 0.0f};
        if (any.grouped && p < P) {
            const int32_t *at = table + (int64_t)p * (ranges + 1) + range;
            c = Place{at[0], at[1], t_best[p]};
        }
        return c;
    };
    // the first 16 rows of each place (few have more) are loaded a step ahead
    auto row_of = [&](const Place &c, int i) {
        const int32_t e = c.e0 + part + 8 * i;
        return e < c.e1 ? rows[e] : make_int2(0, 0);
    };
    auto packed = [&](int2 r) { return ((uint64_t)((uint32_t)r.x >> 6) << 32) | (uint32_t)r.y; };   // index and runtime
    int32_t count = 0;                               // of id `lane` in this wave's problems
    double sum = 0.0;
    Place c = place_of(0), next = place_of(step);
    int2 r0 = row_of(c, 0), r1 = row_of(c, 1);
    for (int32_t p0 = 0; p0 < P; p0 += step) {
        uint64_t (*own)[kRangeIds] = slot + wave * kSumProblems;
#pragma unroll
        for (int i = 0; i < kSumProblems; ++i) own[i][lane] = kAbsent;
        const Place after = place_of(p0 + 2 * step);
        if (any.grouped) {
            // the first row of every id
            auto lower = [&](int2 r) {
                atomicMin(reinterpret_cast<unsigned long long *>(&own[sub][r.x & 63]), packed(r));
            };
            // it puts its y in place.  (No later row of an id takes a y for
            // its own index and runtime: as bits a y is 0 or above 2^57, and
            // only the first row can be row 0.)
            auto settle = [&](int2 r) {
                uint64_t &at = own[sub][r.x & 63];
                if (at == packed(r)) at = __builtin_bit_cast(uint64_t, y_of(c.best, __int_as_float(r.y)));
            };
            if (c.e0 + part < c.e1) lower(r0);
            if (c.e0 + part + 8 < c.e1) lower(r1);
            for (int32_t e = c.e0 + part + 16; e < c.e1; e += 8) lower(rows[e]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            if (c.e0 + part < c.e1) settle(r0);
            if (c.e0 + part + 8 < c.e1) settle(r1);
            for (int32_t e = c.e0 + part + 16; e < c.e1; e += 8) settle(rows[e]);
            r0 = row_of(next, 0);
            r1 = row_of(next, 1);
        } else if (p0 + wave * kSumProblems + sub < P) {
            const int32_t p = p0 + wave * kSumProblems + sub;
            const StaticRows at = static_rows(seg, P, p, n_cfg, table);
            const int32_t *mine = table + (int64_t)p * n_cfg;
            const float fastest = t_best[p];
#pragma unroll
            for (int i = 0; i < kRangeIds / 8; ++i) {
                const int32_t j = at.n > 0 && id0 + 8 * i + part < n_cfg ? mine[id0 + 8 * i + part] : INT_MAX;
                if (j != INT_MAX) own[sub][8 * i + part] = __builtin_bit_cast(uint64_t, y_of(fastest, rt[at.base + j]));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
#pragma unroll
        for (int i = 0; i < kSumProblems; ++i) {
            const bool there = own[i][lane] != kAbsent;
            count += there;
            if (!there) own[i][lane] = 0;
        }
        lds_barrier();
        if (wave == 0) {
            // eight values are read while the eight before are added
            const int steps = P - p0 < step ? (P - p0 + 7) & ~7 : step;
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = __builtin_bit_cast(double, slot[k][lane]);
            for (int i = 0; i < steps; i += 8) {
                const int ahead = i + 8 < steps ? i + 8 : i;
                double u[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) u[k] = __builtin_bit_cast(double, slot[ahead + k][lane]);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    sum += v[k];
                    v[k] = u[k];
                }
            }
        }
        lds_barrier();
        c = next;
        next = after;
    }
    int32_t *counts = reinterpret_cast<int32_t *>(&slot[0][0]);      // [wave][id]
    counts[wave * 64 + lane] = count;
    lds_barrier();
    if (wave == 0) {
        for (int w = 1; w < (int)(blockDim.x >> 6); ++w) count += counts[w * 64 + lane];
        const bool counts_in = count > 0 && 5 * (int64_t)count >= 4 * (int64_t)P;
        const StaticBest v =
            wave_better(StaticBest{counts_in ? sum / (double)count : 0.0, counts_in ? id0 + lane : -1, count});
        if (lane == 0) {
            best_mean[range] = v.mean;
            best_id[range] = v.id;
            best_count[range] = v.count;
        }
    }
}

__global__ __launch_bounds__(1024) void k_static_argmax(const double *__restrict__ best_mean,
                                                        const int32_t *__restrict__ best_id,
                                                        const int32_t *__restrict__ best_count, int32_t ranges,
                                                        int32_t *__restrict__ best, double *__restrict__ mean_y)
{
    __shared__ double mean[16];
    __shared__ int32_t id[16], count[16];
    StaticBest v{0.0, -1, 0};
    for (int32_t r = threadIdx.x; r < ranges; r += 1024) v = better(v, StaticBest{best_mean[r], best_id[r], best_count[r]});
    v = wave_better(v);
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        mean[w] = v.mean;
        id[w] = v.id;
        count[w] = v.count;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) v = better(v, StaticBest{mean[w], id[w], count[w]});
        best[0] = v.id;
        best[1] = v.id < 0 ? 0 : v.count;
        mean_y[0] = v.id < 0 ? __builtin_nan("") : v.mean;
    }
}

size_t up256(size_t v) { return (v + 255) / 256 * 256; }

constexpr size_t eval_workspace_bytes(int64_t P)
{
    return 3 * (((size_t)P * sizeof(double) + 255) / 256 * 256) + ((size_t)P * sizeof(int32_t) + 255) / 256 * 256;
}

// Scratch of hwsel_evaluate_noalloc: the per-problem regrets, y means, order
// statistics and ranks that hwsel_evaluate keeps in the caller's workspace,
// here in a device array of the library's code object (one copy per device,
// held until the process ends).  Every value a call reads is written earlier
// in that same call, so nothing has to be cleared between calls; calls that
// overlap on one device share the array and race.
constexpr size_t kNoAllocScratchBytes = eval_workspace_bytes(HWSEL_EVAL_NOALLOC_MAX_P);
static __device__ __align__(256) uint8_t scratch[kNoAllocScratchBytes];
static_assert(kNoAllocScratchBytes == HWSEL_EVAL_NOALLOC_SCRATCH_BYTES, "scratch size as declared");

}  // namespace

size_t evaluate_workspace_bytes(int32_t P) { return eval_workspace_bytes(P); }

// Device address of this device's scratch copy, looked up (with the device
// current) on the first call on each device and kept.  In host code the
// array's own name is not a device address and is never passed to a kernel.
hipError_t evaluate_noalloc_scratch(void **ptr, size_t *bytes)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *per_device[kMaxDevices];
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        per_device[dev] = p;
    }
    *ptr = per_device[dev];
    *bytes = kNoAllocScratchBytes;
    return hipSuccess;
}

hipError_t launch_evaluate(const float *rt, const int64_t *seg, int32_t P, const int32_t *idx, int32_t k,
                           double *out, double *regret_out, int32_t *rank_out, double *ybar_out, void *ws,
                           hipStream_t s)
{
    uint8_t *w = static_cast<uint8_t *>(ws);
    double *regret = reinterpret_cast<double *>(w);
    double *ybar = reinterpret_cast<double *>(w + up256((size_t)P * 8));
    double *stats = reinterpret_cast<double *>(w + 2 * up256((size_t)P * 8));
    int32_t *rank = reinterpret_cast<int32_t *>(w + 3 * up256((size_t)P * 8));
    each_span(P, [&](int32_t p0, int32_t n) {
        hipLaunchKernelGGL(k_eval_groups, dim3(n), dim3(kEvalThreads), 0, s, rt, seg + p0, n, idx + (int64_t)p0 * k, k,
                           regret + p0, rank + p0, ybar + p0);
    });
    if (P <= kSmallP) {
        hipLaunchKernelGGL(k_eval_small, dim3(1), dim3(kSmallT), 0, s, regret, rank, ybar, P, out, regret_out, rank_out,
                           ybar_out);
    } else {
        hipLaunchKernelGGL(k_eval_select, dim3(1), dim3(kSelectThreads), 0, s, regret, rank, P, stats);
        hipLaunchKernelGGL(k_eval_aggregate, dim3(1), dim3(256), 0, s, regret, rank, ybar, stats, P, out, regret_out,
                           rank_out, ybar_out);
    }
    return hipGetLastError();
}

size_t static_config_workspace_bytes(int32_t P, int32_t n_cfg)
{
    return up256((size_t)P * (size_t)n_cfg * sizeof(int32_t)) + up256((size_t)P * sizeof(float)) +
           up256((size_t)n_cfg * sizeof(int32_t)) + up256((size_t)n_cfg * sizeof(double));
}

hipError_t launch_static_config(const float *rt, const int64_t *seg, int32_t P, const int32_t *cfg, int32_t n_cfg,
                                int32_t *best, double *mean_y, void *ws, hipStream_t s)
{
    uint8_t *w = static_cast<uint8_t *>(ws);
    const size_t table = up256((size_t)P * (size_t)n_cfg * sizeof(int32_t));
    int32_t *groups = reinterpret_cast<int32_t *>(w);
    float *t_best = reinterpret_cast<float *>(w + table);
    // best of every range: 2 ranges <= max(n_cfg, 64) words, ranges doubles
    const int32_t ranges = id_ranges(n_cfg);
    int32_t *id = reinterpret_cast<int32_t *>(w + table + up256((size_t)P * 4)), *count = id + ranges;
    double *mean = reinterpret_cast<double *>(w + table + up256((size_t)P * 4) + up256((size_t)n_cfg * 4));
    const size_t lds = ranges <= kMaxRanges ? (size_t)ranges * 4 : 0;
    each_span(P, [&](int32_t p0, int32_t n) {
        hipLaunchKernelGGL(k_static_group, dim3(n), dim3(kGroupThreads), lds, s, rt, seg, P, p0, cfg, n_cfg, groups, t_best);
    });
    int waves = P < kSumWaves * kSumProblems ? (P + kSumProblems - 1) / kSumProblems : kSumWaves;
    while (waves > 1 && ((int64_t)ranges + 8) * 64 * waves >= (int64_t)1 << 32) waves /= 2;   // threads of a launch
    hipLaunchKernelGGL(k_static_sum, dim3(8 * ((ranges + 7) / 8)), dim3(64 * waves),
                       (size_t)waves * kSumProblems * kRangeIds * 8, s, rt, seg, P, n_cfg, groups, t_best, mean, id, count);
    hipLaunchKernelGGL(k_static_argmax, dim3(1), dim3(1024), 0, s, mean, id, count, ranges, best, mean_y);
    return hipGetLastError();
}

}  // namespace hwsel
