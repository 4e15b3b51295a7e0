// Per-problem selection (top-k by score) and selection regret.
//
// One workgroup per problem segment.  Scores are mapped to 64-bit keys
// (order-preserving score bits << 32 | inverted local index), which makes
// every key unique: "score descending, index ascending" becomes "key
// descending" and the answer is unique.
//
// A segment is read once, kTile rows at a time, the next tile's scores on their
// way while one is worked on.  Of a tile only the keys above a bound are looked
// at further: the k-th best key so far, or, while fewer than k are kept (or too
// many pass), a bound from the tile itself.  Each wave takes the j-th largest of
// its lanes' maxima; if r waves have j lanes each above a value, r j >= k keys
// are, so the r-th largest of those is at most the k-th best.  About k keys pass;
// they meet the kept ones in LDS and every key finds its rank by counting the
// larger ones.  A tile whose keys still do not fit the list gives its best in k
// rounds of a block-wide maximum.
// Bound by latency for one short segment (a load, four barriers) and by the
// score reads for long ones.  Measured against k rounds over all keys (256
// threads): 256 segments of 65,536 rows, k = 16,
// 172 -> 20 us; one of 8,192 rows, k = 10, 19 -> 6 us.
#include "internal.hpp"

namespace hwsel {
namespace {

// rows of a tile: 32 keys per thread of a small workgroup, 8 of a large one
constexpr int kTile = 8192;

// Larger key = better score.  NaN ranks lowest, -0 equals +0.
__device__ __forceinline__ uint32_t desc_bits(float s)
{
    if (s != s) return 0u;
    uint32_t b = __float_as_uint(s);
    if ((b << 1) == 0u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Smaller key = faster runtime.  NaN ranks above +inf, -0 equals +0.
__device__ __forceinline__ uint32_t asc_bits(float t)
{
    if (t != t) return 0xffffffffu;
    uint32_t b = __float_as_uint(t);
    if ((b << 1) == 0u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

template <int CTRL, int ROW_MASK, bool ZERO_FILL>
__device__ __forceinline__ uint32_t dpp_max_u32(uint32_t v)
{
    const uint32_t w = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, ZERO_FILL);
    return w > v ? w : v;
}

// Maximum over the wave of an unsigned 32-bit value (0 is the identity), in
// every lane: scan within rows, row broadcasts to lane 63, then readlane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v)
{
    v = dpp_max_u32<0x111, 0xf, true>(v);
    v = dpp_max_u32<0x112, 0xf, true>(v);
    v = dpp_max_u32<0x114, 0xf, true>(v);
    v = dpp_max_u32<0x118, 0xf, true>(v);
    v = dpp_max_u32<0x142, 0xa, false>(v);
    v = dpp_max_u32<0x143, 0xc, false>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Maximum over the wave of 64-bit keys: the largest high word, then the
// largest low word among the lanes holding it.
__device__ __forceinline__ uint64_t wave_max_key(uint64_t v)
{
    const uint32_t hi = wave_max_u32((uint32_t)(v >> 32));
    const uint32_t lo = wave_max_u32((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0u);
    return ((uint64_t)hi << 32) | lo;
}

// Block maximum with one barrier: the waves' maxima go to sh (a buffer the
// caller alternates between rounds, so no round overwrites one still read).
template <int NT>
__device__ __forceinline__ uint64_t block_max_key(uint64_t v, uint64_t *sh)
{
    v = wave_max_key(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    uint64_t r = sh[0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) r = sh[w] > r ? sh[w] : r;
    return r;
}

__device__ __forceinline__ int64_t seg_len(const int64_t *seg, int32_t p)
{
    int64_t n = seg[p + 1] - seg[p];
    n = n < 0 ? 0 : n;
    return n > 0x7fffffff ? 0x7fffffff : n;
}

__device__ __forceinline__ uint64_t lane_value(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

constexpr int kList = 512;            // keys of one tile that are ranked at once

template <int NT>
struct TopkLds {
    uint64_t top[2][64], cand[kList];                       // kept keys, descending; the tile's
    uint64_t per_wave[2][NT / 64];
    // Keys listed of tiles 0, 3, 6, ..., of tiles 1, 4, ... and of tiles 2, 5, ...
    // Every wave has to read the same count of a tile, and nothing but barriers
    // keeps waves together.  Tile i's count is complete at the barrier after
    // its appends and read before the next tile's; the counter of tile i + 2
    // (tile i - 1's) is cleared between the two: its last reads came before
    // the first, and tile i + 2 appends after the second.
    int32_t n_cand[3];
};

// The k best of one segment by NT threads, TILE rows at a time (lds: for at
// least as many threads).
template <int NT, int TILE, class Lds>
__device__ __forceinline__ void topk_tiles(const float *__restrict__ s, int32_t n, int32_t k, int32_t *__restrict__ idx,
                                           float *__restrict__ vals, Lds &lds)
{
    constexpr int kWaves = NT / 64, kPer = TILE / NT;       // keys per thread and tile
    auto &top = lds.top;
    auto &cand = lds.cand;
    auto &per_wave = lds.per_wave;
    auto &n_cand = lds.n_cand;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // r waves with j lanes each: r at most half the waves
    const int32_t j_of = (k + kWaves / 2 - 1) / (kWaves / 2), r_of = (k + j_of - 1) / j_of;

    float next[kPer];
    auto fetch = [&](int32_t t0) {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t i = (uint32_t)t0 + threadIdx.x + q * NT;
            next[q] = i < (uint32_t)n ? s[i] : 0.0f;
        }
    };
    fetch(0);
    if (threadIdx.x < 3) n_cand[threadIdx.x] = 0;           // (the first bound's barrier follows)
    int32_t kept = 0, cur = 0, turn = 0;                    // block-uniform; turn: the tile's counter
    uint64_t floor = 0;                                     // keys at or below it are out (0: none)
    for (uint32_t t0 = 0; t0 < (uint32_t)n; t0 += TILE) {
        uint32_t hi[kPer];                                  // score bits of the thread's keys
        auto key = [&](int q) -> uint64_t {                 // 0: no row (every real key is > 0)
            const uint32_t i = t0 + threadIdx.x + q * NT;
            return i < (uint32_t)n ? ((uint64_t)hi[q] << 32) | (0xffffffffu - i) : 0ull;
        };
#pragma unroll
        for (int q = 0; q < kPer; ++q) hi[q] = desc_bits(next[q]);
        if (t0 + TILE < (uint32_t)n) fetch(t0 + TILE);
        uint64_t most = 0;                                  // the lane's largest key
#pragma unroll
        for (int q = 0; q < kPer; ++q) most = key(q) > most ? key(q) : most;

        // A key that is at most the k-th best of the tile and of the kept ones.
        auto bound = [&]() -> uint64_t {
            uint64_t m = most, v = 0;
            for (int32_t j = 0; j < j_of; ++j) {
                v = wave_max_key(m);
                m = m == v ? 0ull : m;
            }
            if (lane == 0) per_wave[0][wave] = v;
            __syncthreads();
            const uint64_t mine = lane < kWaves ? per_wave[0][lane] : 0ull;
            int32_t above = 0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint64_t o = lane_value(mine, w);
                above += o > mine || (o == mine && w < lane);
            }
            return lane_value(mine, __builtin_ctzll(__ballot(lane < kWaves && above == r_of - 1)));
        };
        auto append = [&](uint64_t limit) {                 // keys above limit to cand; counted beyond its end too
            if (__ballot(most > limit) == 0) return;
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const uint64_t v = key(q);
                const uint64_t take = __ballot(v > limit);
                if (take == 0) continue;
                int32_t at = 0;
                if (lane == 0) at = atomicAdd(&n_cand[turn], __popcll(take));
                at = __builtin_amdgcn_readfirstlane(at) +
                     (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(take >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)take, 0u));
                if (v > limit && at < kList) cand[at] = v;
            }
        };
        auto raised = [&](uint64_t b) { return b != 0 && b - 1 > floor ? b - 1 : floor; };
        const bool bounded = kept < k;
        if (bounded) append(raised(bound()));
        else append(floor);
        __syncthreads();
        if (threadIdx.x == 0) n_cand[turn == 0 ? 2 : turn - 1] = 0;
        int32_t m = n_cand[turn];
        if (m > kList && !bounded) {                        // far more than k above the floor: bound them
            __syncthreads();                                // all have read the count
            if (threadIdx.x == 0) n_cand[turn] = 0;
            append(raised(bound()));                        // (the bound's barrier comes before)
            __syncthreads();
            m = n_cand[turn];
        }
        turn = turn == 2 ? 0 : turn + 1;
        if (m > kList) {                                    // the tile's best in rounds
            uint64_t prev = ~0ull;
            __syncthreads();
            for (m = 0; m < k; ++m) {                       // block-uniform trip count
                uint64_t best = 0;
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    const uint64_t v = key(q);
                    best = (v < prev && v > floor && v > best) ? v : best;
                }
                best = block_max_key<NT>(best, per_wave[m & 1]);
                if (best == 0) break;
                if (threadIdx.x == 0) cand[m] = best;
                prev = best;
            }
            __syncthreads();
        }
        if (m > 0) {
            // the rank of every kept and every new key among both
            for (int32_t e = threadIdx.x; e < kept + m; e += NT) {
                const uint64_t v = e < kept ? top[cur][e] : cand[e - kept];
                int32_t rank = e < kept ? e : 0;
                if (e >= kept)
                    for (int32_t q = 0; q < kept; ++q) rank += top[cur][q] > v;
                // eight reads in flight (one at a time, 450 keys took 20 us)
#pragma unroll 8
                for (int32_t q = 0; q < m; ++q) rank += cand[q] > v;
                if (rank < k) top[cur ^ 1][rank] = v;
            }
            cur ^= 1;
            kept = kept + m < k ? kept + m : k;
            __syncthreads();
            if (kept == k) floor = top[cur][k - 1];
        }
    }
    for (int32_t j = threadIdx.x; j < k; j += NT) {
        const int32_t li = j < kept ? (int32_t)(0xffffffffu - (uint32_t)top[cur][j]) : -1;
        idx[j] = li;
        if (vals) vals[j] = li < 0 ? -__builtin_inff() : s[li];
    }
}

// By length: up to 64 rows are one wave's, a row per lane, each key's rank by
// counting the larger ones; up to 1,024 are 256 threads' with four keys each
// (the other waves are gone before the first barrier); longer ones take
// tiles.  Going through a whole tile's keys costs a wave over 1,000
// instructions however few the rows: 100,000 segments of 16 rows, k = 4,
// 800 us so and 96 us by length, 3,000 of 300, k = 5, 28 and 12 us.
constexpr int kShort = 1024, kShortThreads = 256;

template <int NT>
__global__ __launch_bounds__(NT) void k_topk(const float *__restrict__ scores, const int64_t *__restrict__ seg, int32_t k,
                                             int32_t *__restrict__ idx, float *__restrict__ vals)
{
    __shared__ TopkLds<NT> lds;
    const int32_t p = blockIdx.x;
    const int32_t n = (int32_t)seg_len(seg, p);
    const float *s = scores + seg[p];
    idx += (int64_t)p * k;
    if (vals) vals += (int64_t)p * k;
    if (n <= 64) {
        const int32_t lane = threadIdx.x;
        if (lane >= 64) return;
        const float v = lane < n ? s[lane] : 0.0f;
        const uint64_t own = lane < n ? ((uint64_t)desc_bits(v) << 32) | (0xffffffffu - (uint32_t)lane) : 0ull;
        int32_t rank = 0;
        for (int32_t l = 0; l < n; ++l) rank += lane_value(own, l) > own;
        const int32_t j = lane < n ? rank : lane;           // past the rows: no pick
        if (j < k) {
            idx[j] = lane < n ? lane : -1;
            if (vals) vals[j] = lane < n ? v : -__builtin_inff();
        }
    } else if (n <= kShort) {
        if (threadIdx.x >= kShortThreads) return;
        topk_tiles<kShortThreads, kShort>(s, n, k, idx, vals, lds);
    } else {
        topk_tiles<NT, kTile>(s, n, k, idx, vals, lds);
    }
}

// 1 - t_star / t_pick in binary64; equal runtimes (inf included) give 0 and a
// NaN runtime (a kernel that never finishes) gives 1.
__device__ __forceinline__ float regret_value(float t_star, float t_pick)
{
    if (t_pick == t_star) return 0.0f;
    if (t_pick != t_pick) return 1.0f;
    return (float)(1.0 - (double)t_star / (double)t_pick);
}

// The runtime whose asc_bits are b (0 for -0).
__device__ __forceinline__ float asc_value(uint32_t b)
{
    return __uint_as_float((b & 0x80000000u) ? b ^ 0x80000000u : ~b);
}

// The fastest row by a block-wide minimum, all of a step's loads in flight;
// up to 512 rows are the first wave's alone, a load per 64 rows that are there.
// The picks' runtimes are fetched by the first wave's lanes meanwhile.
// Bound by the reads (long segments) and latency: 256 segments of
// 65,536 rows 83 -> 14 us (from 128 loads of one row each, one after another);
// 100,000 of 16 rows 66 us then, 91 with eight loads for every lane, now 52.
template <int NT>
__global__ __launch_bounds__(NT) void k_regret(const float *__restrict__ rt, const int64_t *__restrict__ seg,
                                               const int32_t *__restrict__ idx, int32_t k, float *__restrict__ r1,
                                               float *__restrict__ rk, int32_t *__restrict__ best)
{
    __shared__ uint64_t sh[NT / 64];
    const int32_t p = blockIdx.x;
    const int64_t base = seg[p];
    const int64_t n = seg_len(seg, p);
    const float *t = rt + base;
    const int lane = threadIdx.x;
    // lane j < k of the first wave: pick j
    float t_pick = 0.0f;
    uint64_t pick_key = ~0ull;
    bool counted = false;
    if (lane < k) {
        const int32_t c = idx[(int64_t)p * k + lane];
        counted = c >= 0 && c < n;
        if (counted) {
            t_pick = t[c];
            pick_key = ((uint64_t)asc_bits(t_pick) << 32) | (uint64_t)(uint32_t)c;
        }
    }
    constexpr int kIn = NT >= 512 ? 16 : 8;
    constexpr int kFew = 8;
    uint64_t m = ~0ull;
    const bool few = n <= 64 * kFew;                        // the first wave's alone
    if (few) {
        if (threadIdx.x >= 64) return;
#pragma unroll
        for (int q = 0; q < kFew; ++q) {
            if (64 * q >= n) break;                         // (uniform)
            const uint32_t i = lane + 64 * q < n ? lane + 64 * q : lane < n ? lane : 0;
            const uint64_t key = ((uint64_t)asc_bits(t[i]) << 32) | i;
            m = key < m ? key : m;
        }
        m = ~wave_max_key(~m);
    }
    for (int64_t i0 = threadIdx.x; i0 < n && !few; i0 += kIn * NT) {
        float v[kIn];
#pragma unroll
        for (int q = 0; q < kIn; ++q) v[q] = t[i0 + q * NT < n ? i0 + q * NT : i0];
#pragma unroll
        for (int q = 0; q < kIn; ++q) {
            const int64_t i = i0 + q * NT < n ? i0 + q * NT : i0;
            const uint64_t key = ((uint64_t)asc_bits(v[q]) << 32) | (uint64_t)(uint32_t)i;
            m = key < m ? key : m;
        }
    }
    if (!few) m = ~block_max_key<NT>(~m, sh);               // block minimum of the unique keys
    if (threadIdx.x >= 64) return;
    const uint64_t bk = ~wave_max_key(~pick_key);
    // its runtime as it stands (a key does not tell -0 from +0)
    const float t_k = __shfl(t_pick, __builtin_ctzll(__ballot(pick_key == bk)));
    if (threadIdx.x != 0) return;
    if (n == 0) {
        r1[p] = __builtin_nanf("");
        if (rk) rk[p] = __builtin_nanf("");
        if (best) best[p] = -1;
        return;
    }
    const float t_star = (uint32_t)(m >> 32) == 0xffffffffu ? __builtin_nanf("") : asc_value((uint32_t)(m >> 32));
    r1[p] = counted ? regret_value(t_star, t_pick) : __builtin_nanf("");
    if (rk) rk[p] = bk == ~0ull ? __builtin_nanf("") : regret_value(t_star, t_k);
    if (best) best[p] = (int32_t)(uint32_t)m;
}

}  // namespace

// Segment lengths are not known here.  While every problem has a CU to itself,
// a large workgroup has the most loads in flight; beyond that, small ones
// share the CUs better and waste less on short segments.  Top-16 and regret:
// 256 problems of 65,536 rows 39 us large, 67 small; 300 of 50,000 59 and 61;
// 600 of 25,000 50 and 43.  The regret's large ones have 512 threads of twice
// the loads: as fast on long segments as 1,024, and half the waves to start on
// short ones (60 of 8,192 rows 3.7 us, 4.4 with 1,024).
hipError_t launch_topk(const float *scores, const int64_t *seg, int32_t P, int32_t k, int32_t *idx,
                       float *vals, hipStream_t s)
{
    if (P <= compute_units())
        hipLaunchKernelGGL(k_topk<1024>, dim3(P), dim3(1024), 0, s, scores, seg, k, idx, vals);
    else
        each_span(P, [&](int32_t p0, int32_t n) {
            const int64_t o = (int64_t)p0 * k;
            hipLaunchKernelGGL(k_topk<256>, dim3(n), dim3(256), 0, s, scores, seg + p0, k, idx + o, vals ? vals + o : nullptr);
        });
    return hipGetLastError();
}

hipError_t launch_regret(const float *rt, const int64_t *seg, int32_t P, const int32_t *idx,
                         int32_t k, float *r1, float *rk, int32_t *best, hipStream_t s)
{
    if (P <= compute_units())
        hipLaunchKernelGGL(k_regret<512>, dim3(P), dim3(512), 0, s, rt, seg, idx, k, r1, rk, best);
    else
        each_span(P, [&](int32_t p0, int32_t n) {
            hipLaunchKernelGGL(k_regret<256>, dim3(n), dim3(256), 0, s, rt, seg + p0, idx + (int64_t)p0 * k, k, r1 + p0,
                               rk ? rk + p0 : nullptr, best ? best + p0 : nullptr);
        });
    return hipGetLastError();
}

}  // namespace hwsel
