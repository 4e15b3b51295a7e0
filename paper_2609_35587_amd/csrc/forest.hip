// Tree-ensemble scoring: s(x) = base + sum_t leaf_t(x).
//
// Two paths share the decision rule "left iff x < threshold (or NaN with
// the default-left flag)":
//
// Direct path (no packed model): fp32 compares with rows of X and the trees'
// upper levels in LDS, or a row per wave where there are few (see
// k_forest_direct), or a row per thread where there are few trees (see
// rows_visits).  Any forest the header admits runs here.
//
// Packed path (model packed once by hwsel_forest_pack):
//   * Exact binning.  For feature f let U_f be the sorted distinct
//     thresholds the forest uses (at most 255).  With
//     b_f(x) = #{u in U_f : u <= x}, and a node testing x < U_f[j],
//     x < U_f[j]  <=>  b_f(x) <= j,
//     so the traversal compares u8 bins with u8 threshold ranks and gives the
//     same path as the fp32 compares (NaN is binned to 0 when it goes left,
//     255 when it goes right).  A pass writes the bins of every row once:
//     128 bytes per row instead of 512.
//   * Image.  Trees are grouped into image chunks whose nodes (u16 code:
//     feature | rank << 8, heap order, stored as sibling pairs, interleaved by
//     tree, see node_byte) and leaves (fp32, leaf l of tree t at l*TC + t) are
//     stored for the traversal to lay out in LDS.
//   * Trees in LDS.  A workgroup keeps 64 trees (depth <= 8) or 32 trees
//     (depth 9, 10) as two-level groups, one column of banks per tree, plus
//     their leaves; at depth 10 the leaves do not fit next to the groups and
//     go through an 8-tree buffer once per eight tiles (see Walk and
//     k_traverse).
//   * Chunk-stationary, XCD-aware persistent grid.  Each workgroup owns one
//     chunk for a whole row range; each wave owns a slice of every row tile
//     and a private LDS region for its bins, refilled without workgroup
//     barriers while the next slices are fetched into registers.  Workgroup b
//     runs on XCD b % 8; the workgroups of one XCD cover the same rows with
//     different chunks, so a tile is fetched from HBM about once per XCD and
//     re-read from that XCD's L2.
//   * Deterministic sums.  A chunk's per-row sum is a fixed tree of lane folds
//     over its trees, the same for every row, written to a per-chunk partial
//     row; a last pass adds base + partials in chunk order.
#include <algorithm>
#include <cstring>
#include <vector>

#include "internal.hpp"

namespace hwsel {
namespace {

// ---------------------------------------------------------------------------
// Generic path
// ---------------------------------------------------------------------------
struct ForestDev {
    int32_t n_trees, depth, n_features;
    uint32_t nan_left;
    float base;
    const uint8_t *feat;
    const float *thr;
    const float *leaf;
};

__device__ __forceinline__ int32_t walk(const ForestDev &f, const float *__restrict__ x, int32_t t)
{
    const int64_t n_int = ((int64_t)1 << f.depth) - 1;
    const uint8_t *__restrict__ feat = f.feat + t * n_int;
    const float *__restrict__ thr = f.thr + t * n_int;
    int64_t node = 0;
    for (int32_t l = 0; l < f.depth; ++l) {
        int32_t j = feat[node];
        j = j < f.n_features ? j : f.n_features - 1;
        const float v = x[j];
        const bool left = (v < thr[node]) || (f.nan_left && __builtin_isnan(v));
        node = 2 * node + (left ? 1 : 2);
    }
    return (int32_t)(node - n_int);
}

// Sum of a row's eight partial sums (partial i: the leaves of trees i, i + 8,
// ... added in that order), one order for every way a row is scored.
__device__ __forceinline__ float sum_partials(const float (&p)[8], float base)
{
    return base + (((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])));
}

// The leaves of trees t0 .. t0 + CH - 1 for one row, walked in step, added to p.
template <int CH>
__device__ __forceinline__ void add_leaves(const ForestDev &f, const float *__restrict__ x, int32_t t0, float (&p)[8])
{
    const int64_t n_int = ((int64_t)1 << f.depth) - 1, n_leaf = n_int + 1;
    uint32_t node[CH] = {};
    for (int l = 0; l < f.depth; ++l) {
        int j[CH];
        float th[CH], v[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const int64_t first = (t0 + c) * n_int;
            j[c] = (f.feat + first)[node[c]];
            th[c] = (f.thr + first)[node[c]];
        }
#pragma unroll
        for (int c = 0; c < CH; ++c) v[c] = x[j[c] < f.n_features ? j[c] : f.n_features - 1];
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const bool left = (v[c] < th[c]) | (f.nan_left && __builtin_isnan(v[c]));
            node[c] = 2 * node[c] + (left ? 1 : 2);
        }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c)
        p[c] += (f.leaf + (t0 + c) * n_leaf)[node[c] - (uint32_t)n_int];
}

// Direct walk of few trees: a row per thread, up to eight trees in step,
// everything read through the caches and only the columns the nodes name (see
// rows_visits).  Bound by the lines of X it gathers, a line per visit and row:
// 1,500,000 rows of 128 columns, 4 trees of depth 3, 204 us (tiles 421 us; one
// tree after another 307 us).
__global__ __launch_bounds__(256, 8) void k_forest_rows(ForestDev f, const float *__restrict__ X, int64_t R, int64_t ld,
                                                      float *__restrict__ scores)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= R) return;
    const float *__restrict__ x = X + r * ld;
    float p[8] = {};
    for (int32_t t0 = 0; t0 < f.n_trees; t0 += 8) {
        switch (f.n_trees - t0) {
        case 1: add_leaves<1>(f, x, t0, p); break;
        case 2: add_leaves<2>(f, x, t0, p); break;
        case 3: add_leaves<3>(f, x, t0, p); break;
        case 4: add_leaves<4>(f, x, t0, p); break;
        case 5: add_leaves<5>(f, x, t0, p); break;
        case 6: add_leaves<6>(f, x, t0, p); break;
        case 7: add_leaves<7>(f, x, t0, p); break;
        default: add_leaves<8>(f, x, t0, p);
        }
    }
    scores[r] = sum_partials(p, f.base);
}

// Orders a wave's own LDS accesses (its lanes exchange values through LDS).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}

// Direct walk of forests without an image.  A walk is a chain of dependent
// reads (node, then the row's value of the node's feature), scattered from
// the second level on: out of the caches each level costs up to three
// 64-line gathers per wave.  Here a workgroup holds T rows of X (transposed,
// [column][row]: a lane reads its own bank whatever its column) and the first
// kDirLevels levels of 8 C trees in LDS; wave w walks trees w % 8 (+ 8 c) for
// its 64 rows, C chains in flight, while the next trees' nodes are fetched
// into registers.  Leaves are added one group later, so that their gathers
// overlap the next walk.  LDS: 64 KB of X, 80 KB of nodes.  150 trees of depth
// 11 over 65,537 rows of 128 columns: 140 us (a row per thread, everything out
// of the caches: 726 us; 183 us with a test and a byte load per 64 slots in the
// fetch).  A tile takes 64 us, 3.3 us per group of trees: two dependent LDS
// reads per level and the group's 80 KB to fetch and store.
//
// The rows of an incomplete last round of tiles, and calls of few rows, would
// leave compute units idle: the first `tail_blocks` workgroups give such a
// row to one wave, a lane per tree, nodes read from the caches.  Both ways add
// a row's leaves in the same order.
constexpr int kDirLevels = 11;                 // levels in LDS: 8 trees of 2^11 nodes
constexpr int kDirSlots = 8 << kDirLevels;

// LL: the levels in LDS where they are 8 or more (C follows), 0 below.
template <int T, int C, int LL>
__global__ __launch_bounds__(8 * T, 1) void k_forest_direct(ForestDev f, const float *__restrict__ X, int64_t R,
                                                             int64_t ld, int64_t tail_rows, int32_t tail_blocks,
                                                             int32_t tail_per, float *__restrict__ scores)
{
    constexpr int kSlots = LL > 0 ? (8 * C) << LL : (8 * C) << 7;     // at most, of a group
    constexpr int NT = 8 * T, W = NT / 64, PER = kSlots / NT, kXWords = 16384;
    static_assert(PER * NT == kSlots && kSlots <= kDirSlots && PER % 4 == 0 && kXWords / W >= 256 && kDirSlots / W >= 256, "staging");
    __shared__ float xs[kXWords], thr_s[kDirSlots];
    // a tree's feature bytes: 2^L and up to 3 before them, since they are copied
    // as the aligned words they lie in, wherever the tree begins
    __shared__ uint32_t feat_s[kDirSlots / 4 + 8 * C];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n_int = ((int64_t)1 << f.depth) - 1, n_leaf = n_int + 1;
    const int nf = f.n_features;

    if ((int32_t)blockIdx.x < tail_blocks) {
        // no workgroup barrier on this side
        const int64_t i = (int64_t)blockIdx.x * tail_per + wave;
        if (wave >= tail_per || i >= tail_rows) return;
        const int64_t r = R - tail_rows + i;
        float *xw = xs + wave * (kXWords / W), *lw = thr_s + wave * (kDirSlots / W);
        for (int c = lane; c < nf; c += 64) xw[c] = X[r * ld + c];
        wave_lds_sync();
        float acc = 0.0f;                      // lane i < 8: partial i
        for (int32_t t0 = 0; t0 < f.n_trees; t0 += 256) {
            int64_t at[4];
            int32_t node[4] = {0, 0, 0, 0};
            const int chains = f.n_trees - t0 > 192 ? 4 : (f.n_trees - t0 + 63) / 64;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int32_t t = t0 + 64 * c + lane;
                at[c] = t < f.n_trees ? t : f.n_trees - 1;
            }
            for (int l = 0; l < f.depth; ++l) {
                int j[4];
                float th[4];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c < chains) {
                        j[c] = f.feat[at[c] * n_int + node[c]];
                        th[c] = f.thr[at[c] * n_int + node[c]];
                    }
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c < chains) {
                        const float v = xw[j[c] < nf ? j[c] : nf - 1];
                        const bool left = (v < th[c]) || (f.nan_left && __builtin_isnan(v));
                        node[c] = 2 * node[c] + (left ? 1 : 2);
                    }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c < chains) lw[64 * c + lane] = f.leaf[at[c] * n_leaf + (node[c] - n_int)];
            wave_lds_sync();
            const int m = f.n_trees - t0 < 256 ? f.n_trees - t0 : 256;
            if (lane < 8)
                for (int e = lane; e < m; e += 8) acc += lw[e];
            wave_lds_sync();
        }
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = __shfl(acc, e);
        if (lane == 0) scores[r] = sum_partials(p, f.base);
        return;
    }

    const int64_t row0 = (int64_t)((int32_t)blockIdx.x - tail_blocks) * T;
    // X: a wave's load takes 4 columns of 16 rows
    {
        const int quads = (nf + 3) / 4;
        for (int e = wave; e < quads * (T / 16); e += W) {
            const int row = (e % (T / 16)) * 16 + (lane >> 2), col = (e / (T / 16)) * 4 + (lane & 3);
            const int64_t r = row0 + row < R ? row0 + row : R - 1;
            if (col < nf) xs[col * T + row] = X[r * ld + col];
        }
    }
    const int L = LL > 0 ? LL : f.depth;
    const int slots = (8 * C) << L;            // node slots of a group, 2^L a tree
    const int LW = L > 2 ? L - 2 : 0;          // 2^LW words hold 2^L feature bytes
    const int words = (8 * C) << LW, word_stride = (1 << LW) + 1;
    float rt[PER];
    uint32_t rf[PER / 4], rf_last = 0;
    const uint32_t lane_short = lane < 63 ? lane : 62;         // a tree's last slot is no node
    // words of the features of tree t: the aligned word of its first byte, and
    // how far into it that byte is
    auto feat_words = [&](int32_t t, int &skip) {
        const uint8_t *at = f.feat + t * n_int;
        skip = (int)((uintptr_t)at & 3u);
        return reinterpret_cast<const uint32_t *>(at - skip);
    };
    // A group's nodes into registers.  Where all its trees exist the addresses
    // are scalar sums without a branch: tests per load cost as much issue time
    // as the walk.  (Slots of no tree are given nodes of zeros.)
    auto fetch_group = [&]<bool ALL>(int32_t t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e0 = wave * 64 + i * NT;
            if (!ALL) rt[i] = 0.0f;
            if (i * NT >= slots) continue;
            if (L >= 6) {                      // 64 slots of one tree: a scalar base
                const int32_t t = t0 + (e0 >> L);
                const int n0 = e0 & ((1 << L) - 1);
                if (ALL || (e0 < slots && t < f.n_trees))
                    rt[i] = (f.thr + t * n_int + n0)[n0 + 64 == 1 << L ? lane_short : lane];
            } else if (i * NT < 1024) {        // at most 32 trees of 32 slots
                const int32_t t = t0 + ((e0 + lane) >> L);
                const int n = (e0 + lane) & ((1 << L) - 1);
                if (e0 < slots && t < f.n_trees && n < (1 << L) - 1) rt[i] = f.thr[t * n_int + n];
            }
        }
        // a tree's first 2^LW words
#pragma unroll
        for (int i = 0; i < PER / 4; ++i) {
            const int e0 = wave * 64 + i * NT;
            int skip;
            if (!ALL) rf[i] = 0;
            if (i * NT >= words) continue;
            if (LW >= 6) {
                const int32_t t = t0 + (e0 >> LW);
                if (ALL || (e0 < words && t < f.n_trees)) rf[i] = (feat_words(t, skip) + (e0 & ((1 << LW) - 1)))[lane];
            } else if (i * NT < 1024) {
                const int32_t t = t0 + ((e0 + lane) >> LW);
                if (e0 + lane < words && t < f.n_trees) rf[i] = feat_words(t, skip)[(e0 + lane) & ((1 << LW) - 1)];
            }
        }
        // the word after those, where nodes reach into it
        const int32_t t = t0 + (int32_t)threadIdx.x;
        rf_last = 0;
        if (threadIdx.x < 8 * C && t < f.n_trees) {
            int skip;
            const uint32_t *w = feat_words(t, skip);
            if ((4 << LW) < skip + (1 << L) - 1) rf_last = w[1 << LW];
        }
    };
    auto fetch = [&](int32_t t0) __attribute__((always_inline)) {
        // (LL > 0: every slot and word of a whole group is some wave's)
        if (LL > 0 && t0 + 8 * C <= f.n_trees) fetch_group.template operator()<true>(t0);
        else fetch_group.template operator()<false>(t0);
    };
    auto store = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (i * NT < slots) {
                const int e0 = wave * 64 + i * NT;
                if (LL > 0 || e0 < slots) thr_s[e0 + lane] = rt[i];
            }
#pragma unroll
        for (int i = 0; i < PER / 4; ++i)
            if (i * NT < words) {
                const int e = wave * 64 + i * NT + lane;
                if (LL > 0 || e < words) feat_s[(e >> LW) * word_stride + (e & ((1 << LW) - 1))] = rf[i];
            }
        if (threadIdx.x < 8 * C) feat_s[threadIdx.x * word_stride + (1 << LW)] = rf_last;
    };
    fetch(0);
    store();
    lds_barrier();
    const int g = wave & 7, row = (wave >> 3) * 64 + lane;
    float acc = 0.0f, pend[C];
#pragma unroll
    for (int c = 0; c < C; ++c) pend[c] = 0.0f;
    for (int32_t t0 = 0; t0 < f.n_trees; t0 += 8 * C) {
        const bool more = t0 + 8 * C < f.n_trees;
        if (more) fetch(t0 + 8 * C);
        // chains past the last tree walk nodes of zeros and read no leaf
        int32_t node[C];
        const uint8_t *feat[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            int skip;
            feat_words(t0 + 8 * c + g, skip);
            node[c] = 0;
            feat[c] = reinterpret_cast<const uint8_t *>(feat_s + (8 * c + g) * word_stride) + skip;
        }
#pragma unroll 1
        for (int l = 0; l < L; ++l) {
            float th[C], v[C];
            int j[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                j[c] = feat[c][node[c]];
                th[c] = thr_s[((8 * c + g) << L) + node[c]];
            }
#pragma unroll
            for (int c = 0; c < C; ++c) v[c] = xs[(j[c] < nf ? j[c] : nf - 1) * T + row];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const bool left = (v[c] < th[c]) | (f.nan_left && __builtin_isnan(v[c]));
                node[c] = 2 * node[c] + (left ? 1 : 2);
            }
        }
#pragma unroll
        for (int c = 0; c < C; ++c) acc += pend[c];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int32_t t = t0 + 8 * c + g;
            pend[c] = 0.0f;
            if (t < f.n_trees) {
                for (int l = L; l < f.depth; ++l) {            // below the staged levels
                    int j = f.feat[t * n_int + node[c]];
                    j = j < nf ? j : nf - 1;
                    const float v = xs[j * T + row];
                    const bool left = (v < f.thr[t * n_int + node[c]]) || (f.nan_left && __builtin_isnan(v));
                    node[c] = 2 * node[c] + (left ? 1 : 2);
                }
                pend[c] = f.leaf[t * n_leaf + (node[c] - n_int)];
            }
        }
        lds_barrier();                         // every wave is done with these trees
        if (more) store();
        lds_barrier();
    }
#pragma unroll
    for (int c = 0; c < C; ++c) acc += pend[c];
    thr_s[g * T + row] = acc;
    lds_barrier();
    if ((int)threadIdx.x < T && row0 + threadIdx.x < R - tail_rows) {
        float p[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) p[e] = thr_s[e * T + threadIdx.x];
        scores[row0 + threadIdx.x] = sum_partials(p, f.base);
    }
}

__global__ __launch_bounds__(256) void k_forest_leaves(ForestDev f, const float *__restrict__ X, int64_t R,
                                                        int64_t ld, const int64_t *__restrict__ rows,
                                                        int64_t n_rows, uint16_t *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_rows) return;
    int64_t r = rows[i];
    r = r < 0 ? 0 : (r >= R ? R - 1 : r);
    const float *x = X + r * ld;
    for (int32_t t = 0; t < f.n_trees; ++t) out[i * f.n_trees + t] = (uint16_t)walk(f, x, t);
}

ForestDev to_dev(const hwsel_forest_t &f)
{
    return ForestDev{f.n_trees, f.depth, f.n_features, f.flags & 1u, f.base_score,
                     f.node_feature, f.node_threshold, f.leaf_value};
}

// ---------------------------------------------------------------------------
// Packed path: layout
// ---------------------------------------------------------------------------
constexpr int kBinSlots = 256;        // thresholds per feature incl. padding
// Bin table in LDS: threshold i of feature f at word
// (f / 32) * 32 * kBinSlots + 32 * i + f % 32, so the 32 features searched by
// a half-wave each stay on their own bank whatever their search positions.
__host__ __device__ constexpr int bin_table_index(int f, int i) { return (f >> 5) * 32 * kBinSlots + 32 * i + (f & 31); }
constexpr int kWaves = 16;            // waves per traversal workgroup
constexpr int kSliceRows = 16;        // rows of a tile per wave
constexpr int kTileRows = kWaves * kSliceRows;
constexpr int kXcds = 8;
constexpr int kSlotsPerXcd = 32;      // one workgroup per CU
constexpr int kBinThreads = 1024;

// Node codes (u16: feature | rank << 8) are stored in the image as sibling
// pairs: the 4-byte word of pair p holds nodes 2p (low half) and 2p + 1 (high
// half), so one word holds both children of node p (pair 0 holds the root in
// its high half).  Pair p of every tree sits in row p, tree t in 4-byte column
// t; with 16 trees per image chunk (depth 10) every tree is stored twice, in
// columns t and 16 + t: the walk reads the first copy only, the second keeps
// the format that saved images have.
__host__ __device__ constexpr int node_copies(int tc) { return tc == 16 ? 2 : 1; }
__host__ __device__ constexpr uint32_t pair_row_bytes(int tc) { return tc == 64 ? 256u : 128u; }

__host__ __device__ inline uint32_t node_byte(uint32_t n, int t, int copy, int tc)
{
    return (n >> 1) * pair_row_bytes(tc) + 4u * (uint32_t)(copy * 16 + t) + 2u * (n & 1u);
}

struct PackGeom {
    int tc, n_chunks, slots, stride;      // trees per chunk, chunks, heap slots (2^D), bin row bytes
    size_t thr_bytes, chunk_bytes, node_bytes, total;
};

// Trees per image chunk: about 96 KB of nodes (2 B) and leaves (4 B).
int trees_per_chunk(int depth)
{
    int tc = 64;
    while (tc > 1 && (size_t)tc * ((size_t)6 << depth) > 96 * 1024) tc >>= 1;
    return tc;
}

PackGeom geometry(const hwsel_forest_t &f)
{
    PackGeom g;
    g.tc = trees_per_chunk(f.depth);
    g.n_chunks = (f.n_trees + g.tc - 1) / g.tc;
    g.slots = 1 << f.depth;
    g.stride = (f.n_features + 15) / 16 * 16;
    g.thr_bytes = (size_t)f.n_features * kBinSlots * sizeof(float);
    g.node_bytes = (size_t)g.slots * g.tc * 2 * node_copies(g.tc);
    g.chunk_bytes = g.node_bytes + (size_t)g.slots * g.tc * 4;
    g.total = 256 + g.thr_bytes + (size_t)g.n_chunks * g.chunk_bytes;
    return g;
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

constexpr int32_t kImageMagic = 0x48575346;   // "FSWH"
constexpr int32_t kImageVersion = 2;

ImageId image_id(const hwsel_forest_t &f, const PackGeom &g)
{
    return ImageId{kImageMagic, kImageVersion, f.n_trees, f.depth, f.n_features, g.tc, g.n_chunks};
}

// Check outputs of the packed traversal (hwsel_forest_score_checked).
struct LeafHook {
    uint64_t *hash;          // [R] or null: leaf-path fingerprint per row
    uint16_t *idx;           // [n_rows][n_trees] or null: leaf indices of rows [row0, row0 + n_rows)
    int64_t row0, n_rows;
    int32_t n_trees;
};

// 64-bit finaliser of SplitMix64 (Steele, Lea and Flood, OOPSLA 2014): a
// bijection, so the fingerprint sum changes whenever one leaf does.
__device__ __forceinline__ uint64_t leaf_mix(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// Wrapping sum of a 64-bit value over the TC consecutive lanes of a group.
template <int TC>
__device__ __forceinline__ uint64_t group_sum_u64(uint64_t h)
{
#pragma unroll
    for (int o = 1; o < TC; o <<= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)h, o, 64), hi = __shfl_xor((uint32_t)(h >> 32), o, 64);
        h += ((uint64_t)hi << 32) | lo;
    }
    return h;
}

__global__ void k_fill_u64(uint64_t *__restrict__ a, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0;
}

// ---------------------------------------------------------------------------
// Packed path: kernels
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBinThreads, 1) void k_bin(const float *__restrict__ X, int64_t R, int64_t ld,
                                                         const void *__restrict__ packed, ImageId id, int nf,
                                                         uint32_t nan_bin, uint8_t *__restrict__ Xb, int stride)
{
    if (!image_matches(packed, id)) return;
    const float *__restrict__ U = reinterpret_cast<const float *>(static_cast<const uint8_t *>(packed) + 256);
    // thresholds as order-preserving keys; index i of feature f at
    // bin_table_index(f, i), so each searched feature stays on its own bank
    __shared__ uint32_t u[128 * kBinSlots];
    for (int e = threadIdx.x; e < nf * kBinSlots; e += kBinThreads)
        u[bin_table_index(e >> 8, e & 255)] = order_key(U[e]);
    __syncthreads();
    const int f = threadIdx.x & 127;
    // 8 row lanes per block; a wave's 64 threads share one, so the row
    // arithmetic below stays scalar
    const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
    if (f >= stride) return;
    const uint8_t *uf = reinterpret_cast<const uint8_t *>(u + bin_table_index(f, 0));
    constexpr int kRowsPerThread = 8;                 // independent searches in flight
    const int64_t step_rows = (int64_t)gridDim.x * 8 * kRowsPerThread;
    // the next group's values are requested before this group's searches,
    // so the trip to HBM overlaps them
    // Branch-free: rows past R read row R - 1 and columns past nf read
    // column nf - 1 (R, nf >= 1); neither result is stored as such.
    const int fc = f < nf ? f : nf - 1;
    auto fetch = [&](int64_t r0, float (&x)[kRowsPerThread]) {
#pragma unroll
        for (int q = 0; q < kRowsPerThread; ++q) {
            const int64_t r = r0 + q;
            x[q] = X[(r < R ? r : R - 1) * ld + fc];
        }
    };
    float xn[kRowsPerThread];
    fetch(((int64_t)blockIdx.x * 8 + sub) * kRowsPerThread, xn);
    for (int64_t r0 = ((int64_t)blockIdx.x * 8 + sub) * kRowsPerThread; r0 < R; r0 += step_rows) {
        float x[kRowsPerThread];
        uint32_t kx1[kRowsPerThread], b[kRowsPerThread];
#pragma unroll
        for (int q = 0; q < kRowsPerThread; ++q) x[q] = xn[q];
        fetch(r0 + step_rows, xn);
#pragma unroll
        for (int q = 0; q < kRowsPerThread; ++q) {
            kx1[q] = order_key(x[q] == 0.0f ? 0.0f : x[q]) + 1u;
            b[q] = 0;
        }
        // b = #{u <= x} built from the top bit: at step k the probe is
        // threshold (b << (k + 1)) + 2^k - 1 (rows of 32 words, 128 bytes)
#pragma unroll
        for (int k = 7; k >= 0; --k) {
#pragma unroll
            for (int q = 0; q < kRowsPerThread; ++q) {
                const uint32_t key_u =
                    *reinterpret_cast<const uint32_t *>(uf + (b[q] << (k + 8)) + 128u * ((1u << k) - 1u));
                b[q] = search_step(b[q], key_u, kx1[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < kRowsPerThread; ++q) {
            if (r0 + q >= R) break;
            uint32_t v = b[q];
            if (x[q] != x[q]) v = nan_bin;
            if (f >= nf) v = 0;
            Xb[(r0 + q) * stride + f] = (uint8_t)v;
        }
    }
}

// One level of a walk: node <- 2*node + (bin > rank), with node the index
// among its level's nodes (0 at the root, the leaf's index at the end) and
// rank the high byte of the node code.  Subtract-with-borrow leaves (bin > rank) in VCC and
// add-with-carry folds it in: two VALU instructions per visit.
__device__ __forceinline__ int descend(int node, uint32_t code, uint32_t bin)
{
    int out;
    asm("v_sub_co_u32_sdwa %0, vcc, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t"
        "v_addc_co_u32_e32 %0, vcc, %3, %3, vcc"
        : "=&v"(out)
        : "v"(code), "v"(bin), "v"(node)
        : "vcc");
    return out;
}

// The first level of a group (x: root code | left child's << 16, y: right
// child's code): descend() that also takes the chosen child's code with the
// same carry.
__device__ __forceinline__ uint32_t descend_group(int &node, uint32_t x, uint32_t y, uint32_t bin)
{
    int n_out;
    uint32_t code, scratch;
    asm("v_sub_co_u32_sdwa %2, vcc, %3, %5 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_1 src1_sel:DWORD\n\t"
        "v_cndmask_b32_sdwa %1, %3, %4, vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_0\n\t"
        "v_addc_co_u32_e32 %0, vcc, %6, %6, vcc"
        : "=&v"(n_out), "=&v"(code), "=&v"(scratch)
        : "v"(x), "v"(y), "v"(bin), "v"(node)
        : "vcc");
    node = n_out;
    return code;
}

// 32 * (low or high 16 bits of p) + c, one instruction.
template <int HIGH>
__device__ __forceinline__ uint32_t mad32_u16(uint32_t p, uint32_t c)
{
    uint32_t out;
    if constexpr (HIGH)
        asm("v_mad_u32_u16 %0, %1, 32, %2 op_sel:[1,0,0,0]" : "=v"(out) : "v"(p), "v"(c));
    else
        asm("v_mad_u32_u16 %0, %1, 32, %2" : "=v"(out) : "v"(p), "v"(c));
    return out;
}

// Rows of two registers gathered: a keeps its even 16-lane rows and takes b's
// even rows into its odd ones; b gets the odd rows of both.
__device__ __forceinline__ void swap16(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

__device__ __forceinline__ void swap32(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// lanes (l & BIT) == 0: a[l] + a[partner], the others: b[l] + b[partner]; the
// partner is l ^ 8 (row_ror:8) for BIT = 8 and the mirror in 8 lanes for BIT = 4.
template <int BIT>
__device__ __forceinline__ float fold(float a, float b, bool upper)
{
    const float own = upper ? b : a, other = upper ? a : b;
    return own + dpp_f32<BIT == 8 ? 0x128 : 0x141>(other);
}

// Sum over the four lanes of a quad, in all of them.
__device__ __forceinline__ float quad_total(float v)
{
    v += dpp_f32<0xb1>(v);        // quad_perm [1,0,3,2]
    return v + dpp_f32<0x4e>(v);  // quad_perm [2,3,0,1]
}

// The walk of one packed chunk by one wave: shapes, all known from the depth.
//   * A wave takes its 16 rows at a time, in sets of 8 registers of walks,
//     each 64 / TC rows x TC trees.  Register a of a set, half s (TC = 32) walks row
//       TC = 64: 4 (a & 1) + 2 (a >> 1 & 1) + (a >> 2)           of 8,
//       TC = 32: 8 s + 4 (a & 1) + 2 (a >> 1 & 1) + (a >> 2)     of 16,
//     the order in which the row sums come out of the lane folds below.
//   * Levels go two at a time: a group is a node and its two children, 6 of
//     8 bytes, read at once; tree t's groups are in 8-byte column t of rows
//     of 8 TC bytes, so the lanes of a half-wave hit distinct banks.  Two levels
//     cost eight VALU instructions (bin address, compare, child's code, node
//     index; bin address, compare, node index; group address) and three LDS
//     reads, against ten and four when a level reads its sibling pair alone.
//     The root group (the root alone when the depth is odd) sits in registers.
//   * With TC = 64 or 32 a half-wave reads the bins of one row, whose 32
//     words lie on the 32 banks (two rows of 16 trees, as a chunk of 16
//     depth-10 trees with its leaves would give, meet on almost every read:
//     2 passes instead of 1).
// Bound by VALU issue, then LDS.  Measured, against one level per step, 16-tree
// chunks at depth 10 and every row's sum folded on its own: 4,915,200 rows x
// 2,000 trees of depth 10, whole call 20.40 -> 16.35 ms; 1,000,003 rows x 500
// trees of depth 8 on 96 columns 1.02 -> 0.79 ms.
template <int D>
struct Walk {
    static constexpr int TC = D <= 8 ? 64 : 32;
    static constexpr bool DEFER = D == 10;              // leaves do not fit next to the groups
    static constexpr int RPI = 64 / TC;
    static constexpr int STEP_ROWS = 8 * RPI;           // rows of one 8-register set
    static constexpr int STEPS = kSliceRows / STEP_ROWS;
    static constexpr int NS = 1 << D;
    static constexpr int L0 = D & 1;                    // first level that is in a group
    static constexpr int PAIRS = D / 2;
    static constexpr int start(int p) { return (L0 ? 2 : 1) * ((1 << (2 * p)) - 1) / 3; }   // first group row of pair p
    static constexpr int first(int p) { return 1 << (L0 + 2 * p); }                         // its first node
    static constexpr int GROUPS = start(PAIRS);
    static constexpr int ROW_SHIFT = TC == 64 ? 9 : 8;  // 8 TC bytes per group row
    static constexpr int GROUP_B = GROUPS << ROW_SHIFT;
    static constexpr int LEAF_TREES = DEFER ? 8 : TC;   // trees whose leaves are in LDS at a time
    static constexpr int LEAF_B = NS * LEAF_TREES * 4;
    static constexpr int BINS_AT = GROUP_B + LEAF_B;
    static constexpr int LDS_B = BINS_AT + kWaves * kSliceRows * 128;
    static_assert(LDS_B <= 160 * 1024, "LDS");
    // Leaf parts cost a pass over their trees' leaves and two barriers each:
    // with deferred leaves a wave holds the leaf indices of several tiles (two
    // per register) before the parts go through LDS, kDefer where it has them.
    static constexpr int kDefer = DEFER ? 8 : 1;
};

// Chunks the traversal takes the trees in: at depth 10 two of the image's
// 16-tree chunks at a time.
constexpr int walk_chunks(int depth, int image_chunks) { return depth == 10 ? (image_chunks + 1) / 2 : image_chunks; }

// KD: tiles whose leaves are deferred together.  Eight keep every register in
// use and spill some, which a bulk of rows does not notice; but the first
// accesses to spilled registers go to memory, and an item of one tile (32 trees
// of depth 10) took 15 us.  With the kernel for one tile it takes 10 us; items
// of up to four have one as well (60,000 rows, 64 trees: 53 -> 48 us a call).
template <int D, bool HOOK, int KD>
__global__ __launch_bounds__(64 * kWaves, 1) void k_traverse(const void *__restrict__ packed, ImageId id,
                                                              const uint8_t *__restrict__ chunks, int image_chunks,
                                                              int n_chunks, const uint8_t *__restrict__ Xb, int64_t R,
                                                              int stride, int domains, int groups,
                                                              int64_t rows_per_group, float *__restrict__ partial,
                                                              LeafHook hook)
{
    if (!image_matches(packed, id)) return;
    using W = Walk<D>;
    constexpr int TC = W::TC, NS = W::NS;
    constexpr bool kFew = KD < W::kDefer;                  // few tiles per item: latency counts
    __shared__ __attribute__((aligned(16))) uint8_t lds[W::LDS_B];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = lane % TC, s = lane / TC;
    const bool up8 = (lane & 8) != 0, up4 = (lane & 4) != 0;
    // Domain 8: workgroup b is on XCD b % 8 and the XCD's workgroups take its
    // row groups in turn, neighbours with different chunks.  Domain 1: the
    // rows fit in every L2 and neighbours take one chunk's row groups.
    const int xcd = blockIdx.x % kXcds;
    const int slot = domains == 1 ? xcd * kSlotsPerXcd + blockIdx.x / kXcds : blockIdx.x / kXcds;
    const int slots = domains == 1 ? gridDim.x : gridDim.x / kXcds;
    const int items = n_chunks * groups;
    // Each wave owns kSliceRows rows of every tile and a private LDS region
    // for their bins, which it refills on its own (no workgroup barrier
    // between tiles).
    constexpr int kVec = kSliceRows * 8 / 64;             // uint4 per lane, 128-byte rows
    const uint32_t region = W::BINS_AT + wave * kSliceRows * 128;
    const uint32_t row_base = region + s * 8 * 128;       // the lane's row 0 (see Walk)
    const int vpr = stride >> 4;                          // uint4 per bin row
    uint32_t put_at[kVec];
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        const int e = lane + 64 * q;
        put_at[q] = region + (e / vpr) * 128 + 16 * (e % vpr);
    }
    const int n_vec = kSliceRows * vpr;                   // uint4 of a whole slice

    for (int item = slot; item < items; item += slots) {
        const int c = domains == 1 ? item / groups : item % n_chunks;
        const int64_t g = domains == 1 ? item % groups : (int64_t)xcd * groups + item / n_chunks;
        const int64_t r_begin = g * rows_per_group;
        const int64_t r_end = r_begin + rows_per_group < R ? r_begin + rows_per_group : R;
        if (r_begin >= r_end) continue;                   // workgroup-uniform
        // the image's chunk(s) of these trees: node pairs, then leaves
        constexpr int ITC = D <= 8 ? 64 : D == 9 ? 32 : 16;
        constexpr int kPairRow = pair_row_bytes(ITC), kImageNodes = NS * ITC * 2 * node_copies(ITC);
        constexpr int kImageChunk = kImageNodes + NS * ITC * 4;
        constexpr int kSub = TC / ITC;                    // image chunks per chunk
        const uint8_t *image = chunks + (size_t)c * kSub * kImageChunk;
        const int have = image_chunks - c * kSub < kSub ? image_chunks - c * kSub : kSub;
        // The code of node n (1 at the root, children 2n and 2n + 1) and its
        // children's codes, for the chunk's tree tt; trees past the image's
        // chunks read an earlier chunk (in bounds) and become 0.
        auto node_at = [&](int tt) { return image + (tt / ITC < have ? tt / ITC : 0) * kImageChunk; };
        auto node_code = [&](uint32_t n, int tt) -> uint32_t {
            const uint32_t v = *reinterpret_cast<const uint16_t *>(node_at(tt) + node_byte(n, tt % ITC, 0, ITC));
            return tt / ITC < have ? v : 0u;
        };
        auto node_pair = [&](uint32_t n, int tt) -> uint32_t {
            const uint32_t v = *reinterpret_cast<const uint32_t *>(node_at(tt) + n * kPairRow + 4 * (tt % ITC));
            return tt / ITC < have ? v : 0u;
        };
        uint4 preA[kVec], preB[kVec];
        auto fetch = [&](int64_t t0, uint4 (&pre)[kVec]) {
            const int64_t w0 = t0 + wave * kSliceRows;
            const uint4 *slice = reinterpret_cast<const uint4 *>(Xb + w0 * stride);    // wave-uniform
            const int64_t left = (r_end - w0) * vpr;                                  // uint4 left
            if (n_vec == 64 * kVec && left >= n_vec) {
#pragma unroll
                for (int q = 0; q < kVec; ++q) pre[q] = slice[lane + 64 * q];
            } else {
                const int n = left < 0 ? 0 : left < n_vec ? (int)left : n_vec;
#pragma unroll
                for (int q = 0; q < kVec; ++q)
                    pre[q] = lane + 64 * q < n ? slice[lane + 64 * q] : make_uint4(0, 0, 0, 0);
            }
        };
        uint32_t root_x, root_y;                          // the root group is the same for every row
        auto fetch_root = [&]() {
            const uint32_t kids = D >= 2 ? node_pair(1, t) : 0u;
            root_x = node_code(1, t) | (kids << 16);
            root_y = kids >> 16;
        };
        // Two tiles in flight: a tile's bins are requested two tiles before
        // they are written to LDS, alternating between two register buffers.
        auto fetch_first = [&]() {
            fetch(r_begin, preA);
            if (KD > 1 || !W::DEFER) fetch(r_begin + kTileRows, preB);
        };
        auto first_node = [&](int row) {                  // of a group
            uint32_t n = row - W::start(0) + W::first(0);
#pragma unroll
            for (int p = 1; p < W::PAIRS; ++p)
                if (row >= W::start(p)) n = row - W::start(p) + W::first(p);
            return n;
        };
        __syncthreads();                                  // the previous item's LDS is no longer read
        // a thread's groups are all of one tree
        constexpr int kRowsAtOnce = 64 * kWaves / TC;
        const int tree = threadIdx.x % TC, row0 = threadIdx.x / TC;
        const uint8_t *const base = node_at(tree) + 4 * (tree % ITC);
        const bool there = tree / ITC < have;
#pragma unroll 4
        for (int row = row0; row < W::GROUPS; row += kRowsAtOnce) {
            const uint32_t n = first_node(row);
            uint32_t own = *reinterpret_cast<const uint16_t *>(base + (n >> 1) * kPairRow + 2 * (n & 1));
            uint32_t kids = *reinterpret_cast<const uint32_t *>(base + n * kPairRow);
            own = there ? own : 0u;
            kids = there ? kids : 0u;
            *reinterpret_cast<uint2 *>(lds + (row << W::ROW_SHIFT) + 8 * tree) = make_uint2(own | (kids << 16), kids >> 16);
        }
        // the leaves of part q (deferred) as a thread stages them
        constexpr int kLeafVec = (W::LEAF_B / 16 + 64 * kWaves - 1) / (64 * kWaves);
        uint4 leaf_pre[kFew ? 4 : 1][W::DEFER ? kLeafVec : 1];
        auto fetch_leaves = [&](int q) {
            if constexpr (W::DEFER) {
                const int sub = q * W::LEAF_TREES / ITC;
#pragma unroll
                for (int i = 0; i < kLeafVec; ++i) {
                    const int e = threadIdx.x + i * 64 * kWaves;      // 16 bytes: half of a leaf's 8 trees
                    leaf_pre[kFew ? q : 0][i] = *reinterpret_cast<const uint4 *>(image + (sub < have ? sub : 0) * kImageChunk + kImageNodes +
                                                                   (e >> 1) * (ITC * 4) +
                                                                   (q * W::LEAF_TREES % ITC) * 4 + (e & 1) * 16);
                    if (sub >= have) leaf_pre[kFew ? q : 0][i] = make_uint4(0, 0, 0, 0);
                }
            }
        };
        if constexpr (!W::DEFER) {
            const uint4 *src = reinterpret_cast<const uint4 *>(image + kImageNodes);
            uint4 *dst = reinterpret_cast<uint4 *>(lds + W::GROUP_B);
#pragma unroll 4
            for (int e = threadIdx.x; e < W::LEAF_B / 16; e += 64 * kWaves) dst[e] = src[e];
        }
        fetch_root();
        __syncthreads();

        // packed leaf indices of the deferred steps, and their sums
        uint32_t held[KD][4];

        // One slice of rows: bins to LDS, then the walks, all sets in step.
        auto slice = [&](int64_t t0, uint4 (&pre)[kVec], uint32_t (&hold)[4]) {
            const int64_t w0 = t0 + wave * kSliceRows;
            // The previous rows' reads have all returned (their results were
            // used), so the region can be overwritten.
#pragma unroll
            for (int q = 0; q < kVec; ++q)
                if (lane + 64 * q < n_vec) *reinterpret_cast<uint4 *>(lds + put_at[q]) = pre[q];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the region is written before any lane reads it
            fetch(t0 + 2 * kTileRows, pre);
            if (w0 >= r_end) return;                              // wave-uniform: no rows left here
            {
                constexpr int NW = 8 * W::STEPS;
                int node[NW];
                uint32_t x[NW], y[NW], bin[NW];
                auto bin_at = [&](int a, uint32_t code) -> uint32_t {
                    return lds[row_base + (code & 0xffu) + (4 * (a & 1) + 2 * ((a >> 1) & 1) + ((a >> 2) & 1) + (a >> 3) * W::STEP_ROWS) * 128];
                };
#pragma unroll
                for (int a = 0; a < NW; ++a) {
                    node[a] = 0;
                    x[a] = root_x;
                    y[a] = root_y;
                }
                if constexpr (W::L0) {
#pragma unroll
                    for (int a = 0; a < NW; ++a) bin[a] = bin_at(a, x[a]);
#pragma unroll
                    for (int a = 0; a < NW; ++a) node[a] = descend(node[a], x[a], bin[a]);
                }
#pragma unroll
                for (int p = 0; p < W::PAIRS; ++p) {
                    if (W::L0 || p > 0) {
#pragma unroll
                        for (int a = 0; a < NW; ++a) {
                            const uint2 gr = *reinterpret_cast<const uint2 *>(
                                lds + ((uint32_t)node[a] << W::ROW_SHIFT) + 8 * t + (W::start(p) << W::ROW_SHIFT));
                            x[a] = gr.x;
                            y[a] = gr.y;
                        }
                    }
#pragma unroll
                    for (int a = 0; a < NW; ++a) bin[a] = bin_at(a, x[a]);
#pragma unroll
                    for (int a = 0; a < NW; ++a) x[a] = descend_group(node[a], x[a], y[a], bin[a]);
#pragma unroll
                    for (int a = 0; a < NW; ++a) bin[a] = bin_at(a, x[a]);
#pragma unroll
                    for (int a = 0; a < NW; ++a) node[a] = descend(node[a], x[a], bin[a]);
                }
#pragma unroll
                for (int it = 0; it < W::STEPS; ++it) {
                    const int *nd = node + 8 * it;
                    const int64_t step0 = w0 + it * W::STEP_ROWS;
                    if constexpr (HOOK) {
#pragma unroll
                        for (int a = 0; a < 8; ++a) {
                            const int64_t row = step0 + 8 * s + 4 * (a & 1) + 2 * ((a >> 1) & 1) + (a >> 2);
                            const int32_t tree = c * TC + t;
                            const uint32_t leaf = (uint32_t)nd[a];
                            const bool real = row < r_end && tree < hook.n_trees;   // padding trees count for nothing
                            const uint64_t h =
                                group_sum_u64<TC>(real ? leaf_mix(((uint64_t)tree << 32) | leaf) : 0ull);
                            if (hook.hash && t == 0 && row < r_end)
                                atomicAdd(reinterpret_cast<unsigned long long *>(hook.hash + row), (unsigned long long)h);
                            if (hook.idx && real && row >= hook.row0 && row < hook.row0 + hook.n_rows)
                                hook.idx[(row - hook.row0) * hook.n_trees + tree] = (uint16_t)leaf;
                        }
                    }
                    if constexpr (W::DEFER) {
                        // Registers a and a + 4 share one; then the lanes of
                        // trees 0-7, 8-15, 16-23, 24-31 are gathered into one
                        // register each: 8-lane group i of hold[q] is row 2i (low
                        // half) and row 2i + 1 (high half) for trees 8q .. 8q + 7.
                        uint32_t p[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) p[j] = ((uint32_t)nd[j + 4] << 16) | (uint32_t)nd[j];
                        swap16(p[0], p[1]);
                        swap16(p[2], p[3]);
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            hold[2 * j] = (uint32_t)__builtin_amdgcn_update_dpp((int)p[j], (int)p[j + 2], 0x128, 0xf, 0xc,
                                                                                false);
                            hold[2 * j + 1] = (uint32_t)__builtin_amdgcn_update_dpp((int)p[j + 2], (int)p[j], 0x128, 0xf,
                                                                                    0x3, false);
                        }
                    } else {
                        // Leaves of all walks first, then the sums over the
                        // trees: every fold halves the registers, so eight
                        // rows' sums of 64 trees cost 18 instructions (48 with
                        // each reduced on its own).
                        float v[8];
#pragma unroll
                        for (int a = 0; a < 8; ++a)
                            v[a] = *reinterpret_cast<const float *>(lds + (uint32_t)nd[a] * (TC * 4) + 4 * t + W::GROUP_B);
                        auto add_swapped = [&](float a, float b) {
                            uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
                            if constexpr (TC == 64) swap32(ua, ub);
                            else swap16(ua, ub);
                            return __uint_as_float(ua) + __uint_as_float(ub);
                        };
                        float w[4];
#pragma unroll
                        for (int m = 0; m < 4; ++m) w[m] = add_swapped(v[2 * m], v[2 * m + 1]);
                        float *out = partial + (int64_t)c * R + step0;
                        if constexpr (TC == 64) {
                            // 16-lane rows: registers 0 2 1 3 (4 6 5 7)
                            auto add16 = [&](float a, float b) {
                                uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
                                swap16(ua, ub);
                                return __uint_as_float(ua) + __uint_as_float(ub);
                            };
                            float z = fold<8>(add16(w[0], w[1]), add16(w[2], w[3]), up8);
                            z = quad_total(z + dpp_f32<0x141>(z));
                            if ((lane & 7) == 0 && step0 + (lane >> 3) < r_end) out[lane >> 3] = z;
                        } else {
                            const float z = quad_total(fold<4>(fold<8>(w[0], w[1], up8), fold<8>(w[2], w[3], up8), up4));
                            if ((lane & 3) == 0 && step0 + (lane >> 2) < r_end) out[lane >> 2] = z;
                        }
                    }
                }
            }
        };
        fetch_first();
        if constexpr (!W::DEFER) {
            for (int64_t t0 = r_begin; t0 < r_end; t0 += 2 * kTileRows) {
                slice(t0, preA, held[0]);
                if (t0 + kTileRows < r_end) slice(t0 + kTileRows, preB, held[0]);
            }
        } else {
            const uint32_t leaf0 = W::GROUP_B + 4 * (lane & 7);
            for (int64_t t0 = r_begin; t0 < r_end; t0 += KD * kTileRows) {
#pragma unroll
                for (int k = 0; k < KD; ++k) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) held[k][q] = 0u;             // rows past the end: leaf 0
                    if (k == KD - 1) fetch_leaves(0);
                    if (t0 + k * kTileRows < r_end) slice(t0 + k * kTileRows, k % 2 ? preB : preA, held[k]);
                }
                // The parts' leaves go through LDS in turn; every wave adds
                // its held walks' leaves of the part.
                float lo[KD], hi[KD];
                if (kFew) {
                    __builtin_amdgcn_sched_barrier(0);               // after the walks, whose registers they take
#pragma unroll
                    for (int q = 1; q < 4; ++q) fetch_leaves(q);
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    lds_barrier();                         // the buffer's last readers are done
#pragma unroll
                    for (int i = 0; i < kLeafVec; ++i)
                        *reinterpret_cast<uint4 *>(lds + W::GROUP_B + (threadIdx.x + i * 64 * kWaves) * 16) = leaf_pre[kFew ? q : 0][i];
                    if (!kFew && q < 3) fetch_leaves(q + 1);
                    lds_barrier();
                    float vl[KD], vh[KD];
#pragma unroll
                    for (int k = 0; k < KD; ++k) {
                        vl[k] = *reinterpret_cast<const float *>(lds + mad32_u16<0>(held[k][q], leaf0));
                        vh[k] = *reinterpret_cast<const float *>(lds + mad32_u16<1>(held[k][q], leaf0));
                    }
#pragma unroll
                    for (int k = 0; k < KD; ++k) {
                        lo[k] = q == 0 ? vl[k] : lo[k] + vl[k];
                        hi[k] = q == 0 ? vh[k] : hi[k] + vh[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < KD; ++k) {
                    const float z = quad_total(fold<4>(lo[k], hi[k], up4));
                    // 8-lane group i holds rows 2i (lower quad) and 2i + 1
                    const int64_t row = t0 + k * kTileRows + wave * kSliceRows + (lane >> 2);
                    if ((lane & 3) == 0 && row < r_end) partial[(int64_t)c * R + row] = z;
                }
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_reduce(const void *__restrict__ packed, ImageId id,
                                                 const float *__restrict__ partial, int n_chunks, int64_t R,
                                                 float base, float *__restrict__ scores)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    if (!image_matches(packed, id)) {
        scores[r] = __builtin_nanf("");
        return;
    }
    float acc = base;
    for (int c = 0; c < n_chunks; ++c) acc += partial[(int64_t)c * R + r];
    scores[r] = acc;
}

// Four rows per thread with 16-byte loads (R % 4 == 0, so every chunk's
// partial row starts 16-byte aligned); same chunk order per row.
__global__ __launch_bounds__(256) void k_reduce4(const void *__restrict__ packed, ImageId id,
                                                  const float *__restrict__ partial, int n_chunks, int64_t R,
                                                  float base, float *__restrict__ scores)
{
    const int64_t r = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (r >= R) return;
    if (!image_matches(packed, id)) {
        const float q = __builtin_nanf("");
        *reinterpret_cast<float4 *>(scores + r) = make_float4(q, q, q, q);
        return;
    }
    float4 acc = make_float4(base, base, base, base);
#pragma unroll 8
    for (int c = 0; c < n_chunks; ++c) {
        const float4 v = *reinterpret_cast<const float4 *>(partial + (int64_t)c * R + r);
        acc.x += v.x;
        acc.y += v.y;
        acc.z += v.z;
        acc.w += v.w;
    }
    *reinterpret_cast<float4 *>(scores + r) = acc;
}

// How a call's rows and chunks are shared out.  An item is one chunk over one
// group of rows; it costs the load of the chunk, its tiles and (deferred
// leaves) the leaf parts of every kDefer tiles, in units of one tile.
struct Split {
    int domains, groups;
    int64_t rows;                     // per group, whole tiles
};

inline Split split_rows(int n_chunks, int64_t R, int stride, int defer)
{
    const int64_t tiles = (R + kTileRows - 1) / kTileRows;
    Split best{};
    double best_cost = 0;
    // Domain 1 reads every row group from every XCD: only while the bins fit
    // in each 4 MB L2 next to the chunk images.
    for (const int domains : {kXcds, 1}) {
        if (domains == 1 && R * stride > (int64_t)2 << 20) break;
        const int slots = kXcds * kSlotsPerXcd / domains;
        const int64_t in_domain = (tiles + domains - 1) / domains;
        const int cap = (int)(in_domain < slots ? in_domain : slots);
        for (int g = 1; g <= cap; ++g) {
            const int64_t per = (in_domain + g - 1) / g;
            const int64_t rounds = ((int64_t)n_chunks * g + slots - 1) / slots;
            const double cost = (double)rounds * (1.5 + (double)per + (defer > 1 ? 1.3 * (double)((per + defer - 1) / defer) : 0.0));
            if (best.groups == 0 || cost < 0.995 * best_cost) best_cost = cost, best = Split{domains, g, per * kTileRows};
        }
    }
    return best;
}

template <int D>
hipError_t launch_traverse_d(const void *packed, ImageId id, const uint8_t *chunks, int image_chunks,
                             const uint8_t *Xb, int64_t R, int stride, float *partial, const LeafHook &hook,
                             hipStream_t s)
{
    const int n_chunks = walk_chunks(D, image_chunks);
    const Split sp = split_rows(n_chunks, R, stride, Walk<D>::kDefer);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(kXcds * kSlotsPerXcd), dim3(64 * kWaves), 0, s, packed, id, chunks, image_chunks,
                           n_chunks, Xb, R, stride, sp.domains, sp.groups, sp.rows, partial, hook);
    };
    constexpr int KD = Walk<D>::kDefer;
    if (hook.hash || hook.idx) {
        launch(k_traverse<D, true, KD>);
    } else if constexpr (Walk<D>::DEFER) {
        if (sp.rows <= kTileRows) launch(k_traverse<D, false, 1>);
        else if (sp.rows <= 4 * kTileRows) launch(k_traverse<D, false, 4>);
        else launch(k_traverse<D, false, KD>);
    } else {
        launch(k_traverse<D, false, KD>);
    }
    return hipGetLastError();
}

hipError_t launch_traverse(int depth, const void *packed, ImageId id, const uint8_t *chunks, int image_chunks,
                           const uint8_t *Xb, int64_t R, int stride, float *partial, const LeafHook &hook,
                           hipStream_t s)
{
#define HWSEL_TRAVERSE(D_) \
    return launch_traverse_d<D_>(packed, id, chunks, image_chunks, Xb, R, stride, partial, hook, s)
    switch (depth) {
    case 1: HWSEL_TRAVERSE(1);
    case 2: HWSEL_TRAVERSE(2);
    case 3: HWSEL_TRAVERSE(3);
    case 4: HWSEL_TRAVERSE(4);
    case 5: HWSEL_TRAVERSE(5);
    case 6: HWSEL_TRAVERSE(6);
    case 7: HWSEL_TRAVERSE(7);
    case 8: HWSEL_TRAVERSE(8);
    case 9: HWSEL_TRAVERSE(9);
    case 10: HWSEL_TRAVERSE(10);
    default: return hipErrorInvalidValue;
    }
#undef HWSEL_TRAVERSE
}

}  // namespace

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Rows per compute unit up to which the direct walk gives rows to single waves,
// not to tiles.  150 trees of depth 11, 128 columns: 3,000 rows 31 us against
// 64 us, 4,096 rows 37 against 64; 150 of depth 8: 3,000 rows 21 us against 23,
// 4,096 rows 26 against 23.  A wave's time grows with its rows, a tile takes
// what its trees take: the two cross between 14 rows and 30.
constexpr int64_t kDirTailPerCu = 16;

// Node visits per row (trees x depth) up to which a row per thread is quicker
// than tiles, which read and transpose every column of X and have a fixed cost
// per group of trees.  1,500,000 rows, us a row per thread / in tiles, at the
// limit and beyond it:
//   128 columns  8 trees x depth 3  317 / 422,  16 x 2  440 / 414
//    64 columns  8 x 3  176 / 270,  16 x 2  233 / 261,  8 x 6  330 / 314
//     4 columns  8 x 6  102 / 200,  10 x 6  126 / 200,  30 x 3  165 / 160
//   256 columns  16 x 3  922 / 1270,  20 x 3  1215 / 1284,  30 x 3  1575 / 1283
// 10,000 rows, one round of tiles: 4 columns  8 x 3  4.3 / 4.6,  16 x 2  5.7 / 4.4.
// 3,000 rows, which take a wave each instead of a tile: 128 columns  1 x 12
// 4.8 / 5.5,  4 x 3  3.7 / 3.6,  8 x 2  4.5 / 3.4;  256 columns  3 x 8  6.1 / 7.1,
// 16 x 2  7.3 / 5.0.  40,000 rows, a second round of tiles begun: 64 columns
// 5 x 5  6.5 / 11.8.
static int64_t rows_visits(int n_features, int64_t R, int64_t n_cu)
{
    if (R <= kDirTailPerCu * n_cu) return n_features <= 128 ? 12 : 24;
    if (n_features > 128) return 48;
    const int64_t rounds = (R - 1) / (128 * n_cu);          // full rounds of tiles before the last
    if (n_features <= 32) return rounds > 0 ? 64 : 24;
    return rounds > 0 && rounds < 4 ? 32 : 24;
}

static hipError_t launch_direct(const hwsel_forest_t &f, const float *X, int64_t R, int64_t ld, float *scores,
                                int64_t n_cu, hipStream_t s)
{
    if ((int64_t)f.n_trees * f.depth <= rows_visits(f.n_features, R, n_cu)) {
        hipLaunchKernelGGL(k_forest_rows, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, s, to_dev(f), X, R, ld, scores);
        return hipGetLastError();
    }
    // T rows per workgroup, so that n_features columns fit 64 KB (and below C
    // chains per lane, so that 8 C trees fit the node slots)
    const int T = f.n_features <= 128 ? 128 : 64;
    const int64_t round = T * n_cu;
    int64_t tail = R % round;                      // rows of the incomplete round
    if (tail > kDirTailPerCu * n_cu) tail = 0;
    const int64_t tiles = (R - tail + T - 1) / T;
    int32_t per = 1, tail_blocks = 0;
    if (tail > 0) {
        per = (int32_t)((tail + n_cu - 1) / n_cu);
        per = per < T / 8 ? per : T / 8;           // a row per wave
        tail_blocks = (int32_t)((tail + per - 1) / per);
    }
    const dim3 grid((unsigned)(tail_blocks + tiles)), block(8 * T);
#define HWSEL_DIRECT(CC, LL)                                                                                        \
    do {                                                                                                           \
        if (T == 128)                                                                                              \
            hipLaunchKernelGGL((k_forest_direct<128, CC, LL>), grid, block, 0, s, to_dev(f), X, R, ld, tail,       \
                               tail_blocks, per, scores);                                                          \
        else                                                                                                       \
            hipLaunchKernelGGL((k_forest_direct<64, CC, LL>), grid, block, 0, s, to_dev(f), X, R, ld, tail,        \
                               tail_blocks, per, scores);                                                          \
    } while (0)
    if (f.depth >= 11) HWSEL_DIRECT(1, 11);
    else if (f.depth == 10) HWSEL_DIRECT(2, 10);
    else if (f.depth == 9) HWSEL_DIRECT(4, 9);
    else if (f.depth == 8) HWSEL_DIRECT(4, 8);
    else HWSEL_DIRECT(4, 0);
#undef HWSEL_DIRECT
    return hipGetLastError();
}

hipError_t launch_forest_score(const hwsel_forest_t &f, const float *X, int64_t R, int64_t ld,
                               float *scores, hipStream_t s)
{
    // A launch has fewer than 2^32 threads; a tile has eight a row.
    constexpr int64_t kSpan = (int64_t)1 << 28;
    const int64_t n_cu = compute_units();
    for (int64_t r0 = 0; r0 < R; r0 += kSpan) {
        const hipError_t e = launch_direct(f, X + r0 * ld, R - r0 < kSpan ? R - r0 : kSpan, ld, scores + r0, n_cu, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_forest_leaves(const hwsel_forest_t &f, const float *X, int64_t R, int64_t ld,
                                const int64_t *rows, int64_t n_rows, uint16_t *leaf_idx,
                                hipStream_t s)
{
    const dim3 grid((unsigned)((n_rows + 255) / 256)), block(256);
    hipLaunchKernelGGL(k_forest_leaves, grid, block, 0, s, to_dev(f), X, R, ld, rows, n_rows, leaf_idx);
    return hipGetLastError();
}

bool packable(const hwsel_forest_t &f) { return f.depth >= 1 && f.depth <= 10 && f.n_features <= 128; }

size_t packed_bytes(const hwsel_forest_t &f) { return geometry(f).total; }

// Bins, then room for a partial sum per row and image chunk.  The walk writes
// one per chunk of its own, at depth 10 of two image chunks and so half as
// many; the size stays what callers were told.
size_t packed_workspace_bytes(const hwsel_forest_t &f, int64_t R)
{
    const PackGeom g = geometry(f);
    return align256((size_t)R * g.stride) + (size_t)g.n_chunks * (size_t)R * sizeof(float);
}

// The packed image of a forest whose arrays are in host memory, written to
// img (host memory of packed_bytes(f) bytes): per-feature sorted distinct
// thresholds, then the chunks of sibling-pair codes and leaves.
PackStatus build_image(const hwsel_forest_t &f, const uint8_t *feat, const float *thr, const float *leaf,
                       uint8_t *img_out)
{
    const PackGeom g = geometry(f);
    const int64_t n_int = ((int64_t)1 << f.depth) - 1;
    const int64_t nn = n_int * f.n_trees;
    // distinct thresholds per feature
    std::vector<std::vector<float>> U(f.n_features);
    for (int64_t e = 0; e < nn; ++e) {
        if (feat[e] >= f.n_features) return PackStatus::bad_feature;
        if (thr[e] != thr[e]) return PackStatus::nan_threshold;
        U[feat[e]].push_back(thr[e] == 0.0f ? 0.0f : thr[e]);
    }
    std::vector<uint8_t> img(g.total, 0);
    float *table = reinterpret_cast<float *>(img.data() + 256);
    for (int j = 0; j < f.n_features; ++j) {
        auto &u = U[j];
        std::sort(u.begin(), u.end());
        u.erase(std::unique(u.begin(), u.end()), u.end());
        if (u.size() > 255) return PackStatus::too_many_thresholds;
        for (int k = 0; k < kBinSlots; ++k)
            table[j * kBinSlots + k] = k < (int)u.size() ? u[k] : __builtin_inff();
    }
    uint8_t *chunk0 = img.data() + 256 + g.thr_bytes;
    for (int c = 0; c < g.n_chunks; ++c) {
        uint8_t *nodes = chunk0 + (size_t)c * g.chunk_bytes;
        float *leaves = reinterpret_cast<float *>(chunk0 + (size_t)c * g.chunk_bytes + g.node_bytes);
        for (int tt = 0; tt < g.tc; ++tt) {
            const int64_t tree = (int64_t)c * g.tc + tt;
            if (tree >= f.n_trees) continue;   // padding trees: zero codes, zero leaves
            for (int64_t n = 0; n < n_int; ++n) {
                const uint8_t fj = feat[tree * n_int + n];
                float v = thr[tree * n_int + n];
                v = v == 0.0f ? 0.0f : v;
                const auto &u = U[fj];
                const int rank = (int)(std::lower_bound(u.begin(), u.end(), v) - u.begin());
                const uint16_t code = (uint16_t)(fj | (rank << 8));
                for (int copy = 0; copy < node_copies(g.tc); ++copy)
                    std::memcpy(nodes + node_byte((uint32_t)(n + 1), tt, copy, g.tc), &code, 2);
            }
            for (int64_t l = 0; l <= n_int; ++l) leaves[l * g.tc + tt] = leaf[tree * (n_int + 1) + l];
        }
    }
    const ImageId id = image_id(f, g);
    std::memcpy(img.data(), &id, sizeof id);
    std::memcpy(img_out, img.data(), g.total);
    return PackStatus::ok;
}

// Copy the forest to the host, build the image there, upload it.
PackStatus pack_forest(const hwsel_forest_t &f, void *packed, hipStream_t s)
{
    const PackGeom g = geometry(f);
    const int64_t n_int = ((int64_t)1 << f.depth) - 1;
    const int64_t nn = n_int * f.n_trees, nl = (n_int + 1) * f.n_trees;
    std::vector<uint8_t> feat(nn), img(g.total);
    std::vector<float> thr(nn), leaf(nl);
    if (hipMemcpyAsync(feat.data(), f.node_feature, nn, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(thr.data(), f.node_threshold, nn * 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(leaf.data(), f.leaf_value, nl * 4, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return PackStatus::hip_error;
    const PackStatus st = build_image(f, feat.data(), thr.data(), leaf.data(), img.data());
    if (st != PackStatus::ok) return st;
    if (hipMemcpyAsync(packed, img.data(), g.total, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return PackStatus::hip_error;
    return PackStatus::ok;
}

ImageId packed_image_id(const hwsel_forest_t &f) { return image_id(f, geometry(f)); }

int packed_bin_stride(const hwsel_forest_t &f) { return geometry(f).stride; }

uint32_t packed_nan_bin(const hwsel_forest_t &f) { return (f.flags & 1u) ? 0u : 255u; }

namespace {

hipError_t traverse_and_reduce(const hwsel_forest_t &f, const void *packed, int64_t R, float *scores,
                               void *workspace, const LeafHook &hook, hipStream_t s)
{
    const PackGeom g = geometry(f);
    const ImageId id = image_id(f, g);
    const uint8_t *chunks = static_cast<const uint8_t *>(packed) + 256 + g.thr_bytes;
    const uint8_t *Xb = static_cast<const uint8_t *>(workspace);
    float *partial = reinterpret_cast<float *>(static_cast<uint8_t *>(workspace) + align256((size_t)R * g.stride));
    hipError_t e = launch_traverse(f.depth, packed, id, chunks, g.n_chunks, Xb, R, g.stride, partial, hook, s);
    if (e != hipSuccess) return e;
    const int n_chunks = walk_chunks(f.depth, g.n_chunks);
    if (R % 4 == 0 && ((uintptr_t)scores & 15u) == 0)
        hipLaunchKernelGGL(k_reduce4, dim3((unsigned)((R / 4 + 255) / 256)), dim3(256), 0, s, packed, id, partial,
                           n_chunks, R, f.base_score, scores);
    else
        hipLaunchKernelGGL(k_reduce, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, s, packed, id, partial,
                           n_chunks, R, f.base_score, scores);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_forest_packed(const hwsel_forest_t &f, const void *packed, const float *X, int64_t R,
                                int64_t ld, float *scores, void *workspace, hipStream_t s)
{
    return launch_forest_checked(f, packed, X, R, ld, scores, workspace, nullptr, nullptr, 0, 0, s);
}

hipError_t launch_forest_checked(const hwsel_forest_t &f, const void *packed, const float *X, int64_t R,
                                 int64_t ld, float *scores, void *workspace, uint64_t *leaf_hash,
                                 uint16_t *leaf_idx, int64_t leaf_row0, int64_t leaf_rows, hipStream_t s)
{
    const PackGeom g = geometry(f);
    uint8_t *Xb = static_cast<uint8_t *>(workspace);
    hipLaunchKernelGGL(k_bin, dim3(compute_units()), dim3(kBinThreads), 0, s, X, R, ld, packed, image_id(f, g), f.n_features,
                       packed_nan_bin(f), Xb, g.stride);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (leaf_hash) {
        hipLaunchKernelGGL(k_fill_u64, dim3(1024), dim3(256), 0, s, leaf_hash, R);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const LeafHook hook{leaf_hash, leaf_idx, leaf_row0, leaf_idx ? leaf_rows : 0, f.n_trees};
    return traverse_and_reduce(f, packed, R, scores, workspace, hook, s);
}

// Traversal and reduction of bins already in the workspace.
hipError_t launch_forest_from_bins(const hwsel_forest_t &f, const void *packed, int64_t R, float *scores,
                                   void *workspace, hipStream_t s)
{
    return traverse_and_reduce(f, packed, R, scores, workspace, LeafHook{nullptr, nullptr, 0, 0, f.n_trees}, s);
}

}  // namespace hwsel
