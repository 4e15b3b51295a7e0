// Configuration catalogue (section "Configuration Space", Table
// "Configuration knobs") and its static validity mask (section "Validity
// Constraints", Table "Static validity constraints").
//
// A point index decodes to its knobs by mixed radix (first knob slowest), so
// the mask pass never stores the catalogue: each thread decodes one group of
// 18 consecutive points (the three fastest knobs' combinations) once and
// derives the 18 from four tests; a block's mask bytes leave LDS as whole
// words.  The compaction is an ordered scan over a problem's mask, split over
// several workgroups where there are few problems.
#include "internal.hpp"

namespace hwsel {
namespace {

constexpr int64_t kCat = HWSEL_CATALOGUE_SIZE;
__constant__ int16_t kTileM[4] = {64, 128, 192, 256};
__constant__ int16_t kTileN[9] = {16, 32, 48, 64, 80, 96, 128, 192, 256};
__constant__ int16_t kTileK[5] = {32, 64, 128, 256, 512};
// (C_M, C_N) in {1,2,4,8,16}^2 with C_M C_N <= 16, C_M slower
__constant__ uint8_t kClusterM[15] = {1, 1, 1, 1, 1, 2, 2, 2, 2, 4, 4, 4, 8, 8, 16};
__constant__ uint8_t kClusterN[15] = {1, 2, 4, 8, 16, 1, 2, 4, 8, 1, 2, 4, 1, 2, 1};

struct Knobs {
    int32_t tm, tn, tk, st, cm, cn, ks, es, ts;
};

// Point index -> knobs (the index fits in 32 bits, so the divisions by
// constants are 32-bit multiply-shifts).
__device__ __forceinline__ Knobs decode(int64_t index)
{
    uint32_t i = (uint32_t)index;
    Knobs k;
    k.ts = (int32_t)(i % 2u); i /= 2u;
    k.es = (int32_t)(i % 3u); i /= 3u;
    k.ks = (int32_t)(i % 3u); i /= 3u;
    const uint32_t cl = i % 15u; i /= 15u;
    k.st = 2 + (int32_t)(i % 11u); i /= 11u;
    k.tk = kTileK[i % 5u]; i /= 5u;
    k.tn = kTileN[i % 9u]; i /= 9u;
    k.tm = kTileM[i];
    k.cm = kClusterM[cl];
    k.cn = kClusterN[cl];
    return k;
}

// Validity of the 18 points of a group, whose knobs but the three fastest are
// k's.  The tile and stage rules of a point depend on the epilogue schedule
// alone (e[es]); of the others, Stream-K (ts 1) needs the cooperative schedule
// (ks 2), which needs T_M to split in two (coop).
struct GroupValid {
    uint32_t e[3], coop;                       // 0 or 1
};

__device__ __forceinline__ GroupValid group_valid(const HwDev &h, const hwsel_problem_t &pb, uint32_t flags,
                                                  const Knobs &k)
{
    const int layout = pb.layout < 3 ? pb.layout : 3;
    const int32_t b = (pb.dtype < 2 ? pb.dtype : 2) == 2 ? 1 : 2;
    const int32_t frag = (k.tm < 64 ? k.tm : 64) * (k.tn < 32 ? k.tn : 32) * 2;
    const int64_t smem = (int64_t)(k.st * (k.tm + k.tn) * k.tk * b) + h.smem_rsv;
    bool ok = true;
    if (layout == 2 || layout == 3) ok &= k.tk <= 256 * k.cn;           // A column-major
    if (layout == 1 || layout == 3) ok &= k.tk <= 256 * k.cm;           // B row-major
    if (flags & 1u) {
        const int64_t M = pb.M > 1 ? pb.M : 1, N = pb.N > 1 ? pb.N : 1;
        ok &= k.tn <= 2 * M && k.tn <= 2 * N;
    }
    GroupValid v;
    v.e[0] = ok && smem <= h.smem_block;
    v.e[1] = ok && smem + 2 * frag <= h.smem_block;
    v.e[2] = ok && smem + 4 * frag <= h.smem_block;
    v.coop = k.tm % 128 == 0;
    return v;
}

__global__ void k_zero_i64(int64_t *__restrict__ a, int32_t n)
{
    const int32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = 0;
}

constexpr int kMaskThreads = 256;
constexpr int64_t kWords = (kCat + 3) / 4;
// The three fastest knobs (tile scheduler, epilogue, kernel schedule) take
// 2 x 3 x 3 = 18 values; the 18 consecutive points of a group share every
// other knob, decoded once.
constexpr int kGroup = 18;
constexpr int64_t kGroups = kCat / kGroup;
static_assert(kCat % kGroup == 0 && kCat % 4 == 0, "catalogue groups");
constexpr int kBlockBytes = kMaskThreads * kGroup;           // points (mask bytes) per block

// The 18 validities are 9 two-byte stores: the two tile schedulers of (kernel
// schedule, epilogue).  Testing every point by itself cost about 25
// instructions a point and 26 us for 61 problems; the bytes alone take about 8.
__global__ __launch_bounds__(kMaskThreads) void k_catalogue_mask(HwDev h, const hwsel_problem_t *__restrict__ probs,
                                                                 int32_t P, uint32_t flags, int32_t pieces,
                                                                 uint8_t *__restrict__ mask,
                                                                 int64_t *__restrict__ n_valid)
{
    __shared__ __align__(16) uint16_t stage_h[kBlockBytes / 2];
    __shared__ int32_t wave_cnt[kMaskThreads / 64];
    typedef uint32_t __attribute__((may_alias)) pair_t;
    const pair_t *stage = reinterpret_cast<const pair_t *>(stage_h);
    for (int32_t p = blockIdx.y; p < P; p += gridDim.y) {
        const hwsel_problem_t pb = probs[p];
        float cnt = 0.0f;
        for (int32_t piece = blockIdx.x * pieces; piece < (int32_t)(blockIdx.x + 1) * pieces; ++piece) {
            const int64_t g = (int64_t)piece * kMaskThreads + threadIdx.x;    // this thread's group
            const int64_t point0 = (int64_t)piece * kBlockBytes;
            if (point0 >= kCat) break;
            const int bytes = (int)(kCat - point0 < kBlockBytes ? kCat - point0 : kBlockBytes);
            if (g < kGroups) {
                const GroupValid v = group_valid(h, pb, flags, decode(g * kGroup));   // its first point: fast knobs 0
#pragma unroll
                for (int es = 0; es < 3; ++es) {
                    const uint16_t both = (uint16_t)(v.e[es] * v.coop * 0x0101u);
                    stage_h[threadIdx.x * 9 + es] = (uint16_t)v.e[es];
                    stage_h[threadIdx.x * 9 + 3 + es] = (uint16_t)v.e[es];
                    stage_h[threadIdx.x * 9 + 6 + es] = both;
                }
                cnt += (float)((v.e[0] + v.e[1] + v.e[2]) * (2 + 2 * v.coop));
            }
            __syncthreads();
            uint32_t *row = reinterpret_cast<uint32_t *>(mask + (int64_t)p * kCat + point0);
            for (int e = threadIdx.x; e < bytes / 4; e += kMaskThreads) row[e] = stage[e];
            lds_barrier();                               // stage is reused for the next piece
        }
        // per-wave totals (exact: below 2^24 in fp32), then one LDS step
        float tot[1] = {cnt};
        group_totals<64, 1>(tot);
        if ((threadIdx.x & 63) == 63) wave_cnt[threadIdx.x >> 6] = (int32_t)tot[0];
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t t = 0;
#pragma unroll
            for (int i = 0; i < kMaskThreads / 64; ++i) t += wave_cnt[i];
            if (t) atomicAdd(reinterpret_cast<unsigned long long *>(n_valid + p), (unsigned long long)t);
        }
        __syncthreads();                                 // wave_cnt is reused for the next problem
    }
}

// seg[0] = 0, seg[p + 1] = seg[p] + max(n_valid[p], 0): one workgroup, each
// thread summing a contiguous range of problems, the range sums scanned in
// LDS (exact integer sums, so the order is free).
constexpr int kOffsetThreads = 1024;

__global__ __launch_bounds__(kOffsetThreads) void k_catalogue_offsets(const int64_t *__restrict__ n_valid, int32_t P,
                                                                      int64_t *__restrict__ seg)
{
    __shared__ int64_t part[kOffsetThreads];
    const int t = threadIdx.x;
    const int64_t per = ((int64_t)P + kOffsetThreads - 1) / kOffsetThreads;
    const int64_t lo = t * per < P ? t * per : P, hi = lo + per < P ? lo + per : P;
    int64_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += n_valid[i] > 0 ? n_valid[i] : 0;
    part[t] = s;
    __syncthreads();
    for (int d = 1; d < kOffsetThreads; d <<= 1) {      // inclusive scan of the range sums
        const int64_t v = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t acc = t > 0 ? part[t - 1] : 0;
    if (t == 0) seg[0] = 0;
    for (int64_t i = lo; i < hi; ++i) {
        acc += n_valid[i] > 0 ? n_valid[i] : 0;
        seg[i + 1] = acc;
    }
}

constexpr int kCompactThreads = 1024;

// Ordered compaction of one problem's mask.  A step covers kBlocks consecutive
// blocks of 1,024 four-byte words (4 points each); thread i takes word i of
// every block, all loads issued together.  Within a wave, the valid points of
// lower lanes are counted from one ballot per byte position (mbcnt); across
// the 16 waves and the blocks, the wave totals meet in LDS.  Two barriers per
// step of 16,384 points.
//
// A step takes about 3 us, a problem 33 steps.  Where there are few problems,
// each is split: part y takes the steps [y, y + 1) * steps and finds
// its first place by counting the words before them, which runs at the rate
// of the caches (at most 0.5 MB, 4 us).
constexpr int kBlocks = 4;
constexpr int32_t kStepWords = kBlocks * kCompactThreads;
constexpr int32_t kSteps = (int32_t)((kWords + kStepWords - 1) / kStepWords);

__global__ __launch_bounds__(kCompactThreads) void k_catalogue_compact(const uint8_t *__restrict__ mask,
                                                                       const int64_t *__restrict__ seg,
                                                                       int32_t *__restrict__ point, int64_t cap,
                                                                       int32_t P, int32_t split, int32_t steps)
{
    constexpr int kWavesC = kCompactThreads / 64;
    static_assert(kBlocks * kWavesC == 64, "a lane per wave and block");
    __shared__ int32_t wave_total[kBlocks][kWavesC], list[kWavesC][256];
    // one problem's workgroups run on one XCD (blockIdx % 8), whose L2 then
    // holds the mask they count
    const int32_t p = (int32_t)(blockIdx.x % 8) + 8 * (int32_t)(blockIdx.x / 8 / split);
    const int32_t part = (int32_t)(blockIdx.x / 8) % split;
    if (p >= P) return;
    const int wave = threadIdx.x >> 6;
    const uint32_t *row = reinterpret_cast<const uint32_t *>(mask + (int64_t)p * kCat);
    int64_t out = seg[p];
    const int32_t w_lo = part * steps * kStepWords;
    if (w_lo > 0) {
        int32_t before = 0;
#pragma unroll 16
        for (int32_t w = 0; w < w_lo; w += kCompactThreads) before += __popc(row[w + threadIdx.x] & 0x01010101u);
        for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
        if ((threadIdx.x & 63) == 0) wave_total[0][wave] = before;
        lds_barrier();
#pragma unroll
        for (int i = 0; i < kWavesC; ++i) out += wave_total[0][i];
        lds_barrier();
    }
    const int64_t w_hi = w_lo + steps * kStepWords < kWords ? w_lo + steps * kStepWords : kWords;
    uint32_t ahead[kBlocks];             // the next step's words
    auto fetch = [&](int64_t w0) {
#pragma unroll
        for (int k = 0; k < kBlocks; ++k) {
            const int64_t w = w0 + k * kCompactThreads + threadIdx.x;
            ahead[k] = w < kWords ? row[w] : 0u;
        }
    };
    fetch(w_lo);
    for (int64_t w0 = w_lo; w0 < w_hi; w0 += kStepWords) {
        uint32_t word[kBlocks];
#pragma unroll
        for (int k = 0; k < kBlocks; ++k) word[k] = ahead[k];
        if (w0 + kStepWords < w_hi) fetch(w0 + kStepWords);
        int32_t below[kBlocks];              // valid points of block k in lower lanes of this wave
        int32_t count[kBlocks];              // and in all its lanes
#pragma unroll
        for (int k = 0; k < kBlocks; ++k) {
            int32_t bl = 0, total = 0;
            // nine in ten points are invalid, in long runs: most waves' words are 0
            if (__ballot(word[k] & 0x01010101u))
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint64_t b = __ballot((word[k] >> (8 * q)) & 1u);
                bl += (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                total += __popcll(b);
            }
            below[k] = bl;
            count[k] = total;
            if ((threadIdx.x & 63) == 0) wave_total[k][wave] = total;
        }
        lds_barrier();
        // the 64 totals, a lane each in point order, summed up to each lane
        // (a step's 16,384 points are exact in fp32)
        float upto[1] = {(float)wave_total[(threadIdx.x & 63) / kWavesC][threadIdx.x % kWavesC]};
        const int32_t own = (int32_t)upto[0];
        group_totals<64, 1>(upto);
        const int32_t before = (int32_t)upto[0] - own;
#pragma unroll
        for (int k = 0; k < kBlocks; ++k) {
            if (count[k] == 0) continue;
            // gathered in LDS, so that they leave as whole lines (written
            // from where they stand they touch every line four times)
            int32_t at = below[k];
            const int32_t p0 = (int32_t)(4 * (w0 + k * kCompactThreads + threadIdx.x));
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((word[k] >> (8 * q)) & 1u) list[wave][at++] = p0 + q;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
            const int64_t to = out + __shfl(before, k * kWavesC + wave);
            for (int32_t e = threadIdx.x & 63; e < count[k]; e += 64)
                if (to + e < cap) point[to + e] = list[wave][e];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        }
        out += __shfl((int32_t)upto[0], 63);
        lds_barrier();                        // wave_total is rewritten by the next step
    }
}

__global__ void k_catalogue_candidates(const hwsel_problem_t *__restrict__ probs, int32_t P,
                                       const int64_t *__restrict__ seg, const int32_t *__restrict__ point, int64_t R,
                                       hwsel_cands_out_t out)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // the wave's first row (wave-uniform): one scalar search per wave
    const int64_t r_first = (int64_t)blockIdx.x * blockDim.x + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    if (r >= R) return;
    const int32_t p = segment_of_row_after(seg, P, r, r_first);
    int64_t i = point ? (int64_t)point[r] : r - seg[p];
    i = i < 0 ? 0 : (i >= kCat ? kCat - 1 : i);
    const Knobs k = decode(i);
    const int dt = probs[p].dtype < 2 ? probs[p].dtype : 2;
    out.tile_m[r] = (uint16_t)k.tm;
    out.tile_n[r] = (uint16_t)k.tn;
    out.tile_k[r] = (uint16_t)k.tk;
    out.inst_n[r] = (uint16_t)k.tn;
    out.stages[r] = (uint8_t)k.st;
    out.cluster_m[r] = (uint8_t)k.cm;
    out.cluster_n[r] = (uint8_t)k.cn;
    out.swizzle[r] = 1;
    out.inst_m_div16[r] = 4;
    out.inst_k[r] = dt == 2 ? 32 : 16;
    out.kernel_sched[r] = (uint8_t)k.ks;
    out.epi_sched[r] = (uint8_t)k.es;
    out.tile_sched[r] = (uint8_t)k.ts;
}

// Four consecutive rows per thread, each field written with one 4-byte
// (8-bit fields) or 8-byte (16-bit fields) store; taken when every field
// array is aligned for that (the rows of a partial last quad are stored one
// by one).
__global__ void k_catalogue_candidates4(const hwsel_problem_t *__restrict__ probs, int32_t P,
                                        const int64_t *__restrict__ seg, const int32_t *__restrict__ point,
                                        int64_t R, hwsel_cands_out_t out)
{
    const int64_t r0 = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    const int64_t r_first = 4 * ((int64_t)blockIdx.x * blockDim.x + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u));
    if (r0 >= R) return;
    int32_t p = segment_of_row_after(seg, P, r0, r_first);
    uint32_t tm[4], tn[4], tk[4], st[4], cm[4], cn[4], ik[4], ks[4], es[4], ts[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int64_t r = r0 + j < R ? r0 + j : R - 1;
        while (p + 1 < P && seg[p + 1] <= r) ++p;
        int64_t i = point ? (int64_t)point[r] : r - seg[p];
        i = i < 0 ? 0 : (i >= kCat ? kCat - 1 : i);
        const Knobs k = decode(i);
        const int dt = probs[p].dtype < 2 ? probs[p].dtype : 2;
        tm[j] = (uint32_t)k.tm; tn[j] = (uint32_t)k.tn; tk[j] = (uint32_t)k.tk; st[j] = (uint32_t)k.st;
        cm[j] = (uint32_t)k.cm; cn[j] = (uint32_t)k.cn; ik[j] = dt == 2 ? 32u : 16u;
        ks[j] = (uint32_t)k.ks; es[j] = (uint32_t)k.es; ts[j] = (uint32_t)k.ts;
    }
    if (r0 + 3 < R) {
        auto p16 = [](const uint32_t (&v)[4]) {
            return make_uint2(v[0] | (v[1] << 16), v[2] | (v[3] << 16));
        };
        auto p8 = [](const uint32_t (&v)[4]) { return v[0] | (v[1] << 8) | (v[2] << 16) | (v[3] << 24); };
        *reinterpret_cast<uint2 *>(out.tile_m + r0) = p16(tm);
        *reinterpret_cast<uint2 *>(out.tile_n + r0) = p16(tn);
        *reinterpret_cast<uint2 *>(out.tile_k + r0) = p16(tk);
        *reinterpret_cast<uint2 *>(out.inst_n + r0) = p16(tn);
        *reinterpret_cast<uint32_t *>(out.stages + r0) = p8(st);
        *reinterpret_cast<uint32_t *>(out.cluster_m + r0) = p8(cm);
        *reinterpret_cast<uint32_t *>(out.cluster_n + r0) = p8(cn);
        *reinterpret_cast<uint32_t *>(out.swizzle + r0) = 0x01010101u;
        *reinterpret_cast<uint32_t *>(out.inst_m_div16 + r0) = 0x04040404u;
        *reinterpret_cast<uint32_t *>(out.inst_k + r0) = p8(ik);
        *reinterpret_cast<uint32_t *>(out.kernel_sched + r0) = p8(ks);
        *reinterpret_cast<uint32_t *>(out.epi_sched + r0) = p8(es);
        *reinterpret_cast<uint32_t *>(out.tile_sched + r0) = p8(ts);
    } else {
        for (int j = 0; j < 4 && r0 + j < R; ++j) {
            const int64_t r = r0 + j;
            out.tile_m[r] = (uint16_t)tm[j];
            out.tile_n[r] = (uint16_t)tn[j];
            out.tile_k[r] = (uint16_t)tk[j];
            out.inst_n[r] = (uint16_t)tn[j];
            out.stages[r] = (uint8_t)st[j];
            out.cluster_m[r] = (uint8_t)cm[j];
            out.cluster_n[r] = (uint8_t)cn[j];
            out.swizzle[r] = 1;
            out.inst_m_div16[r] = 4;
            out.inst_k[r] = (uint8_t)ik[j];
            out.kernel_sched[r] = (uint8_t)ks[j];
            out.epi_sched[r] = (uint8_t)es[j];
            out.tile_sched[r] = (uint8_t)ts[j];
        }
    }
}

}  // namespace

hipError_t launch_catalogue_mask(const HwDev &h, const hwsel_problem_t *probs, int32_t P, uint32_t flags,
                                 uint8_t *mask, int64_t *n_valid, hipStream_t s)
{
    hipLaunchKernelGGL(k_zero_i64, dim3((P + 255) / 256), dim3(256), 0, s, n_valid, P);
    // The counts meet in atomics on few cache lines, which complete one by one
    // (7,076 of them take 26 us): a block takes several pieces of a problem,
    // as many as leave four blocks per compute unit.
    constexpr int32_t kPieces = (int32_t)((kGroups + kMaskThreads - 1) / kMaskThreads);
    int32_t pieces = (int32_t)((int64_t)P * kPieces / 1024);
    pieces = pieces < 1 ? 1 : (pieces > 15 ? 15 : pieces);
    const dim3 grid((unsigned)((kPieces + pieces - 1) / pieces), (unsigned)(P < 65535 ? P : 65535));
    hipLaunchKernelGGL(k_catalogue_mask, grid, dim3(kMaskThreads), 0, s, h, probs, P, flags, pieces, mask, n_valid);
    return hipGetLastError();
}

hipError_t launch_catalogue_compact(const uint8_t *mask, const int64_t *n_valid, int32_t P, int64_t *seg,
                                    int32_t *point, int64_t cap, hipStream_t s)
{
    hipLaunchKernelGGL(k_catalogue_offsets, dim3(1), dim3(kOffsetThreads), 0, s, n_valid, P, seg);
    // about 512 workgroups (61 problems: 31 us, 35 us with 1,024, 48 us with 2,048)
    int32_t split = 512 / P < 1 ? 1 : (512 / P > kSteps ? kSteps : 512 / P);
    const int32_t steps = (kSteps + split - 1) / split;
    split = (kSteps + steps - 1) / steps;
    hipLaunchKernelGGL(k_catalogue_compact, dim3(8 * ((P + 7) / 8) * split), dim3(kCompactThreads), 0, s, mask, seg, point, cap,
                       P, split, steps);
    return hipGetLastError();
}

hipError_t launch_catalogue_candidates(const hwsel_problem_t *probs, int32_t P, const int64_t *seg,
                                       const int32_t *point, int64_t R, const hwsel_cands_out_t &out, hipStream_t s)
{
    auto al = [](const void *q, uintptr_t a) { return ((uintptr_t)q & (a - 1)) == 0; };
    const bool packed = al(out.tile_m, 8) && al(out.tile_n, 8) && al(out.tile_k, 8) && al(out.inst_n, 8) &&
                        al(out.stages, 4) && al(out.cluster_m, 4) && al(out.cluster_n, 4) && al(out.swizzle, 4) &&
                        al(out.inst_m_div16, 4) && al(out.inst_k, 4) && al(out.kernel_sched, 4) &&
                        al(out.epi_sched, 4) && al(out.tile_sched, 4);
    if (packed) {
        const int64_t quads = (R + 3) / 4;
        hipLaunchKernelGGL(k_catalogue_candidates4, dim3((unsigned)((quads + 255) / 256)), dim3(256), 0, s, probs, P,
                           seg, point, R, out);
    } else {
        hipLaunchKernelGGL(k_catalogue_candidates, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, s, probs, P,
                           seg, point, R, out);
    }
    return hipGetLastError();
}

}  // namespace hwsel
