// Feature kernel: x = phi(p, c, h) for every (problem, candidate) row.
//
// One thread per row; a wave owns 64 consecutive rows.  The candidate record
// is read as coalesced struct-of-arrays streams (17 B/row), the problem record
// once per row from a tiny L2-resident table.  The map hands its columns to a
// sink in order; the feature kernel's sink transposes them through LDS 32 at a
// time so that every global store is a 16-byte vector store into a contiguous
// 128-byte row segment (8 rows per wave instruction).
//
// Numeric contract (same as the definition the oracle follows):
//   integer columns  - exact int64 values, one conversion to fp32 (RNE);
//   ratio columns    - one binary64 division of two exact int64 values, then
//                      fp32;
//   composite columns- a fixed short sequence of binary64 operations;
//   log2 columns     - binary64 log2, then fp32.
// This translation unit is compiled with -ffp-contract=off so no multiply-add
// is fused behind the sequence's back.
//
// Number types.  The map is written once over a number type T.  T = double
// holds the integers exactly (rows whose integers all stay below 2^52, which a
// row checks on its own, see Phi::plain): binary64 multiplies and adds run at
// the full vector rate, an integer division is a multiply by a reciprocal and a
// truncation, and quotients by one denominator share its reciprocal.  T =
// int64_t takes the rows beyond that, whose 64-bit products wrap as they
// always did, and every row when a hardware field is too large (HwPhi::plain).
// Measured, 4,915,200 rows x 128 columns: 538 -> 444 us (5.9 TB/s of output;
// one fill kernel writes 6.9), with 1,100 vector instructions per wave instead
// of 2,900; every column bit-identical.
#include "internal.hpp"

#include <math.h>

#include <type_traits>

namespace hwsel {
namespace {

// ---------------------------------------------------------------------------
// Exact integers in two number types
// ---------------------------------------------------------------------------
__device__ __forceinline__ float exact(int64_t v) { return (float)v; }
__device__ __forceinline__ float exact(double v) { return (float)v; }
__device__ __forceinline__ float exact(int v) { return (float)v; }
__device__ __forceinline__ float exact(uint32_t v) { return (float)v; }
__device__ __forceinline__ float exact(bool v) { return v ? 1.0f : 0.0f; }
__device__ __forceinline__ int64_t max_of(int64_t a, int64_t b) { return a > b ? a : b; }
__device__ __forceinline__ int64_t min_of(int64_t a, int64_t b) { return a < b ? a : b; }
__device__ __forceinline__ double max_of(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ double min_of(double a, double b) { return __builtin_fmin(a, b); }

// Reciprocal of a non-zero integer below 2^63 in magnitude: the hardware's
// approximation and two Newton steps, the same steps a binary64 division takes
// (whose scaling steps change nothing in this range).
__device__ __forceinline__ double reciprocal(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
}

// A denominator: its value and, for T = double, its reciprocal.
template <class T>
struct Den;
template <>
struct Den<double> {
    double v, r;
};
template <>
struct Den<int64_t> {
    int64_t v;
};

template <class T>
__device__ __forceinline__ Den<T> den(T v);
template <>
__device__ __forceinline__ Den<double> den<double>(double v) { return Den<double>{v, reciprocal(v)}; }
template <>
__device__ __forceinline__ Den<int64_t> den<int64_t>(int64_t v) { return Den<int64_t>{v}; }

// A denominator whose reciprocal is at hand.
template <class T>
__device__ __forceinline__ Den<T> den_with(T v, double r)
{
    if constexpr (sizeof(Den<T>) == 16) return Den<T>{v, r};
    else return Den<T>{v};
}

template <class T>
__device__ __forceinline__ double recip_of(const Den<T> &d)
{
    if constexpr (sizeof(Den<T>) == 16) return d.r;
    else return 0.0;
}

// n / d in binary64, correctly rounded: with r the rounded reciprocal, n r is
// within an ulp and one residual step rounds it right (Markstein, IBM Journal
// of Research and Development 34, 1990).
__device__ __forceinline__ double ratio(double n, const Den<double> &d)
{
    const double q = n * d.r;
    return __builtin_fma(__builtin_fma(-q, d.v, n), d.r, q);
}
__device__ __forceinline__ double ratio(int64_t n, const Den<int64_t> &d) { return (double)n / (double)d.v; }
template <class T>
__device__ __forceinline__ float quot(T n, const Den<T> &d) { return (float)ratio(n, d); }

// floor(n / d) and ceil(n / d) for 0 <= n (1 <= n) < 2^50: (n + 1/2) / d is at
// least 1 / (2 d) from an integer, and the product's error is below that.
__device__ __forceinline__ double floor_div(double n, const Den<double> &d)
{
    return __builtin_trunc(__builtin_fma(n, d.r, 0.5 * d.r));
}
__device__ __forceinline__ int64_t floor_div(int64_t n, const Den<int64_t> &d) { return n / d.v; }
__device__ __forceinline__ double ceil_div(double n, const Den<double> &d) { return floor_div(n - 1.0, d) + 1.0; }
__device__ __forceinline__ int64_t ceil_div(int64_t n, const Den<int64_t> &d) { return (n + d.v - 1) / d.v; }

// ceil(a / b) of two 16-bit values: (a - 1/2) / b is at least 1 / (2 b) from an
// integer, and the fp32 product's error (2^-22 of at most 2^16) below that.
__device__ __forceinline__ uint32_t ceil_div16(uint32_t a, uint32_t b)
{
    return (uint32_t)(((float)a - 0.5f) * __builtin_amdgcn_rcpf((float)b)) + 1u;
}

__device__ __forceinline__ float lg(int64_t v) { return (float)log2((double)v); }
__device__ __forceinline__ float lg(double v) { return (float)log2(v); }

__device__ __forceinline__ int64_t cdiv64(int64_t a, int64_t b) { return (a + b - 1) / b; }
__device__ __forceinline__ int64_t max64(int64_t a, int64_t b) { return a > b ? a : b; }

// Knob codes.
constexpr int kWS = 0, kCoop = 2;
constexpr int eNone = 0, eTma = 1;
constexpr int tStreamK = 1;
constexpr int dFp16 = 1, dFp8 = 2, dFp32 = 3;
constexpr int lNN = 2, lNT = 3, lTT = 1;

// Analytic sampling score (section "Candidate Sampling"): the cluster-wave
// fill n_c / (W S_SM c_M c_N) times S sqrt(T_M T_N T_K), in binary64.
__device__ __forceinline__ float sampling_score(int64_t clusters, int64_t cwaves, int64_t cslots, int64_t cm,
                                                int64_t cn, int64_t st, int64_t tm, int64_t tn, int64_t tk)
{
    const double fill = (double)(clusters * st) / (double)(cwaves * cslots * cm * cn);
    return (float)(fill * sqrt((double)(tm * tn * tk)));
}

// The hardware as the map reads it, prepared on the host.
template <class T>
struct HwPhi {
    T n_sm, smem_sm, smem_block, smem_rsv, regs_sm, regs_thread_max, llc, bw, threads_sm_max;
    T by_arch_ws, by_arch;                         // blocks the thread and block limits allow: 256 and 384 threads
    T peak[3];
    double r_nsm, r_smem, r_llc, r_bw, r_threads;  // reciprocals, for T = double
    float x59, x60, x61, x62, x63, x78;
};

struct HwBoth {
    HwPhi<double> d;
    HwPhi<int64_t> i;
    int32_t plain;                                 // every field small enough for T = double
};

template <class T>
HwPhi<T> hw_phi(const HwDev &h)
{
    HwPhi<T> o{};
    o.n_sm = (T)h.n_sm; o.smem_sm = (T)h.smem_sm; o.smem_block = (T)h.smem_block; o.smem_rsv = (T)h.smem_rsv;
    o.regs_sm = (T)h.regs_sm; o.regs_thread_max = (T)h.regs_thread_max; o.llc = (T)h.llc; o.bw = (T)h.bw;
    o.threads_sm_max = (T)h.threads_sm_max;
    auto arch = [&](int64_t threads) {
        const int64_t v = h.threads_sm_max / threads;
        return (T)(h.blocks_sm_max < v ? h.blocks_sm_max : v);
    };
    o.by_arch_ws = arch(256); o.by_arch = arch(384);
    for (int i = 0; i < 3; ++i) o.peak[i] = (T)h.peak[i];
    o.r_nsm = 1.0 / (double)h.n_sm; o.r_smem = 1.0 / (double)h.smem_sm; o.r_llc = 1.0 / (double)h.llc;
    o.r_bw = 1.0 / (double)h.bw; o.r_threads = 1.0 / (double)h.threads_sm_max;
    o.x59 = (float)h.n_sm; o.x60 = (float)h.smem_sm; o.x61 = (float)h.regs_sm; o.x62 = (float)h.llc;
    o.x63 = (float)h.bw; o.x78 = (float)h.arch_id;
    return o;
}

HwBoth hw_both(const HwDev &h)
{
    const int64_t big = (int64_t)1 << 40;
    const int64_t fields[] = {h.n_sm, h.smem_sm, h.smem_block, h.smem_rsv, h.regs_sm, h.regs_thread_max, h.blocks_sm_max,
                              h.threads_sm_max, h.llc, h.bw, h.peak[0], h.peak[1], h.peak[2]};
    int32_t plain = 1;
    for (int64_t f : fields) plain &= f <= big;
    return HwBoth{hw_phi<double>(h), hw_phi<int64_t>(h), plain};
}

constexpr double kPlainMost = 1125899906842624.0;  // 2^50

// What the feature map needs of a problem alone: its integer terms and the
// columns that depend on nothing else, computed once per problem rather than
// once per row (the same operations, so the same values).
template <class T>
struct ProbTerms {
    Den<T> M, N, K, pk, ab, mnk;                   // ab: operand bytes; mnk: M N K
    T a_bytes, b_bytes, epi_traffic, conv;
    int32_t layout, dtype, eb, out_dtype;
    // columns 0-3, 43, 46, 49, 80, 81, 88, 119-123
    float lg_m, lg_n, lg_k, lg_flops, x43, x46, x49, x80, x81, x88, x119, x120, x121, x122, x123;
};

template <class T>
__device__ __forceinline__ ProbTerms<T> problem_terms(const HwPhi<T> &h, const hwsel_problem_t &pb)
{
    ProbTerms<T> t;
    const T M = (T)(pb.M > 1 ? pb.M : 1), N = (T)(pb.N > 1 ? pb.N : 1), K = (T)(pb.K > 1 ? pb.K : 1);
    const int dtype = pb.dtype < 2 ? pb.dtype : 2;
    const int eb = dtype == dFp8 ? 1 : 2;              // input element bytes (A and B)
    const T ob = 2;                                    // output / C element bytes
    const int out_dtype = dtype == dFp16 ? dFp16 : 0;
    t.layout = pb.layout < 3 ? pb.layout : 3;
    t.dtype = dtype; t.eb = eb; t.out_dtype = out_dtype;
    t.a_bytes = (T)eb * M * K;
    t.b_bytes = (T)eb * K * N;
    t.epi_traffic = (T)2 * ob * M * N;                 // D written + C read
    t.conv = out_dtype != dtype ? M * N * ob : (T)0;
    const T gemm_flops = (T)2 * M * N * K;
    t.M = den<T>(M); t.N = den<T>(N); t.K = den<T>(K); t.pk = den<T>(h.peak[dtype]);
    t.ab = den<T>(t.a_bytes + t.b_bytes);
    t.mnk = den<T>(M * N * K);
    const Den<T> all = den<T>(t.a_bytes + t.b_bytes + t.epi_traffic);
    const Den<T> llc = den_with<T>(h.llc, h.r_llc), bw = den_with<T>(h.bw, h.r_bw);
    t.lg_m = lg(M); t.lg_n = lg(N); t.lg_k = lg(K); t.lg_flops = lg(gemm_flops);
    const double intensity = ratio(gemm_flops, all), ridge = ratio(t.pk.v, bw);
    t.x43 = (float)intensity;
    t.x46 = quot(t.ab.v, llc);
    t.x49 = exact(t.epi_traffic);
    t.x80 = (float)ridge;
    t.x81 = (float)(intensity / ridge);
    t.x88 = exact(t.conv);
    t.x119 = quot(t.a_bytes, llc);
    t.x120 = quot(t.b_bytes, llc);
    t.x121 = quot(ob * M * N, llc);
    t.x122 = quot(M, t.N);
    t.x123 = quot(K, M > N ? t.M : t.N);
    return t;
}

// One row's candidate record.
struct Cand {
    uint16_t tile_m, tile_n, tile_k, inst_n;
    uint8_t stages, cluster_m, cluster_n, swizzle, inst_m_div16, inst_k, kernel_sched, epi_sched, tile_sched;
};

__device__ __forceinline__ Cand load_cand(const CandsDev &c, int64_t r)
{
    return Cand{c.tile_m[r], c.tile_n[r], c.tile_k[r], c.inst_n[r], c.stages[r], c.cluster_m[r], c.cluster_n[r], c.swizzle[r],
                c.inst_m_div16[r], c.inst_k[r], c.kernel_sched[r], c.epi_sched[r], c.tile_sched[r]};
}

// The feature map of one row: out(j, x_j) for the columns j < F in order.
// Returns whether every integer of the row stayed below 2^52, so that T = double held it
// exactly (the bounds below cover the others: sums and differences of them,
// and products by at most 4).
template <int F, class T, class Out>
__device__ __forceinline__ bool phi(const HwPhi<T> &h, const ProbTerms<T> &pt, const Cand &c, Out &&out)
{
    // ---- problem ----
    const T M = pt.M.v, N = pt.N.v, K = pt.K.v;
    const int layout = pt.layout;
    const T eb = (T)pt.eb, ob = 2;                     // element bytes: inputs, output and C

    // ---- candidate ----
    auto at_least_1 = [](uint32_t v) { return v > 1u ? v : 1u; };
    const uint32_t utm = at_least_1(c.tile_m), utn = at_least_1(c.tile_n), utk = at_least_1(c.tile_k);
    const uint32_t ucm = at_least_1(c.cluster_m), ucn = at_least_1(c.cluster_n), ust = at_least_1(c.stages);
    const T tm = (T)utm, tn = (T)utn, tk = (T)utk, st = (T)ust, cm = (T)ucm, cn = (T)ucn;
    const int ks = c.kernel_sched < 2 ? c.kernel_sched : 2;
    const int es = c.epi_sched < 2 ? c.epi_sched : 2;
    const int ts = c.tile_sched < 1 ? c.tile_sched : 1;

    // ---- schedule: warpgroups ----
    const bool ws = ks == kWS;
    const Den<T> threads = den_with<T>(ws ? 256 : 384, ws ? 1.0 / 256 : 1.0 / 384);   // producer + 1 or 2 consumer warpgroups
    const T consumers = ks == kCoop ? 2 : 1;           // consumer warpgroups on one tile

    // ---- work decomposition ----
    const T gm = ceil_div(M, den<T>(tm)), gn = ceil_div(N, den<T>(tn)), gk = ceil_div(K, den<T>(tk));
    const Den<T> ntile = den<T>(gm * gn);

    // ---- shared memory, registers, residency ----
    const T stage_bytes = (tm + tn) * tk * eb;
    const T main_bytes = st * stage_bytes;
    const T frag = (T)(utm < 64 ? utm : 64) * (T)(utn < 32 ? utn : 32) * ob;
    const T epi_bytes = es == eNone ? (T)0 : (es == eTma ? 2 * frag : 4 * frag);
    const T smem = (ws ? max_of(main_bytes, epi_bytes) : main_bytes + epi_bytes) + h.smem_rsv;
    const T by_smem = floor_div(h.smem_sm, den<T>(smem));
    const T regs = min_of(h.regs_thread_max, ceil_div(tm * tn, threads) + 32);
    const T by_regs = floor_div(h.regs_sm, den<T>(regs * threads.v));
    const T by_arch = ws ? h.by_arch_ws : h.by_arch;
    const T resident = min_of(min_of(by_smem, by_regs), by_arch);
    const bool fits = main_bytes + epi_bytes + h.smem_rsv <= h.smem_block;

    // ---- waves over resident slots ----
    const T slot_count = h.n_sm * max_of(resident, (T)1);
    const T waves = ceil_div(ntile.v, den<T>(slot_count));
    const Den<T> wave_cap = den<T>(waves * slot_count);

    // ---- clusters (ceil(M / (cm tm)) = ceil(gm / cm)) ----
    const Den<T> dcm = den<T>(cm), dcn = den<T>(cn), dst = den<T>(st);
    const T cmn = cm * cn;
    const T clusters = ceil_div(gm, dcm) * ceil_div(gn, dcn);
    const Den<T> cslots = den<T>(max_of(floor_div(h.n_sm, den_with<T>(cmn, recip_of(dcm) * recip_of(dcn))), (T)1));
    const T cwaves = ceil_div(clusters, cslots);
    const Den<T> ccap = den<T>(cwaves * cslots.v);

    // ---- bytes ----
    const T loads = gn * pt.a_bytes + gm * pt.b_bytes; // every tile loads its panels
    const T tile_flops = (T)2 * tm * tn * tk;
    const Den<T> n_sm = den_with<T>(h.n_sm, h.r_nsm), smem_sm = den_with<T>(h.smem_sm, h.r_smem);
    const Den<T> llc = den_with<T>(h.llc, h.r_llc), bw = den_with<T>(h.bw, h.r_bw);
    const Den<T> rate = den_with<T>(consumers * pt.pk.v, ks == kCoop ? 0.5 * recip_of(pt.pk) : recip_of(pt.pk));

    // ---- tier 1 ----
    out(0, pt.lg_m); out(1, pt.lg_n); out(2, pt.lg_k); out(3, pt.lg_flops);
    out(4, exact(utm)); out(5, exact(utn)); out(6, exact(utk)); out(7, exact(ust));
    out(8, exact(ucm)); out(9, exact(ucn)); out(10, exact(ucm * ucn)); out(11, exact((uint32_t)c.swizzle));
    out(12, exact(gm)); out(13, exact(gn)); out(14, exact(gk)); out(15, exact(ntile.v));
    out(16, quot(gm * tm - M, pt.M));
    out(17, quot(gn * tn - N, pt.N));
    out(18, quot(gk * tk - K, pt.K));
    out(19, quot(ntile.v, n_sm));
    out(20, exact(ws ? 256 : 384));
    out(21, quot(tm * tn, threads));
    out(22, exact(regs));
    out(23, exact(by_regs));
    out(24, exact(stage_bytes));
    out(25, exact(main_bytes));
    out(26, exact(epi_bytes));
    out(27, exact(smem));
    out(28, quot(smem, smem_sm));
    out(29, exact(by_smem));
    out(30, exact(by_arch));
    out(31, exact(resident));
    out(32, exact(fits));
    out(33, exact(waves));
    out(34, quot(ntile.v, wave_cap));
    const float x35 = quot(wave_cap.v - ntile.v, wave_cap);
    out(35, x35);
    out(36, exact(clusters));
    out(37, exact(cslots.v));
    out(38, exact(cwaves));
    out(39, quot(clusters, ccap));
    out(40, quot(gm, dcm));
    out(41, quot(gn, dcn));
    out(42, exact(cm > gm || cn > gn));
    out(43, pt.x43);
    out(44, quot((T)2 * tm * tn, den<T>((tm + tn) * eb)));
    out(45, quot(loads, pt.ab));
    out(46, pt.x46);
    out(47, quot((tm + tn) * K * eb, llc));
    out(48, exact(loads));
    out(49, pt.x49);
    const double t_load = ratio(h.n_sm * stage_bytes, bw);
    const double t_mma = ratio(tile_flops * h.n_sm, rate);
    out(50, (float)t_load);
    out(51, (float)t_mma);
    out(52, quot(tile_flops * h.bw, den<T>(rate.v * stage_bytes)));
    out(53, quot(min_of(st, gk), dst));
    out(54, quot(gk, dst));
    out(55, quot(st * smem, smem_sm));
    out(56, exact(utk * ust));
    out(57, exact(st * resident));
    const double volume_root = sqrt((double)(tm * tn * tk));
    out(58, (float)(ratio(clusters * st, den<T>(ccap.v * cm * cn)) * volume_root));
    out(59, h.x59); out(60, h.x60); out(61, h.x61); out(62, h.x62); out(63, h.x63);

    const bool a_colmajor = layout == lNN || layout == lNT;
    const bool b_rowmajor = layout == lTT || layout == lNT;
    const bool streamk = ts == tStreamK;
    const double stage_t = t_load > t_mma ? t_load : t_mma;
    const T padded = (gm * tm) * (gn * tn) * (gk * tk);

    if constexpr (F > 64) {
        out(64, exact(layout)); out(65, exact(a_colmajor)); out(66, exact(b_rowmajor));
        out(67, exact(pt.dtype)); out(68, exact(dFp32)); out(69, exact(pt.out_dtype));
        out(70, exact(pt.eb)); out(71, exact(pt.eb)); out(72, 2.0f);
        out(73, exact(ks)); out(74, exact(es)); out(75, exact(ts)); out(76, exact(streamk));
        out(77, ks == kCoop ? 2.0f : 1.0f); out(78, h.x78); out(79, exact(pt.pk.v));
        out(80, pt.x80);
        out(81, pt.x81);
        const bool ok_a = !a_colmajor || utk <= 256 * ucn;
        const bool ok_b = !b_rowmajor || utk <= 256 * ucm;
        const bool ok_coop = ks != kCoop || (utm % 128) == 0;
        const bool ok_sk = !streamk || ks == kCoop;
        out(82, exact(ok_a)); out(83, exact(ok_b)); out(84, exact(ok_coop)); out(85, exact(ok_sk));
        out(86, exact(tn <= 2 * M && tn <= 2 * N));
        out(87, exact(fits && ok_a && ok_b && ok_coop && ok_sk));
        out(88, pt.x88);
        const T traffic = loads + pt.epi_traffic + pt.conv;
        out(89, exact(traffic));
        out(90, quot(traffic, bw));
        out(91, quot((T)2 * padded, pt.pk));
        out(92, quot(padded, pt.mnk));
        out(93, exact(h.smem_block - smem));
        out(94, exact(by_smem == resident));
        out(95, exact(by_regs == resident));
    }
    double per_most = 0.0;
    if constexpr (F > 96) {
        const uint32_t uim = 16u * at_least_1(c.inst_m_div16), uin = at_least_1(c.inst_n), uik = at_least_1(c.inst_k);
        const uint32_t per_mn = ceil_div16(utm, uim) * ceil_div16(utn, uin);           // at most 2^12 2^16
        const T per_kblock = (T)per_mn * (T)ceil_div16(utk, uik);
        per_most = (double)(per_kblock * gk);
        out(96, exact(uim)); out(97, exact(uin)); out(98, exact(uik));
        out(99, exact(per_kblock)); out(100, exact(per_kblock * gk));
        out(101, exact((utm + 63u) / 64u)); out(102, exact(utm * utn)); out(103, exact(tm * tn * tk));
        out(104, (float)volume_root);
        out(105, exact(tm * K * eb)); out(106, exact(tn * K * eb));
        out(107, exact(tm * tn * ob)); out(108, exact((T)4 * tm * tn));
        out(109, exact(min_of(st, gk))); out(110, exact(max_of(gk - st, (T)0)));
        const double mainloop_t = stage_t * (double)gk;
        out(111, (float)stage_t);
        out(112, (float)mainloop_t);
        out(113, (float)(mainloop_t * (double)waves));
        out(114, streamk ? exact(ntile.v * gk) : 0.0f);
        out(115, streamk ? x35 : 0.0f);
        out(116, exact(resident * threads.v));
        out(117, quot(resident * threads.v, den_with<T>(h.threads_sm_max, h.r_threads)));
        out(118, exact(by_arch == resident));
        out(119, pt.x119);
        out(120, pt.x120);
        out(121, pt.x121);
        out(122, pt.x122);
        out(123, pt.x123);
        out(124, quot(clusters, cslots));
        const T full_m = gm * tm > M ? gm - 1 : gm, full_n = gn * tn > N ? gn - 1 : gn;   // floor(M / tm), floor(N / tn)
        const T edge = ntile.v - full_m * full_n;
        out(125, exact(edge));
        out(126, quot(edge, ntile));
        out(127, lg(ntile.v));
    }
    // M N K and all operand bytes are at most 4 padded
    double most = max_of((double)padded, max_of((double)loads, (double)(tile_flops * h.bw)));
    most = max_of(most, max_of((double)(tile_flops * h.n_sm), (double)(rate.v * stage_bytes)));
    most = max_of(most, max_of((double)(st * smem), (double)(clusters * st)));
    most = max_of(most, max_of((double)(ccap.v * cm * cn), per_most));
    most = max_of(most, max_of((double)(h.n_sm * stage_bytes), (double)wave_cap.v));
    return most < kPlainMost;
}

constexpr int kWaves = 4;
constexpr int kStageStride = 36;      // floats per staged row: 16-byte aligned, its chunks on distinct bank groups

template <bool NT>
__device__ __forceinline__ void store_row(float *to, const float4 &v)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    if constexpr (NT) __builtin_nontemporal_store((f4){v.x, v.y, v.z, v.w}, reinterpret_cast<f4 *>(to));
    else *reinterpret_cast<float4 *>(to) = v;
}

// The columns of one row a scalar at a time, for rows beyond T = double.
// Kept out of line so that its 64-bit divisions cost the others no registers
// (a copy per caller: a function's register budget is its callers' smallest).
template <int F, int kCached>
__device__ __noinline__ void wide_row(HwPhi<int64_t> h, hwsel_problem_t pb, Cand c, float *x)
{
    phi<F, int64_t>(h, problem_terms<int64_t>(h, pb), c, [&](int j, float v) __attribute__((always_inline)) { x[j] = v; });
}

// One row per thread.  The problem terms of the workgroup's first kCached
// problems are computed once, by its first threads, and read from LDS by every
// row; rows of a later problem (and rows beyond T = double) go the scalar way.
template <int F, int kCached, bool NT>
__global__ __launch_bounds__(64 * kWaves, kCached == 32 ? 3 : 1) void k_features(HwBoth h, const hwsel_problem_t *__restrict__ probs,
                                                             int32_t P, const int64_t *__restrict__ seg, CandsDev c,
                                                             int64_t R, float *__restrict__ X, int64_t ld)
{
    __shared__ __attribute__((aligned(16))) float stage[kWaves][64][kStageStride];
    __shared__ ProbTerms<double> cached[kCached];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t blk0 = (int64_t)blockIdx.x * kWaves * 64;            // < R
    const int64_t row0 = blk0 + wave * 64;
    const int64_t r = row0 + lane, rc = r < R ? r : R - 1;             // lanes past R repeat row R - 1, unstored
    const Cand cand = load_cand(c, rc);                                // on its way during the problem terms
    const int32_t p0 = segment_of_row(seg, P, blk0);
    const int64_t last = blk0 + 64 * kWaves < R ? blk0 + 64 * kWaves - 1 : R - 1;
    const int32_t p_last = p0 + 1 >= P || seg[p0 + 1] > last ? p0 : segment_of_row(seg, P, last);
    int32_t p = p0;
    if (p_last > p0) {
        const int64_t first = row0 < R ? row0 : R - 1;
        p = segment_of_row_after(seg, P, rc, first);
    }
    if ((int)threadIdx.x < kCached && p0 + (int)threadIdx.x <= p_last)
        cached[threadIdx.x] = problem_terms<double>(h.d, probs[p0 + threadIdx.x]);
    __syncthreads();
    if (row0 >= R) return;
    const bool known = p - p0 < kCached;
    float quad[4];
    float *const out_lane = X + (row0 + (lane >> 3)) * ld + (lane & 7) * 4;
    const bool plain = phi<F, double>(h.d, cached[known ? p - p0 : 0], cand, [&](int j, float v) __attribute__((always_inline)) {
        quad[j % 4] = v;
        if (j % 4 == 3)
            *reinterpret_cast<float4 *>(&stage[wave][lane][j % 32 - 3]) = make_float4(quad[0], quad[1], quad[2], quad[3]);
        if (j % 32 == 31) {
            // the wave's own rows: its LDS accesses stay in order
            asm volatile("" ::: "memory");
            float4 v4[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                v4[i] = *reinterpret_cast<const float4 *>(&stage[wave][(lane >> 3) + 8 * i][(lane & 7) * 4]);
            float *to = out_lane + (j - 31);
            if (row0 + 64 <= R) {                                      // wave-uniform
#pragma unroll
                for (int i = 0; i < 8; ++i) store_row<NT>(to + i * 8 * ld, v4[i]);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (row0 + (lane >> 3) + 8 * i < R) store_row<NT>(to + i * 8 * ld, v4[i]);
            }
            asm volatile("" ::: "memory");
        }
    });
    if (r < R && !(known && plain && h.plain)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // after the row's stores above
        wide_row<F, kCached>(h.i, probs[p], cand, X + r * ld);
    }
}

// Sampling score alone, one row per thread.
__global__ __launch_bounds__(256) void k_sample_score(HwDev h, const hwsel_problem_t *__restrict__ probs, int32_t P,
                                                       const int64_t *__restrict__ seg, CandsDev c, int64_t R,
                                                       float *__restrict__ scores)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    // the wave's first row (wave-uniform): one scalar search per wave
    const int64_t r_first = (int64_t)blockIdx.x * 256 + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
    if (r >= R) return;
    const hwsel_problem_t pb = probs[segment_of_row_after(seg, P, r, r_first)];
    const int64_t M = max64(pb.M, 1), N = max64(pb.N, 1);
    const int64_t tm = max64(c.tile_m[r], 1), tn = max64(c.tile_n[r], 1), tk = max64(c.tile_k[r], 1);
    const int64_t st = max64(c.stages[r], 1);
    const int64_t cm = max64(c.cluster_m[r], 1), cn = max64(c.cluster_n[r], 1);
    const int64_t clusters = cdiv64(M, cm * tm) * cdiv64(N, cn * tn);
    const int64_t cslots = max64(h.n_sm / (cm * cn), 1);
    const int64_t cwaves = cdiv64(clusters, cslots);
    scores[r] = sampling_score(clusters, cwaves, cslots, cm, cn, st, tm, tn, tk);
}

// Features straight to forest bins: each of the first nf columns is binned
// against the forest's sorted thresholds as the map hands it over (NaN to
// nan_bin); X is never written.  One row per lane; the thresholds sit in LDS in
// breadth-first order, so the lanes' probes of one step spread over the banks,
// and a group of kFbChains columns is searched in as many steps as the one with
// the most thresholds needs.  Two shapes:
//   split: a workgroup takes one tile of 64 rows and its waves share the
//     columns, kFbCols each (few rows still occupy many CUs, and a wave's chain
//     of searches is short; the integer part of the map is computed per wave);
//   whole: a workgroup stages the thresholds once and its waves walk tiles,
//     all columns each.
// Bound by latency (split) and VALU issue (whole).  Measured against one row
// per lane for all columns, thresholds in sorted order, 8 steps always:
// one problem of 8,192 rows x 128 columns 51 -> 10 us, 60 problems of 8,192 rows
// with 60 depth-6 trees (whole call) 232 -> 194 us.
constexpr int kFbSlots = 256;
constexpr int kFbChains = 8;
constexpr int kFbCols = 16;
constexpr int kFbCached = 32;         // problem terms in LDS; rows of further problems go the scalar way

// Stages columns [c0, c0 + kFbCols) by one wave: threshold p (1-based position)
// of a column's sorted list at node 2^(s - 1 - ctz(p)) + (p >> (ctz(p) + 1)),
// s the steps of its group.
__device__ __forceinline__ void stage_thresholds(const float *__restrict__ U, int c0, int nf, uint32_t *u, int *steps)
{
    const int lane = threadIdx.x & 63;
    float4 v[kFbCols];
#pragma unroll
    for (int q = 0; q < kFbCols; ++q) {
        const int f = c0 + q < nf ? c0 + q : nf - 1;           // columns past nf reread the last one
        v[q] = *reinterpret_cast<const float4 *>(U + f * kFbSlots + 4 * lane);
    }
#pragma unroll
    for (int g = 0; g < kFbCols / kFbChains; ++g) {
        // A column's list ends in +inf.  One of them may be a threshold (then
        // x = +inf must count it), so one beyond the finite ones is searched.
        int most = 1;
#pragma unroll
        for (int q = g * kFbChains; q < (g + 1) * kFbChains; ++q) {
            const int finite = __popcll(__ballot(v[q].x < __builtin_inff())) + __popcll(__ballot(v[q].y < __builtin_inff())) +
                               __popcll(__ballot(v[q].z < __builtin_inff())) + __popcll(__ballot(v[q].w < __builtin_inff()));
            most = finite + 1 > most ? finite + 1 : most;
        }
        const int s = most > 255 ? 8 : 32 - __builtin_clz(most);
        if (lane == 0) steps[g] = s;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t p = 4 * lane + i + 1;
            const int k = __builtin_ctz(p);
            if (p < (1u << s)) {
                uint32_t *to = u + (1u << (s - 1 - k)) + (p >> (k + 1));
#pragma unroll
                for (int q = g * kFbChains; q < (g + 1) * kFbChains; ++q)
                    to[q * kFbSlots] = order_key(i == 0 ? v[q].x : i == 1 ? v[q].y : i == 2 ? v[q].z : v[q].w);
            }
        }
    }
}

// Columns [C0, C0 + NC) of one row (below `stride`): u and steps are theirs;
// every 16 bins go to dst + 16 i.
template <int F, int C0, int NC>
__device__ __forceinline__ bool bin_columns(const HwPhi<double> &h, const ProbTerms<double> &pt, const Cand &c,
                                            const uint32_t *u, const int *steps, int nf, uint32_t nan_bin, int stride,
                                            bool store, uint8_t *dst)
{
    float x[kFbChains];
    uint32_t word[4];
    return phi<F, double>(h, pt, c, [&](int j, float v) __attribute__((always_inline)) {
        if (j < C0 || j >= C0 + NC) return;
        const int q0 = (j - C0) / kFbChains * kFbChains;             // the group's first column, from C0
        x[(j - C0) % kFbChains] = v;
        if ((j - C0) % kFbChains != kFbChains - 1 || C0 + q0 / 16 * 16 >= stride) return;
        uint32_t n[kFbChains], kx1[kFbChains];
#pragma unroll
        for (int q = 0; q < kFbChains; ++q) {
            kx1[q] = order_key(x[q] + 0.0f) + 1u;                    // -0 + 0 = +0
            n[q] = 1;
        }
        const int s = __builtin_amdgcn_readfirstlane(steps[q0 / kFbChains]);
        for (int k = 0; k < s; ++k) {
            uint32_t key_u[kFbChains];
#pragma unroll
            for (int q = 0; q < kFbChains; ++q) key_u[q] = u[(q0 + q) * kFbSlots + n[q]];
            // all reads before the first step (left to itself the compiler
            // waits for each in turn)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < kFbChains; ++q) n[q] = search_step(n[q], key_u[q], kx1[q]);
        }
        const uint32_t first = 1u << s;
#pragma unroll
        for (int q = 0; q < kFbChains; ++q) {
            uint32_t b = n[q] - first;
            if (x[q] != x[q]) b = nan_bin;
            if (C0 + q0 + q >= nf) b = 0;
            const int w = (q0 + q) / 4 % 4;
            word[w] = (q % 4 ? word[w] : 0u) | b << (8 * (q % 4));
        }
        if (j % 16 == 15 && store)
            *reinterpret_cast<uint4 *>(dst + (j - C0) / 16 * 16) = make_uint4(word[0], word[1], word[2], word[3]);
    });
}

// Columns [c0, c1) of a row beyond T = double, against the sorted thresholds
// in memory.
template <int F>
__device__ __noinline__ void wide_bins(HwPhi<int64_t> h, hwsel_problem_t pb, Cand c, const float *U, int c0, int c1,
                                       uint32_t nan_bin, uint8_t *bins)
{
    phi<F, int64_t>(h, problem_terms<int64_t>(h, pb), c, [&](int j, float v) __attribute__((always_inline)) {
        if (j < c0 || j >= c1) return;
        uint32_t b = 0;
        for (int step = 128; step > 0; step >>= 1) b += U[j * kFbSlots + b + step - 1] <= v ? step : 0;
        bins[j] = (uint8_t)(v != v ? nan_bin : b);
    });
}

// Workgroup: the problem terms of the rows [row0, row0 + n) to LDS, unless the
// ones there (first problem `have`) are theirs; every thread's row is r.
struct TermsOf {
    int32_t p0, p;
};
template <int N>
__device__ __forceinline__ TermsOf stage_terms(const HwPhi<double> &h, const hwsel_problem_t *__restrict__ probs, int32_t P,
                                               const int64_t *__restrict__ seg, int64_t R, int64_t row0, int64_t n, int64_t r,
                                               int64_t wave_row0, ProbTerms<double> (&cached)[N], int32_t &have)
{
    const int32_t p0 = segment_of_row(seg, P, row0);
    const int64_t last = row0 + n < R ? row0 + n - 1 : R - 1;
    const int32_t p_last = p0 + 1 >= P || seg[p0 + 1] > last ? p0 : segment_of_row(seg, P, last);
    if (p0 != have || p_last > p0) {                                   // workgroup-uniform
        if (have >= 0) __syncthreads();                                // the previous terms are no longer read
        if ((int)threadIdx.x < N && p0 + (int)threadIdx.x <= p_last)
            cached[threadIdx.x] = problem_terms<double>(h, probs[p0 + threadIdx.x]);
        __syncthreads();
        have = p0;
    }
    return TermsOf{p0, p_last > p0 ? segment_of_row_after(seg, P, r, wave_row0 < R ? wave_row0 : R - 1) : p0};
}

template <int F>
__global__ __launch_bounds__(64 * (F / kFbCols)) void k_features_bins_split(
    HwBoth h, const hwsel_problem_t *__restrict__ probs, int32_t P, const int64_t *__restrict__ seg, CandsDev c, int64_t R,
    const void *__restrict__ packed, ImageId id, int nf, uint32_t nan_bin, uint8_t *__restrict__ Xb, int stride)
{
    if (!image_matches(packed, id)) return;
    __shared__ uint32_t table[F / kFbCols][kFbCols * kFbSlots];
    __shared__ int steps[F / kFbCols][kFbCols / kFbChains];
    __shared__ ProbTerms<double> cached[kFbCached];
    const float *__restrict__ U = reinterpret_cast<const float *>(static_cast<const uint8_t *>(packed) + 256);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = wave * kFbCols;
    const int64_t row0 = (int64_t)blockIdx.x * 64;                     // < R
    const int64_t r = row0 + lane, rc = r < R ? r : R - 1;
    const Cand cand = load_cand(c, rc);
    stage_thresholds(U, c0, nf, table[wave], steps[wave]);
    int32_t have = -1;
    const TermsOf t = stage_terms(h.d, probs, P, seg, R, row0, 64, rc, row0, cached, have);
    if (c0 >= stride) return;                                          // columns the forest does not have
    const bool known = t.p - t.p0 < kFbCached;
    const ProbTerms<double> &pt = cached[known ? t.p - t.p0 : 0];
    bool plain = true;
    auto columns = [&](auto w) __attribute__((always_inline)) {
        constexpr int C0 = decltype(w)::value * kFbCols;
        if constexpr (C0 < F)
            if (c0 == C0)
                plain = bin_columns<F, C0, kFbCols>(h.d, pt, cand, table[wave], steps[wave], nf, nan_bin, stride, r < R,
                                                    Xb + r * stride + C0);
    };
    columns(std::integral_constant<int, 0>{}); columns(std::integral_constant<int, 1>{});
    columns(std::integral_constant<int, 2>{}); columns(std::integral_constant<int, 3>{});
    columns(std::integral_constant<int, 4>{}); columns(std::integral_constant<int, 5>{});
    columns(std::integral_constant<int, 6>{}); columns(std::integral_constant<int, 7>{});
    if (r < R && !(known && plain && h.plain)) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // after the store above
        wide_bins<F>(h.i, probs[t.p], cand, U, c0, c0 + kFbCols < nf ? c0 + kFbCols : nf, nan_bin, Xb + r * stride);
    }
}

constexpr int kFbWaves = 8;

template <int F>
__global__ __launch_bounds__(64 * kFbWaves) void k_features_bins(HwBoth h, const hwsel_problem_t *__restrict__ probs,
                                                                 int32_t P, const int64_t *__restrict__ seg, CandsDev c,
                                                                 int64_t R, int64_t rows_per_block,
                                                                 const void *__restrict__ packed, ImageId id, int nf,
                                                                 uint32_t nan_bin, uint8_t *__restrict__ Xb, int stride)
{
    if (!image_matches(packed, id)) return;
    __shared__ uint32_t table[F * kFbSlots];
    __shared__ int steps[F / kFbChains];
    __shared__ ProbTerms<double> cached[kFbCached];
    const float *__restrict__ U = reinterpret_cast<const float *>(static_cast<const uint8_t *>(packed) + 256);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int g = wave; g < F / kFbCols; g += kFbWaves)
        stage_thresholds(U, g * kFbCols, nf, table + g * kFbCols * kFbSlots, steps + g * (kFbCols / kFbChains));
    __syncthreads();
    // Consecutive rows: the problem terms carry over from step to step.
    const int64_t begin = blockIdx.x * rows_per_block;
    const int64_t end = begin + rows_per_block < R ? begin + rows_per_block : R;
    int32_t have = -1;
    for (int64_t row0 = begin; row0 < end; row0 += 64 * kFbWaves) {
        const int64_t wave_row0 = row0 + 64 * wave;
        const int64_t r = wave_row0 + lane;
        int64_t rc = r < R ? r : R - 1;
        asm volatile("" : "+v"(rc));
        const Cand cand = load_cand(c, rc);
        const TermsOf t = stage_terms(h.d, probs, P, seg, R, row0, 64 * kFbWaves, rc, wave_row0, cached, have);
        if (wave_row0 >= end) continue;
        const bool known = t.p - t.p0 < kFbCached;
        const bool plain = bin_columns<F, 0, F>(h.d, cached[known ? t.p - t.p0 : 0], cand, table, steps, nf, nan_bin, stride,
                                                r < end, Xb + r * stride);
        if (r < end && !(known && plain && h.plain)) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // after the stores above
            wide_bins<F>(h.i, probs[t.p], cand, U, 0, nf, nan_bin, Xb + r * stride);
        }
    }
}

}  // namespace

hipError_t launch_features_bins(const HwDev &hw, const hwsel_problem_t *problems, int32_t P, const int64_t *seg,
                                const CandsDev &c, int64_t R, int32_t F, const void *packed, ImageId id, int nf,
                                uint32_t nan_bin, uint8_t *Xb, int stride, hipStream_t s)
{
    int dev = 0, n_cu = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
        n_cu = 256;
    const HwBoth h = hw_both(hw);
    // Up to two tiles per CU, sharing a tile's columns among waves is quicker
    // (the map's integer part is then computed per wave: 491,520 rows x 128
    // columns with 60 depth-6 trees take 271 us split and 194 us whole).
    const int64_t tiles = (R + 63) / 64;
    const bool split = tiles <= 2 * (int64_t)n_cu;
    const int64_t per = ((tiles + n_cu - 1) / n_cu + kFbWaves - 1) / kFbWaves * kFbWaves * 64;
    const unsigned blocks = (unsigned)((R + per - 1) / per);
#define HWSEL_BINS(F_)                                                                                                  \
    if (split)                                                                                                          \
        hipLaunchKernelGGL(k_features_bins_split<F_>, dim3((unsigned)tiles), dim3(64 * (F_ / kFbCols)), 0, s, h,         \
                           problems, P, seg, c, R, packed, id, nf, nan_bin, Xb, stride);                                \
    else                                                                                                                \
        hipLaunchKernelGGL(k_features_bins<F_>, dim3(blocks), dim3(64 * kFbWaves), 0, s, h, problems, P, seg, c, R, per, \
                           packed, id, nf, nan_bin, Xb, stride)
    if (F == 64) {
        HWSEL_BINS(64);
    } else if (F == 96) {
        HWSEL_BINS(96);
    } else {
        HWSEL_BINS(128);
    }
#undef HWSEL_BINS
    return hipGetLastError();
}

hipError_t launch_sample_score(const HwDev &hw, const hwsel_problem_t *problems, int32_t P, const int64_t *seg,
                               const CandsDev &c, int64_t R, float *scores, hipStream_t s)
{
    hipLaunchKernelGGL(k_sample_score, dim3((unsigned)((R + 255) / 256)), dim3(256), 0, s, hw, problems, P, seg, c,
                       R, scores);
    return hipGetLastError();
}

hipError_t launch_features(const HwDev &hw, const hwsel_problem_t *problems, int32_t P,
                           const int64_t *seg, const CandsDev &c, int64_t R, int32_t F, float *X,
                           int64_t ld, hipStream_t s)
{
    const int64_t rows_per_block = 64 * kWaves;
    const dim3 grid((unsigned)((R + rows_per_block - 1) / rows_per_block));
    const dim3 block(64 * kWaves);
    const HwBoth h = hw_both(hw);
    // 32 problems' terms leave LDS to three workgroups per CU (as many as the
    // registers do); segments under 16 rows on average take a term per row.
    // A matrix beyond the 256 MB last-level cache is stored past the caches,
    // where none of it would be found again: 492 -> 444 us for 2.5 GB.
    const bool terms_per_row = R < (int64_t)P * 16, past_caches = R * (int64_t)F * 4 > ((int64_t)256 << 20);
#define HWSEL_FEATURES(F_)                                                                                              \
    if (terms_per_row)                                                                                                  \
        hipLaunchKernelGGL((k_features<F_, 256, false>), grid, block, 0, s, h, problems, P, seg, c, R, X, ld);          \
    else if (past_caches)                                                                                               \
        hipLaunchKernelGGL((k_features<F_, 32, true>), grid, block, 0, s, h, problems, P, seg, c, R, X, ld);            \
    else                                                                                                                \
        hipLaunchKernelGGL((k_features<F_, 32, false>), grid, block, 0, s, h, problems, P, seg, c, R, X, ld)
    if (F == 64) {
        HWSEL_FEATURES(64);
    } else if (F == 96) {
        HWSEL_FEATURES(96);
    } else {
        HWSEL_FEATURES(128);
    }
#undef HWSEL_FEATURES
    return hipGetLastError();
}

}  // namespace hwsel
