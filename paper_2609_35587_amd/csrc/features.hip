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
// row checks before its columns, see phi): binary64 multiplies and adds run at
// the full vector rate, an integer division is a multiply by a reciprocal and a
// truncation, and quotients by one denominator share its reciprocal.  T =
// int64_t takes the rows beyond that, whose 64-bit products wrap as they
// always did, and every row when a hardware field is too large (HwBoth::plain):
// 491,520 such rows 57 us, 46 us plain ones.
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

// The feature map of one row: start(plain), then out(j, x_j) for the columns
// j < F in order if it returns true (wave-uniform).  plain: every integer of
// the row stays below 2^52, so that T = double holds it exactly (the bounds
// checked cover the others: sums and differences of them, and products by at
// most 4).
template <int F, class T, class Start, class Out>
__device__ __forceinline__ void phi(const HwPhi<T> &h, const ProbTerms<T> &pt, const Cand &c, Start &&start, Out &&out)
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

    const T padded = (gm * tm) * (gn * tn) * (gk * tk);
    const uint32_t uim = 16u * at_least_1(c.inst_m_div16), uin = at_least_1(c.inst_n), uik = at_least_1(c.inst_k);
    T per_kblock = 0;
    if constexpr (F > 96)                              // instructions of a tile's plane: at most 2^12 2^16
        per_kblock = (T)(ceil_div16(utm, uim) * ceil_div16(utn, uin)) * (T)ceil_div16(utk, uik);

    if constexpr (std::is_same_v<T, double>) {
        // M N K and all operand bytes are at most 4 padded
        double most = max_of((double)padded, max_of((double)loads, (double)(tile_flops * h.bw)));
        most = max_of(most, max_of((double)(tile_flops * h.n_sm), (double)(rate.v * stage_bytes)));
        most = max_of(most, max_of((double)(st * smem), (double)(clusters * st)));
        most = max_of(most, max_of((double)(ccap.v * cm * cn), (double)(per_kblock * gk)));
        most = max_of(most, max_of((double)(h.n_sm * stage_bytes), (double)wave_cap.v));
        if (!start(most < kPlainMost)) return;
    } else {
        if (!start(true)) return;
    }

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
    if constexpr (F > 96) {
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
}

constexpr int kWaves = 4;
constexpr int kStageStride = 36;      // floats per staged row: 16-byte aligned, its chunks on distinct bank groups
typedef float Staged[64][kStageStride];
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <class T>
using lds_ptr = __attribute__((address_space(3))) T *;
template <class T>
using arg_ptr = const __attribute__((address_space(4))) T *;

// The kernel's arguments in a function that is not inlined, whose parameters
// come in vector registers: read as scalars again.
template <class T>
__device__ __forceinline__ const T &args_of(arg_ptr<T> p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return *(const T *)(arg_ptr<T>)(((uint64_t)hi << 32) | lo);
}

// Problems of rows first .. last and the lane's own, of row r between them: two
// scalar searches (one, where all are of one problem), then one per lane
// between their results.  p0 <= p whatever the offsets hold.
struct Problems {
    int32_t p0, p_last, p;
};
__device__ __forceinline__ Problems problems_of(const int64_t *__restrict__ seg, int32_t P, int64_t first, int64_t last, int64_t r)
{
    const int32_t p0 = segment_of_row(seg, P, first);
    if (p0 + 1 >= P || seg[p0 + 1] > last) return Problems{p0, p0, p0};
    const int32_t p_last = segment_of_row(seg, P, last);
    int32_t lo = p0, hi = p_last + 1;
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (seg[mid] <= r) lo = mid; else hi = mid;
    }
    return Problems{p0, p_last, lo};
}

template <bool NT>
__device__ __forceinline__ void store_row(float *to, f32x4 v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<f32x4 *>(to));
    else *reinterpret_cast<f32x4 *>(to) = v;
}

// The columns of a wave's rows by way of LDS to X; `want`: the lane has a row.
// Returns the rows stored: those wanted whose integers T holds.
template <int F, bool NT, class T>
__device__ __forceinline__ uint64_t write_rows(const HwPhi<T> &h, const ProbTerms<T> &pt, const Cand &cand, bool want,
                                               Staged &stage, float *x0, int64_t ld)
{
    const int lane = threadIdx.x & 63;
    uint64_t done = 0;
    float quad[4];
    float *const out_lane = x0 + (lane >> 3) * ld + (lane & 7) * 4;
    phi<F, T>(h, pt, cand,
              [&](bool plain) __attribute__((always_inline)) {
                  done = __ballot(want && plain);
                  return done != 0;
              },
              [&](int j, float v) __attribute__((always_inline)) {
        quad[j % 4] = v;
        if (j % 4 == 3)
            *reinterpret_cast<float4 *>(&stage[lane][j % 32 - 3]) = make_float4(quad[0], quad[1], quad[2], quad[3]);
        if (j % 32 == 31) {
            // the wave's own rows: its LDS accesses stay in order
            asm volatile("" ::: "memory");
            auto row = [&](int i) { return *reinterpret_cast<const f32x4 *>(&stage[(lane >> 3) + 8 * i][(lane & 7) * 4]); };
            const f32x4 v0 = row(0), v1 = row(1), v2 = row(2), v3 = row(3), v4 = row(4), v5 = row(5), v6 = row(6), v7 = row(7);
            float *const to = out_lane + (j - 31);
            // (straight on where all are: code not fetched yet is slow)
            if (__builtin_expect(done == ~0ull, 1)) {                  // wave-uniform
                store_row<NT>(to, v0); store_row<NT>(to + 8 * ld, v1); store_row<NT>(to + 16 * ld, v2);
                store_row<NT>(to + 24 * ld, v3); store_row<NT>(to + 32 * ld, v4); store_row<NT>(to + 40 * ld, v5);
                store_row<NT>(to + 48 * ld, v6); store_row<NT>(to + 56 * ld, v7);
            } else {
                const uint64_t mine = done >> (lane >> 3);
                if (mine & 1) store_row<NT>(to, v0);
                if (mine >> 8 & 1) store_row<NT>(to + 8 * ld, v1);
                if (mine >> 16 & 1) store_row<NT>(to + 16 * ld, v2);
                if (mine >> 24 & 1) store_row<NT>(to + 24 * ld, v3);
                if (mine >> 32 & 1) store_row<NT>(to + 32 * ld, v4);
                if (mine >> 40 & 1) store_row<NT>(to + 40 * ld, v5);
                if (mine >> 48 & 1) store_row<NT>(to + 48 * ld, v6);
                if (mine >> 56 & 1) store_row<NT>(to + 56 * ld, v7);
            }
            asm volatile("" ::: "memory");
        }
    });
    return done;
}

// The rows a wave has left: `later`, whose problems' terms are not in LDS (a
// row computes them for itself), then what is beyond T = double.  Kept out of
// line so that the 64-bit divisions cost the others no registers (a copy per
// caller: a function's register budget is its callers' smallest).
template <int F, bool NT, bool OWN>
__device__ __noinline__ void write_rest(arg_ptr<HwBoth> args, const hwsel_problem_t *__restrict__ probs, int32_t p, Cand cand,
                                        uint64_t left, uint64_t later, lds_ptr<Staged> stage, float *x0, int64_t ld)
{
    const HwBoth &h = args_of(args);
    const int lane = threadIdx.x & 63;
    const hwsel_problem_t pb = probs[p];
    if (later)
        left &= ~write_rows<F, NT, double>(h.d, problem_terms<double>(h.d, pb), cand, later >> lane & 1, *(Staged *)stage, x0, ld);
    if (left)
        write_rows<F, NT, int64_t>(h.i, problem_terms<int64_t>(h.i, pb), cand, left >> lane & 1, *(Staged *)stage, x0, ld);
}

// One row per thread.  The terms of the workgroup's first kTerms problems are
// computed by its first threads and read from LDS by the rows (each wave for
// itself took 2 us longer on few rows); with OWN every row computes its
// problem's for itself.
constexpr int kTerms = 64;

template <int F, bool OWN, bool NT>
__global__ __launch_bounds__(64 * kWaves, OWN ? 2 : 3) void k_features(HwBoth h, const hwsel_problem_t *__restrict__ probs,
                                                             int32_t P, const int64_t *__restrict__ seg, CandsDev c,
                                                             int64_t R, float *__restrict__ X, int64_t ld)
{
    __shared__ __attribute__((aligned(16))) Staged stage[kWaves];
    __shared__ ProbTerms<double> terms[OWN ? 1 : kTerms];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t blk0 = (int64_t)blockIdx.x * kWaves * 64, row0 = blk0 + wave * 64;      // blk0 < R
    const int64_t r = row0 + lane, rc = r < R ? r : R - 1;             // lanes past R repeat row R - 1, unstored
    const Cand cand = load_cand(c, rc);                                // on its way during the problem terms
    const Problems at = problems_of(seg, P, blk0, blk0 + 64 * kWaves <= R ? blk0 + 64 * kWaves - 1 : R - 1, rc);
    if constexpr (!OWN) {
        if ((int)threadIdx.x < kTerms && at.p0 + (int)threadIdx.x <= at.p_last)
            terms[threadIdx.x] = problem_terms<double>(h.d, probs[at.p0 + threadIdx.x]);
        __syncthreads();
    }
    if (row0 >= R) return;
    uint64_t left = __ballot(r < R), later = 0;
    float *const x0 = X + row0 * ld;
    if (h.plain) {
        if constexpr (OWN) {
            left &= ~write_rows<F, NT, double>(h.d, problem_terms<double>(h.d, probs[at.p]), cand, r < R, stage[wave], x0, ld);
        } else {
            const bool in = r < R && at.p - at.p0 < kTerms;
            later = left & ~__ballot(in);
            left &= ~write_rows<F, NT, double>(h.d, terms[in ? at.p - at.p0 : 0], cand, in, stage[wave], x0, ld);
        }
    }
    if (left)                                                          // (h is the kernel's first argument)
        write_rest<F, NT, OWN>((arg_ptr<HwBoth>)__builtin_amdgcn_kernarg_segment_ptr(), probs, at.p, cand, left, later,
                               (lds_ptr<Staged>)&stage[wave], x0, ld);
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
// per lane for all columns, thresholds in sorted order, 8 steps always, with
// 2,000 trees of depth 6: 8,192 rows x 128 columns 42 -> 10 us, 491,520 rows
// 156 -> 77 us, 4,915,200 rows 1.26 -> 0.78 ms; with 2,000 trees of depth 10
// (8 steps for every column that varies) 1.25 -> 0.94 ms.
constexpr int kFbSlots = 256;
constexpr int kFbChains = 8;
constexpr int kFbCols = 16;

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

// Columns [c0, c0 + NC) of a wave's rows (those below `stride`): u and steps
// are theirs; every 16 bins go to dst + 16 i.  Returns the rows stored: those
// wanted whose integers T holds.
template <int F, int NC, class T>
__device__ __forceinline__ uint64_t write_bins(const HwPhi<T> &h, const ProbTerms<T> &pt, const Cand &c, bool want, int c0,
                                               const uint32_t *u, const int *steps, int nf, uint32_t nan_bin, int stride,
                                               uint8_t *dst)
{
    const int lane = threadIdx.x & 63;
    uint64_t done = 0;
    float x[kFbChains];
    uint32_t word[4];
    phi<F, T>(h, pt, c,
              [&](bool plain) __attribute__((always_inline)) {
                  done = __ballot(want && plain);
                  return done != 0;
              },
              [&](int j, float v) __attribute__((always_inline)) {
        x[j % kFbChains] = v;
        if (j % kFbChains != kFbChains - 1) return;
        const int f0 = j - (kFbChains - 1), q0 = NC == F ? f0 : f0 - c0;          // the group's first column, from c0
        if (q0 < 0 || q0 >= NC || f0 / 16 * 16 >= stride) return;
        uint32_t n[kFbChains], kx1[kFbChains];
#pragma unroll
        for (int q = 0; q < kFbChains; ++q) {
            kx1[q] = order_key(x[q] + 0.0f) + 1u;                    // -0 + 0 = +0
            n[q] = 1;
        }
        const int s = __builtin_amdgcn_readfirstlane(steps[q0 / kFbChains]);
        const uint32_t *const ug = u + q0 * kFbSlots;
        for (int k = 0; k < s; ++k) {
            uint32_t key_u[kFbChains];
#pragma unroll
            for (int q = 0; q < kFbChains; ++q) key_u[q] = ug[q * kFbSlots + n[q]];
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
            const int w = (f0 + q) / 4 % 4;
            word[w] = (q % 4 ? word[w] : 0u) | b << (8 * (q % 4));
        }
        if (f0 + kFbChains > nf) {                                   // columns past the forest's: 0
#pragma unroll
            for (int i = 0; i < kFbChains / 4; ++i) {
                const int n_in = nf - (f0 + 4 * i);
                word[f0 / 4 % 4 + i] &= n_in >= 4 ? ~0u : n_in <= 0 ? 0u : (1u << (8 * n_in)) - 1u;
            }
        }
        if (j % 16 == 15 && (done >> lane & 1))
            *reinterpret_cast<uint4 *>(dst + (q0 & ~15)) = make_uint4(word[0], word[1], word[2], word[3]);
    });
    return done;
}

struct BinsArgs {
    HwBoth h;
    CandsDev c;
    const hwsel_problem_t *probs;
    const int64_t *seg;
    const void *packed;
    uint8_t *Xb;
    ImageId id;
    int32_t P, nf, stride;
    uint32_t nan_bin;
    int64_t R, rows_per_block;
};

// The bins of the rows a wave has left (see write_rest), columns [c0, c0 + NC).
template <int F, int NC>
__device__ __noinline__ void bins_rest(arg_ptr<BinsArgs> args, int32_t p, Cand cand, uint64_t left, uint64_t later, int c0,
                                       lds_ptr<const uint32_t> u, lds_ptr<const int> steps, uint8_t *dst)
{
    const BinsArgs &a = args_of(args);
    const int lane = threadIdx.x & 63;
    c0 = __builtin_amdgcn_readfirstlane(c0);
    const hwsel_problem_t pb = a.probs[p];
    if (later)
        left &= ~write_bins<F, NC, double>(a.h.d, problem_terms<double>(a.h.d, pb), cand, later >> lane & 1, c0, (const uint32_t *)u,
                                           (const int *)steps, a.nf, a.nan_bin, a.stride, dst);
    if (left)
        write_bins<F, NC, int64_t>(a.h.i, problem_terms<int64_t>(a.h.i, pb), cand, left >> lane & 1, c0, (const uint32_t *)u,
                                   (const int *)steps, a.nf, a.nan_bin, a.stride, dst);
}

template <int F>
__global__ __launch_bounds__(64 * (F / kFbCols)) void k_features_bins_split(BinsArgs a)
{
    if (!image_matches(a.packed, a.id)) return;
    __shared__ uint32_t table[F / kFbCols][kFbCols * kFbSlots];
    __shared__ int steps[F / kFbCols][kFbCols / kFbChains];
    __shared__ ProbTerms<double> terms[kTerms];
    const float *__restrict__ U = reinterpret_cast<const float *>(static_cast<const uint8_t *>(a.packed) + 256);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c0 = wave * kFbCols;
    const int64_t row0 = (int64_t)blockIdx.x * 64;                     // < R
    const int64_t r = row0 + lane, rc = r < a.R ? r : a.R - 1;
    const Cand cand = load_cand(a.c, rc);
    stage_thresholds(U, c0, a.nf, table[wave], steps[wave]);
    const Problems at = problems_of(a.seg, a.P, row0, row0 + 63 < a.R ? row0 + 63 : a.R - 1, rc);
    if ((int)threadIdx.x < kTerms && at.p0 + (int)threadIdx.x <= at.p_last)
        terms[threadIdx.x] = problem_terms<double>(a.h.d, a.probs[at.p0 + threadIdx.x]);
    __syncthreads();
    if (c0 >= a.stride) return;                                        // columns the forest does not have
    uint8_t *const dst = a.Xb + rc * a.stride + c0;
    uint64_t left = __ballot(r < a.R), later = 0;
    if (a.h.plain) {
        const bool in = r < a.R && at.p - at.p0 < kTerms;
        const ProbTerms<double> &pt = terms[in ? at.p - at.p0 : 0];
        later = left & ~__ballot(in);
        auto columns = [&](auto w) __attribute__((always_inline)) {
            constexpr int C0 = decltype(w)::value * kFbCols;
            if constexpr (C0 < F)
                if (c0 == C0)
                    left &= ~write_bins<F, kFbCols, double>(a.h.d, pt, cand, in, C0, table[wave], steps[wave], a.nf, a.nan_bin,
                                                            a.stride, dst);
        };
        columns(std::integral_constant<int, 0>{}); columns(std::integral_constant<int, 1>{});
        columns(std::integral_constant<int, 2>{}); columns(std::integral_constant<int, 3>{});
        columns(std::integral_constant<int, 4>{}); columns(std::integral_constant<int, 5>{});
        columns(std::integral_constant<int, 6>{}); columns(std::integral_constant<int, 7>{});
    }
    if (left)
        bins_rest<F, kFbCols>((arg_ptr<BinsArgs>)__builtin_amdgcn_kernarg_segment_ptr(), at.p, cand, left, later, c0,
                              (lds_ptr<const uint32_t>)&table[wave][0], (lds_ptr<const int>)&steps[wave][0], dst);
}

constexpr int kFbWaves = 8;
constexpr int kWaveTerms = 16;        // problems' terms a wave keeps in LDS

template <int F>
__global__ __launch_bounds__(64 * kFbWaves) void k_features_bins(BinsArgs first)
{
    if (!image_matches(first.packed, first.id)) return;
    __shared__ uint32_t table[F * kFbSlots];
    __shared__ int steps[F / kFbChains];
    __shared__ ProbTerms<double> terms[kFbWaves][kWaveTerms];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    {
        const float *__restrict__ U = reinterpret_cast<const float *>(static_cast<const uint8_t *>(first.packed) + 256);
        for (int g = wave; g < F / kFbCols; g += kFbWaves)
            stage_thresholds(U, g * kFbCols, first.nf, table + g * kFbCols * kFbSlots, steps + g * (kFbCols / kFbChains));
    }
    __syncthreads();
    // Consecutive rows: the problem terms carry over from step to step.
    const int64_t begin = blockIdx.x * first.rows_per_block;
    const int64_t end = begin + first.rows_per_block < first.R ? begin + first.rows_per_block : first.R;
    int32_t have0 = 0, have1 = 0;
    arg_ptr<BinsArgs> args = (arg_ptr<BinsArgs>)__builtin_amdgcn_kernarg_segment_ptr();
    for (int64_t row0 = begin + 64 * wave; row0 < end; row0 += 64 * kFbWaves) {
        // The arguments are read again in every step (scalar loads that hit):
        // kept through the loop, they and what follows from them spill 340
        // scalar registers.
        asm volatile("" : "+s"(args));
        const BinsArgs &a = *(const BinsArgs *)args;
        const int64_t r = row0 + lane;
        int64_t rc = r < end ? r : end - 1;
        asm volatile("" : "+v"(rc));
        const Cand cand = load_cand(a.c, rc);
        const Problems at = problems_of(a.seg, a.P, row0, row0 + 63 < end ? row0 + 63 : end - 1, rc);
        uint8_t *const dst = a.Xb + rc * a.stride;
        uint64_t left = __ballot(r < end), later = 0;
        if (a.h.plain) {
            // the terms of the wave's first problems, unless they are there
            if (at.p0 < have0 || (at.p_last < at.p0 + kWaveTerms ? at.p_last + 1 : at.p0 + kWaveTerms) > have1) {
                have0 = at.p0;
                have1 = at.p_last < at.p0 + kWaveTerms ? at.p_last + 1 : at.p0 + kWaveTerms;
                if (lane < have1 - have0) terms[wave][lane] = problem_terms<double>(a.h.d, a.probs[have0 + lane]);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                __builtin_amdgcn_wave_barrier();
            }
            const bool in = r < end && at.p < have1;
            later = left & ~__ballot(in);
            left &= ~write_bins<F, F, double>(a.h.d, terms[wave][in ? at.p - have0 : 0], cand, in, 0, table, steps, a.nf, a.nan_bin,
                                              a.stride, dst);
        }
        if (left)
            bins_rest<F, F>(args, at.p, cand, left, later, 0, (lds_ptr<const uint32_t>)&table[0], (lds_ptr<const int>)&steps[0], dst);
    }
}

}  // namespace

hipError_t launch_features_bins(const HwDev &hw, const hwsel_problem_t *problems, int32_t P, const int64_t *seg,
                                const CandsDev &c, int64_t R, int32_t F, const void *packed, ImageId id, int nf,
                                uint32_t nan_bin, uint8_t *Xb, int stride, hipStream_t s)
{
    const int n_cu = compute_units();
    const HwBoth h = hw_both(hw);
    // Up to two tiles per CU, sharing a tile's columns among waves is quicker
    // (the map's integer part is then computed per wave).  Whole call, 128
    // columns, 64 trees of depth 6, split / whole: 8,192 rows 23 / 36 us,
    // 32,768 32 / 38, 49,152 41 / 39, 131,072 92 / 49.
    const int64_t tiles = (R + 63) / 64;
    const bool split = tiles <= 2 * (int64_t)n_cu;
    const int64_t per = ((tiles + n_cu - 1) / n_cu + kFbWaves - 1) / kFbWaves * kFbWaves * 64;
    const unsigned blocks = (unsigned)((R + per - 1) / per);
    const BinsArgs a{h, c, problems, seg, packed, Xb, id, P, nf, stride, nan_bin, R, per};
#define HWSEL_BINS(F_)                                                                                                  \
    if (split) hipLaunchKernelGGL(k_features_bins_split<F_>, dim3((unsigned)tiles), dim3(64 * (F_ / kFbCols)), 0, s, a);  \
    else hipLaunchKernelGGL(k_features_bins<F_>, dim3(blocks), dim3(64 * kFbWaves), 0, s, a)
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
    // kTerms problems' terms leave LDS to three workgroups per CU (as many as
    // the registers do) and cover a workgroup's rows at four rows per problem
    // on average; with fewer, every row computes its own: 500,000 rows, shared /
    // own, 1 row per problem 86 / 69 us, 3 83 / 67, 4 59 / 65, 16 53 / 57.
    // A matrix beyond the 256 MB last-level cache is stored past the caches,
    // where none of it would be found again: 492 -> 444 us for 2.5 GB.
    const bool terms_per_row = R < (int64_t)P * 4, past_caches = R * (int64_t)F * 4 > ((int64_t)256 << 20);
#define HWSEL_FEATURES(F_)                                                                                              \
    if (terms_per_row)                                                                                                  \
        hipLaunchKernelGGL((k_features<F_, true, false>), grid, block, 0, s, h, problems, P, seg, c, R, X, ld);          \
    else if (past_caches)                                                                                               \
        hipLaunchKernelGGL((k_features<F_, false, true>), grid, block, 0, s, h, problems, P, seg, c, R, X, ld);            \
    else                                                                                                                \
        hipLaunchKernelGGL((k_features<F_, false, false>), grid, block, 0, s, h, problems, P, seg, c, R, X, ld)
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
