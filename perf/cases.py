"""The work that users of this library have it do, as cases that can be timed and checked.

A selector ranks GEMM kernel configurations: problems and candidate rows go
through the feature map, a tree ensemble, an MLP or a cheap scorer rank the
rows, the best candidates of every problem are picked, and the picks are judged
against runtimes.  Each case is one such call or short chain of calls through
the public binding, with its inputs, model and buffers already in device
memory.  Inputs are synthetic: problems, candidates and runtimes of the shapes
the library's own workloads have (the knob grids of the paper, log-uniform
GEMM shapes), forests whose thresholds are quantiles of the features they
test, Kaiming MLP weights.

`features64` states the feature map in plain torch, int64 and binary64; it
makes the feature matrices the scorers read and the exact values of the
feature cases.
"""
from __future__ import annotations

import math

import torch

from paper_2609_35587_amd import hwsel

DEV = "cuda"

# The target hardware of the ranked kernels (a GH200: the workloads' own).
HW = dict(n_sm=132, smem_per_sm=233472, smem_per_block_max=232448, smem_reserved=2048, regs_per_sm=65536,
          max_regs_per_thread=255, max_blocks_per_sm=32, max_threads_per_sm=2048, arch_id=90, llc_bytes=52428800,
          hbm_bw_gbps=4000, peak_gflops=(989500, 989500, 1979000))


def listed():
    return [
        # One GEMM shape ranked over a short list of configurations with a
        # small ensemble, while the caller waits: the smallest call.
        dict(name="select-small", kind="select", P=1, C=512, F=64, trees=100, depth=6, k=5, grid="tiny", ragged=False),
        # One GEMM shape ranked with the full ensemble: a selector deployed in
        # front of a GEMM library.
        dict(name="select-online", kind="select", P=1, C=8192, F=128, trees=2000, depth=10, k=10, grid="full",
             ragged=False),
        # The feature matrix of the whole data set (600 problems x 8,192).
        dict(name="features-bulk", kind="features", P=600, C=8192, F=128, grid="full", ragged=False),
        # The full ensemble over the whole data set.
        dict(name="forest-bulk", kind="forest", R=4_915_200, F=128, trees=2000, depth=10),
        # A shallower ensemble on 96 columns over an odd number of rows.
        dict(name="forest-medium", kind="forest", R=1_000_003, F=96, trees=500, depth=8),
        # A forest too deep for the packed image, walked directly.
        dict(name="forest-direct", kind="direct", R=65_537, F=128, trees=150, depth=11),
        # The neural ranker over the whole data set, and over one problem's rows.
        dict(name="mlp-bulk", kind="mlp", R=4_915_200),
        dict(name="mlp-small", kind="mlp", R=3_001),
        # The cheap scorers (ridge model, analytic sampling score) over the data set.
        dict(name="scorers", kind="scorers", P=600, C=8192, F=128, grid="full", ragged=False),
        # A scorer judged on the data set: picks, regret, metrics, static baseline.
        dict(name="evaluate", kind="evaluate", P=600, C=8192, k=10, grid="full", ragged=True),
        # Picks and regret over the whole 65,536-point grid of 256 problems.
        dict(name="rank-long", kind="rank", P=256, C=65_536, k=16),
        # The valid configurations of 61 problems listed from the catalogue.
        dict(name="catalogue", kind="catalogue", P=61, guard=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["select", "select", "features", "forest", "forest", "direct", "mlp", "mlp", "scorers",
                       "evaluate", "rank", "catalogue"])
    if kind == "select":
        c = dict(kind=kind, P=_log(rng, 1, 64), C=_log(rng, 64, 8192), F=rng.choice([64, 96, 128]),
                 trees=_log(rng, 50, 2000), depth=rng.randint(5, 10), k=rng.randint(1, 32),
                 grid=rng.choice(["full", "paper"]), ragged=rng.random() < 0.5)
    elif kind in ("features", "scorers"):
        c = dict(kind=kind, P=_log(rng, 1, 600), C=_log(rng, 64, 8192), F=rng.choice([64, 96, 128]),
                 grid=rng.choice(["full", "paper"]), ragged=rng.random() < 0.5)
    elif kind == "forest":
        c = dict(kind=kind, R=_log(rng, 2000, 4_000_000), F=rng.choice([64, 96, 128]), trees=_log(rng, 50, 2000),
                 depth=rng.randint(4, 10))
    elif kind == "direct":
        c = dict(kind=kind, R=_log(rng, 1000, 100_000), F=rng.choice([64, 128]), trees=_log(rng, 20, 150),
                 depth=rng.randint(6, 12))
    elif kind == "mlp":
        c = dict(kind=kind, R=_log(rng, 500, 4_900_000))
    elif kind == "evaluate":
        c = dict(kind=kind, P=_log(rng, 20, 1000), C=_log(rng, 200, 8000), k=rng.randint(1, 32), grid="full",
                 ragged=rng.random() < 0.5)
    elif kind == "rank":
        P = _log(rng, 1, 256)
        c = dict(kind=kind, P=P, C=_log(rng, 5_000, min(500_000, 16_000_000 // P)), k=rng.randint(1, 64))
    else:
        c = dict(kind=kind, P=_log(rng, 1, 120), guard=rng.random() < 0.5)
    return c


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------
class Gen:
    """Seeded draws on the device."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def uniform(self, *shape, dtype=torch.float64):
        return torch.rand(shape, generator=self.g, device=DEV, dtype=dtype)

    def normal(self, *shape, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device=DEV, dtype=dtype)

    def integers(self, lo, hi, *shape):
        return torch.randint(lo, hi, shape, generator=self.g, device=DEV)


def make_problems(g, P, mixed):
    """M, N, K log-uniform in [16, 16384], a tenth of the Ks in [32768,
    131072], multiples of 8; any layout; with `mixed` any input type."""
    size = lambda lo, hi: (8 * torch.round(torch.exp(math.log(lo) + g.uniform(P) * math.log(hi / lo)) / 8)) \
        .clamp(min=8).long()  # noqa: E731
    M, N, K, deep = size(16, 16384), size(16, 16384), size(16, 16384), size(32776, 131072)
    K = torch.where(g.uniform(P) < 0.1, deep, K)
    layout = g.integers(0, 4, P)
    dtype = g.integers(0, 3, P) if mixed else torch.zeros(P, dtype=torch.long, device=DEV)
    rec = torch.zeros(P, 16, dtype=torch.uint8, device=DEV)
    for i, v in enumerate((M, N, K)):
        rec[:, 4 * i:4 * i + 4] = v.to(torch.int32).view(P, 1).view(torch.uint8)
    rec[:, 12], rec[:, 13] = layout.to(torch.uint8), dtype.to(torch.uint8)
    return dict(M=M, N=N, K=K, layout=layout, dtype=dtype, rec=rec)


_TN = [16, 32, 48, 64, 96, 128, 192, 256]
_PAIRS = [(m, n) for m in (1, 2, 4, 8, 16) for n in (1, 2, 4, 8, 16) if m * n <= 16]
# name -> axes, first slowest (a joint axis is a tuple of names)
GRIDS = {
    "tiny": [("tile_m", [64, 128, 256]), ("tile_n", [64, 128, 256]), ("tile_k", [32, 64]), ("stages", [2, 3, 4, 5]),
             ("cluster_m", [1, 2]), ("cluster_n", [1, 2]), ("swizzle", [1, 2, 4])],
    "full": [("tile_m", [64, 128, 192, 256]), ("tile_n", _TN), ("tile_k", [32, 64, 128, 256]), ("half", [0, 1]),
             ("stages", list(range(2, 10))), (("kernel_sched", "epi_sched"), [(0, 0), (0, 1), (1, 1), (2, 2)]),
             ("cluster_m", [1, 2]), ("cluster_n", [1, 2]), ("tile_sched", [0, 1])],
    "paper": [("tile_m", [64, 128, 192, 256]), ("tile_n", [16, 32, 48, 64, 80, 96, 128, 192, 256]),
              ("tile_k", [32, 64, 128, 256, 512]), ("stages", list(range(2, 13))),
              (("cluster_m", "cluster_n"), _PAIRS), ("kernel_sched", [0, 1, 2]), ("epi_sched", [0, 1, 2]),
              ("tile_sched", [0, 1])],
}


def decode(grid, index):
    """Knob values (int64) of grid points."""
    out, i = {}, index
    for name, values in reversed(GRIDS[grid]):
        d = i % len(values)
        i = i // len(values)
        for j, n in enumerate(name if isinstance(name, tuple) else (name,)):
            col = [v[j] if isinstance(v, tuple) else v for v in values]
            out[n] = torch.tensor(col, device=DEV)[d]
    if "half" in out:
        out["inst_n"] = torch.where(out.pop("half") == 1, out["tile_n"] // 2, out["tile_n"])
    out.setdefault("inst_n", out["tile_n"])
    one = torch.ones_like(index)
    out.setdefault("swizzle", one)
    for n, v in (("kernel_sched", 0), ("epi_sched", 1), ("tile_sched", 0)):
        out.setdefault(n, v * one)
    return out


def grid_size(grid):
    n = 1
    for _, values in GRIDS[grid]:
        n *= len(values)
    return n


def valid_points(k, layout, dtype, M=None, N=None):
    """The static validity constraints (ints or tensors that broadcast)."""
    b = 1 if dtype == 2 else 2
    frag = k["tile_m"].clamp(max=64) * k["tile_n"].clamp(max=32) * 2
    epi = torch.where(k["epi_sched"] == 0, 0, torch.where(k["epi_sched"] == 1, 2 * frag, 4 * frag))
    ok = (k["tile_sched"] != 1) | (k["kernel_sched"] == 2)
    ok &= (k["kernel_sched"] != 2) | (k["tile_m"] % 128 == 0)
    ok &= k["stages"] * (k["tile_m"] + k["tile_n"]) * k["tile_k"] * b + epi + HW["smem_reserved"] \
        <= HW["smem_per_block_max"]
    if layout in (2, 3):
        ok &= k["tile_k"] <= 256 * k["cluster_n"]
    if layout in (1, 3):
        ok &= k["tile_k"] <= 256 * k["cluster_m"]
    if M is not None:
        ok &= (k["tile_n"] <= 2 * M) & (k["tile_n"] <= 2 * N)
    return ok


def make_rows(g, probs, lens, grid):
    """Per problem a sorted draw of valid grid points (each at most once while
    there are enough).  Returns (seg int64 [P+1], row's problem, row's grid
    index)."""
    P = len(lens)
    knobs = decode(grid, torch.arange(grid_size(grid), device=DEV))
    lists, of, at = [], {}, 0
    key = (probs["layout"] * 3 + probs["dtype"]).tolist()
    for kk in sorted(set(key)):
        v = valid_points(knobs, kk // 3, kk % 3).nonzero().flatten()
        of[kk] = (at, len(v))
        lists.append(v)
        at += len(v)
    first = torch.tensor([of[k][0] for k in key], device=DEV)
    count = torch.tensor([of[k][1] for k in key], device=DEV)
    lens = torch.tensor(lens, device=DEV)
    seg = torch.zeros(P + 1, dtype=torch.long, device=DEV)
    seg[1:] = torch.cumsum(lens, 0)
    R = int(seg[-1])
    pid = torch.repeat_interleave(torch.arange(P, device=DEV), lens)
    j = torch.arange(R, device=DEV) - seg[pid]
    n, c = count[pid].double(), lens[pid].double()
    pos = torch.floor((j + g.uniform(R)) * n / c).long()
    pos = torch.minimum(pos, count[pid] - 1)
    return seg, pid, torch.cat(lists)[first[pid] + pos]


def make_cands(grid, index, dtype_row):
    k = decode(grid, index)
    k["inst_m_div16"] = torch.full_like(index, 4)
    k["inst_k"] = torch.where(dtype_row == 2, 32, 16)
    wide = ("tile_m", "tile_n", "tile_k", "inst_n")
    return {n: k[n].to(torch.int16 if n in wide else torch.uint8) for n in hwsel.CAND_FIELDS}


def make_lens(g, P, C, ragged):
    """Rows per problem: C, or spread evenly over [C/2, 3C/2] in seeded order."""
    if not ragged:
        return [C] * P
    even = C // 2 + torch.arange(P, device=DEV) * C // max(P - 1, 1)
    return even[torch.argsort(g.uniform(P))].clamp(min=1).tolist()


def make_input(g, P, C, grid, ragged, mixed):
    """Problems, segments and candidates of one batch."""
    probs = make_problems(g, P, mixed)
    seg, pid, index = make_rows(g, probs, make_lens(g, P, C, ragged), grid)
    cands = make_cands(grid, index, probs["dtype"][pid])
    return dict(probs=probs, seg=seg, pid=pid, index=index, cands=cands, R=int(seg[-1]), P=P)


def features64(inp, F, rows=None):
    """phi(p, c, h) in int64 and binary64, [R][F] float64 (rows: a slice)."""
    rows = rows or slice(0, inp["R"])
    pid = inp["pid"][rows]
    p = {n: inp["probs"][n][pid] for n in ("M", "N", "K", "layout", "dtype")}
    c = {n: v[rows].long() & (0xffff if v.dtype == torch.int16 else 0xff) for n, v in inp["cands"].items()}
    h = HW
    M, N, K = p["M"], p["N"], p["K"]
    q = lambda a, b: (a.double() if torch.is_tensor(a) else float(a)) / (b.double() if torch.is_tensor(b) else float(b))  # noqa: E731
    cd = lambda a, b: (a + b - 1) // b  # noqa: E731
    lg = lambda a: torch.log2(a.double())  # noqa: E731
    sel = lambda cond, a, b: torch.where(cond, a, b)  # noqa: E731
    tm, tn, tk, st = c["tile_m"], c["tile_n"], c["tile_k"], c["stages"]
    cm, cn, ks, es, ts = c["cluster_m"], c["cluster_n"], c["kernel_sched"], c["epi_sched"], c["tile_sched"]
    im, in_, ik = 16 * c["inst_m_div16"], c["inst_n"], c["inst_k"]
    eb = sel(p["dtype"] == 2, 1, 2)
    ob = 2
    od = sel(p["dtype"] == 1, 1, 0)
    pk = torch.tensor(h["peak_gflops"], device=DEV)[p["dtype"]]
    threads = sel(ks == 0, 256, 384)
    cons = sel(ks == 2, 2, 1)
    gm, gn, gk = cd(M, tm), cd(N, tn), cd(K, tk)
    nt = gm * gn
    stage = (tm + tn) * tk * eb
    main = st * stage
    frag = tm.clamp(max=64) * tn.clamp(max=32) * ob
    epi = sel(es == 0, 0 * frag, sel(es == 1, 2 * frag, 4 * frag))
    smem = sel(ks == 0, torch.maximum(main, epi), main + epi) + h["smem_reserved"]
    by_smem = h["smem_per_sm"] // smem
    regs = (cd(tm * tn, threads) + 32).clamp(max=h["max_regs_per_thread"])
    by_regs = h["regs_per_sm"] // (regs * threads)
    by_arch = (h["max_threads_per_sm"] // threads).clamp(max=h["max_blocks_per_sm"])
    res = torch.minimum(torch.minimum(by_smem, by_regs), by_arch)
    fits = main + epi + h["smem_reserved"] <= h["smem_per_block_max"]
    slots = h["n_sm"] * res.clamp(min=1)
    waves = cd(nt, slots)
    cap = waves * slots
    cl = cd(M, cm * tm) * cd(N, cn * tn)
    cs = (h["n_sm"] // (cm * cn)).clamp(min=1)
    cw = cd(cl, cs)
    ab, bb = eb * M * K, eb * K * N
    epit = 2 * ob * M * N
    loads = gn * ab + gm * bb
    conv = sel(od != p["dtype"], M * N * ob, torch.zeros_like(M))
    gf = 2 * M * N * K
    tf = 2 * tm * tn * tk
    llc, bw, sm = h["llc_bytes"], h["hbm_bw_gbps"], h["n_sm"]
    full = torch.ones_like(M)
    x = [lg(M), lg(N), lg(K), lg(gf), tm, tn, tk, st, cm, cn, cm * cn, c["swizzle"], gm, gn, gk, nt,
         q(gm * tm - M, M), q(gn * tn - N, N), q(gk * tk - K, K), q(nt, sm), threads, q(tm * tn, threads), regs,
         by_regs, stage, main, epi, smem, q(smem, h["smem_per_sm"]), by_smem, by_arch, res, fits, waves, q(nt, cap),
         q(cap - nt, cap), cl, cs, cw, q(cl, cw * cs), q(gm, cm), q(gn, cn), (cm > gm) | (cn > gn),
         q(gf, ab + bb + epit), q(2 * tm * tn, (tm + tn) * eb), q(loads, ab + bb), q(ab + bb, llc),
         q((tm + tn) * K * eb, llc), loads, epit, q(sm * stage, bw), q(tf * sm, cons * pk),
         q(tf * bw, cons * pk * stage), q(torch.minimum(st, gk), st), q(gk, st), q(st * smem, h["smem_per_sm"]),
         tk * st, st * res, q(cl * st, cw * cs * cm * cn) * torch.sqrt((tm * tn * tk).double()), full * sm,
         full * h["smem_per_sm"], full * h["regs_per_sm"], full * llc, full * bw]
    if F > 64:
        acol = (p["layout"] == 2) | (p["layout"] == 3)
        brow = (p["layout"] == 1) | (p["layout"] == 3)
        ok = [~acol | (tk <= 256 * cn), ~brow | (tk <= 256 * cm), (ks != 2) | (tm % 128 == 0), (ts != 1) | (ks == 2)]
        traffic = loads + epit + conv
        padded = (gm * tm) * (gn * tn) * (gk * tk)
        x += [p["layout"], acol, brow, p["dtype"], full * 3, od, eb, eb, full * ob, ks, es, ts, ts == 1, cons,
              full * h["arch_id"], pk, q(pk, bw), q(gf, ab + bb + epit) / q(pk, bw), *ok, (tn <= 2 * M) & (tn <= 2 * N),
              fits & ok[0] & ok[1] & ok[2] & ok[3], conv, traffic, q(traffic, bw), q(2 * padded, pk),
              q(padded, M * N * K), h["smem_per_block_max"] - smem, by_smem == res, by_regs == res]
    if F > 96:
        per = cd(tm, im) * cd(tn, in_) * cd(tk, ik)
        t_st = torch.maximum(q(sm * stage, bw), q(tf * sm, cons * pk))
        edge = nt - (M // tm) * (N // tn)
        x += [im, in_, ik, per, per * gk, cd(tm, 64), tm * tn, tm * tn * tk, torch.sqrt((tm * tn * tk).double()),
              tm * K * eb, tn * K * eb, tm * tn * ob, 4 * tm * tn, torch.minimum(st, gk), (gk - st).clamp(min=0), t_st,
              t_st * gk.double(), t_st * gk.double() * waves.double(), sel(ts == 1, nt * gk, 0 * nt),
              sel(ts == 1, q(cap - nt, cap), torch.zeros_like(t_st)), res * threads,
              q(res * threads, h["max_threads_per_sm"]), by_arch == res, q(ab, llc), q(bb, llc), q(ob * M * N, llc),
              q(M, N), q(K, torch.maximum(M, N)), q(cl, cs), edge, q(edge, nt), lg(nt)]
    out = torch.empty(len(M), F, dtype=torch.float64, device=DEV)
    for i, v in enumerate(x[:F]):
        out[:, i] = v
    return out


def matrix(inp, F):
    """The fp32 feature matrix, a million rows at a time."""
    X = torch.empty(inp["R"], F, dtype=torch.float32, device=DEV)
    for lo in range(0, inp["R"], 1 << 20):
        rows = slice(lo, min(lo + (1 << 20), inp["R"]))
        X[rows] = features64(inp, F, rows)
    return X


def make_matrix(g, R, F):
    """R rows of features: problems of up to 8,192 candidates each."""
    P = -(-R // 8192)
    lens = [8192] * (P - 1) + [R - 8192 * (P - 1)]
    probs = make_problems(g, P, False)
    seg, pid, index = make_rows(g, probs, lens, "full")
    inp = dict(probs=probs, seg=seg, pid=pid, index=index, cands=make_cands("full", index, probs["dtype"][pid]),
               R=int(seg[-1]), P=P)
    return matrix(inp, F)


def make_cuts(g, X):
    """Per column up to 255 split candidates: midpoints of neighbouring
    distinct values at its quantiles."""
    R, F = X.shape
    S = X[g.integers(0, R, min(4 * R, 16384))]
    S = torch.sort(S, dim=0).values
    n = S.shape[0]
    at = (torch.arange(1, 256, device=DEV) * n // 256).clamp(min=1)
    lo, hi = S[at - 1], S[at]                       # [255][F]
    mid = (0.5 * (lo.double() + hi.double())).float()
    ok = (hi > lo) & (mid > lo)
    order = torch.sort((~ok).int(), dim=0, stable=True).indices
    return torch.gather(mid, 0, order).t().contiguous(), ok.sum(0)


def make_forest(g, X, trees, depth):
    """Node features uniform over the columns that vary, thresholds uniform
    over the column's split candidates, leaves N(0, 0.1^2)."""
    cuts, n = make_cuts(g, X)
    cols = n.nonzero().flatten()
    n_int = (1 << depth) - 1
    feat = cols[g.integers(0, len(cols), trees, n_int)]
    j = (g.uniform(trees, n_int) * n[feat]).long()
    return dict(n_trees=trees, depth=depth, n_features=X.shape[1], flags=1, base_score=0.5,
                node_feature=feat.to(torch.uint8), node_threshold=cuts[feat, j].contiguous(),
                leaf_value=0.1 * g.normal(trees, 1 << depth))


MLP_WIDTHS = (128, 512, 512, 256, 1)


def make_mlp(g, X):
    m = {}
    for l in range(4):
        fi, fo = MLP_WIDTHS[l], MLP_WIDTHS[l + 1]
        m["W%d" % (l + 1)] = (g.normal(fo, fi) * math.sqrt(2 / fi)).bfloat16().view(torch.int16)
        m["b%d" % (l + 1)] = ((2 * g.uniform(fo) - 1) / math.sqrt(fi)).float()
    S = X[: 1 << 16].double()
    sd = S.std(0)
    m["mean"] = S.mean(0).float()
    m["inv_std"] = torch.where(sd > 0, 1 / sd, 0).nan_to_num(0, 0, 0).float()
    return m


def make_linear(g, X):
    F = X.shape[1]
    S = X[: 1 << 16].double()
    sd = S.std(0)
    return dict(n_features=F, bias=float(2 * g.uniform(1) - 1), mean=S.mean(0).float(),
                inv_std=torch.where(sd > 0, 1 / sd, 0).nan_to_num(0, 0, 0).float(), w=g.normal(F) / math.sqrt(F),
                w_onehot=0.1 * g.normal(12))


def make_times(g, pid, P):
    """Runtimes in seconds: a base per problem times lognormal noise; one in
    fifty candidates never runs."""
    base = 1e-6 * torch.exp(6 * g.uniform(P))
    t = (base[pid] * torch.exp(0.5 * g.normal(len(pid)).double())).float()
    t[g.uniform(len(pid)) < 0.02] = float("inf")
    return t


def make_scores(g, R):
    """Scores as an ensemble gives them: normal, some of them equal."""
    s = g.normal(R)
    return torch.where(g.uniform(R) < 0.1, torch.round(s * 64) / 64, s)


# ----------------------------------------------------------------------------
# Cases
# ----------------------------------------------------------------------------
def prepare(case, seed):
    g, kind = Gen(seed), case["kind"]
    s = dict(case=case)
    if kind in ("select", "features", "scorers"):
        inp = make_input(g, case["P"], case["C"], case["grid"], case["ragged"], case["grid"] == "paper")
        s.update(inp=inp, problems=inp["probs"]["rec"], seg=inp["seg"], cands=inp["cands"])
        R, F = inp["R"], case["F"]
    if kind == "select":
        f = make_forest(g, matrix(inp, F), case["trees"], case["depth"])
        s.update(forest=f, packed=hwsel.hwsel_forest_pack(f),
                 ws=torch.empty(hwsel.hwsel_select_forest_workspace_bytes(f, R), dtype=torch.uint8, device=DEV),
                 scores=torch.empty(R, device=DEV))
    elif kind == "features":
        s["X"] = torch.empty(R, F, device=DEV)
    elif kind == "scorers":
        s["X"] = matrix(inp, F)
        s.update(lin=make_linear(g, s["X"]), out=[torch.empty(R, device=DEV) for _ in range(2)])
    elif kind in ("forest", "direct"):
        s["X"] = make_matrix(g, case["R"], case["F"])
        f = s["forest"] = make_forest(g, s["X"], case["trees"], case["depth"])
        s["scores"] = torch.empty(case["R"], device=DEV)
        s["packed"] = s["ws"] = None
        if kind == "forest":
            s["packed"] = hwsel.hwsel_forest_pack(f)
            s["ws"] = torch.empty(hwsel.hwsel_forest_workspace_bytes(f, case["R"]), dtype=torch.uint8, device=DEV)
    elif kind == "mlp":
        s["X"] = make_matrix(g, case["R"], 128)
        m = s["mlp"] = make_mlp(g, s["X"])
        s.update(packed=hwsel.hwsel_mlp_pack(m), scores=torch.empty(case["R"], device=DEV))
    elif kind == "evaluate":
        probs = make_problems(g, case["P"], False)
        seg, pid, index = make_rows(g, probs, make_lens(g, case["P"], case["C"], case["ragged"]), case["grid"])
        s.update(seg=seg, pid=pid, ids=index.int(), n_cfg=grid_size(case["grid"]), scores=make_scores(g, len(pid)),
                 times=make_times(g, pid, case["P"]))
    elif kind == "rank":
        P, C = case["P"], case["C"]
        pid = torch.repeat_interleave(torch.arange(P, device=DEV), C)
        s.update(seg=torch.arange(P + 1, device=DEV) * C, pid=pid, scores=make_scores(g, P * C),
                 times=make_times(g, pid, P))
    elif kind == "catalogue":
        # the same problems for every seed, in another order: as many valid points
        probs = make_problems(Gen(case["P"]), case["P"], True)
        s.update(problems=probs["rec"][torch.argsort(g.uniform(case["P"]))].contiguous(),
                 mask=torch.empty(case["P"], hwsel.HWSEL_CATALOGUE_SIZE, dtype=torch.uint8, device=DEV))
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "select":
        return hwsel.hwsel_select_forest(HW, s["problems"], s["seg"], s["cands"], c["F"], s["forest"], s["packed"],
                                         c["k"], workspace=s["ws"], scores=s["scores"])
    if kind == "features":
        return hwsel.hwsel_features(HW, s["problems"], s["seg"], s["cands"], c["F"], X=s["X"])
    if kind == "scorers":
        return (hwsel.hwsel_linear_score(s["lin"], s["X"], scores=s["out"][0]),
                hwsel.hwsel_sample_score(HW, s["problems"], s["seg"], s["cands"], scores=s["out"][1]))
    if kind in ("forest", "direct"):
        return hwsel.hwsel_forest_score(s["forest"], s["X"], scores=s["scores"], packed=s["packed"],
                                        workspace=s["ws"])
    if kind == "mlp":
        return hwsel.hwsel_mlp_score(s["mlp"], s["X"], scores=s["scores"], packed=s["packed"])
    if kind == "evaluate":
        idx, vals = hwsel.hwsel_topk_per_problem(s["scores"], s["seg"], c["k"])
        return (idx, vals, hwsel.hwsel_regret(s["times"], s["seg"], idx),
                hwsel.hwsel_evaluate(s["times"], s["seg"], idx),
                hwsel.hwsel_static_config(s["times"], s["seg"], s["ids"], s["n_cfg"]))
    if kind == "rank":
        idx, vals = hwsel.hwsel_topk_per_problem(s["scores"], s["seg"], c["k"])
        return idx, vals, hwsel.hwsel_regret(s["times"], s["seg"], idx)
    if kind == "catalogue":
        # the list's length decides the buffers: a caller has to read it back
        mask, n = hwsel.hwsel_catalogue_mask(HW, s["problems"], int(c["guard"]), mask=s["mask"])
        total = int(n.sum())
        seg, point = hwsel.hwsel_catalogue_compact(mask, n, total)
        return mask, n, seg, point, hwsel.hwsel_catalogue_candidates(s["problems"], seg, total, point=point)
    raise ValueError(kind)


def work(case):
    """Inputs read once, outputs written once, and the arithmetic: a compare
    per node visited and an add per tree, two operations per weight."""
    kind = case["kind"]
    R = case.get("R", case.get("P", 0) * case.get("C", 0))
    if kind == "features":
        return {"bytes": R * (17 + 4 * case["F"]), "flops": 0}
    if kind == "scorers":
        return {"bytes": R * (17 + 4 * case["F"] + 8), "flops": R * 3 * case["F"]}
    if kind in ("forest", "direct", "select"):
        T, D = case["trees"], case["depth"]
        model = T * ((1 << D) - 1) * 5 + T * (1 << D) * 4
        row = 17 + 4 if kind == "select" else 4 * case["F"] + 4
        return {"bytes": R * row + model, "flops": R * T * (D + 1)}
    if kind == "mlp":
        return {"bytes": R * (4 * 128 + 4) + 917504, "flops": R * 918016}
    if kind == "evaluate":
        return {"bytes": R * 12, "flops": 0}
    if kind == "rank":
        return {"bytes": R * 8, "flops": 0}
    valid = 60_000 * case["P"]                # about as many points are valid
    return {"bytes": case["P"] * hwsel.HWSEL_CATALOGUE_SIZE + valid * (4 + 17), "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind in ("features", "catalogue"):
        return "exact"                        # whole numbers, and quotients rounded once
    if kind in ("forest", "direct"):
        return {"rel": 2e-6, "max": 2e-5}
    if kind == "select":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}
    if kind == "mlp":
        return {"rel": 1e-2, "max": 0.2}
    if kind == "scorers":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 1e-7, "max": 1e-6}         # picks are exact; regrets are one quotient


# ----------------------------------------------------------------------------
# 64-bit values
# ----------------------------------------------------------------------------
def forest64(f, X):
    """Every tree walked, leaves added in binary64."""
    T, D = f["n_trees"], f["depth"]
    n_int, R = (1 << D) - 1, X.shape[0]
    feat, thr = f["node_feature"].flatten(), f["node_threshold"].flatten()
    leaf = f["leaf_value"].flatten()
    out = torch.full((R,), float(f["base_score"]), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // R)
    for t0 in range(0, T, step):
        t = torch.arange(t0, min(T, t0 + step), device=DEV)
        node = torch.zeros(R, len(t), dtype=torch.long, device=DEV)
        for _ in range(D):
            at = node + t * n_int
            x = torch.gather(X, 1, feat[at].long())
            node = 2 * node + 2 - (x < thr[at]).long()
        out += leaf[node - n_int + t * (n_int + 1)].double().sum(1)
    return out


def mlp64(m, X):
    out = torch.empty(X.shape[0], dtype=torch.float64, device=DEV)
    W = [m["W%d" % l].view(torch.bfloat16).double().t().contiguous() for l in range(1, 5)]
    for lo in range(0, len(out), 1 << 18):
        h = (X[lo:lo + (1 << 18)].double() - m["mean"].double()) * m["inv_std"].double()
        for l in range(4):
            h = h @ W[l] + m["b%d" % (l + 1)].double()
            if l < 3:
                h = 0.5 * h * (1 + torch.erf(h * math.sqrt(0.5)))
        out[lo:lo + (1 << 18)] = h[:, 0]
    return out


def linear64(m, X):
    out = torch.empty(X.shape[0], dtype=torch.float64, device=DEV)
    F = m["n_features"]
    w = m["w"].double().clone()
    cat = {64: (0, 4), 73: (4, 3), 74: (7, 3), 75: (10, 2)} if F > 64 else {}
    for c in cat:
        w[c] = 0
    for lo in range(0, len(out), 1 << 20):
        x = X[lo:lo + (1 << 20)].double()
        y = ((x - m["mean"].double()) * m["inv_std"].double()) @ w + m["bias"]
        for c, (slot, levels) in cat.items():
            for l in range(levels):
                y += torch.where(x[:, c] == l, m["w_onehot"][slot + l].double(), 0.0)
        out[lo:lo + (1 << 20)] = y
    return out


def picks64(s, k):
    """Top k by score then index, and best-of-k regrets; equal segments are
    not assumed."""
    seg, scores, times, pid = s["seg"], s["scores"], s["times"], s["pid"]
    P, R = len(seg) - 1, len(scores)
    key = torch.sort(-scores, stable=True).indices            # by score, ties by row
    order = key[torch.sort(pid[key], stable=True).indices]    # within each problem
    at = seg[:-1, None] + torch.arange(k, device=DEV)
    there = at < seg[1:, None]
    row = order[at.clamp(max=R - 1)]
    idx = torch.where(there, row - seg[:-1, None], -1)
    vals = torch.where(there, scores[row].double(), -math.inf)
    t = torch.where(there, times[row].double(), math.inf)
    best = torch.full((P,), math.inf, dtype=torch.float64, device=DEV)
    best.scatter_reduce_(0, pid, times.double(), "amin")
    y = lambda a, b: torch.where(a == b, 1.0, a / b)  # noqa: E731
    return idx, vals, 1 - y(best, t[:, 0]), 1 - y(best, t.min(1).values), best, t[:, 0]


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "features":
        return features64(s["inp"], case["F"])
    if kind == "select":
        X = matrix(s["inp"], case["F"])
        sc = forest64(s["forest"], X)
        P, k = case["P"], case["k"]
        vals = torch.full((P, k), -math.inf, dtype=torch.float64, device=DEV)
        for p, (a, b) in enumerate(zip(s["seg"][:-1].tolist(), s["seg"][1:].tolist())):
            n = min(k, b - a)
            vals[p, :n] = torch.topk(sc[a:b], n).values
        return None, vals, sc
    if kind in ("forest", "direct"):
        return forest64(s["forest"], s["X"])
    if kind == "mlp":
        return mlp64(s["mlp"], s["X"])
    if kind == "scorers":
        step, sample = 1 << 20, []
        for lo in range(0, s["inp"]["R"], step):
            sample.append(features64(s["inp"], 64, slice(lo, min(lo + step, s["inp"]["R"])))[:, 58].clone())
        return linear64(s["lin"], s["X"]), torch.cat(sample)
    if kind in ("evaluate", "rank"):
        idx, vals, r1, rk, best, t1 = picks64(s, case["k"])
        got = (idx, vals, (r1, rk, None))
        if kind == "rank":
            return got
        seg, pid, times = s["seg"], s["pid"], s["times"].double()
        y = torch.where(times == best[pid], 1.0, best[pid] / times)
        n = (seg[1:] - seg[:-1]).double()
        zero = torch.zeros(len(n), dtype=torch.float64, device=DEV)
        ybar = zero.index_add(0, pid, y) / n
        rank = 1 + zero.index_add(0, pid, (times < t1[pid]).double())
        q = torch.quantile(r1, torch.tensor([0.5, 0.95], dtype=torch.float64, device=DEV))
        out = torch.stack([r1.mean(), q[0], q[1], r1.max(), (rank == 1).double().mean(), (rank <= 5).double().mean(),
                           (r1 <= 0.05).double().mean(), (1 - ybar).mean(), torch.tensor(float(len(n)), device=DEV,
                                                                                     dtype=torch.float64)])
        return (*got, (out, r1, rank.int(), ybar), None)
    return None                               # the catalogue is whole numbers
