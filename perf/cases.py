"""What the speed of this library is measured on.

Every case goes through the public entry points of `paper_2310_05037_amd.lib`
on inputs shaped like the ones `workloads.py` draws (random reference, 6-mer
levels, reads with skips and dwells, true and decoy candidates), drawn here on
the GPU so that making them is quick.  Case fields:

  kind      batch | extend | bnb | span | path | band | band_chains | anchored
  pairs     (read, candidate region) pairs; candidate chains for the last two
  median, sigma, n_lo, n_hi
            read lengths (events): clip(round(LogNormal(ln median, sigma)))
  flat      read lengths uniform in [n_lo, n_hi] instead
  cands     most candidates per read, uniform in 1..cands (fixed: exactly it)
  ratio_lo, ratio_hi
            region levels per event, uniform
  band      band half-width as a fraction of the levels
  reads, chunk, chunks, serving
            streaming: reads in one tick, events per chunk, most chunks per
            read, and whether the serving launch options are used
"""
import math

import numpy as np
import torch

from paper_2310_05037_amd import lib, workloads

DEV = "cuda" if torch.cuda.is_available() else "cpu"
SKIP, DWELL, NOISE = workloads.SKIP_P, workloads.DWELL_P, workloads.NOISE_SD
EVENTS_PER_KMER = (1 - SKIP) / DWELL
B_MATCH = workloads.SYNTHETIC_B_MATCH
THRESHOLD = 20.0
UNEVEN = dict(median=1500, sigma=0.6, n_lo=100, n_hi=8000, cands=50, ratio_lo=1.2, ratio_hi=3.0)


def listed():
    return [
        # One read against its ten candidates, as a mapper that takes reads
        # one by one calls it: latency.
        dict(name="single_read", kind="batch", pairs=10, median=1566, sigma=0.0, n_lo=1, n_hi=8000, cands=10, fixed=True,
             ratio_lo=0.5716, ratio_hi=0.5716),
        # A Read Until tick at 2,000 reads/s: the chunks of the few reads
        # that became ready in half a millisecond, with the serving options.
        dict(name="serving_tick", kind="extend", reads=4, cands=50, chunk=400, chunks=10, serving=True, ratio_lo=1.2,
             ratio_hi=3.0),
        # A tick after a stall: hundreds of reads wait, library defaults.
        dict(name="serving_backlog", kind="extend", reads=160, cands=50, chunk=400, chunks=10, serving=False, ratio_lo=1.2,
             ratio_hi=3.0),
        # The plain batch of moderate reads, ten candidates each.
        dict(name="plain_batch", kind="batch", pairs=4096, flat=True, n_lo=200, n_hi=2000, cands=10, fixed=True,
             ratio_lo=1.2, ratio_hi=2.0),
        # Throughput mapping: the uneven batch (the benchmark's headline).
        dict(UNEVEN, name="uneven_batch", kind="batch", pairs=100_000),
        # Few, long problems (ultra-long reads).
        dict(name="long_regions", kind="batch", pairs=1024, median=10_000, sigma=0.0, n_lo=1, n_hi=10_000, cands=1,
             fixed=True, ratio_lo=2.0, ratio_hi=2.0),
        # Mapping with early termination, candidates in chaining order.
        dict(UNEVEN, name="early_termination", kind="bnb", pairs=20_000),
        # Scores, ends and starts (mapping positions).
        dict(UNEVEN, name="alignment_start", kind="span", pairs=10_000),
        # Warping paths of reads against their accepted candidate.
        dict(UNEVEN, name="warping_path", kind="path", pairs=500, cands=1, fixed=True),
        # Banded alignment of whole chains (20% band, more events than levels).
        dict(UNEVEN, name="banded_chains", kind="band_chains", pairs=40_000, band=0.2),
        # Banded alignment of candidate regions (20% band, more levels than events).
        dict(UNEVEN, name="banded_regions", kind="band", pairs=10_000, band=0.2),
        # Anchor-guided alignment: the gaps of 100,000 chains, their sums and
        # the decision.
        dict(UNEVEN, name="anchored_chains", kind="anchored", pairs=100_000),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["batch", "batch", "long", "extend", "extend", "bnb", "span", "path", "band", "band_chains",
                       "anchored"])
    if kind == "extend":
        lo = round(rng.uniform(1.0, 2.0), 3)
        return dict(kind=kind, reads=_log_uniform(rng, 1, 160), cands=rng.randint(1, 50), chunk=_log_uniform(rng, 100, 800),
                    chunks=rng.randint(1, 10), serving=rng.random() < 0.5, ratio_lo=lo,
                    ratio_hi=round(lo + rng.uniform(0.0, 1.5), 3))
    most = {"batch": 50_000, "long": 1024, "bnb": 20_000, "span": 10_000, "path": 500, "band": 10_000,
            "band_chains": 40_000, "anchored": 100_000}[kind]
    least = {"batch": 3, "long": 16, "path": 5}.get(kind, 40)
    c = dict(kind="batch" if kind == "long" else kind, pairs=_log_uniform(rng, least, most))
    if kind == "long":
        c.update(median=_log_uniform(rng, 3000, 10_000), sigma=0.0, n_lo=1, n_hi=10_000, cands=1, fixed=True)
        lo = round(rng.uniform(1.2, 2.0), 3)
        c.update(ratio_lo=lo, ratio_hi=lo)
    else:
        lo = round(rng.uniform(0.5, 1.5), 3)
        c.update(median=_log_uniform(rng, 150, 1500), sigma=round(rng.uniform(0.0, 0.6), 3), n_lo=60, n_hi=8000,
                 cands=1 if kind == "path" else rng.randint(1, 50), ratio_lo=lo,
                 ratio_hi=round(lo + rng.uniform(0.0, 1.5), 3))
    if kind in ("band", "band_chains"):
        c["band"] = round(rng.uniform(0.05, 0.25), 3)
    return c


# ---- shapes (host; the same for every seed, which draws the values) ------------------

REF_BASES = 10_000_000


def _shapes(c):
    """Read lengths, candidates per read, owning read and region length of
    every pair, and how many events of each read are aligned already."""
    g = np.random.Generator(np.random.PCG64(20))
    if c["kind"] == "extend":
        R = c["reads"]
        total = g.integers(1, c["chunks"] + 1, size=R)          # chunks of the whole read
        at = (g.random(R) * total).astype(np.int64)              # chunks already aligned
        k = g.integers(1, c["cands"] + 1, size=R)
        own = np.repeat(np.arange(R), k)
        m = np.maximum(np.floor(c["chunk"] * total[own] * g.uniform(c["ratio_lo"], c["ratio_hi"], len(own))), 1)
        return (at + 1) * c["chunk"], k, own, m.astype(np.int64), at * c["chunk"]
    P = c["pairs"]
    k = np.full(P, c["cands"]) if c.get("fixed") else g.integers(1, c["cands"] + 1, size=P)
    R = int(np.searchsorted(np.cumsum(k), P)) + 1
    k = k[:R].copy()
    k[-1] -= int(k.sum()) - P
    if c.get("flat"):
        n = g.integers(c["n_lo"], c["n_hi"] + 1, size=R)
    else:
        n = np.clip(np.round(g.lognormal(math.log(c["median"]), c["sigma"], R)), c["n_lo"], c["n_hi"]).astype(np.int64)
    own = np.repeat(np.arange(R), k)
    m = np.maximum(np.floor(n[own] * g.uniform(c["ratio_lo"], c["ratio_hi"], P)), 1).astype(np.int64)
    return n, k, own, m, None


def work(c):
    n, k, own, m, _ = _shapes(c)
    P, kind = len(own), c["kind"]
    qn = n[own]
    if kind in ("anchored", "band_chains"):
        # a decoy chain spans 0.6 of its read on average; anchors cover 8
        # k-mers and gaps 12 (sum of squares 276) on average
        kmers = float((qn * np.where(np.r_[True, own[1:] != own[:-1]], 1.0, 0.6)).sum()) / EVENTS_PER_KMER
        if kind == "anchored":
            gaps = kmers / 20.0
            return {"bytes": 4.0 * gaps * 12 * (1 + EVENTS_PER_KMER) + 28 * gaps + 24 * P + 24 * len(n),
                    "flops": 4.0 * gaps * 276 * EVENTS_PER_KMER}
        km = qn * np.where(np.r_[True, own[1:] != own[:-1]], 1.0, 0.6) / EVENTS_PER_KMER
        return {"bytes": float(4 * km.sum() * (1 + EVENTS_PER_KMER) + 36 * P),
                "flops": float(4.0 * (2 * c["band"] * km * km * EVENTS_PER_KMER).sum())}
    tables = 24 * P + 8 * P + 24 * len(n)
    if kind == "extend":
        return {"bytes": float(4 * c["chunk"] * len(n) + 12 * m.sum() + tables + 9 * P), "flops": 4.0 * c["chunk"] * float(m.sum())}
    b = float(4 * n.sum() + 4 * m.sum() + tables)
    cells = float((qn * m).sum())
    if kind == "bnb":   # at least each read's winning candidate
        cells = float((qn * m)[np.r_[True, own[1:] != own[:-1]]].sum())
    elif kind == "band":
        w = np.ceil(c["band"] * m)
        cells = float((qn * np.minimum(m, 2 * w * (1 - c["band"] / 2) + 1)).sum())
    elif kind == "span":   # the table, and the read against its own span backwards
        cells += float((qn * qn / EVENTS_PER_KMER).sum())
    elif kind == "path":
        cells += float((qn * qn / EVENTS_PER_KMER).sum())
        b += 8.0 * float(qn.sum())
    return {"bytes": b, "flops": 4.0 * cells}


# ---- inputs ------------------------------------------------------------------------

def _segments(counts):
    """(owner, position within owner) of a ragged layout with these counts."""
    own = torch.repeat_interleave(torch.arange(len(counts), device=DEV), counts)
    first = torch.cumsum(counts, 0) - counts
    return own, torch.arange(len(own), device=DEV) - first[own], first


def _dwells(gen, size):
    u = torch.rand(size, generator=gen, device=DEV, dtype=torch.float64).clamp_(min=1e-12)
    d = torch.ceil(torch.log(u) / math.log(1 - DWELL)).clamp_(min=1).to(torch.int64)
    return torch.where(torch.rand(size, generator=gen, device=DEV) < SKIP, torch.zeros_like(d), d)


def _inputs(c, seed):
    """Reference levels, reads and candidate regions (host index arrays)."""
    n, k, own, m, pre = _shapes(c)
    g = np.random.Generator(np.random.PCG64(seed))
    gen, form = torch.Generator(device=DEV), torch.Generator(device=DEV)
    gen.manual_seed(1_000_003 * seed + 17)
    form.manual_seed(20)   # dwells and anchors: part of the shapes
    model = torch.randn(workloads.N_KMERS, generator=gen, device=DEV)
    bases = torch.randint(0, 4, (REF_BASES,), generator=gen, device=DEV)
    L = REF_BASES - workloads.K + 1
    idx = torch.zeros(L, dtype=torch.int64, device=DEV)
    for t in range(workloads.K):
        idx = idx * 4 + bases[t:t + L]
    r = model[idx]
    start = g.integers(0, L - 4 * int(n.max()) - 256, size=len(n))
    nd = torch.from_numpy(n).to(DEV)
    kk = nd // 2 + 64
    ro, pos, first = _segments(kk)
    d = _dwells(form, len(ro))
    cs = torch.cumsum(d, 0)
    upto = cs - (cs[first] - d[first])[ro]                       # events up to and with this k-mer
    upto = torch.minimum(upto, nd[ro])
    upto = torch.where(pos == kk[ro] - 1, nd[ro], upto)
    before = torch.where(pos == 0, torch.zeros_like(upto), torch.roll(upto, 1))
    lv = r[torch.from_numpy(start).to(DEV)[ro] + pos]
    q = torch.repeat_interleave(lv, upto - before)
    q = (q + NOISE * torch.randn(len(q), generator=gen, device=DEV)).contiguous()
    used = torch.zeros(len(n), dtype=torch.int64, device=DEV).index_add_(0, ro, (before < nd[ro]).to(torch.int64))
    span = used.cpu().numpy()
    q_start = np.concatenate([[0], np.cumsum(n)[:-1]])
    m = np.minimum(m, L)
    true = np.r_[True, own[1:] != own[:-1]]
    off = (g.random(len(own)) * (L - m + 1)).astype(np.int64)
    slack = np.maximum(m - span[own], 0)
    t_off = start[own] - (g.random(len(own)) * (slack + 1)).astype(np.int64)
    off = np.where(true, np.clip(t_off, 0, L - m), off)
    return dict(q=q, r=r, n=n, k=k, own=own, m=m, off=off, q_start=q_start, start=start, span=span, g=g, form=form, pre=pre,
                kmer_events=before, kmer_first=first.cpu().numpy(), L=L)


def _t(x, dt):
    return torch.from_numpy(np.ascontiguousarray(x).astype(dt)).to(DEV)


def _pairs(c, seed):
    """Plain values of every pair: slices of q and r, candidates of each read."""
    x = _inputs(c, seed)
    first = np.concatenate([[0], np.cumsum(x["k"])[:-1]])
    if c["kind"] == "bnb":   # chaining puts the true candidate first for nine reads in ten
        swap = np.nonzero((x["g"].random(len(first)) >= 0.9) & (x["k"] > 1))[0]
        other = first[swap] + 1 + (x["g"].random(len(swap)) * (x["k"][swap] - 1)).astype(np.int64)
        for key in ("off", "m"):
            a = x[key]
            a[first[swap]], a[other] = a[other].copy(), a[first[swap]].copy()
    p = dict(q=x["q"], r=x["r"], q_off=x["q_start"][x["own"]], q_len=x["n"][x["own"]], r_off=x["off"], r_len=x["m"],
             cand_off=first, cand_cnt=x["k"], n_events=x["n"], pre=x["pre"], own=x["own"])
    if c["kind"] == "extend":   # the chunk's events; the ones before it are aligned already
        p["q_all"], p["q_all_len"] = p["q_off"], p["q_len"]
        p["done"] = x["pre"][x["own"]]
        p["q_off"], p["q_len"] = p["q_off"] + p["done"], p["q_len"] - p["done"]
    if c["kind"] in ("band", "band_chains"):
        p["band"] = np.ceil(c["band"] * p["r_len"])
    return p


def _chains(c, seed):
    """Chains of anchors of 4..12 k-mers, gaps of a geometric number (mean 12)
    of k-mers between them: the true candidate's on the read's source path,
    a decoy's pairing a random stretch of the read with a random stretch of
    the reference."""
    x = _inputs(c, seed)
    g, form, own, n, L = x["g"], x["form"], x["own"], x["n"], x["L"]
    sizes = np.random.Generator(np.random.PCG64(21))
    P = len(own)
    true = np.r_[True, own[1:] != own[:-1]]
    span = np.where(true, n[own], np.maximum(1, (n[own] * sizes.uniform(0.2, 1.0, P)).astype(np.int64)))
    e0 = np.where(true, 0, (g.random(P) * (n[own] - span + 1)).astype(np.int64))
    kmers = np.where(true, x["span"][own], np.maximum(1, (span / EVENTS_PER_KMER).astype(np.int64)))
    l0 = np.where(true, x["start"][own], (g.random(P) * (L - kmers + 1)).astype(np.int64))
    # a decoy's events per k-mer are fresh dwells, the true chain's are its read's
    kd, td = torch.from_numpy(kmers).to(DEV), torch.from_numpy(true).to(DEV)
    ko, kpos, kfirst = _segments(kd + 1)
    dw = torch.cumsum(_dwells(form, len(ko)), 0)
    fresh = torch.minimum(torch.roll(dw, 1) - torch.roll(dw, 1)[kfirst][ko], torch.from_numpy(span).to(DEV)[ko])
    fresh = torch.where(kpos == 0, torch.zeros_like(fresh), fresh)
    at = torch.from_numpy(x["kmer_first"][own]).to(DEV)[ko] + kpos
    read_ev = torch.where(kpos == kd[ko], torch.from_numpy(n[own]).to(DEV)[ko],
                          x["kmer_events"][at.clamp(max=len(x["kmer_events"]) - 1)])
    ev = torch.where(td[ko], read_ev, fresh)                  # events before k-mer kpos of the chain
    # alternating anchors and gaps
    uo, upos, ufirst = _segments(kd // 8 + 4)
    a = torch.randint(4, 13, (len(uo),), generator=form, device=DEV)
    u = torch.rand(len(uo), generator=form, device=DEV, dtype=torch.float64).clamp_(min=1e-12)
    gap = torch.ceil(torch.log(u) / math.log(1 - 1 / workloads.GAP_MEAN_KMERS)).clamp_(min=1).to(torch.int64)
    step = torch.where(upos == 0, torch.randint(0, 3, (len(uo),), generator=form, device=DEV), torch.roll(a + gap, 1))
    cs = torch.cumsum(step, 0)
    a0 = cs - (cs[ufirst] - step[ufirst])[uo]                   # first k-mer of the anchor
    ok = a0 + a <= kd[uo]
    uo, a0, a1 = uo[ok], a0[ok], (a0 + a)[ok]
    es, ee = ev[kfirst[uo] + a0], ev[kfirst[uo] + a1]
    # an anchor that follows a gap without events is dropped: the gap runs on
    same = torch.zeros_like(uo, dtype=torch.bool)
    same[1:] = uo[1:] == uo[:-1]
    keep = ~(same & (es == torch.roll(ee, 1)))
    uo, a0, a1, es, ee = uo[keep], a0[keep], a1[keep], es[keep], ee[keep]
    same = torch.zeros_like(uo, dtype=torch.bool)
    same[1:] = uo[1:] == uo[:-1]
    qb = torch.from_numpy(x["q_start"][own] + e0).to(DEV)
    rb = torch.from_numpy(l0).to(DEV)
    h = torch.nonzero(same).reshape(-1)
    gaps = dict(q_off=qb[uo[h]] + ee[h - 1], q_len=es[h] - ee[h - 1], r_off=rb[uo[h]] + a1[h - 1], r_len=a0[h] - a1[h - 1])
    cnt = torch.bincount(uo[h], minlength=P)
    lead = torch.nonzero(~same).reshape(-1)
    last = torch.cat([lead[1:] - 1, torch.tensor([len(uo) - 1], device=DEV)])
    zeros = torch.zeros(P, dtype=torch.int64, device=DEV)
    fe, le = zeros.clone(), zeros.clone()
    fl, ll = zeros.clone(), zeros.clone()
    fe[uo[lead]], le[uo[lead]], fl[uo[lead]], ll[uo[lead]] = es[lead], ee[last], a0[lead], a1[last]
    first = np.concatenate([[0], np.cumsum(x["k"])[:-1]])
    return dict(q=x["q"], r=x["r"], gaps=gaps, gap_cnt=cnt, gap_off=torch.cumsum(cnt, 0) - cnt, events=le - fe,
                levels=ll - fl, seg_q=qb + fe, seg_r=rb + fl, cand_off=first, cand_cnt=x["k"])


def _segment_pairs(c, seed):
    x = _chains(c, seed)
    lv = x["levels"].cpu().numpy()
    return dict(q=x["q"], r=x["r"], q_off=x["seg_q"].cpu().numpy(), q_len=x["events"].cpu().numpy(),
                r_off=x["seg_r"].cpu().numpy(), r_len=lv, band=np.ceil(c["band"] * lv), cand_off=x["cand_off"],
                cand_cnt=x["cand_cnt"], n_events=None)


# ---- state and one pass --------------------------------------------------------------

def _empty(n, dt):
    return torch.empty(int(n), dtype=dt, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "anchored":
        x = _chains(case, seed)
        gp, P, R = x["gaps"], len(x["events"]), len(x["cand_off"])
        i64, i32 = torch.int64, torch.int32
        return dict(kind=kind, q=x["q"], r=x["r"],
                    gaps=tuple(gp[k].to(t).contiguous() for k, t in (("q_off", i64), ("q_len", i32), ("r_off", i64), ("r_len", i32))),
                    chains=(x["gap_off"].to(i64).contiguous(), x["gap_cnt"].to(i32).contiguous(), x["events"].to(i32).contiguous()),
                    reads=(_t(x["cand_off"], np.int64), _t(x["cand_cnt"], np.int32)),
                    cost=_empty(len(gp["q_off"]), torch.float32), chain_cost=_empty(P, torch.float32), best=_empty(R, i32),
                    best_score=_empty(R, torch.float64), mapped=_empty(R, torch.uint8))
    p = _segment_pairs(case, seed) if kind == "band_chains" else _pairs(case, seed)
    P, R = len(p["q_off"]), len(p["cand_off"])
    s = dict(kind=kind, q=p["q"], r=p["r"], q_off=_t(p["q_off"], np.int64), q_len=_t(p["q_len"], np.int32),
             r_off=_t(p["r_off"], np.int64), r_len=_t(p["r_len"], np.int32), cand_off=_t(p["cand_off"], np.int64),
             cand_cnt=_t(p["cand_cnt"], np.int32), score=_empty(P, torch.float32), end=_empty(P, torch.int32))
    if kind in ("batch", "extend", "bnb"):
        s.update(n_events=_t(p["n_events"], np.int32), best=_empty(R, torch.int32), best_score=_empty(R, torch.float64),
                 mapped=_empty(R, torch.uint8))
    if kind in ("span", "path"):
        s["start"] = _empty(P, torch.int32)
    if kind in ("extend", "bnb"):
        s["row_off"] = _t(np.concatenate([[0], np.cumsum(p["r_len"])[:-1]]), np.int64)
        s["rows"] = torch.zeros(int(p["r_len"].sum()), dtype=torch.float32, device=DEV)
    if kind == "bnb":
        s["max_query"] = int(p["q_len"].max())
    if kind == "path":
        off, words = lib.path_workspace(p["q_len"], p["r_len"])
        s["dir_off"], s["dirs"] = _t(off, np.int64), _empty(words, torch.int64)
        s["path_off"] = _t(np.concatenate([[0], np.cumsum(p["q_len"])[:-1]]), np.int64)
        s["lo"], s["hi"] = _empty(p["q_len"].sum(), torch.int32), _empty(p["q_len"].sum(), torch.int32)
    if kind in ("band", "band_chains"):
        s["band"] = _t(p["band"], np.int32)
    if kind == "extend":
        s["opts"] = lib.make_opts(streams=3, single_max=2048, long_kernel=lib.LONG_PIPELINE,
                                  pipe_waves=8) if case["serving"] else None
        s["first"] = _t(p["done"] == 0, np.uint8)
        # the resident rows hold the chunks aligned so far
        lib.rawalign_dtw_extend(s["q"], _t(p["q_all"], np.int64), _t(p["done"], np.int32), s["r"], s["r_off"], s["r_len"],
                                s["rows"], s["row_off"], torch.ones_like(s["first"]), s["score"], s["end"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "anchored":
        lib.rawalign_dtw_global_batch(s["q"], *s["gaps"][:2], s["r"], *s["gaps"][2:], s["cost"])
        lib.rawalign_chain_decide(s["cost"], *s["chains"], *s["reads"], s["chain_cost"], s["best"], s["best_score"],
                                  s["mapped"], b_match=B_MATCH, threshold=THRESHOLD)
        return s["cost"], s["chain_cost"], s["best"], s["best_score"], s["mapped"]
    a = (s["q"], s["q_off"], s["q_len"], s["r"], s["r_off"], s["r_len"])
    if kind == "batch":
        lib.rawalign_dtw_batch_ex(*a, s["score"], s["end"])
    elif kind == "extend":
        lib.rawalign_dtw_extend(*a, s["rows"], s["row_off"], s["first"], s["score"], s["end"], opts=s["opts"])
    elif kind == "bnb":
        lib.rawalign_map_bnb(*a, s["cand_off"], s["cand_cnt"], s["n_events"], s["rows"], s["row_off"], s["score"], s["end"],
                             s["best"], s["best_score"], s["mapped"], s["max_query"], b_match=B_MATCH, threshold=THRESHOLD)
        # which hopeless candidates are dropped before their end depends on
        # timing, so the pairs' own scores are not results here
        return s["best"], s["best_score"], s["mapped"]
    elif kind == "span":
        lib.rawalign_dtw_span(*a, s["score"], s["end"], s["start"])
        return s["score"], s["end"], s["start"]
    elif kind == "path":
        lib.rawalign_dtw_path(*a, s["dir_off"], s["dirs"], s["path_off"], s["lo"], s["hi"], s["score"], s["end"], s["start"])
        return s["score"], s["end"], s["start"], s["lo"], s["hi"]
    else:
        lib.rawalign_dtw_band(*a, s["band"], s["score"], s["end"])
        return s["score"], s["end"]
    lib.rawalign_decide(s["score"], s["cand_off"], s["cand_cnt"], s["n_events"], s["best"], s["best_score"], s["mapped"],
                        b_match=B_MATCH, threshold=THRESHOLD)
    out = s["score"], s["end"], s["best"], s["best_score"], s["mapped"]
    return out + (s["rows"],) if kind == "extend" else out


# ---- the same in 64 bits -------------------------------------------------------------

def _slices(flat, off, length, width):
    """(pairs, width) matrix of the slices, zero past their ends, in 64 bits."""
    ix = torch.arange(width, device=DEV)
    x = flat[(off[:, None] + ix).clamp(max=len(flat) - 1)].double()
    return torch.where(ix < length[:, None], x, torch.zeros((), dtype=torch.float64, device=DEV))


def _dtw64(q, q_off, q_len, r, r_off, r_len, band=None, corners=False, want_row=False):
    """C_DTW of every pair by anti-diagonals; corners: from (0, 0) to (n-1,
    m-1) instead; want_row: also the last row of every pair, end to end."""
    inf = math.inf
    q_off, q_len, r_off, r_len = (torch.as_tensor(np.asarray(v, dtype=np.int64), device=DEV) for v in (q_off, q_len, r_off, r_len))
    w = None if band is None else torch.as_tensor(np.asarray(band, dtype=np.int64), device=DEV)
    P = len(q_len)
    out = torch.zeros(P, dtype=torch.float64, device=DEV)
    rows = torch.zeros(int(r_len.sum()), dtype=torch.float64, device=DEV) if want_row else None
    row_at = torch.cumsum(r_len, 0) - r_len
    order = torch.argsort(q_len * (1 << 20) + r_len, descending=True)
    sizes = (q_len + r_len)[order].cpu().numpy()
    lens = q_len[order].cpu().numpy()
    at = 0
    while at < P:
        take, width, most = 0, int(lens[at]), (1 << 24)
        while at + take < P and (take + 1) * max(width, 1) <= most and (take < 256 or lens[at + take] * 4 >= width):
            take += 1
            if want_row and (take + 1) * int(sizes[at:at + take].max()) > most:
                break
        ids = order[at:at + max(take, 1)]
        at += max(take, 1)
        n, m = q_len[ids], r_len[ids]
        empty = (n == 0) | (m == 0)
        N, M = max(int(n.max()), 1), max(int(m.max()), 1)
        Q = _slices(q, q_off[ids], n, N)
        F = _slices(r, r_off[ids], m, M).flip(1)
        k = len(ids)
        buf = [torch.full((k, N + 1), inf, dtype=torch.float64, device=DEV) for _ in range(3)]
        best = torch.full((k,), inf, dtype=torch.float64, device=DEV)
        last = torch.full((k, N + M), inf, dtype=torch.float64, device=DEV) if want_row else None
        i_all = torch.arange(N, device=DEV)
        c_all = None if w is None else (i_all * m[:, None]) // n.clamp(min=1)[:, None]
        nn = n.clamp(min=1)[:, None]
        start = torch.full((k,), inf, dtype=torch.float64, device=DEV) if corners else torch.zeros(k, dtype=torch.float64, device=DEV)
        for d in range(N + M - 1):
            lo, hi = max(0, d - (M - 1)), min(N - 1, d)
            cur, p1, p2 = buf[d % 3], buf[(d - 1) % 3], buf[(d - 2) % 3]
            p1[:, 0] = start
            p2[:, 0] = 0.0 if corners and d == 0 else start
            x = torch.minimum(p1[:, lo + 1:hi + 2], p1[:, lo:hi + 1])
            torch.minimum(x, p2[:, lo:hi + 1], out=x)
            x += (Q[:, lo:hi + 1] - F[:, M - 1 - d + lo:M - d + hi]).abs_()
            if w is not None:
                x.masked_fill_(((d - i_all[lo:hi + 1]) - c_all[:, lo:hi + 1]).abs_() > w[ids][:, None], inf)
            cur[:, lo + 1:hi + 2] = x
            v = cur.gather(1, nn)[:, 0]
            j = d - (n - 1)
            inside = (j == m - 1) if corners else ((j >= 0) & (j < m))
            best = torch.where(inside, torch.minimum(best, v), best)
            if want_row:
                last[:, d] = v
        if corners:
            best = torch.where(empty, torch.where((n == 0) & (m == 0), 0.0, inf).double(), best)
        else:
            best = torch.where(n == 0, torch.zeros_like(best), best)
        out[ids] = best
        if want_row:
            own, pos, _ = _segments(m)
            rows[row_at[ids][own] + pos] = last[own, (n - 1)[own] + pos]
    return (out, rows) if want_row else out


def _best64(score, cand_off, cand_cnt, events):
    """Best Score of every read: the largest b * events - cost of its candidates."""
    own, pos, _ = _segments(torch.as_tensor(np.asarray(cand_cnt, dtype=np.int64), device=DEV))
    v = B_MATCH * events - score
    best = torch.full((len(cand_off),), -math.inf, dtype=torch.float64, device=DEV)
    return best.scatter_reduce(0, own, v, "amax")


def exact(case, seed):
    kind = case["kind"]
    if kind == "anchored":
        x = _chains(case, seed)
        gp = {k: v.cpu().numpy() for k, v in x["gaps"].items()}
        cost = _dtw64(x["q"], gp["q_off"], gp["q_len"], x["r"], gp["r_off"], gp["r_len"], corners=True)
        own, _, _ = _segments(x["gap_cnt"])
        total = torch.zeros(len(x["events"]), dtype=torch.float64, device=DEV).index_add_(0, own, cost)
        return cost, total, None, _best64(total, x["cand_off"], x["cand_cnt"], x["events"].double()), None
    p = _segment_pairs(case, seed) if kind == "band_chains" else _pairs(case, seed)
    n_all = p["q_all_len"] if kind == "extend" else p["q_len"]
    if float((n_all * p["r_len"]).sum()) > 3e11:   # more than about 20 seconds
        return None
    if kind == "extend":
        score, rows = _dtw64(p["q"], p["q_all"], p["q_all_len"], p["r"], p["r_off"], p["r_len"], want_row=True)
    else:
        score = _dtw64(p["q"], p["q_off"], p["q_len"], p["r"], p["r_off"], p["r_len"], band=p.get("band"))
    if kind in ("span", "band", "band_chains"):
        return (score, None, None) if kind == "span" else (score, None)
    if kind == "path":
        return score, None, None, None, None
    best = _best64(score, p["cand_off"], p["cand_cnt"],
                   torch.as_tensor(np.repeat(p["n_events"], p["cand_cnt"]), device=DEV).double())
    if kind == "bnb":
        return None, best, None
    out = score, None, None, best, None
    return out + (rows,) if kind == "extend" else out
