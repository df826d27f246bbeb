"""Work that programs built on this library have it do, as cases to be timed.

A case is one call (or the short chain of calls a program makes) through the
public entry points: aligning a batch, the captured paired step, locate,
mate rescue and mapping quality, the request server, indexing a reference.
The sizes are those of the library's workloads (`gen/configs.py`, `bench.py`)
-- 36 bp reads on 1 Mbp (C1), 2 x 100 bp pairs on 100 Mbp (C2), ragged
36-150 bp pairs with per-read budgets (C3), serving requests of 76-150 bp
(C4), 250 bp reads with 6 differences (C5) -- and smaller ones.

Inputs are drawn on the GPU: references of GC 41% with 40% repeat copies of
5-20% divergence, and reads from either strand with substitutions, short
indels and a few N.  A reference and its index are made once per process
and size, as a program does that aligns many batches to one reference;
reads, requests and handles are new for each seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1505_07855_amd as bw

DEV = "cuda"
# search parameters of the workloads
PARAMS = {
    "C1": dict(max_diff=2, max_gapo=0, seed_len=0),
    "C2": dict(max_diff=4, max_gapo=1, seed_len=32, seed_diff=2),
    "C5": dict(max_diff=6, max_gapo=1, seed_len=0),
}
# index layouts: the default one, C1's (a checkpoint every 128 rows), and
# the three the autotuner chooses from
LAYOUT = {
    "default": dict(line_bytes=128),
    "planes128": dict(line_bytes=64, bases_per_line=128),
    "planes192": dict(line_bytes=64, bases_per_line=192),
    "sub64": dict(line_bytes=64, bases_per_line=160, rank_format=bw.RANK_SUBCOUNTS),
    "sub128": dict(line_bytes=128, bases_per_line=384, rank_format=bw.RANK_SUB128),
}
WINDOW = dict(lo=180, hi=420, mu=300)  # inserts ~ N(300, 30)
MAX_OCC = 100000
RAGGED = (36, 51, 76, 100, 150)
ERR = {"C1": (0.02, 0.0), "C2": (0.01, 0.001), "C3": (0.016, 0.0018), "C4": (0.01, 0.001), "C5": (0.03, 0.003)}


def listed():
    return [
        # one pair at a time: a tool that looks pairs up interactively
        dict(name="pair_one", kind="chain", ref=1_000_000, layout="default", n=1, length=100, params="C2", rescue=0),
        # C1: short single-end reads, few mismatches, no gaps
        dict(name="se36_10k", kind="align", ref=1_000_000, layout="planes128", n=10_000, length=36, params="C1",
             mode="best", form="batched"),
        # every placement within the budget (ALL mode), an odd number of reads
        dict(name="all36_25k", kind="align", ref=16_000_000, layout="planes192", n=25_001, length=36, params="C1",
             mode="all", form="batched"),
        # an ordinary batch of 2 x 100 bp pairs: align, pair, rescue, MAPQ
        dict(name="pairs100_30k", kind="chain", ref=100_000_000, layout="sub128", n=30_000, length=100, params="C2",
             rescue=1),
        # ragged lengths with per-read budgets (C3) on a reference whose
        # index no longer fits the last-level cache
        dict(name="ragged_150k", kind="chain", ref=500_000_000, layout="sub128", n=150_001, length=0, params="C2",
             rescue=1),
        # the headline step: 1M pairs of 2 x 100 bp, captured once, replayed
        dict(name="step100_1M", kind="step", ref=100_000_000, layout="sub128", n=1_000_000, length=100, params="C2"),
        # C5: long noisy single-end reads, 6 differences with a gap
        dict(name="se250_150k", kind="align", ref=100_000_000, layout="sub128", n=150_000, length=250, params="C5",
             mode="best", form="batched"),
        # the plain form, one lane per read
        dict(name="plain100_20k", kind="align", ref=100_000_000, layout="sub64", n=20_000, length=100, params="C2",
             mode="best", form="plain"),
        # positions of every hit of a large batch
        dict(name="locate_400k", kind="locate", ref=100_000_000, layout="sub128", n=400_000, length=36),
        # mate rescue and mapping quality of a large ragged batch
        dict(name="rescue_300k", kind="rescue", ref=100_000_000, layout="sub128", n=300_000, length=0),
        # a burst of requests to the server (host buffers in, records out)
        dict(name="serve_8", kind="serve", ref=100_000_000, layout="sub128", n=40_000, requests=8),
        # a new reference: index it on the device and align a first batch
        dict(name="index_16M", kind="index", ref=16_000_003, layout="sub128", n=2_000, length=100, params="C2"),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["chain", "chain", "align", "align", "align", "step", "locate", "rescue", "serve", "index"])
    ref = rng.choice([1_000_000, 16_000_000, 100_000_000])
    layout = rng.choice(sorted(LAYOUT))
    if kind == "chain":
        return dict(kind=kind, ref=ref, layout=layout, n=size(1, 100_000), length=rng.choice([0, 36, 75, 100, 101, 150]),
                    params="C2", rescue=rng.choice([0, 1]))
    if kind == "align":
        what = rng.choice(["C1", "C2", "C5"])
        form = rng.choice(["batched", "batched", "plain"])
        if what == "C1":
            return dict(kind=kind, ref=ref, layout=layout, n=size(100, 200_000), length=rng.choice([32, 36, 50]),
                        params="C1", mode=rng.choice(["best", "all"]), form=form)
        if what == "C2":
            return dict(kind=kind, ref=ref, layout=layout, n=size(100, 30_000 if form == "plain" else 500_000),
                        length=rng.choice([0, 36, 75, 100, 125, 151]), params="C2", mode="best", form=form)
        return dict(kind=kind, ref=ref, layout=layout, n=size(100, 100_000), length=rng.choice([201, 250, 300]),
                    params="C5", mode="best", form="batched")
    if kind == "step":
        return dict(kind=kind, ref=ref, layout=layout, n=size(100, 400_000), length=rng.choice([0, 75, 100, 150]),
                    params="C2")
    if kind == "locate":
        return dict(kind=kind, ref=ref, layout=layout, n=size(1_000, 400_000), length=rng.choice([36, 50, 100]))
    if kind == "rescue":
        return dict(kind=kind, ref=ref, layout=layout, n=size(1_000, 300_000), length=rng.choice([0, 36, 100, 150, 250]))
    if kind == "serve":
        return dict(kind=kind, ref=ref, layout=layout, n=size(1_000, 60_000), requests=rng.randint(1, 16))
    return dict(kind="index", ref=size(50_000, 16_000_000), layout=layout, n=size(100, 2_000), length=100, params="C2")


# ------------------------------------------------------------------ inputs

_REFS: dict = {}
_INDEXES: dict = {}


def _rng(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _iid(n, g):
    u = torch.rand(n, generator=g, device=DEV)
    return ((u >= 0.295).to(torch.uint8) + (u >= 0.5).to(torch.uint8) + (u >= 0.705).to(torch.uint8))


def _make_ref(n):
    """n bases: 60% i.i.d. at GC 41%, 40% diverged copies of repeat families."""
    g = _rng(77 + n)
    ref = _iid(n, g)
    fam = max(4, min(500, n // 20_000))
    flen = torch.exp(torch.empty(fam, device=DEV).uniform_(math.log(300), math.log(6000), generator=g)).long()
    fbase = torch.cumsum(flen, 0) - flen
    cons = _iid(int(flen.sum()), g)
    k = int(0.4 * n / float(flen.double().mean()) * 1.2) + 8
    which = torch.randint(0, fam, (k,), generator=g, device=DEV)
    clen = flen[which]
    keep = torch.cumsum(clen, 0) <= int(0.4 * n)
    which, clen = which[keep], clen[keep]
    k = int(which.numel())
    if k == 0:
        return ref
    cum = torch.cumsum(clen, 0)
    total = int(cum[-1])
    cuts = torch.sort(torch.randint(0, n - total + 1, (k,), generator=g, device=DEV)).values
    start = cuts + cum - clen
    div = torch.empty(k, device=DEV).uniform_(0.05, 0.20, generator=g)
    rc = torch.rand(k, generator=g, device=DEV) < 0.5
    cid = torch.repeat_interleave(torch.arange(k, device=DEV), clen)
    off = torch.arange(total, device=DEV) - (cum - clen)[cid]
    src = torch.where(rc[cid], clen[cid] - 1 - off, off) + fbase[which][cid]
    b = cons[src]
    b = torch.where(rc[cid], 3 - b, b)
    sub = torch.rand(total, generator=g, device=DEV) < div[cid]
    b = torch.where(sub, (b + torch.randint(1, 4, (total,), generator=g, device=DEV, dtype=torch.uint8)) & 3, b)
    ref[start[cid] + off] = b
    return ref


def _ref(n):
    if n not in _REFS:
        r = _make_ref(n)
        _REFS[n] = (r, r.cpu().numpy())
    return _REFS[n]


def _index(n, layout):
    if (n, layout) not in _INDEXES:
        _INDEXES[n, layout] = bw.Index.build_device(_ref(n)[1], **LAYOUT[layout])
    return _INDEXES[n, layout]


def _sequence(ref, start, lens, strand, sub, indel, g):
    """Reads of the given starts, lengths and strands: flat bases and CSR
    offsets.  A read has at most one indel event (1-3 bases)."""
    n, m = lens.numel(), ref.numel()
    offs = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lens, 0, out=offs[1:])
    total = int(offs[-1])
    rid = torch.repeat_interleave(torch.arange(n, device=DEV), lens)
    j = torch.arange(total, device=DEV) - offs[rid]
    j = torch.where(strand[rid], lens[rid] - 1 - j, j)
    u = torch.rand(n, generator=g, device=DEV)
    ev = u < indel * lens  # an indel in this read
    size = torch.randint(1, 4, (n,), generator=g, device=DEV)
    at = 6 + (torch.rand(n, generator=g, device=DEV) * (lens - 15).clamp(min=1)).long()
    dele = ev & (u < 0.5 * indel * lens)
    at_, size_ = at[rid], size[rid]
    shift = torch.where(dele[rid] & (j >= at_), size_, 0)
    ins = (ev & ~dele)[rid]
    shift = torch.where(ins & (j >= at_ + size_), -size_, shift)
    inserted = ins & (j >= at_) & (j < at_ + size_)
    src = (start[rid] + j + shift).clamp(0, m - 1)
    del shift, ins, at_, size_
    b = ref[src]
    r = torch.rand(total, generator=g, device=DEV)
    e = torch.randint(1, 4, (total,), generator=g, device=DEV, dtype=torch.uint8)
    b = torch.where((r < sub[rid]) | inserted, (b + e) & 3, b)
    b = torch.where(strand[rid], 3 - b, b)
    b = torch.where(r > 1.0 - 2e-4, torch.full_like(b, 4), b)  # a few N
    return b, offs


def _lengths(case, n, g):
    if case["length"]:
        return torch.full((n,), case["length"], dtype=torch.int64, device=DEV)
    return torch.tensor(RAGGED, device=DEV)[torch.randint(0, len(RAGGED), (n,), generator=g, device=DEV)]


def _single(case, workload, g):
    ref = _ref(case["ref"])[0]
    n = case["n"]
    lens = _lengths(case, n, g)
    start = (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * (ref.numel() - lens - 4)).long()
    strand = torch.rand(n, generator=g, device=DEV) < 0.5
    sub = torch.full((n,), ERR[workload][0], device=DEV)
    return _sequence(ref, start, lens, strand, sub, ERR[workload][1], g)


def _pairs(ref, lens, workload, g):
    """End 1's reads, then end 2's: FR pairs of fragments ~ N(300, 30)."""
    n = lens.numel()
    frag = (300 + 30 * torch.randn(n, generator=g, device=DEV)).round().long()
    frag = torch.maximum(frag, torch.clamp(lens + 24, min=100))
    start = (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * (ref.numel() - frag - 4)).long()
    flip = torch.rand(n, generator=g, device=DEV) < 0.5  # end 1 is the fragment's right end
    left, right = start, start + frag - lens
    s1, s2 = torch.where(flip, right, left), torch.where(flip, left, right)
    rate, indel = ERR[workload]
    sub = torch.full((2 * n,), rate, device=DEV)
    if workload == "C3":  # per-read error rates 0.5-3%
        sub = torch.empty(2 * n, device=DEV).uniform_(0.9 * 0.005, 0.9 * 0.03, generator=g)
    return _sequence(ref, torch.cat([s1, s2]), torch.cat([lens, lens]), torch.cat([flip, ~flip]), sub, indel, g)


def _budgets(offs):
    rule = torch.tensor([bw.max_diff_rule(m) for m in range(513)], dtype=torch.uint8, device=DEV)
    return rule[offs[1:] - offs[:-1]]


def _params(case):
    form = bw.FORM_PLAIN if case.get("form") == "plain" else bw.FORM_BATCHED
    mode = bw.MODE_ALL if case.get("mode") == "all" else bw.MODE_BEST
    return bw.Params(**PARAMS[case["params"]], form=form, mode=mode)


def _max_len(case):
    return case["length"] or max(RAGGED)


def _out(reads, per_read):
    """Result buffers a program keeps for its batches; hits past the last
    offset stay zero."""
    def z(*shape, dtype=torch.int32):
        return torch.zeros(shape, dtype=dtype, device=DEV)

    return bw.AlignResult(z(reads + 1, dtype=torch.int64), z(per_read * reads + 4096, 4), z(reads), z(reads),
                          z(reads, dtype=torch.uint8), reads)


def prepare(case, seed):
    g = _rng(1_000_003 * seed + 17)
    kind = case["kind"]
    s = dict(case=case)
    if kind == "index":
        s["ref"] = np.random.default_rng(seed).permutation(4).astype(np.uint8)[_ref(case["ref"])[1]]
        r = torch.from_numpy(s["ref"]).to(DEV)
        lens = torch.full((case["n"],), case["length"], dtype=torch.int64, device=DEV)
        start = (torch.rand(case["n"], generator=g, device=DEV, dtype=torch.float64) * (r.numel() - 110)).long()
        s["bases"], s["offs"] = _sequence(r, start, lens, torch.rand(case["n"], generator=g, device=DEV) < 0.5,
                                          torch.full((case["n"],), 0.01, device=DEV), 0.001, g)
        s["p"] = _params(case)
        s["out"] = _out(case["n"], 8)
        return s
    ix = s["ix"] = _index(case["ref"], case["layout"])
    if kind == "align":
        s["bases"], s["offs"] = _single(case, case["params"], g)
        s["p"] = _params(case)
        s["out"] = _out(case["n"], 16)
        return s
    if kind == "locate":
        # hits of reads within one mismatch, repeats included
        bases, offs = _single(case, "C2", g)
        s["res"] = bw.align_batch(ix, bases, offs, bw.Params(max_diff=1, max_gapo=0, max_best=1000),
                                  max_len=_max_len(case))
        # a program's position buffers, whole; past the last entry they stay zero
        s["po"] = torch.zeros(8 * case["n"] + 4096, dtype=torch.int64, device=DEV)
        s["pos"] = torch.zeros(32 * case["n"] + 65536, dtype=torch.int32, device=DEV)
        return s
    n = case["n"]
    ref = _ref(case["ref"])[0]
    if kind == "serve":
        cuts = sorted(np.random.default_rng(n).integers(1, n, case["requests"] - 1).tolist())  # sizes as the case has them
        s["reqs"] = []
        for a, b in zip([0] + cuts, cuts + [n]):
            if b == a:
                continue
            lens = torch.randint(76, 151, (b - a,), generator=g, device=DEV)
            bases, offs = _pairs(ref, lens, "C4", g)
            h, o = bases.cpu().numpy(), offs.cpu().numpy().astype(np.uint64)
            k = b - a
            s["reqs"].append((h[:int(o[k])].copy(), o[:k + 1].copy(), h[int(o[k]):].copy(), (o[k:] - o[k]).copy()))
        s["srv"] = bw.Server(ix, bw.Params(**PARAMS["C2"]), **WINDOW, max_occ=MAX_OCC, arena_bytes=64 << 20,
                             step_pairs=16384, max_len=150, budget_rule=True, rescue_mapq=True)
        return s
    lens = _lengths(case, n, g)
    ragged = not case["length"]
    s["bases"], s["offs"] = _pairs(ref, lens, "C3" if ragged else "C2", g)
    s["md"] = _budgets(s["offs"]) if ragged else None
    s["p"] = bw.Params(**PARAMS["C2"])
    if kind == "step":
        s["pl"] = bw.Pipeline(ix, s["p"], **WINDOW, max_occ=MAX_OCC, max_pairs=n, max_len=_max_len(case),
                              hit_capacity=8 * n + 4096, pos_capacity=64 * n + 65536)
        s["out"] = _out(2 * n, 4)
        s["po"] = torch.zeros(8 * n + 4097, dtype=torch.int64, device=DEV)
        s["pos"] = torch.zeros(64 * n + 65536, dtype=torch.int32, device=DEV)
        s["pairs"] = torch.zeros((n, bw.PAIR_DTYPE.itemsize), dtype=torch.uint8, device=DEV)
        return s
    s["out"] = _out(2 * n, 8)
    # both ends as ragged batches of their own (rescue takes them apart)
    b1 = int(s["offs"][n])
    s["ends"] = [(s["bases"][:b1].clone(), s["offs"][:n + 1].clone()), (s["bases"][b1:].clone(), s["offs"][n:] - b1)]
    if kind == "rescue":
        res = bw.align_batch(ix, s["bases"], s["offs"], s["p"], max_diff=s["md"], max_len=_max_len(case))
        s["r"] = (res.window(0, n), res.window(n, 2 * n))
        s["pairs"] = bw.pair_reads(ix, *s["r"], **WINDOW, max_occ=MAX_OCC)
        # a tenth of the pairs as if end 2 had found nothing, so that its
        # mate is looked for near end 1
        rec = s["pairs"].view(torch.int32)
        lost = torch.rand(n, generator=g, device=DEV) < 0.1
        flags = s["pairs"][:, 22]
        flags[lost] = flags[lost] & 2
        rec[lost, 1] = -1
    return s


# ------------------------------------------------------------------ one pass


def _aligned(res):
    """An alignment's outputs; the status's upper bits only say how the
    search was scheduled."""
    return [res.hit_offsets, res.hits, res.c1, res.c2, res.status & 7]


def _mates(s, pairs):
    ml = _max_len(s["case"])
    n = s["case"]["n"]
    resc = bw.rescue_mates(s["ix"], s["ends"][0], s["ends"][1], pairs, WINDOW["lo"], WINDOW["hi"], max_len=ml)
    md = s["md"]
    mq = bw.mapq(*s["r"], pairs, rescue=resc, budgets1=md[:n] if md is not None else None,
                 budgets2=md[n:] if md is not None else None)
    return [resc, mq]


def run(s):
    case = s["case"]
    kind, n = case["kind"], case["n"]
    if kind == "align":
        return _aligned(bw.align_batch(s["ix"], s["bases"], s["offs"], s["p"], max_len=_max_len(case), out=s["out"]))
    if kind == "chain":
        res = bw.align_batch(s["ix"], s["bases"], s["offs"], s["p"], max_diff=s["md"], max_len=_max_len(case),
                             out=s["out"])
        s["r"] = (res.window(0, n), res.window(n, 2 * n))
        pairs = bw.pair_reads(s["ix"], *s["r"], **WINDOW, max_occ=MAX_OCC)
        return _aligned(res) + [pairs] + (_mates(s, pairs) if case["rescue"] else [])
    if kind == "step":
        pl = s["pl"]
        pl.set_reads(s["bases"], s["offs"], n, _max_len(case), max_diff=s["md"])
        pl.run()
        st = pl.finish()
        if st["error"]:
            raise RuntimeError(f"step capacities too small: {st}")
        r1, r2, pairs, po, pos = pl.results()
        # taken out of the pipeline's own buffers, which its next run (or
        # its end) takes back
        o, nh, np_ = s["out"], st["n_hits"], st["n_positions"]
        for e, r in enumerate((r1, r2)):
            o.hit_offsets[e * n:(e + 1) * n + 1].copy_(r.hit_offsets)
            o.c1[e * n:(e + 1) * n].copy_(r.c1)
            o.c2[e * n:(e + 1) * n].copy_(r.c2)
            o.status[e * n:(e + 1) * n].copy_(r.status)
        o.hits[:nh].copy_(r1.hits[:nh])
        s["po"][:nh + 1].copy_(po)
        s["pos"][:np_].copy_(pos[:np_])
        s["pairs"].copy_(pairs)
        return _aligned(o) + [s["po"], s["pos"], s["pairs"]]
    if kind == "locate":
        po, pos = bw.locate(s["ix"], s["res"], MAX_OCC)
        s["po"][:po.numel()].copy_(po)
        s["pos"][:pos.numel()].copy_(pos)
        return [s["po"], s["pos"]]
    if kind == "rescue":
        return _mates(s, s["pairs"])
    if kind == "serve":
        tickets = [s["srv"].submit(*q) for q in s["reqs"]]
        out = []
        for t, q in zip(tickets, s["reqs"]):
            pairs, resc, mq, _ = s["srv"].wait(t, len(q[1]) - 1, extras=True)
            out += [pairs.view(np.uint8), resc.view(np.uint8), mq]
        return out
    ix = bw.Index.build_device(s["ref"], **LAYOUT[case["layout"]])
    res = bw.align_batch(ix, s["bases"], s["offs"], s["p"], max_len=case["length"], out=s["out"])
    info = ix.info()
    return [ix.sa_samples(0), ix.sa_samples(1), np.array(info["primary"] + info["C"][0] + info["C"][1], np.int64)] \
        + _aligned(res)


# ------------------------------------------------------------------ work


def work(case):
    """Bytes that go in and out once: reads, results, and of the index at
    most a rank line per base looked up, at most all of it.  The search is
    integer work; rescue counts its cells' 12 operations."""
    n, kind = case["n"], case["kind"]
    length = case.get("length") or 83
    index_bytes = 2 * case["ref"] * (128 / 384 + 4 / 32)
    ends = 1 if kind in ("align", "index", "locate") else 2
    reads = ends * n
    if kind == "serve":
        length = 113
    if kind == "index":
        return dict(bytes=case["ref"] + 2 * index_bytes + n * (length + 50), flops=0)
    if kind == "locate":
        return dict(bytes=n * (16 + 8 + 4) + min(index_bytes, n * 128), flops=0)
    if kind == "rescue":
        cells = 0.1 * n * length * 400
        return dict(bytes=n * (24 + 16 + 2 + 2 * 60) + 0.1 * n * (length + 100), flops=12 * cells)
    out = reads * (8 + 9 + 1.5 * 16) + (n * 24 if ends == 2 else 0)
    return dict(bytes=reads * (length + 8) + out + min(index_bytes, reads * length * 128), flops=0)


def exact(case, seed):
    """No output here has a value in 64 bits that it rounds: all are whole
    numbers and records, defined exactly."""
    return None
