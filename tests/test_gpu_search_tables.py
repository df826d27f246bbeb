"""The search and locate with every depth of their tables -- none (rank lines
and SA samples only), a few levels, the library's rule, deeper than many reads
are long -- in every rank-line format and form, against the oracle; the depth
changed under captured steps and under calls of another thread."""
from __future__ import annotations

import threading

import numpy as np
import pytest

import gen
import oracle
import paper_1505_07855_amd as bw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LEVELS = (0, 1, 2, 6, -1, 12)
LAYOUTS = [(32, 0, 4, bw.RANK_PLANES), (64, 192, 32, bw.RANK_PLANES), (128, 0, 64, bw.RANK_PLANES),
           (64, 0, 16, bw.RANK_SUBCOUNTS), (128, 0, 32, bw.RANK_SUB128)]
MAX_OCC = 1 << 20


@pytest.fixture(scope="module")
def case():
    """Reads of 1-150 bases, some with N, on a text whose families reach the
    second pass in ALL mode, with the oracle's answers."""
    g = gen.genome_repeats(61, 60_000, repeat_frac=0.6, n_fam=3, min_len=100, max_len=300, div_lo=0.0, div_hi=0.03)
    lens = np.random.default_rng(61).integers(1, 151, 500).astype(np.int32)
    r = gen.reads_se(62, g, 500, lens, ps=0.03, indel_ratio=0.2)
    bases = r.bases.copy()
    bases[np.random.default_rng(63).random(len(bases)) < 0.002] = 4
    ox = oracle.Index(g.seq)
    want = {}
    for name, kw in (("best", dict(max_diff=3, max_gapo=1, seed_len=16, seed_diff=2)),
                     ("all", dict(max_diff=2, mode=bw.MODE_ALL))):
        o = oracle.align(ox, bases, r.offsets, oracle.Params(**kw), threads=8)
        want[name] = (kw, o, oracle.locate(ox, o.hits, MAX_OCC))
    return g, bases, r.offsets, want


def _check(ix, case, bt, ot, form, split):
    for name, (kw, o, (opo, opos)) in case[3].items():
        p = bw.Params(**kw, form=form, split_budget=split)
        res = bw.align_batch(ix, bt, ot, p, max_len=150)
        ho, hits, c1, c2, st = res.to_numpy()
        assert np.array_equal(ho, o.hit_off), name
        assert np.array_equal(hits.view(np.uint8), o.hits.view(np.uint8)), name
        assert np.array_equal(c1, o.c1) and np.array_equal(c2, o.c2) and np.array_equal(st & 7, o.status), name
        if name == "all":
            assert (st & 8).any(), "no read reached the second pass"
        po, pos = bw.locate(ix, res, MAX_OCC)
        assert np.array_equal(po.cpu().numpy().view(np.uint64), opo), name
        assert np.array_equal(pos.cpu().numpy().view(np.uint32), opos), name


@pytest.mark.parametrize("layout", LAYOUTS)
def test_every_depth_equals_the_oracle(case, layout):
    g, bases, offsets, _ = case
    lb, bpl, sas, fmt = layout
    ix = bw.Index(g.seq, line_bytes=lb, bases_per_line=bpl, sa_sample=sas, rank_format=fmt)
    ix.search_tables(LEVELS[0]).upload()  # asked for before the upload
    bt, ot = torch.from_numpy(bases).cuda(), torch.from_numpy(offsets.view(np.int64)).cuda()
    bare = ix.info()["device_bytes"]
    for K in LEVELS:
        ix.search_tables(K)
        info = ix.info()
        deep = 9 if K < 0 else K  # the least d with 4^d >= 120,000
        assert info["search_levels"] == deep
        table = 2 * (-(-8 * (4 + (4 ** (deep + 1) - 4) // 3) // 256) * 256 + 8 * (len(g.seq) + 1)) if deep else 0
        assert info["device_bytes"] == bare + table
        for form, split in ((bw.FORM_BATCHED, 0), (bw.FORM_BATCHED, 16), (bw.FORM_PLAIN, 0)):
            print("levels", K, "form", form, "split", split, flush=True)
            _check(ix, case, bt, ot, form, split)


@pytest.mark.parametrize("n", [1, 7, 40])
def test_tiny_texts(n):
    """Tables deeper than the text is long."""
    text = np.random.default_rng(n).integers(0, 4, n).astype(np.uint8)
    reads = [text[:k] for k in range(1, min(n, 6) + 1)] + [np.array([0, 1, 2, 3], np.uint8)]
    off = np.cumsum([0] + [len(r) for r in reads]).astype(np.uint64)
    b = np.concatenate(reads)
    ox = oracle.Index(text)
    o = oracle.align(ox, b, off, oracle.Params(max_diff=1))
    opo, opos = oracle.locate(ox, o.hits, MAX_OCC)
    ix = bw.Index(text, sa_sample=1).upload()
    for K in (0, 3, 9, -1):
        ix.search_tables(K)
        for form in (bw.FORM_BATCHED, bw.FORM_PLAIN):
            res = bw.align_batch(ix, torch.from_numpy(b).cuda(), torch.from_numpy(off.view(np.int64)).cuda(),
                                 bw.Params(max_diff=1, form=form), max_len=8)
            ho, hits, c1, c2, st = res.to_numpy()
            assert np.array_equal(ho, o.hit_off) and np.array_equal(hits.view(np.uint8), o.hits.view(np.uint8)), K
            po, pos = bw.locate(ix, res, MAX_OCC)
            assert np.array_equal(pos.cpu().numpy().view(np.uint32), opos), K


@pytest.mark.parametrize("fmt,lb", [(bw.RANK_PLANES, 64), (bw.RANK_SUB128, 128)])
def test_captured_steps_follow_the_tables(case, fmt, lb):
    """Every run after a change gives the results of the runs before: a graph
    that holds released tables is captured again."""
    g, bases, offsets, want = case
    kw, o, (_, opos) = want["best"]
    ix = bw.Index(g.seq, line_bytes=lb, rank_format=fmt).upload()
    n = len(offsets) - 1
    pl = bw.Pipeline(ix, bw.Params(**kw), 0, 500, 250, MAX_OCC, max_pairs=n, max_len=150, paired=False,
                     hit_capacity=len(o.hits) + 8, pos_capacity=len(opos) + 8)
    pl.set_reads(torch.from_numpy(bases).cuda(), torch.from_numpy(offsets.view(np.int64)).cuda(), n, max_len=150)
    for K in (None, 0, 3, -1, 0):
        if K is not None:
            ix.search_tables(K)
        for graph in (True, True, False):
            pl.run(graph=graph)
            st = pl.finish()
            assert st["error"] == 0 and (st["n_hits"], st["n_positions"]) == (len(o.hits), len(opos)), K
            r, _, _, _, pos = pl.results()
            assert np.array_equal(r.to_numpy()[1].view(np.uint8), o.hits.view(np.uint8)), K
            assert np.array_equal(pos[:len(opos)].cpu().numpy().view(np.uint32), opos), K
    pl.close()


def test_changed_under_calls_of_another_thread(case):
    g, bases, offsets, want = case
    kw, o, _ = want["best"]
    ix = bw.Index(g.seq, line_bytes=64).upload()
    bt, ot = torch.from_numpy(bases).cuda(), torch.from_numpy(offsets.view(np.int64)).cuda()
    torch.cuda.synchronize()
    bad = []

    def calls():
        s = torch.cuda.Stream()
        for i in range(20):
            res = bw.align_batch(ix, bt, ot, bw.Params(**kw), max_len=150, stream=s)
            with torch.cuda.stream(s):
                if not np.array_equal(res.to_numpy()[1].view(np.uint8), o.hits.view(np.uint8)):
                    bad.append(i)

    t = threading.Thread(target=calls)
    t.start()
    for i in range(12):
        ix.search_tables((0, -1, 4)[i % 3])
    t.join()
    assert not bad


def test_errors():
    ix = bw.Index(gen.genome_iid(64, 3000, 0.5).seq)
    for bad in (-2, 16):
        with pytest.raises(bw.BwfmError):
            ix.search_tables(bad)
    ix.upload()
    for bad in (-2, 16):
        with pytest.raises(bw.BwfmError):
            ix.search_tables(bad)
    assert ix.info()["search_levels"] == 7  # the least d with 4^d >= 6000
