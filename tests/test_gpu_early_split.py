"""Early splits go by the reads, not by the length the caller declares: a
batch of short reads is not split because max_len is generous, one of long
reads is, and the results are the same."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1505_07855_amd as bw
from gen import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(ix, r, p, max_len, lengths=None):
    res = bw.align_batch(ix, torch.from_numpy(r.bases).cuda(), torch.from_numpy(r.offsets.view(np.int64)).cuda(), p,
                         max_len=max_len)
    ho, hits, c1, c2, st = res.to_numpy()
    return [ho, hits.view(np.uint8), c1, c2, st & 7], int(((st & bw.ST_SPLIT) != 0).sum())


def test_declared_length_does_not_split_short_reads():
    g = configs.c2_genome(2_000_000, seed=171)
    r = configs.c2_pairs(g, 40_000, seed=172).end1
    ix = bw.Index(g.seq, **configs.LAYOUT["C2"]).upload()
    p = bw.Params(**configs.PARAMS["C2"])
    want, split = _run(ix, r, p, 100)
    for declared in (199, 200, 256):
        got, s = _run(ix, r, p, declared)
        assert all(np.array_equal(a, b) for a, b in zip(want, got)), declared
        print("declared", declared, "split", s, "against", split, flush=True)
        assert s <= split + 40, declared


def test_long_reads_are_split_early_and_equal_the_oracle():
    g = configs.c2_genome(2_000_000, seed=173)
    r = configs.c5_reads(g, 3000, seed=174)
    ix = bw.Index(g.seq, **configs.LAYOUT["C2"]).upload()
    p = bw.Params(**configs.PARAMS["C5"])
    got, split = _run(ix, r, p, 250)
    assert split > 0
    o = oracle.align(oracle.Index(g.seq), r.bases, r.offsets, oracle.Params(**configs.PARAMS["C5"]), threads=8)
    want = [o.hit_off, o.hits.view(np.uint8), o.c1, o.c2, o.status]
    assert all(np.array_equal(a, b) for a, b in zip(want, got))


def test_every_long_read_in_flight_finds_room():
    """At the smallest split budget more of a batch is split than one read in
    eight, the room that batches of short reads have."""
    n = 3000
    g = configs.c2_genome(2_000_000, seed=173)
    r = configs.c5_reads(g, n, seed=174)
    ix = bw.Index(g.seq, **configs.LAYOUT["C2"]).upload()
    want, _ = _run(ix, r, bw.Params(**configs.PARAMS["C5"], split_budget=-1), 250)
    got, split = _run(ix, r, bw.Params(**configs.PARAMS["C5"], split_budget=16), 250)
    assert split > n // 8
    assert all(np.array_equal(a, b) for a, b in zip(want, got))
