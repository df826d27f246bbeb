"""Batches of fewer reads than the device has lanes: each wave takes an equal
share of the reads at once and its other lanes help.  Sizes around one wave,
one block and the number of resident waves, against the oracle bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import gen
import oracle
import paper_1505_07855_amd as bw
from gen import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def setup():
    g = configs.c2_genome(1_000_000, seed=301)
    reads = gen.reads_se(302, g, 5000, np.random.default_rng(303).integers(20, 121, 5000).astype(np.int32), ps=0.015,
                         indel_ratio=0.1)
    kw = dict(max_diff=3, max_gapo=1, seed_len=32, seed_diff=2)
    ores = oracle.align(oracle.Index(g.seq), reads.bases, reads.offsets, oracle.Params(**kw), threads=8)
    ix = bw.Index(g.seq, **configs.LAYOUT["C2"]).upload()
    return reads, kw, ores, ix


@pytest.mark.parametrize("split", [0, 64, -1])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 257, 4095, 4097, 5000])
def test_small_batches(setup, n, split):
    reads, kw, ores, ix = setup
    off = reads.offsets[:n + 1]
    b = torch.from_numpy(reads.bases[:int(off[-1])]).cuda()
    o = torch.from_numpy(off.view(np.int64)).cuda()
    res = bw.align_batch(ix, b, o, bw.Params(**kw, split_budget=split), max_len=120)
    ho, hits, c1, c2, st = res.to_numpy()
    h = int(ores.hit_off[n])
    assert np.array_equal(ho, ores.hit_off[:n + 1])
    assert np.array_equal(hits.view(np.uint8), ores.hits[:h].view(np.uint8))
    assert np.array_equal(c1, ores.c1[:n]) and np.array_equal(c2, ores.c2[:n])
    assert np.array_equal(st & 7, ores.status[:n])


@pytest.mark.parametrize("n", [1, 65, 700])
def test_small_batches_of_long_reads(n):
    """250 bp reads: few reads with large trees, whose parts are split early
    once half of the waves have ended."""
    g = configs.c2_genome(1_000_000, seed=311)
    reads = configs.c5_reads(g, n, seed=312)
    kw = configs.PARAMS["C5"]
    ores = oracle.align(oracle.Index(g.seq), reads.bases, reads.offsets, oracle.Params(**kw), threads=8)
    ix = bw.Index(g.seq, **configs.LAYOUT["C5"]).upload()
    b = torch.from_numpy(reads.bases).cuda()
    o = torch.from_numpy(reads.offsets.view(np.int64)).cuda()
    ho, hits, c1, c2, st = bw.align_batch(ix, b, o, bw.Params(**kw), max_len=250).to_numpy()
    assert np.array_equal(ho, ores.hit_off) and np.array_equal(hits.view(np.uint8), ores.hits.view(np.uint8))
    assert np.array_equal(c1, ores.c1) and np.array_equal(c2, ores.c2) and np.array_equal(st & 7, ores.status)
