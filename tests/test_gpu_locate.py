"""Locate of hits of every width class -- one row, a few (one lane each), up
to thousands (a wave each) and more (the whole grid) -- against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1505_07855_amd as bw
from gen import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("fmt", [0, 1, 2])
def test_widths(fmt):
    rng = np.random.default_rng(331)
    unit = rng.integers(0, 4, 40).astype(np.uint8)
    parts, reads = [], [unit[5:35]]
    for copies in (2, 8, 9, 64, 65, 2048, 2049, 6000):
        u = rng.integers(0, 4, 30).astype(np.uint8)
        reads.append(u)
        for _ in range(copies):
            parts += [u, rng.integers(0, 4, 3).astype(np.uint8)]
    ref = np.concatenate([unit] + parts + [rng.integers(0, 4, 1000).astype(np.uint8)])
    bases = np.concatenate([r for r in reads for _ in range(3)] + [3 - reads[4][::-1]])
    offs = np.arange(0, len(bases) + 1, 30).astype(np.uint64)
    kw = dict(max_diff=0, max_gapo=0)
    ores = oracle.align(oracle.Index(ref), bases, offs, oracle.Params(**kw), threads=2)
    ix = bw.Index(ref, **configs.FORMAT_LAYOUT[fmt]).upload()
    res = bw.align_batch(ix, torch.from_numpy(bases).cuda(), torch.from_numpy(offs.view(np.int64)).cuda(),
                         bw.Params(**kw), max_len=30)
    ox = oracle.Index(ref)
    for max_occ in (100000, 2048, 8):
        po, pos = bw.locate(ix, res, max_occ)
        opo, opos = oracle.locate(ox, ores.hits, max_occ)
        assert np.array_equal(po.cpu().numpy().view(np.uint64), opo)
        assert np.array_equal(pos.cpu().numpy().view(np.uint32), opos)
    assert np.diff(opo.astype(np.int64)).max() <= 8
