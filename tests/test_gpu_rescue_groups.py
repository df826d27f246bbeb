"""Mate rescue over every way its mates are spread over lanes -- one, two or
four to a wave, every number of rows a lane -- and at the edges of the
records a block takes, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import gen
import oracle
import paper_1505_07855_amd as bw
from gen import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,max_len,hi", [(1, 256, 500), (4, 256, 500), (5, 64, 64), (9, 128, 300), (17, 256, 500),
                                          (18, 512, 500), (129, 512, 8192), (257, 256, 8192), (9000, 128, 300),
                                          (9000, 256, 300)])
def test_spread(n, max_len, hi):
    rng = np.random.default_rng(4100 + n + max_len)
    g = gen.genome_iid(41, 20_000, 0.45)
    ix = bw.Index(g.seq, **configs.FORMAT_LAYOUT[2]).upload()
    # mates of every length up to max_len, some of no length, cut from the
    # reference with changes
    m = rng.integers(0, max_len + 1, n)
    m[0] = max_len
    offs = np.concatenate([[0], np.cumsum(m)]).astype(np.uint64)
    rec = np.zeros(n, oracle.PAIR_DTYPE)
    rec["len1"] = 50
    rec["flags"] = np.where(rng.random(n) < (0.2 if n > 1000 else 0.9), oracle.PF_MAPPED1, 0)
    rec["flags"][0] = oracle.PF_MAPPED1
    rec["pos1"] = rng.integers(0, len(g.seq) - 50, n)
    rec["strand1"] = rng.integers(0, 2, n)
    rec["pos2"] = 0xFFFFFFFF
    bases = np.empty(int(offs[-1]), np.uint8)
    for i in range(n):
        at = int(rec["pos1"][i]) + int(rng.integers(-40, max(hi // 2, 1))) - (hi // 2 if rec["strand1"][i] else 0)
        at = int(np.clip(at, 0, len(g.seq) - m[i]))
        b = g.seq[at:at + m[i]].copy()
        b[rng.random(m[i]) < 0.05] = rng.integers(0, 5)
        if rec["strand1"][i] == 0:
            b = np.where(b < 4, 3 - b, b)[::-1]
        bases[int(offs[i]):int(offs[i + 1])] = b
    none, empty = np.zeros(n + 1, np.uint64), np.zeros(1, np.uint8)
    want = oracle.rescue(g.seq, (empty, none), (bases, offs), rec, 0, hi)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    got = bw.rescue_numpy(bw.rescue_mates(ix, (d(empty), d(none.view(np.int64))), (d(bases), d(offs.view(np.int64))),
                                          d(rec.view(np.uint8)), 0, hi, max_len))[:n]
    assert n < 17 or (want["end"] != 0).any()
    for f in want.dtype.names:
        assert np.array_equal(got[f], want[f]), f
