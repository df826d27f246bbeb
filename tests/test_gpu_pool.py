"""Indexes made and given back in turn share the library's pool of device
blocks: results stay those of a first index, also with two threads at it."""
from __future__ import annotations

import threading

import numpy as np
import pytest

import gen
import paper_1505_07855_amd as bw
from gen import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("threads", [1, 2])
def test_blocks_are_reused(threads):
    work = []
    for k, n in enumerate((400_000, 900_001)):
        g = configs.c2_genome(n, seed=321 + k)
        r = gen.reads_se(323 + k, g, 300, 60, ps=0.02)
        work.append((g, torch.from_numpy(r.bases).cuda(), torch.from_numpy(r.offsets.view(np.int64)).cuda()))
    torch.cuda.synchronize()

    def once(g, b, o, stream):
        ix = bw.Index.build_device(g.seq, stream=stream)
        res = bw.align_batch(ix, b, o, bw.Params(max_diff=2), max_len=60, stream=stream)
        with torch.cuda.stream(stream):
            out = [a.copy() for a in res.to_numpy()]
        sa = ix.sa_samples(1)
        ix.close()
        return [out[0], out[1].view(np.uint8), out[2], out[3], out[4] & 7, sa]

    first = [once(*w, torch.cuda.Stream()) for w in work]
    bad = []

    def loop():
        s = torch.cuda.Stream()
        for i in range(6):
            if not all(np.array_equal(x, y) for x, y in zip(first[i % 2], once(*work[i % 2], s))):
                bad.append(i)

    ts = [threading.Thread(target=loop) for _ in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
