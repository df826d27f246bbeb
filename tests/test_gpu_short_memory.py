"""Small batches of long reads where the device has little memory left: the
call and the captured step take a smaller workspace, with the same results."""
from __future__ import annotations

import numpy as np
import pytest

import gen
import paper_1505_07855_amd as bw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GB = 1 << 30


def _leave(n_bytes):
    """Tensors that hold all of the device's memory but about n_bytes."""
    spare = torch.empty(n_bytes, dtype=torch.uint8, device="cuda")
    held, size = [], 16 * GB
    while size >= GB // 8:
        try:
            held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            size //= 2
    del spare
    torch.cuda.empty_cache()
    return held


def test_a_smaller_workspace_is_taken():
    """1,000 reads declared as up to 512 bases: 5 GB of buffers where there is
    room, 1.4 GB where 3 GB are free."""
    n, L = 1000, 512
    g = gen.genome_iid(81, 300_000, 0.45)
    r = gen.reads_se(82, g, n, 150, ps=0.02, indel_ratio=0.1)
    b, o = torch.from_numpy(r.bases).cuda(), torch.from_numpy(r.offsets.view(np.int64)).cuda()
    p = bw.Params(max_diff=4)

    def align(ix):
        return [a.copy() for a in bw.align_batch(ix, b, o, p, max_len=L).to_numpy()]

    ix = bw.Index(g.seq, line_bytes=64).upload()
    want = align(ix)
    roomy = ix.info()["ws_bytes"]
    assert roomy > 4.5 * GB
    ix.close()
    ix = bw.Index(g.seq, line_bytes=64).upload()
    few = bw.align_batch(ix, b, o[:5], p, max_len=L)  # the kernels are loaded before memory is short
    assert np.array_equal(few.to_numpy()[0], want[0][:5])
    bw.release_cached()
    fill = _leave(3 * GB)
    try:
        got = align(ix)
        lean = ix.info()["ws_bytes"]
        print("workspace", roomy, "short of memory", lean, flush=True)
        pl = bw.Pipeline(ix, p, 0, 500, 250, 1000, max_pairs=n, max_len=L, paired=False)
        pl.set_reads(b, o, n, max_len=L)
        pl.run()
        st = pl.finish()
        hits = pl.results()[0].to_numpy()[1].copy()
        pl.close()
    finally:
        del fill
        torch.cuda.empty_cache()
    assert lean < 2 * GB
    for x, y in zip(want[:4], got):
        assert np.array_equal(x, y)
    assert np.array_equal(want[4] & 7, got[4] & 7)
    assert st["error"] == 0 and np.array_equal(hits, want[1])
