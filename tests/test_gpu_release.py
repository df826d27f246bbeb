"""Device blocks the library keeps for later use go back to the driver when
the caller asks for them."""
from __future__ import annotations

import pytest

import gen
import paper_1505_07855_amd as bw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_release_cached():
    g = gen.genome_iid(91, 4_000_000, 0.5)
    bw.release_cached()
    torch.cuda.synchronize()
    ix = bw.Index.build_device(g.seq)
    held = ix.info()["device_bytes"]  # tables of 4^12 strings, suffix arrays, lines: 430 MB
    ix.close()
    before = torch.cuda.mem_get_info()[0]
    bw.release_cached()
    assert torch.cuda.mem_get_info()[0] - before >= held // 2
    ix = bw.Index.build_device(g.seq)  # and the library takes new ones
    assert ix.info()["device_bytes"] == held
