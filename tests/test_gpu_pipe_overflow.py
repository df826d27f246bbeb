"""A captured step whose hits or positions outgrow their capacities by far:
nothing past the arrays is touched, the need is reported, every pair record
is an unplaced pair's (so that rescue and MAPQ enqueued behind the step leave
it alone), and the next batch that fits equals the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1505_07855_amd as bw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

COPIES, UNIT, L, N = 3000, 300, 100, 120
LO, HI, MU, MAX_OCC = 200, 400, 300, 100_000


def _pairs(text, starts):
    """Fragments of UNIT bases at starts, both ends error-free."""
    one, two = [], []
    for s in starts:
        f = text[s:s + UNIT]
        one.append(f[:L])
        two.append(3 - f[::-1][:L])
    return np.concatenate(one + two).astype(np.uint8), np.arange(0, 2 * len(starts) + 1, dtype=np.uint64) * L


@pytest.fixture(scope="module")
def setup():
    """300 kbp without repeats, then one unit 3,000 times with random bases
    between: a read of it has one hit of 3,000 rows."""
    rng = np.random.default_rng(5)
    unit = rng.integers(0, 4, UNIT)
    parts = [rng.integers(0, 4, 300_000)]
    first = 300_000 + (UNIT + 30) * np.arange(COPIES)
    for _ in range(COPIES):
        parts += [unit, rng.integers(0, 4, 30)]
    text = np.concatenate(parts).astype(np.uint8)
    assert np.array_equal(text[first[7]:first[7] + UNIT], unit)
    single = rng.integers(0, 290_000, N)
    wide = single.copy()
    wide[::3] = rng.choice(first, len(wide[::3]))
    ox = oracle.Index(text)
    out = {}
    for name, at in (("single", single), ("wide", wide)):
        b, o = _pairs(text, at)
        ends = [oracle.align(ox, b[e * N * L:(e + 1) * N * L], o[:N + 1], oracle.Params(max_diff=2), threads=8)
                for e in (0, 1)]
        locs = [oracle.locate(ox, r.hits, MAX_OCC) for r in ends]
        pr = oracle.pair(ends[0], locs[0][0], locs[0][1], ends[1], locs[1][0], locs[1][1], LO, HI, MU)
        out[name] = dict(b=torch.from_numpy(b).cuda(), o=torch.from_numpy(o.view(np.int64)).cuda(), host=(b, o),
                         hits=sum(len(r.hits) for r in ends), pos=sum(len(x[1]) for x in locs), pairs=pr)
    assert out["wide"]["pos"] > 200_000 and out["single"]["pos"] < 2_000
    return text, out


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("short", ["positions", "hits"])
def test_step_over_its_capacities(setup, short, graph):
    text, runs = setup
    ix = bw.Index(text, line_bytes=64).upload()
    p = bw.Params(max_diff=2)
    caps = dict(pos_capacity=2_000) if short == "positions" else dict(hit_capacity=8)
    pl = bw.Pipeline(ix, p, LO, HI, MU, MAX_OCC, max_pairs=N, max_len=L, **caps)
    ends = [(runs["wide"]["b"][e * N * L:(e + 1) * N * L].contiguous(), runs["wide"]["o"][:N + 1]) for e in (0, 1)]
    for _ in range(2):
        w = runs["wide"]
        pl.set_reads(w["b"], w["o"], N, max_len=L)
        pl.run(graph=graph)
        r1, r2, prs, _, _ = pl.results()
        resc = bw.rescue_mates(ix, ends[0], ends[1], prs, LO, HI, max_len=L)
        q = bw.mapq(r1, r2, prs, rescue=resc, max_diff=2).cpu().numpy()
        st = pl.finish()
        if short == "positions":
            assert st["error"] == bw.PIPE_E_POSITIONS
            assert (st["n_hits"], st["n_positions"]) == (w["hits"], w["pos"])
        else:
            assert st["error"] & bw.PIPE_E_HITS and st["n_hits"] == w["hits"]
        got = bw.pairs_numpy(prs)[:N]
        assert (got["flags"] == 0).all() and (got["pos1"] == 0xFFFFFFFF).all() and (got["pos2"] == 0xFFFFFFFF).all()
        assert not bw.rescue_numpy(resc)[:N].view(np.uint8).any() and not q.any()
        if short == "positions":  # a batch that fits
            s = runs["single"]
            pl.set_reads(s["b"], s["o"], N, max_len=L)
            pl.run(graph=graph)
            st = pl.finish()
            assert st["error"] == 0 and (st["n_hits"], st["n_positions"]) == (s["hits"], s["pos"])
            assert np.array_equal(bw.pairs_numpy(pl.results()[2])[:N].view(np.uint8), s["pairs"].view(np.uint8))
    pl.close()


@pytest.mark.parametrize("levels", [0, -1])
def test_no_room_for_positions(setup, levels):
    """pos_capacity 0, with and without the search's tables: a batch without
    hits runs, one with hits is reported."""
    text, runs = setup
    ix = bw.Index(text, line_bytes=64).search_tables(levels).upload()
    pl = bw.Pipeline(ix, bw.Params(max_diff=2), LO, HI, MU, MAX_OCC, max_pairs=N, max_len=L, pos_capacity=0)
    b = torch.full((2 * N * L,), 4, dtype=torch.uint8, device="cuda")
    for graph in (False, True):
        pl.set_reads(b, runs["single"]["o"], N, max_len=L)
        pl.run(graph=graph)
        st = pl.finish()
        assert (st["error"], st["n_hits"], st["n_positions"]) == (0, 0, 0)
        pl.set_reads(runs["single"]["b"], runs["single"]["o"], N, max_len=L)
        pl.run(graph=graph)
        st = pl.finish()
        assert (st["error"], st["n_positions"]) == (bw.PIPE_E_POSITIONS, runs["single"]["pos"])
    pl.close()


def test_served_steps_over_their_capacities(setup):
    """A server whose steps outgrow the capacities it starts with redoes
    them: records equal the oracle's."""
    text, runs = setup
    ix = bw.Index(text, line_bytes=64).upload()
    srv = bw.Server(ix, bw.Params(max_diff=2), LO, HI, MU, MAX_OCC, arena_bytes=4 << 20, step_pairs=64, max_len=L,
                    budget_rule=False, rescue_mapq=True)
    tickets = []
    for name in ("wide", "single", "wide"):
        b, o = runs[name]["host"]
        tickets.append((name, srv.submit(b[:N * L], o[:N + 1], b[N * L:], o[:N + 1])))
    for name, t in tickets:
        rec, _ = srv.wait(t, N)
        assert np.array_equal(rec.view(np.uint8).reshape(-1), runs[name]["pairs"].view(np.uint8).reshape(-1)), name
    srv.close()
