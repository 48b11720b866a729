"""Bottom-up levels of job launches (several graphs in one launch, the serving
queue): they are counted in the statistics, and pull_alpha and pull_beta
decide them as in a query of its own (0: none)."""

import ctypes

import numpy as np
import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


def wide():
    """A graph whose frontiers soon hold most arcs, so that levels run bottom up."""
    return synth.erdos_renyi(1500, 30, 7)


def check(res, ref):
    assert res.ids.tolist() == ref["ids"].tolist()
    assert res.farness.tolist() == ref["f"].tolist() and res.reach.tolist() == ref["r"].tolist()


@pytest.mark.parametrize("width", [64, 256])
def test_launch_counts_bottom_up_levels(width):
    g = wide()
    ref = oracle.topk(g, 5)
    with bc.Graph(g.row_ptr, g.col) as G:
        for r in bc.topk_multi([G, G], [5, 5], width=width):
            check(r, ref)
            assert 0 < r.stats["pull_levels"] <= r.stats["levels"]


def test_queue_counts_bottom_up_levels():
    g = wide()
    ref = oracle.topk(g, 5)
    with bc.Server(lanes=2, queue=True) as S:
        gid = S.add_graph(g.row_ptr, g.col)
        t = S.submit(gid, 5, mode="batched")
        assert S.wait(t, 60000)
        r = S.poll(t)
    check(r, ref)
    assert 0 < r.stats["pull_levels"] <= r.stats["levels"]


def launch(graphs, k, width, **kw):
    """bc_topk_multi with any options; the results and statistics of every query."""
    keep, m = [], len(graphs)
    o = bc.make_opts(max(g.n for g in graphs), keep, mode="batched", width=width, **kw)
    hs = (ctypes.c_void_p * m)(*[g._h.value for g in graphs])
    ks = np.full(m, k, np.int32)
    ids, far, rea = np.zeros(m * k, np.int32), np.zeros(m * k, np.uint64), np.zeros(m * k, np.uint32)
    cnt, sts = np.zeros(m, np.int32), (bc.Stats * m)()
    for st in sts:
        st.size = ctypes.sizeof(bc.Stats)
    bc._check(bc.load_library().bc_topk_multi(hs, m, bc._ptr(ks), ctypes.byref(o), bc._ptr(ids), bc._ptr(far),
                                              bc._ptr(rea), bc._ptr(cnt), ctypes.cast(sts, ctypes.c_void_p)))
    return [bc.TopK(ids[i * k:(i + 1) * k], far[i * k:(i + 1) * k], rea[i * k:(i + 1) * k], sts[i].as_dict())
            for i in range(m)]


@pytest.mark.parametrize("width", [64, 128, 256])
def test_launch_takes_the_direction_it_is_told(width):
    g = wide()
    ref = oracle.topk(g, 5)
    with bc.Graph(g.row_ptr, g.col) as G:
        never, auto, always = [launch([G, G], 5, width, **kw) for kw in
                               (dict(pull_alpha=0.0), dict(), dict(pull_alpha=1e9, pull_beta=1e9))]
    for r in never + auto + always:
        check(r, ref)
    assert all(r.stats["pull_levels"] == 0 for r in never)
    assert all(0 < r.stats["pull_levels"] < r.stats["levels"] for r in auto)
    assert sum(r.stats["pull_levels"] for r in always) > sum(r.stats["pull_levels"] for r in auto)


def test_queue_takes_the_direction_it_is_told():
    g = wide()
    ref = oracle.topk(g, 5)
    with bc.Server(lanes=2, queue=True) as S:
        gid = S.add_graph(g.row_ptr, g.col)
        tickets = [S.submit(gid, 5, mode="batched", pull_alpha=a) for a in (0.0, 3.0)]
        got = []
        for t in tickets:
            assert S.wait(t, 60000)
            got.append(S.poll(t))
    for r in got:
        check(r, ref)
    assert got[0].stats["pull_levels"] == 0 and got[1].stats["pull_levels"] > 0
