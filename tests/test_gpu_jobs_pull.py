"""Bottom-up levels of job launches (several graphs in one launch, the serving
queue): they are counted in the statistics."""

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
