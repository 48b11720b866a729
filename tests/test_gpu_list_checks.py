"""The level loop with the lists checked where its narrow kernel hands them to
the host, in every way a query comes to it."""

import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("make", [lambda: synth.path(9), lambda: synth.star(20_000), lambda: synth.empty(5),
                                  lambda: synth.barabasi_albert(30_000, 4, 31), lambda: synth.erdos_renyi(9000, 12, 2),
                                  lambda: synth.rmat(14, 8, 0.57, 0.19, 0.19, 32)])
def test_lists_handed_back_by_the_narrow_kernel(make, monkeypatch):
    monkeypatch.setenv("BC_CHECK_LISTS", "2")
    g = make()
    ref = oracle.topk(g, 7)
    with bc.Graph(g.row_ptr, g.col, directed=g.directed) as G:
        for kw in (dict(mode="plain", width=64), dict(mode="plain", width=256, pull_alpha=1e9, pull_beta=1e-9),
                   dict(mode="batched", width=64, defer_arcs=1), dict(mode="batched", width=64, defer_arcs=1,
                                                                      defer_width=64)):
            r = G.topk(7, **kw)
            assert r.ids.tolist() == ref["ids"].tolist() and r.farness.tolist() == ref["f"].tolist(), kw
            assert r.reach.tolist() == ref["r"].tolist(), kw
