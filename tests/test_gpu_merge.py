"""The merge of completed sources into the top-k list at its edges: k below,
at and above the workgroup's 1,024 threads (the list then shifts in several
chunks) and above n, on graphs where every source ties, where most do, and
where none does.  Against the oracle, exact, in every mode."""

import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu

GRAPHS = [lambda: synth.cycle(2300), lambda: synth.disjoint_union(synth.star(900), synth.path(700), synth.cycle(800)),
          lambda: synth.barabasi_albert(2500, 3, 41), lambda: synth.rmat(11, 4, 0.57, 0.19, 0.19, 42)]
MODES = [dict(mode="plain", width=64), dict(mode="plain", width=256), dict(mode="batched", width=64),
         dict(mode="batched", width=256), dict(mode="batched", width=64, defer_arcs=50)]


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("k", [1, 63, 257, 1023, 1024, 1025, 2049, 4000])
def test_list_merge(gi, k):
    g = GRAPHS[gi]()
    ref = oracle.topk(g, k)
    print(f"[merge] graph {gi} n={g.n} k={k}", flush=True)
    with bc.Graph(g.row_ptr, g.col, directed=g.directed) as G:
        got = [G.topk(k, **kw) for kw in MODES] + bc.topk_multi([G, G], [k, k])
    for r in got:
        assert r.ids.tolist() == ref["ids"].tolist()
        assert r.farness.tolist() == ref["f"].tolist() and r.reach.tolist() == ref["r"].tolist()
