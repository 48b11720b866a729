"""Bottom-up steps on graphs whose nodes all have long lists of in-arcs."""

import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


def test_bottom_up_pays_on_a_dense_graph():
    """The seed batch is faster with bottom-up levels than without (it was 1.45
    times as slow while the step's grid was sized by the nodes alone)."""
    g = synth.erdos_renyi(3000, 600, 4)
    ref = oracle.topk(g, 10)
    with bc.Graph(g.row_ptr, g.col) as G:
        def best(alpha):
            runs = [G.topk(10, mode="batched", pull_alpha=alpha) for _ in range(12)]
            for r in runs:
                assert r.ids.tolist() == ref["ids"].tolist() and r.farness.tolist() == ref["f"].tolist()
            return min(r.stats["seed_ms"] for r in runs)
        pull, push = best(3.0), best(0.0)
    print(f"[dense] seed batch {pull:.3f} ms bottom up, {push:.3f} ms top down", flush=True)
    assert pull < push


@pytest.mark.parametrize("levels", [0, 3, -1])
@pytest.mark.parametrize("width", [64, 256])
def test_dense_graph_in_every_level_driver(width, levels):
    g = synth.erdos_renyi(700, 200, 6)
    ref = oracle.topk(g, 9)
    with bc.Graph(g.row_ptr, g.col) as G:
        r = G.topk(9, mode="plain", width=width, graph_levels=levels, pull_alpha=1e9, pull_beta=1e9)
    assert r.ids.tolist() == ref["ids"].tolist() and r.farness.tolist() == ref["f"].tolist()
    assert r.reach.tolist() == ref["r"].tolist() and r.stats["pull_levels"] > 0
