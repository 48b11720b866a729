"""Graphs of many nodes without arcs, whose batches end at once: bottom-up
steps that pass over every node for a handful of arcs do not run in one
workgroup."""

import numpy as np
import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


def spread(n, core, directed=False):
    """A graph of `core` nodes whose ids are spread over n, the others without arcs."""
    g = synth.barabasi_albert(core, 3, 3)
    src, step = np.repeat(np.arange(g.n), np.diff(g.row_ptr)), n // core
    return synth.from_edges(n, src * step, g.col.astype(np.int64) * step, directed)


@pytest.mark.parametrize("directed", [False, True])
@pytest.mark.parametrize("width", [64, 128, 256])
def test_few_arcs_run_top_down(width, directed):
    g = spread(60_000, 1000, directed)
    ref = oracle.topk(g, 10)
    with bc.Graph(g.row_ptr, g.col, directed=directed) as G:
        res = bc.topk_multi([G, G], [10, 10], width=width)
        res += [G.topk(10, mode="batched", width=width, seed_batches=0, lds_tables=lds) for lds in (True, False)]
    for r in res:
        assert r.ids.tolist() == ref["ids"].tolist() and r.farness.tolist() == ref["f"].tolist()
        assert r.reach.tolist() == ref["r"].tolist() and r.stats["pull_levels"] == 0, r.stats


def test_short_batches_are_claimed_without_contention():
    """6,250 batches, nearly all of which end at once: the launch stays within
    a few times the batched query (it took 40 times as long while its 256
    workgroups claimed by compare-and-exchange)."""
    g = spread(400_000, 1500)
    with bc.Graph(g.row_ptr, g.col) as G:
        query = min(G.topk(10, mode="batched").stats["query_ms"] for _ in range(5))
        M = bc.MultiLaunch([G], [10])
        launch = min(M.run()[0].stats["persistent_ms"] for _ in range(5))
    print(f"[sparse] query {query:.2f} ms, launch {launch:.2f} ms", flush=True)
    assert launch < 8 * query


@pytest.mark.parametrize("capture", [False, True])
@pytest.mark.parametrize("n", [5, 64, 65, 256 * 64 - 1, 256 * 64, 256 * 64 + 1])
def test_every_batch_is_claimed_in_every_run(n, capture):
    """As many batches as workgroups, one less and one more, run after run."""
    g = synth.cycle(n) if n < 1000 else spread(n, 300)
    ref = oracle.topk(g, 4)
    with bc.Graph(g.row_ptr, g.col) as G:
        M = bc.MultiLaunch([G, G], [4, 2], capture=capture)
        for _ in range(3):
            a, b = M.run()
            assert a.ids.tolist() == ref["ids"].tolist() and a.farness.tolist() == ref["f"].tolist()
            assert b.ids.tolist() == ref["ids"].tolist()[:2]
            assert int(a.stats["n_cut"] + a.stats["n_done"] + a.stats["n_trivial"]) == g.n
