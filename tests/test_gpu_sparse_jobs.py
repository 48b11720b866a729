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
