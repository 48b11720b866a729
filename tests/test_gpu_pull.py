"""Bottom-up levels inside the persistent kernels, and lists whose lengths sit
at the edges of what a lane, a group of lanes and a wave take.  Against the
oracle, exact, at every width, whatever direction the levels take."""

import numpy as np
import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


def hubs(n, seed, directed):
    """Nodes joined to (or from) 3, 4, 5, 63, 64, 65, 127, 256 and 1,025 others, on a random tree or arcs."""
    rng = np.random.default_rng(seed)
    src, dst = list(range(1, n)), [int(rng.integers(0, i)) for i in range(1, n)]
    for h, d in enumerate((3, 4, 5, 63, 64, 65, 127, 256, 1025)):
        for w in rng.choice(n - 16, size=d, replace=False):
            src.append(int(w))
            dst.append(n - 1 - h)
            if directed and int(w) % 2:
                src.append(n - 1 - h)
                dst.append(int(w))
    return synth.from_edges(n, src, dst, directed)


GRAPHS = [lambda: hubs(1500, 1, False), lambda: hubs(1537, 2, True), lambda: synth.erdos_renyi(1023, 30, 3),
          lambda: synth.barabasi_albert(2049, 7, 4)]
ALWAYS = dict(pull_alpha=1e9, pull_beta=1e9)
NEVER = dict(pull_alpha=0.0)


@pytest.mark.parametrize("gi", range(len(GRAPHS)))
@pytest.mark.parametrize("width", [64, 128, 256])
def test_bottom_up_levels(gi, width):
    g = GRAPHS[gi]()
    ref = oracle.topk(g, 20)
    print(f"[pull] graph {gi} n={g.n} m={g.m} width={width}", flush=True)
    with bc.Graph(g.row_ptr, g.col, directed=g.directed) as G:
        got = [G.topk(20, mode="batched", width=width, lds_tables=False, seed_batches=0, **kw)
               for kw in (ALWAYS, dict(ALWAYS, order="degree"), dict(), NEVER)]
        pulls = [int(r.stats["pull_levels"]) for r in got]
        if width == 64:  # batches that leave LDS
            lds = G.topk(20, mode="batched", width=64, seed_batches=0, trial=False, **ALWAYS)
            assert int(lds.stats["spills"]) == 0 or int(lds.stats["pull_levels"]) > 0
            got += [lds, G.topk(20, mode="batched", width=64, seed_batches=0, trial=False)]
        got += bc.topk_multi([G, G], [20, 20], width=width)
    assert pulls[0] > 0 and pulls[1] > 0 and pulls[3] == 0, pulls
    for r in got:
        assert r.ids.tolist() == ref["ids"].tolist()
        assert r.farness.tolist() == ref["f"].tolist() and r.reach.tolist() == ref["r"].tolist()


@pytest.mark.parametrize("shape", [(1023, 20), (1600, 7), (3001, 5), (4099, 40)])
@pytest.mark.parametrize("width", [64, 128, 256])
def test_levels_found_by_sweep(shape, width):
    """Top-down levels that reach less and more than a third and a half of the
    nodes, on the node records and, at width 64, after a batch has left LDS."""
    g = synth.erdos_renyi(shape[0], shape[1], 5)
    ref = oracle.topk(g, 33)
    print(f"[sweep] n={g.n} m={g.m} width={width}", flush=True)
    with bc.Graph(g.row_ptr, g.col, directed=g.directed) as G:
        got = [G.topk(33, mode="batched", width=width, lds_tables=lds, seed_batches=sb, **NEVER)
               for lds in ((True, False) if width == 64 else (False,)) for sb in (0, 2)]
        f, r, _ = G.farness_all(width=width)
    for x in got:
        assert x.ids.tolist() == ref["ids"].tolist()
        assert x.farness.tolist() == ref["f"].tolist() and x.reach.tolist() == ref["r"].tolist()
    assert f[ref["ids"]].tolist() == ref["f"].tolist() and r[ref["ids"]].tolist() == ref["r"].tolist()
