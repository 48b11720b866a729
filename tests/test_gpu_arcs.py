"""Arc-parallel pre-processing at its edges: tiles of 2,048 arcs (one short,
exact, one over, several), runs of empty rows inside a tile, rows that span
tiles, rows above the 8,192 arcs that are split over workgroups, components
in each length class of the reach recurrence.  Against the oracle, exact."""

import numpy as np
import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


def star_into_chain(arcs, gap):
    """Node 0 -> `arcs` leaves that sit `gap` ids apart (empty rows between)."""
    n = arcs * gap + 2
    return synth.from_edges(n, np.zeros(arcs, np.int64), 1 + gap * np.arange(arcs), directed=True)


def classes(seed):
    """Components with 3, 17, 5,000 and 9,000 successor components, the
    longest one in a cycle of two nodes."""
    rng = np.random.default_rng(seed)
    n, src, dst = 20_000, [0, 1], [1, 0]
    for u, k in ((0, 9000), (1, 40), (2, 5000), (3, 17), (4, 3)):
        t = rng.choice(np.arange(10, n), k, replace=False)
        src += [u] * k
        dst += t.tolist()
    src += list(range(10, 400))
    dst += rng.integers(400, n, 390).tolist()
    return synth.from_edges(n, src, dst, directed=True)


@pytest.mark.parametrize("make", [
    lambda: star_into_chain(2047, 1), lambda: star_into_chain(2048, 1), lambda: star_into_chain(2049, 3),
    lambda: star_into_chain(8192, 1), lambda: star_into_chain(8193, 2), lambda: synth.directed_path(4097),
    lambda: synth.directed_cycle(2048), lambda: synth.rmat(13, 12, 0.57, 0.19, 0.19, 5), lambda: classes(1),
    lambda: synth.empty(3000, True)])
@pytest.mark.parametrize("big", [False, True])
def test_reach_at_tile_edges(make, big):
    g = make()
    print(f"[arcs] n={g.n} m={g.m} big={big}", flush=True)
    with bc.Graph(g.row_ptr, g.col, directed=True, big_scc=big) as G:
        lo, hi = G.reach()
        rp, col = G.csr()
    a, o = oracle.alpha_omega(g, big)
    assert lo.tolist() == a.tolist() and hi.tolist() == o.tolist()
    assert rp.tolist() == g.row_ptr.tolist() and col.tolist() == g.col.tolist()


@pytest.mark.parametrize("at", [0, 2047, 2048, 4999])
def test_bad_column_is_refused_wherever_it_is(at):
    n = 50
    rp = np.linspace(0, 5000, n + 1).astype(np.int32)
    for bad in (-1, n):
        col = np.tile(np.arange(n, dtype=np.int32), 100)
        col[at] = bad
        with pytest.raises(bc.BcError) as e:
            bc.Graph(rp, col, directed=True)
        assert e.value.status == -2
