"""Narrow levels in job launches: a level of a few nodes is a chain of short
steps, none of which may come to dominate it."""

import pytest

import oracle
import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [64, 128])
def test_build_of_a_narrow_level_is_short(width):
    """On a cycle every level reaches 2 W nodes and nothing is cut.  Setting a
    level's frontier up takes less than half of what expanding and counting it
    takes (it was 0.8 of it while the sum of the frontier's arcs went through a
    loop over the lanes)."""
    g = synth.cycle(4000)
    ref = oracle.topk(g, 3)
    with bc.Graph(g.row_ptr, g.col) as G:
        bc.topk_multi([G], [3], width=width)
        r, = bc.topk_multi([G], [3], width=width)
    assert r.ids.tolist() == ref["ids"].tolist() and r.farness.tolist() == ref["f"].tolist()
    _, expand, cut, build, _ = r.stats["phase_ms"]
    us = [1e3 * x / r.stats["levels"] for x in (expand, cut, build)]
    print(f"[narrow] W = {width}: expand {us[0]:.2f}, cut {us[1]:.2f}, build {us[2]:.2f} us a level", flush=True)
    assert build < 0.5 * expand
