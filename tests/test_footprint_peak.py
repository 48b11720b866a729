"""The admission estimate of a query covers what its slots take at their peak,
for every width of the batches, of the seed batches and of the deferred ones,
and the graph's list of nodes of many in-arcs."""

import itertools

import pytest

import paper_1507_01490_amd as bc

GIB = 1 << 30


def node_bytes(w):
    """seen, nxt and cur, a stamp for more than one word, three lists."""
    return 24 * (w // 64) + (4 if w > 64 else 0) + 12


def deferred_slots(n, w, room):
    slot, lv = n * node_bytes(w), 1
    while lv < 32 and lv < -(-n // w) and 2 * lv * slot <= min(room, GIB):
        lv *= 2
    return lv


def peak(n, w, slots, sw, dw):
    slots = min(slots, -(-n // w))
    pers = slots * n * node_bytes(w)
    widths = [dw] if dw else [64] + [128] * (n > 64) + [256] * (n > 128)
    return n * node_bytes(sw) + max([pers] + [deferred_slots(n, d, pers) * n * node_bytes(d) for d in widths])


@pytest.mark.parametrize("n,m", [(1, 0), (64, 200), (129, 800), (5000, 40_000), (1_000_000, 10_000_000),
                                 (3_000_000, 2_000_000_000)])
def test_query_estimate_covers_its_slots(n, m):
    for w, slots, k, dw in itertools.product((64, 128, 256), (1, 2, 8, 64, 256), (1, 100), (0, 64, 128, 256)):
        opts = dict(mode="batched", width=w)
        sw = 256 if k > w else w
        lists = 4 * n + 24 * n + 4 * n  # order, threshold records, deferred sources
        q = bc.footprint(n, m, k=k, slots=slots, **opts)[2] if dw == 0 else footprint_dw(n, m, k, slots, w, dw)
        assert q >= peak(n, w, slots, sw, dw) + lists + 4 * (m // 65), (w, slots, k, dw)


def footprint_dw(n, m, k, slots, w, dw):
    import ctypes
    keep = []
    o = bc.make_opts(n, keep, mode="batched", width=w)
    o.defer_width = dw
    g, u, q = ctypes.c_uint64(), ctypes.c_uint64(), ctypes.c_uint64()
    bc._check(bc.load_library().bc_footprint(n, m, 0, k, ctypes.byref(o), slots, ctypes.byref(g), ctypes.byref(u),
                                             ctypes.byref(q)))
    return q.value


def test_plain_estimate_covers_the_list_of_heavy_nodes():
    n = 1000
    a, b = [bc.footprint(n, m, k=1, mode="plain")[2] for m in (0, 65_000_000)]
    assert b - a >= 4 * (65_000_000 // 65)
