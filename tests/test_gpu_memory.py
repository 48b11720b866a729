"""Device memory that a graph keeps between queries is bounded."""

import ctypes

import pytest

import paper_1507_01490_amd as bc
from paper_1507_01490_amd import synth

pytestmark = pytest.mark.gpu

GIB = 1 << 30
USED = 7  # hipMemPoolAttrUsedMemCurrent


def pool_used():
    """Bytes that are allocated from the device's default memory pool."""
    import torch
    torch.cuda.synchronize()
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    pool, used = ctypes.c_void_p(), ctypes.c_uint64()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), torch.cuda.current_device()) == 0
    assert hip.hipMemPoolGetAttribute(pool, USED, ctypes.byref(used)) == 0
    return used.value


def test_level_slots_of_all_widths_are_bounded():
    """Deferred re-runs in all three widths, many batches each: the slots kept
    for them take 1 GiB together, not 1 GiB per width."""
    g = synth.barabasi_albert(500_000, 2, 9)
    with bc.Graph(g.row_ptr, g.col) as G:
        ids = G.topk(3, mode="batched", slots=4).ids.tolist()
        before = pool_used()
        for width in (64, 128, 256, 64):
            r = G.topk(3, mode="batched", slots=4, defer_arcs=1, defer_width=width)
            assert r.ids.tolist() == ids and r.stats["n_deferred"] > 32 * width
            kept = pool_used() - before
            print(f"[memory] defer width {width}: {kept / 2**20:.0f} MiB kept", flush=True)
            assert kept <= 1.05 * GIB
