"""Workspace sizes on the host: a caller that sizes a workspace once, for the
capacity of its map, passes it with every smaller n, so no size may fall as n
grows; and gsr_spatial_order accepts what its capacity's workspace holds
(argument checks only: no device work on the accepted path is reached, the
misplaced index pointer is refused after the size is accepted)."""
import ctypes

import pytest

from paper_2601_00705_amd import lib

EDGES = sorted({max(1, e + d) for e in (1, 64, 1024, 4096, 5000, 16384, 131072, 1 << 20, 1_002_433, 1_096_896, 1 << 21,
                                        1 << 22, 1 << 25, 1 << 27, (1 << 31) - 4) for d in (-1025, -65, -1, 0, 1, 63, 1025)
                if 1 <= e + d < 1 << 31} | set(range(1, 40_000, 331)) | set(range(900_000, 1_200_000, 3_001)))


@pytest.mark.parametrize("name", ["gsr_spatial_order_workspace_bytes", "gsr_seed_scale_workspace_bytes",
                                  "gsr_prune_workspace_bytes"])
def test_sizes_grow_with_n(name):
    f = getattr(lib.raw(), name)
    sizes = [f(n) for n in EDGES]
    assert all(s > 0 for s in sizes)
    assert all(a <= b for a, b in zip(sizes, sizes[1:])), [n for n, a, b in zip(EDGES, sizes, sizes[1:]) if a > b][:5]


def test_order_takes_its_capacity_workspace():
    raw = lib.raw()
    have = raw.gsr_spatial_order_workspace_bytes((1 << 20) + 1)
    ws = ctypes.c_void_p(1 << 40)
    for n in (1, 1000, 1_002_433, 1 << 20, (1 << 20) + 1):
        # the index lies inside the workspace: refused, but for that
        assert raw.gsr_spatial_order(n, ctypes.c_void_p(1 << 30), 64, ws, ws, have, None) == lib.EINVAL
        assert b"overlap" in raw.gsr_last_error(), n


def test_direct_search_needs_no_workspace():
    """Up to 16,384 points the searches keep nothing in memory."""
    raw = lib.raw()
    for n in (1, 1000, 16384):
        assert 0 < raw.gsr_seed_scale_workspace_bytes(n) <= 256
    assert raw.gsr_seed_scale_workspace_bytes(16385) > 256
