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


@pytest.mark.parametrize("n", [1, 2_000, 30_000, 120_000, 1_000_000])
@pytest.mark.parametrize("size", [(64, 48), (1920, 1080), (8192, 6000), (16384, 16384)])
def test_count_matrix_of_many_tiles(size, n):
    """A plan's count matrix has a row of one counter per tile for every 256
    Gaussians at most, or 64 MiB where that is less: few Gaussians in a huge
    view do not take 512 rows."""
    from paper_2601_00705_amd.render import Config

    def total(n, w, h):
        plan = lib.gsr_plan_create(n, [{"width": w, "height": h, "fx": 1.0, "fy": 1.0, "cx": 0.0, "cy": 0.0}], Config(), 1000)
        try:
            return lib.gsr_plan_workspace_bytes(plan), lib.gsr_plan_get_info(plan).total_tiles
        finally:
            lib.gsr_plan_destroy(plan)
    have, tiles = total(n, *size)
    fixed, _ = total(0, *size)  # one row
    slots = total(n, 16, 16)[0] - total(0, 16, 16)[0]
    assert have <= fixed + slots + max(4 * tiles * -(-n // 256), 64 << 20) + 4096
