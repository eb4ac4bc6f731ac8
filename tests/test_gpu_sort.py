"""The per-tile sort, exact: one tile's list at the edges of its paths.

A single 16x16 view holds every Gaussian in its one tile, so the list's
length is n; the expected order is numpy's lexicographic sort of (depth
bits, index).  Lengths stand at a round's, a block's and a chunk's edges;
depths are spread, banded with outliers (surfaces), of few values, all equal
(lists that cannot be cut by depth are merged), or spread with one crowded
depth (too many small chunks for the cursors).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2601_00705_amd.render import Config, Renderer


def _depths(kind, n, rng):
    if kind == "spread":
        d = rng.uniform(0.2, 9.0, n)
    elif kind == "bands":
        d = np.where(rng.random(n) < 0.7, 3.0 + 1e-3 * rng.random(n), 5.0 + 1e-4 * rng.standard_normal(n))
        d[rng.random(n) < 0.02] = 0.3
        d[-1] = 900.0
    elif kind == "few":
        d = rng.choice(np.array([0.5, 1.0, np.nextafter(np.float32(1), np.float32(2)), 7.25]), n)
    elif kind == "equal":
        d = np.full(n, 2.5)
    else:  # spread, and 1,200 keys of one depth
        d = rng.uniform(2.0, 3.9, n)
        d[rng.choice(n, min(n, 1200), replace=False)] = 2.5
    return d.astype(np.float32)


@pytest.mark.parametrize("kind,n", [(k, n) for k in ("spread", "bands", "few", "equal")
                                    for n in (1, 2, 64, 255, 257, 513, 2047, 2048, 2049, 4097, 30011)] +
                         [("crowded", 600000)])
def test_one_tile(kind, n):
    print(f"[sort] {kind} n={n}", flush=True)
    rng = np.random.default_rng(n)
    cam = {"width": 16, "height": 16, "fx": 1, "fy": 1, "cx": 0, "cy": 0}
    R = Renderer(n, [cam], Config(), pair_capacity=n)
    d = _depths(kind, n, rng)
    rec = R.records()
    rec["geom"].copy_(torch.tensor([8.0, 8.0, 4.0, 4.0]).expand(n, 4))
    rec["conic_o"][:, :3].copy_(torch.tensor([1.0, 0.0, 1.0]).expand(n, 3))
    rec["qthr"].fill_(16.0)
    rec["rgb_d"][:, 3].copy_(torch.from_numpy(d))
    rec["live_mask"].fill_(-1)
    R.bin()
    M, overflow = R.pair_count()
    assert M == n and not overflow
    keys, vals, ranges = R.sorted_pairs(M)
    want = np.lexsort((np.arange(n), d.view(np.uint32)))
    np.testing.assert_array_equal(vals.cpu().numpy(), want)
    np.testing.assert_array_equal(keys.cpu().numpy(), d.view(np.uint32)[want].astype(np.int64))
    np.testing.assert_array_equal(ranges.cpu().numpy(), [[0, n]])
