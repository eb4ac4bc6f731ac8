"""The per-tile sort where many keys share one coarse depth bin: surfaces seen
head-on with an outlier before or behind them, one or two depths for all,
clusters inside clusters (each half as many points in a thousandth of the
depth, so that the list is cut again and again), beside tiles with ordinary
and with empty lists.  Exact against numpy's order of (depth bits, index);
and such a list takes at most 2.5 times as long as one of spread depths (it is
cut once more, which doubles its passes over memory)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2601_00705_amd.render import Config, Renderer

KINDS = ["near", "far", "equal", "two", "two_near", "nested", "bits"]


def _depths(kind, n, rng):
    if kind == "spread":
        return rng.uniform(2, 4, n).astype(np.float32)
    if kind == "near":
        d = 3.0 + 0.01 * rng.random(n)
        d[0] = 0.2
    elif kind == "far":
        d = 3.0 + 1e-4 * rng.random(n)
        d[n // 2] = 5e4
    elif kind == "equal":
        d = np.full(n, 2.5)
    elif kind == "two":
        d = np.where(rng.random(n) < 0.5, 2.0, 5.0)
    elif kind == "two_near":
        d = np.where(rng.random(n) < 0.3, 2.0, 5.0) + 1e-3 * rng.random(n)
        d[-1] = 0.01
    elif kind == "nested":
        level = np.minimum(rng.geometric(0.5, n) - 1, 7)
        d = 1.0 + rng.random(n) * 10.0 ** (-3.0 * level)
        d[rng.random(n) < 0.2] = 1.0
    else:  # every bit pattern from the least to the greatest finite depth, and a crowd
        d = rng.integers(1, 0x7f7fffff, n).astype(np.uint32).view(np.float32).copy()
        d[: n // 2] = np.float32(1.5)
        return d
    return d.astype(np.float32)


def _plan(lists):
    """One 16-row view of a tile per list; the records of every list's Gaussians, shuffled."""
    n = sum(len(d) for d in lists)
    cam = {"width": 16 * len(lists), "height": 16, "fx": 1, "fy": 1, "cx": 0, "cy": 0}
    R = Renderer(n, [cam], Config(), pair_capacity=n)
    tile = np.repeat(np.arange(len(lists)), [len(d) for d in lists])
    depth = np.concatenate(lists)
    order = np.random.default_rng(n).permutation(n)
    tile, depth = tile[order], depth[order]
    rec = R.records()
    g = torch.full((n, 4), 0.5)
    g[:, 0] = torch.from_numpy(tile * 16.0 + 8.0)
    g[:, 1] = 8.0
    rec["geom"].copy_(g)
    rec["conic_o"][:, :3].copy_(torch.tensor([1.0, 0.0, 1.0]).expand(n, 3))
    rec["qthr"].fill_(0.25)
    rec["rgb_d"][:, 3].copy_(torch.from_numpy(depth))
    rec["live_mask"].fill_(-1)
    return R, tile, depth


def _check(R, tile, depth):
    n = len(depth)
    R.bin()
    M, overflow = R.pair_count()
    assert M == n and not overflow
    keys, vals, ranges = R.sorted_pairs(M)
    want = np.lexsort((np.arange(n), depth.view(np.uint32), tile))
    np.testing.assert_array_equal(vals.cpu().numpy(), want)
    np.testing.assert_array_equal(keys.cpu().numpy(),
                                  (tile[want].astype(np.int64) << 32) | depth.view(np.uint32)[want].astype(np.int64))
    np.testing.assert_array_equal((ranges[:, 1] - ranges[:, 0]).cpu().numpy(),
                                  np.bincount(tile, minlength=R.info.total_tiles))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [2049, 4097, 12_000, 200_003])
def test_one_list(kind, n):
    print(f"[crowded] {kind} n={n}", flush=True)
    _check(*_plan([_depths(kind, n, np.random.default_rng(n))]))


def test_many_lists():
    rng = np.random.default_rng(5)
    lists = []
    for k, kind in enumerate(KINDS * 3):
        lists += [_depths(kind, 2047 + 977 * k, rng), _depths("spread", 1 + 450 * k, rng), np.zeros(0, np.float32)]
    print(f"[crowded] {len(lists)} lists", flush=True)
    _check(*_plan(lists))


@pytest.mark.parametrize("kind", ["near", "far", "equal", "two"])
def test_time(kind):
    n = 200_000
    ms = {}
    for k in ("spread", kind):
        R, _, _ = _plan([_depths(k, n, np.random.default_rng(1))])
        R.bin()
        torch.cuda.synchronize()
        best = np.inf
        for _ in range(4):
            R.set_timing(True)
            R.bin()
            torch.cuda.synchronize()
            best = min(best, R.read_timing()["bin_sort"][0])
        ms[k] = best
    print(f"[crowded] sort of {n} keys: {ms}", flush=True)
    assert ms[kind] <= 2.5 * ms["spread"]
