"""Neighbour searches at what test_gpu_knn.py leaves out: points that are not
finite, whose outputs are those of a point without neighbours, among enough
points and among too few, in the direct search and in the tree."""
import numpy as np
import pytest
import torch

from tests import test_gpu_knn

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2601_00705_amd import maintain, seeding

FLOOR = 1e-6


@pytest.mark.parametrize("n", [4, 900, 16384, 16385, 40000])
@pytest.mark.parametrize("finite", [1, 2, 3, 500])
def test_infinite_points(n, finite):
    print(f"[knn] {n} points, {finite} finite", flush=True)
    rng = np.random.default_rng(n + finite)
    x = rng.uniform(-3, 3, (3, n)).astype(np.float32)
    fine = np.zeros(n, bool)
    fine[rng.permutation(n)[:min(finite, n - 1)]] = True
    far = np.nonzero(~fine)[0]
    x[far % 3, far] = np.where(far % 2 == 0, np.inf, -np.inf)
    x[1, far[::5]] = np.nan
    X, V = torch.from_numpy(x).cuda(), torch.ones(n, dtype=torch.int32, device="cuda")
    nn = maintain.nearest(X, V).cpu().numpy()
    ls = seeding.Scaler(n)(X, V, FLOOR).cpu().numpy()
    lf = np.log(np.float64(np.float32(FLOOR)))
    assert np.all(nn[~fine] == -1)
    assert np.abs(ls[:, ~fine] - lf).max() <= 1e-6 * abs(lf)
    q = np.nonzero(fine)[0]
    pts = x[:, q].astype(np.float64)
    d = np.sqrt(((pts[:, :, None] - pts[:, None, :]) ** 2).sum(0))
    np.fill_diagonal(d, np.inf)
    if len(q) == 1:
        assert nn[q[0]] == -1 and np.abs(ls[:, q] - lf).max() <= 1e-6 * abs(lf)
        return
    assert np.array_equal(nn[q], q[d.argmin(0)])
    want = np.log(np.maximum(np.sort(d, 0)[:min(3, len(q) - 1)].mean(0), FLOOR))
    assert np.all(np.abs(ls[:, q] - want) <= 1e-6 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("n,period,phase", [(1 << 20, 2, 0), (1 << 20, 256, 0), (1 << 17, 2, 1), (40960, 40, 0),
                                            (1 << 22, 256, 0)])
def test_periodic_validity(n, period, phase):
    """Valid points that follow the storage order (every other pixel, all but
    one column): the search is exact, and takes no longer than it does with
    as many valid points in any order.  Valid points that the samples miss
    all land in one bucket and cost tens of times that, so the bound is 5."""
    print(f"[knn] {n} points, all but every {period}th", flush=True)
    rng = np.random.default_rng(period)
    X = torch.from_numpy(rng.uniform(-1, 1, (3, n)).astype(np.float32)).cuda()
    valid = (np.arange(n) % period != phase).astype(np.int32)
    V, W = torch.from_numpy(valid).cuda(), torch.from_numpy(rng.permutation(valid)).cuda()
    out = {}
    for key, v in (("order", V), ("shuffled", W)):
        times = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            nn = maintain.nearest(X, v)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        out[key] = min(times)
        if key == "order":
            got = nn.cpu().numpy()
    print(f"[knn] {out['order']:.3f} ms, shuffled {out['shuffled']:.3f} ms", flush=True)
    assert out["order"] <= 5 * out["shuffled"]
    assert np.all(got[valid == 0] == -1)
    Xd, ok = X.double(), V != 0
    for i in rng.choice(np.nonzero(valid)[0], 40, replace=False):
        d = ((Xd - Xd[:, i:i + 1]) ** 2).sum(0)
        d[~ok] = np.inf
        d[i] = np.inf
        assert int(d.argmin()) == got[i]


def _best_ms(f, reps=4):
    best = np.inf
    for _ in range(reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        out = f()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best, out


@pytest.mark.parametrize("n", [20_000, 150_000])
@pytest.mark.parametrize("far", [1.5e3, 1e6, 1e12, 3e37])
def test_outliers(n, far):
    """Points far outside the others, past and before the extent at which the
    cells follow the logarithm: nearest and scale are exact, and the radius
    search, in which outliers have no part, takes no longer than without them
    (its leaves held points in storage order: tens of times that, hence 5)."""
    print(f"[knn] {n} points, outliers at {far:g}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.uniform(-1, 1, (3, n))
    x[rng.integers(0, 3, n), np.arange(n)] = 1.0  # three faces of a box
    y = x.copy()
    odd = np.array([0, n // 3, n - 1])
    y[:, odd] = far * np.array([[1.0, -0.5, 0.25], [0.5, 1.0, -1.0], [-1.0, 0.1, 0.7]])
    plain, dirty = (torch.from_numpy(a.astype(np.float32)).cuda() for a in (x, y))
    valid = (rng.random(n) < 0.9).astype(np.int32)
    valid[odd] = 1
    V = torch.from_numpy(valid).cuda()
    err, ang = torch.ones(n, device="cuda"), torch.full((n,), 0.1, device="cuda")
    P = np.array([[500.0, 0, 320, 0], [0, 500, 240, 0], [0, 0, 1, 0]]).reshape(-1)
    S = seeding.Scaler(n)
    r = 2.0 * np.sqrt(12 / np.pi / n * 3)
    t0, _ = _best_ms(lambda: S.frame(plain, V, err, ang, P, [0.0, 0, 5.0], r))
    t1, (quat, _) = _best_ms(lambda: S.frame(dirty, V, err, ang, P, [0.0, 0, 5.0], r))
    print(f"[knn] radius search {t0:.3f} ms, with outliers {t1:.3f} ms", flush=True)
    assert t1 <= 5 * t0 and bool(torch.isfinite(quat).all())
    nn = maintain.nearest(dirty, V).cpu().numpy()
    ls = S(dirty, V, FLOOR).cpu().numpy()
    X, ok = dirty.double(), V != 0
    pick = np.concatenate([odd, rng.choice(np.nonzero(valid)[0], 60, replace=False)])
    for i in pick:
        d = ((X - X[:, i:i + 1]) ** 2).sum(0)
        d[~ok] = np.inf
        d[i] = np.inf
        assert int(torch.nonzero(d == d.min())[0]) == nn[i]
        want = float(torch.log(torch.sqrt(torch.sort(d)[0][:3]).mean().clamp_min(FLOOR)))
        assert abs(ls[0, i] - want) <= 1e-6 * max(1.0, abs(want))


@pytest.mark.parametrize("kind,n,share", [(k, n, s) for k, s in (("box", 1.0), ("cluster", 0.95))
                                          for n in (1_049_599, 1_049_600, 1_200_000)])
def test_larger_buckets(kind, n, share):
    """From 1,049,600 points on a bucket is sorted 8192 keys at a time."""
    test_gpu_knn.test_nearest_and_scale(kind, n, share)
