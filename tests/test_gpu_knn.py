"""Neighbour searches (gsr_nearest, gsr_seed_scale, gsr_seed_frame's plane
fit) where they can go wrong: leaf and bucket boundaries, the change from the
direct search to the tree at 16,384 points and to more buckets above 2^21,
duplicates, one dense cluster among far points, few valid points, points that
are not finite.

Bar: the searches decide in double on (squared distance of the FP32 points,
index), so nearest indices equal a float64 brute force exactly; the scale is
the float64 mean distance's logarithm rounded once to FP32 (2^-24 of |log|
up to 16, so 1e-6 absolute).
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2601_00705_amd import maintain, seeding


def _points(kind, n, rng):
    if kind == "box":
        x = rng.uniform(-3, 3, (3, n))
    elif kind == "plane":
        x = rng.uniform(-3, 3, (3, n))
        x[2] = 1.25
    elif kind == "line":
        x = np.zeros((3, n))
        x[0] = rng.uniform(0, 1, n)
    elif kind == "duplicates":
        x = rng.uniform(-1, 1, (3, n))
        x[:, rng.permutation(n)[: n // 2]] = x[:, : n // 2]
        x[:, : min(n, 150)] = 0.5
    elif kind == "cluster":  # two scales and far outliers
        x = rng.uniform(-3, 3, (3, n))
        x[:, : n // 2] = 1.0 + 1e-4 * rng.normal(size=(3, n // 2))
        x[:, -5:] *= 1e5
    elif kind == "nonfinite":
        x = rng.uniform(-3, 3, (3, n))
        x[0, 3::97] = np.nan
        x[1, 5::101] = np.inf
    return np.ascontiguousarray(x, dtype=np.float32)


def _brute(x, valid, q):
    """(distance, index) order of the valid others of the queries q."""
    X = torch.from_numpy(x).cuda().double()
    ok = torch.from_numpy(valid != 0).cuda()
    near, d3 = [], []
    for i in q:
        d = sum((X[c] - X[c, i]) ** 2 for c in range(3))
        d[~ok] = np.inf
        d[i] = np.inf
        d = torch.nan_to_num(d, nan=np.inf, posinf=np.inf)
        near.append(int(torch.nonzero(d == d.min())[0]) if torch.isfinite(d.min()) else -1)
        s = torch.sort(d)[0][:3]
        s = s[torch.isfinite(s)]
        d3.append(float(torch.sqrt(s).mean()) if len(s) else -1.0)
    return np.array(near), np.array(d3)


CASES = [("box", n, 1.0) for n in (1, 2, 3, 63, 64, 65, 1023, 1025, 16383, 16384, 16385, 16449, 70001, 131073)] + [
    ("plane", 40000, 0.8), ("line", 20000, 1.0), ("duplicates", 9000, 1.0), ("duplicates", 33000, 0.9),
    ("cluster", 12000, 1.0), ("cluster", 60000, 0.7), ("box", 30000, 0.0001), ("box", 30000, 0.0),
    ("nonfinite", 5000, 1.0), ("nonfinite", 30000, 0.9), ("box", (2 << 20) + 77, 1.0), ("cluster", (2 << 20) + 1, 0.9)]


@pytest.mark.parametrize("kind,n,share", CASES)
def test_nearest_and_scale(kind, n, share):
    print(f"[knn] {kind} n={n} valid {share}", flush=True)
    rng = np.random.default_rng(n)
    x = _points(kind, n, rng)
    valid = (rng.uniform(size=n) < share).astype(np.int32)
    X, V = torch.from_numpy(x).cuda(), torch.from_numpy(valid).cuda()
    nn = maintain.nearest(X, V).cpu().numpy()
    ls = seeding.Scaler(n)(X, V, 1e-6).cpu().numpy()
    assert np.all(nn[valid == 0] == -1) and np.all(ls[:, valid == 0] == 0.0)
    fine = np.isfinite(x).all(0) & (valid != 0)
    q = np.nonzero(fine)[0]
    q = q if len(q) <= 200 else np.sort(rng.choice(q, 200, replace=False))
    ref, d3 = _brute(x, valid, q)
    if kind != "nonfinite":
        assert np.array_equal(nn[q], ref)
    else:  # an infinite point has no nearest of its own, the others never take it
        assert np.array_equal(nn[q], ref) and np.all(fine[nn[fine & (nn >= 0)]])
    want = np.where(d3 >= 0, np.log(np.maximum(d3, 1e-6)), np.log(1e-6))
    assert np.all(np.abs(ls[:, q] - want) <= 1e-6 * np.maximum(1.0, np.abs(want)))


@pytest.mark.parametrize("n,share", [(1, 1.0), (130, 1.0), (16384, 0.9), (16385, 0.9), (50000, 0.5)])
def test_frame_moments(n, share):
    """Points scattered about planes through them: the normal of the plane
    fit against float64 moments of the neighbours (the second-largest
    eigenvalue stays 100 times the least, so 1e-6 in |cos| leaves room for
    the FP32 quaternion), for sampled points."""
    print(f"[knn] frame n={n}", flush=True)
    rng = np.random.default_rng(n + 1)
    x = rng.uniform(-1, 1, (3, n))
    x[2] = 3.0 + 0.3 * x[0] + 1e-4 * rng.normal(size=n)
    x = np.ascontiguousarray(x, dtype=np.float32)
    valid = (rng.uniform(size=n) < share).astype(np.int32)
    valid[0] = 1
    P = np.array([[500.0, 0, 320, 0], [0, 500, 240, 0], [0, 0, 1, 0]])
    err, ang = rng.uniform(0, 2, n).astype(np.float32), rng.uniform(0.01, 0.3, n).astype(np.float32)
    r = 2.0 * np.sqrt(20 / np.pi / max(n * share, 1))
    dev = [torch.from_numpy(a).cuda() for a in (x, valid, err, ang)]
    quat, ls = (t.cpu().numpy().astype(np.float64) for t in
                seeding.Scaler(n).frame(*dev, P.reshape(-1), [0.0, 0, 0], r))
    assert np.all(quat[0, valid == 0] == 1) and np.all(quat[1:, valid == 0] == 0) and np.all(ls[:, valid == 0] == 0)
    ok = np.nonzero(valid)[0]
    X = x[:, ok].astype(np.float64)
    for i in rng.choice(ok, min(len(ok), 100), replace=False):
        d = x[:, i].astype(np.float64)[:, None]
        pts = X[:, ((X - d) ** 2).sum(0) <= r * r]
        if pts.shape[1] < 8:
            continue
        lam, U = np.linalg.eigh(np.cov(pts))
        if lam[1] < 100 * lam[0]:
            continue
        w, a, b, c = quat[:, i]
        v = np.array([2 * (a * c + w * b), 2 * (b * c - w * a), 1 - 2 * (a * a + b * b)])
        assert abs(abs(v @ U[:, 0]) - 1) <= 1e-6
