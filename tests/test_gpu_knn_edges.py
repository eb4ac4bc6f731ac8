"""Neighbour searches at what test_gpu_knn.py leaves out: points that are not
finite, whose outputs are those of a point without neighbours, among enough
points and among too few, in the direct search and in the tree."""
import numpy as np
import pytest
import torch

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
