"""Triangulation with one, two and four lanes to a pixel: every number of
neighbours whose lanes are not all busy (2, 3, 5, 6, 7 of 4), and pixel counts
that end inside a block or a wave, against the oracle at the tolerances of
the seeding tests."""
import numpy as np
import pytest

from paper_2601_00705_amd import scenes
from tests import test_gpu_seed as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,n", [(2, 301), (3, 257), (5, 77), (6, 129), (7, 1), (4, 65)])
def test_lanes(K, n):
    print(f"[seed] {K} neighbours, {n} pixels", flush=True)
    d = scenes.seed_inputs(40 + K, n, n_views=K + 1, outlier_frac=0.2)
    ref = T.S.seed(d["Ps"], d["centres"], d["images"], d["expo"], d["xr"], d["xn"], d["kappa"], **T.CFG)
    assert T._compare(d, T._gpu(d), ref, np.arange(n)) <= 2
