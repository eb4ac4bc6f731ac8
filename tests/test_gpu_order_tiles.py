"""The spatial order at the edges of its radix tiles (1024 keys, 4096 past
2^20), exact against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_order import O, _gpu_order, _means

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 1023, 1024, 1025, 2049, 30_011, 1 << 20, (1 << 20) + 1])
def test_order_tiles(n):
    print(f"[spatial order] n={n}", flush=True)
    mean = _means(n, n, "dups")
    assert np.array_equal(_gpu_order(mean, 128), O.spatial_order(mean, 128))
