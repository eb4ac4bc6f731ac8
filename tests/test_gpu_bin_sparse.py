"""Binning of views with few live Gaussians, exact: the chunks of the live
list shrink (and the count matrix's column scan takes its rows in passes), so
lengths at the edges of a chunk, of a staged group and of a scan pass are
compared with the oracle's keys, values and ranges."""
import numpy as np
import pytest
import torch

import oracle
from tests.test_gpu_parity import _disc_records, _fill_and_bin

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2601_00705_amd.render import Config, Renderer


@pytest.mark.parametrize("n,live", [(1, 1), (70, 63), (70, 64), (70, 65), (3000, 0), (3000, 129), (3000, 3000),
                                    (40000, 257), (40000, 16385), (40000, 40000), (140000, 140000),
                                    (1100000, 1100000)])
@pytest.mark.parametrize("views", [1, 3])
def test_sparse(n, live, views):
    print(f"[sparse] n={n} live={live} views={views}", flush=True)
    rng = np.random.default_rng(n + live)
    cams = [{"width": w, "height": h, "fx": 1, "fy": 1, "cx": 0, "cy": 0}
            for w, h in ((130, 70), (33, 90), (16, 16))][:views]
    recs = [np.concatenate(x) for x in zip(*(_disc_records(rng, n, c["width"], c["height"], 0.5) for c in cams))]
    for v in range(views):  # all but `live` of the view's Gaussians are culled
        dead = rng.permutation(n)[live:]
        recs[2][v * n + dead] = -1.0
    R = Renderer(n, cams, Config(), pair_capacity=40_000_000)
    M, overflow = _fill_and_bin(R, recs)
    assert not overflow
    keys, vals, ranges = R.sorted_pairs(M)
    k, v, r = oracle.bin_f32(cams, n, *recs, 16, 16)
    assert M == len(k)
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), k)
    np.testing.assert_array_equal(vals.cpu().numpy().view(np.uint32), v)
    np.testing.assert_array_equal(ranges.cpu().numpy().view(np.uint32), r)


@pytest.mark.parametrize("n,live", [(40000, 257), (140000, 8754)])
def test_sparse_live_lists(n, live):
    """The same with the culled Gaussians' liveness bits cleared, as the
    projection leaves them, so that the live list itself is short."""
    rng = np.random.default_rng(live)
    cam = {"width": 130, "height": 70, "fx": 1, "fy": 1, "cx": 0, "cy": 0}
    recs = _disc_records(rng, n, 130, 70, 2.0)
    keep = np.zeros(n, bool)
    keep[rng.permutation(n)[:live]] = True
    recs[2][~keep] = -1.0
    R = Renderer(n, [cam], Config(), pair_capacity=4_000_000)
    _fill_and_bin(R, recs)
    words = np.packbits(np.pad(keep, (0, -n % 64)).reshape(-1, 64), axis=1, bitorder="little").view(np.int64)
    R.records()["live_mask"].reshape(-1).copy_(torch.from_numpy(words.reshape(-1)))
    R.bin()
    M, overflow = R.pair_count()
    keys, vals, _ = R.sorted_pairs(M)
    k, v, _ = oracle.bin_f32([cam], n, *recs, 16, 16)
    assert M == len(k) and not overflow
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), k)
    np.testing.assert_array_equal(vals.cpu().numpy().view(np.uint32), v)
