"""The fixed device array of gsr_prune_noalloc: its size is what gsr.h states,
and the lists are those of gsr_prune and of the rule where the chunks change
(2^20 Gaussians), in large maps and at the largest n it takes."""
import os
import subprocess

import numpy as np
import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_size_is_the_documented_one():
    header = open(os.path.join(ROOT, "include", "gsr.h")).read()
    assert "array of the library (256 KiB, one per GPU" in " ".join(header.split()).replace("* ", "")
    so = os.path.join(ROOT, "paper_2601_00705_amd", "libgsr.so")
    out = subprocess.run(["nm", "-S", so], capture_output=True, text=True, check=True).stdout
    sizes = [int(f[1], 16) for f in (line.split() for line in out.splitlines()) if len(f) == 4 and f[3] == "_ZL7scratch"]
    assert sizes == [256 * 1024]


@pytest.mark.gpu
@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 4000, (1 << 25) - 1, 1 << 25, (1 << 25) + 1, (1 << 27) - 100, 1 << 27])
def test_large_maps(n):
    from paper_2601_00705_amd import lib, maintain
    print(f"[prune] n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    m_obs = torch.randint(0, 6, (n,), generator=g, device="cuda", dtype=torch.int32)
    v_vis = torch.rand(n, generator=g, device="cuda")
    ls = torch.rand(3, n, generator=g, device="cuda") * 4 - 3.5
    logit = torch.randn(n, generator=g, device="cuda") * 2
    keep, kept = maintain.prune(m_obs, v_vis, ls, logit, 2, 0.3, 1.5, 0.05)
    keep_b = torch.empty(n, dtype=torch.int32, device="cuda")
    kept_b = torch.empty(1, dtype=torch.int64, device="cuda")
    cfg = lib.PruneConfig(2, 0.3, 1.5, 0.05)
    lib.gsr_prune_noalloc(n, m_obs, v_vis, ls, logit, cfg, keep_b, kept_b, torch.cuda.current_stream().cuda_stream)
    m = int(kept)
    assert 0 < m < n and int(kept_b) == m
    assert torch.equal(keep[:m], keep_b[:m])
    assert bool((keep[1:m] > keep[:m - 1]).all())
    # the rule in float64, away from its thresholds
    tr = torch.exp(2 * ls.double()).sum(0)
    al = torch.sigmoid(logit.double())
    want = (m_obs >= 2) & (v_vis >= 0.3) & (tr <= 1.5 ** 2) & (al >= 0.05)
    sure = ((tr - 1.5 ** 2).abs() > 1e-6) & ((al - 0.05).abs() > 1e-7) & ((v_vis - 0.3).abs() > 1e-7)
    got = torch.zeros(n, dtype=torch.bool, device="cuda")
    got[keep[:m].long()] = True
    assert bool((got == want)[sure].all())
