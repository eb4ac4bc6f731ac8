"""Compositing of few tiles, bit for bit what it is among many.

A plan of few tiles splits them over more waves than a plan whose tiles fill
the chip.  The same view is rendered and differentiated alone, beside an
empty view that brings the plan into the middle range, and beside one that
brings it past the split: image, T, n_contrib and n_blend must be equal, and
so must the gradients in deterministic mode (order-independent sums).  The
views hold clamped and stopping pixels, rows that entries do not reach, list
lengths off every batch, and one tile with a list long enough to be
composited in parts among many tiles."""
import numpy as np
import pytest
import torch

from paper_2601_00705_amd import scenes
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2601_00705_amd.render import Config, Renderer


def _scene(kind):
    n, w, h = {"one": (1, 21, 18), "few": (7, 21, 18), "long": (9000, 13, 11)}.get(kind, (1500, 61, 45))
    params, cam = scenes.cloud(400, n, w, h, 40.0)
    shift = {"small": -1.0, "large": 0.7, "long": 1.0}.get(kind, 0.0)
    params["log_scale"] = (params["log_scale"] + shift).astype(np.float32)
    if kind == "long":  # faint enough that most pixels reach deep into the list
        params["opacity_logit"] = (params["opacity_logit"] - 4.0).astype(np.float32)
    else:
        params["opacity_logit"][::5] = 6.0  # above alpha_max
    return params, cam


def _run(params, cam, extra, tile, precision):
    cams, poses = [cam], [scenes.identity_pose()]
    if extra is not None:  # looks away: sees nothing
        cams.append(scenes.camera(extra[0], extra[1], 40.0))
        poses.append(scenes.pose_from_centre(np.array([0.0, 0.0, -1.0]), np.pi, 0.0))
    cfg = Config(tile_w=tile[0], tile_h=tile[1], deterministic=True, precision=precision)
    R = Renderer(params["opacity_logit"].shape[0], cams, cfg)
    P, poses_d = to_dev(params), torch.from_numpy(np.asarray(poses, np.float32)).cuda()
    rgb, T, nc, nb = R.forward_all(P, poses_d, want_blend=True)
    hw = cam["width"] * cam["height"]
    dL, dT = torch.zeros(3 * R.total_pixels, device="cuda"), torch.zeros(R.total_pixels, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    dL[:3 * hw] = torch.randn(3 * hw, generator=g, device="cuda")
    dT[:hw] = torch.randn(hw, generator=g, device="cuda")
    grads = {k: torch.empty_like(v) for k, v in P.items()}
    xi = torch.empty(len(cams), 6, device="cuda")
    R.render_bwd(P, poses_d, T, nc, dL, dT, None, grads, xi)
    torch.cuda.synchronize()
    out = {"rgb": rgb[:3 * hw], "T": T[:hw], "n_contrib": nc[:hw], "n_blend": nb[:hw], "xi": xi[0], **grads}
    return R.info.total_tiles, out


@pytest.mark.parametrize("kind,tile,precision", [(k, (16, 16), "fp32") for k in ("one", "few", "small", "large", "long")] +
                         [("mid", t, "fp32") for t in ((8, 8), (16, 8), (32, 8), (32, 16))] +
                         [("small", (16, 16), "mixed"), ("long", (32, 16), "fp32")])
def test_few_equals_many(kind, tile, precision):
    params, cam = _scene(kind)
    tiles, want = _run(params, cam, None, tile, precision)
    assert int(want["n_contrib"].max()) > (4096 if kind == "long" else 0)
    tw, th = tile
    for extra in ((60 * tw, 50 * th), (100 * tw, 90 * th)):
        many, got = _run(params, cam, extra, tile, precision)
        print(f"[few] {kind} {tile} {precision}: {tiles} tiles against {many}", flush=True)
        for k in want:
            assert torch.equal(want[k], got[k]), k
