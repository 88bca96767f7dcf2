"""Backward of one tile at the edges of its batches and lists.

All m Gaussians cover the single tile of a 16 x 12 image (its last rows lie
outside the image), so the tile's list has m entries: around the two entries
taken at a time, the 64 a wave lists at a time and the 256 of a batch, and over
several chunks walked from saved state. Gradients against the float64 oracle at
the bar of tests/test_gpu_backward.py, the image bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import synth
from tests.test_gpu_backward import GROUPS, check_grads, gpu_fwd_bwd, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 2, 3, 63, 64, 65, 255, 256, 257, 513])
def test_one_tile_list_lengths(m):
    rng = np.random.default_rng(m)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 16, 12)
    z = rng.uniform(8, 14, m)
    px, py = rng.uniform(2, 14, m), rng.uniform(2, 10, m)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    # footprints from a pixel to most of the tile
    log_scale = rng.uniform(-0.5, 1.5, (m, 3)) + np.log(z / cam.fx)[:, None]
    prm = oracle.ParamsRef(mean.T, log_scale.T, rng.standard_normal((m, 4)).T, rng.normal(-2.0, 1.0, m),
                           rng.normal(0, 0.3, (m, 16, 3)), 3)
    fwd = oracle.forward32(prm, cam)
    assert fwd["ranges"][0, 1] == m
    w = rng.normal(0, 1, (3, cam.height, cam.width))
    img, g_gpu, _ = gpu_fwd_bwd(prm, cam, w)
    assert np.array_equal(img, fwd["image"])
    _, g64 = oracle.replay64(prm, cam, fwd, dL_dimage=w, want_image=False)
    check_grads(g_gpu, g64)


@pytest.mark.parametrize("sh_degree", [0, 1, 2, 3])
@pytest.mark.parametrize("seen", ["none", "half", "all"])
def test_gradients_of_unselected_are_zero(sh_degree, seen):
    """Gaussians behind the camera are not selected: their gradients are exactly
    zero (also on a second pass into used memory), those of the others at the bar."""
    m = 700
    rng = np.random.default_rng(sh_degree)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 64, 48)
    z = rng.uniform(8, 14, m)
    behind = np.ones(m, bool) if seen == "none" else (np.arange(m) % 3 == 1 if seen == "half" else np.zeros(m, bool))
    px, py = rng.uniform(2, 62, m), rng.uniform(2, 46, m)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, np.where(behind, -z, z)], 1)
    log_scale = rng.uniform(-0.5, 1.0, (m, 3)) + np.log(z / cam.fx)[:, None]
    prm = oracle.ParamsRef(mean.T, log_scale.T, rng.standard_normal((m, 4)).T, rng.normal(-2.0, 1.0, m),
                           rng.normal(0, 0.3, (m, (sh_degree + 1) ** 2, 3)), sh_degree)
    fwd = oracle.forward32(prm, cam)
    w = rng.normal(0, 1, (3, cam.height, cam.width))
    img, g_gpu, r = gpu_fwd_bwd(prm, cam, w)
    again = r.backward(*to_dev(prm), cam, torch.from_numpy(w.astype(np.float32)).cuda())
    assert np.array_equal(img, fwd["image"])
    for g in (g_gpu, {k: v.cpu().numpy() for k, v in zip(GROUPS, again)}):
        for k in ("mean", "log_scale", "quat"):
            assert np.all(g[k][:, behind] == 0)
        assert np.all(g["logit"][behind] == 0) and np.all(g["sh"][behind] == 0)
    if seen != "none":
        _, g64 = oracle.replay64(prm, cam, fwd, dL_dimage=w, want_image=False)
        check_grads(g_gpu, g64)
