"""KPC of one tile, bit for bit: a pair's sum is one fixed float32 tree, in both
walks and in every run.

All n splats cover the single tile of a 16 x 12 image (its last rows lie outside
the image), n around the 64 splats a wave lists at a time, the 128 of a batch
and the 256 of a chunk. The terms alpha * T come from the oracle's renderer
with colours that single out one splat per channel; the tree is quads of
four pixels, rows of four quads, waves of four rows, then the waves in order."""
import numpy as np
import pytest

import oracle
from paper_2603_23891_amd import fg, synth
from tests.helpers import flat_tree
from tests.test_gpu_gtc import gpu_view

pytestmark = pytest.mark.gpu


def pair_terms(sp, vals, ranges, cam):
    """[n, 16, 16] alpha * T of each pair and pixel of the tile (0 outside the image)."""
    n = vals.size
    py, px = np.mgrid[0:cam.height, 0:cam.width]
    out = np.zeros((n, 16, 16), np.float32)
    for k0 in range(0, n, 3):
        s = sp.copy()
        for f in "rgb":
            s[f] = 0.0
        for c, k in enumerate(range(k0, min(k0 + 3, n))):
            for f in "rgb":
                s[f][vals[k]] = 1.0 if f == "rgb"[c] else 0.0
        rgb, _, _ = oracle.render_pixels(s, vals, ranges, cam, px.ravel(), py.ravel())
        for c, k in enumerate(range(k0, min(k0 + 3, n))):
            out[k, :cam.height, :cam.width] = rgb[:, c].reshape(cam.height, cam.width)
    return out


def tree_sum(t):
    def pairwise(x):  # (0 + 1) + (2 + 3) over the last axis
        return (x[..., 0] + x[..., 1]) + (x[..., 2] + x[..., 3])
    rows = pairwise(pairwise(t.reshape(-1, 16, 4, 4)))
    waves = pairwise(rows.reshape(-1, 4, 4))
    k = np.zeros(t.shape[0], np.float32)
    for w in range(4):
        k = k + waves[:, w]
    return k


@pytest.mark.parametrize("opacity_logit_mu", [-2.0, 2.0])
@pytest.mark.parametrize("n", [1, 5, 64, 127, 128, 129, 256, 257, 400])
def test_kpc_is_one_tree(n, opacity_logit_mu):
    rng = np.random.default_rng(n)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 16, 12)
    z = rng.uniform(20, 60, n)
    px, py = rng.uniform(0, 16, n), rng.uniform(0, 12, n)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    scale = np.exp(rng.uniform(-2.5, 2.5, (n, 3))) * z[:, None] / cam.fx
    q = rng.standard_normal((n, 4))
    op = 1 / (1 + np.exp(-rng.normal(opacity_logit_mu, 1.5, n)))
    tree = flat_tree(mean, scale, q / np.linalg.norm(q, axis=1, keepdims=True), op, rng.normal(0, 0.3, (n, 1, 3)))
    _, sel = oracle.filter(tree, cam, 3.0)
    sp = oracle.preprocess(tree, cam, 0.0, sel)
    _, vals, ranges = oracle.sort(sp, cam)
    assert vals.size == n
    want = tree_sum(pair_terms(sp, vals, ranges, cam))
    dt = fg.DeviceTree(tree)
    fb = fg.FrameBuffers(dt, cam.width, cam.height, n, 4 * n)
    for chunked in (False, True, True):
        g = gpu_view(dt, cam, fb, 3.0, hist=False, chunked=chunked)
        assert np.array_equal(g["vals"], vals)
        assert np.array_equal(g["kpc"].astype(np.float32), want)
