"""KPC of one tile at the edges of its batches and lists, both walks.

All n splats cover the single tile of a 16 x 12 image (its last rows lie outside
the image), so its list has n entries: around the four entries taken at a
time, the 64 a wave lists at a time and the 256 of a batch or chunk. A pair's sum
is 8 terms in a tree of depth 3 and at most 32 such block sums in sequence: at
most 34 float32 roundings, 34 * 2^-24 = 2.03e-6 of the sum, the relative bar."""
import numpy as np
import pytest

from paper_2603_23891_amd import fg, synth
from tests.helpers import flat_tree
from tests.test_gpu_gtc import ATOL, gpu_view, oracle_view

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 64, 65, 255, 256, 257, 513])
def test_one_tile_list_lengths(n):
    rng = np.random.default_rng(n)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 16, 12)
    z = rng.uniform(20, 60, n)
    px, py = rng.uniform(0, 16, n), rng.uniform(0, 12, n)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    scale = np.exp(rng.uniform(-2.5, 1.0, (n, 3))) * z[:, None] / cam.fx
    q = rng.standard_normal((n, 4))
    op = 1 / (1 + np.exp(-rng.normal(-2.0, 1.5, n)))
    tree = flat_tree(mean, scale, q / np.linalg.norm(q, axis=1, keepdims=True), op, rng.normal(0, 0.3, (n, 1, 3)))
    o = oracle_view(tree, cam, 3.0)
    assert o["kpc"].size == n
    dt = fg.DeviceTree(tree)
    fb = fg.FrameBuffers(dt, cam.width, cam.height, n, 4 * n)
    for chunked in (False, True):
        g = gpu_view(dt, cam, fb, 3.0, hist=False, chunked=chunked)
        assert np.array_equal(g["vals"], o["vals"])
        assert np.all(np.abs(g["kpc"] - o["kpc"]) <= 34 * 2.0**-24 * o["kpc"] + ATOL)
        assert abs(g["tile"][0] - o["tile"][0]) <= 35 * 2.0**-24 * o["tile"][0] + ATOL
        assert g["view"][1] == 1
