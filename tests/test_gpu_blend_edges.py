"""Blend of one tile at the edges of its batches, chunks and paths.

All n splats cover the single tile of a 16 x 12 image (its last rows lie
outside the image), so the tile's list has n entries: around the 64 splats a wave
lists at a time, the 256 of a batch or chunk, and the 12 chunks from which a
tile is always walked from pass masks. mask_items = 1 leaves no room for a long
tile's masks, so the same lists are blended batch by batch instead. Both
must equal the oracle: contributor counts exactly, colours within 1e-4 (the
bar of every frame parity test)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth
from tests.gpu_util import assert_frame_parity, read_frame
from tests.helpers import flat_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [128, 256, 512])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 512, 513, 3073])
def test_one_tile_list_lengths(n, chunk):
    rng = np.random.default_rng(n)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 16, 12)
    z = rng.uniform(20, 60, n)
    px, py = rng.uniform(0, 16, n), rng.uniform(0, 12, n)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    # from sub-pixel to tile-sized footprints, some elongated
    scale = np.exp(rng.uniform(-2.5, 1.0, (n, 3))) * z[:, None] / cam.fx
    q = rng.standard_normal((n, 4))
    op = 1 / (1 + np.exp(-rng.normal(-3.0, 1.5, n)))
    tree = flat_tree(mean, scale, q / np.linalg.norm(q, axis=1, keepdims=True), op, rng.normal(0, 0.3, (n, 1, 3)))
    o = oracle.render_frame(tree, cam, 3.0, 0.0)
    assert o["ranges"][0, 1] == n
    dt = fg.DeviceTree(tree)
    fb = fg.FrameBuffers(dt, cam.width, cam.height, n, 4 * n)
    for mask_items in (0, 1):
        fg.render_frame(dt, cam, fb, 3.0, 0.0, tune=fg.tune_struct(chunk, 0, mask_items=mask_items))
        torch.cuda.synchronize()
        assert_frame_parity(read_frame(fb, tree.n_nodes), o)
