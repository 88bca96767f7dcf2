"""Pixels of tiles that hold no splat: runs of four empty tiles inside the image,
runs cut by a row's end, by the image's border or by a tile that holds splats, and
image widths that allow no 16-byte stores. One small splat in a corner tile (or
none): every other pixel is background, T = 1, no contributor. Above 32768 tiles four
are written at a time."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth
from tests.gpu_util import assert_frame_parity, read_frame
from tests.helpers import flat_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(64, 16), (64, 17), (128, 48), (80, 64), (144, 33), (129, 40), (130, 40), (20, 9),
                                  (1024, 64), (4112, 2064), (4108, 2060), (4114, 2064)])
@pytest.mark.parametrize("at", [(3.0, 3.0), (-100.0, 3.0)])
def test_background(size, at):
    cam = synth.make_camera(np.eye(3), (0, 0, 0), *size)
    z = 20.0
    mean = np.array([[(at[0] - cam.cx) * z / cam.fx, (at[1] - cam.cy) * z / cam.fy, z]])
    tree = flat_tree(mean, np.full((1, 3), 1.5 * z / cam.fx), np.array([[1.0, 0, 0, 0]]), np.array([0.9]),
                     np.full((1, 1, 3), 0.3))
    bg = (0.25, 0.5, 0.75)
    o = oracle.render_frame(tree, cam, 3.0, 0.0, bg=bg)
    dt = fg.DeviceTree(tree)
    fb = fg.FrameBuffers(dt, cam.width, cam.height, 1, 4096)
    for t in (fb.image, fb.final_T):
        t.fill_(float("nan"))
    fb.n_contrib.fill_(-1)
    fg.render_frame(dt, cam, fb, 3.0, 0.0, bg=bg)
    torch.cuda.synchronize()
    assert_frame_parity(read_frame(fb, tree.n_nodes), o)
