"""Sort at the edges of its blocks, slices and dispatches.

n splats around one block of the emission (1024) and one histogram tile, from
sub-tile to image-sized, so that a block holds from fewer to 100 times the 2048
pairs that a workgroup emits. A selection capacity above 256 histogram tiles takes
the scanned rows, one below the rows summed in the scatter. Keys, values and
ranges must equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth
from tests.gpu_util import assert_frame_parity, read_frame
from tests.helpers import flat_tree

pytestmark = pytest.mark.gpu


def scene(n, log_scale_hi):
    rng = np.random.default_rng(n)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 520, 260)
    z = rng.uniform(5, 60, n)
    px, py = rng.uniform(0, 520, n), rng.uniform(0, 260, n)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    scale = np.exp(rng.uniform(-1.0, log_scale_hi, (n, 3))) * z[:, None] / cam.fx
    q = rng.standard_normal((n, 4))
    op = 1 / (1 + np.exp(-rng.normal(-3.0, 1.0, n)))
    return flat_tree(mean, scale, q / np.linalg.norm(q, axis=1, keepdims=True), op, rng.normal(0, 0.3, (n, 1, 3))), cam


@pytest.mark.parametrize("cap_sel", [4096, 1 << 19])
@pytest.mark.parametrize("n,log_scale_hi", [(1, 4.0), (1, 1.0), (1023, 1.0), (1024, 4.0), (1025, 4.0), (3000, 2.0)])
def test_blocks_and_slices(n, log_scale_hi, cap_sel):
    tree, cam = scene(n, log_scale_hi)
    o = oracle.render_frame(tree, cam, 3.0, 0.0)
    if log_scale_hi == 4.0 and n >= 1024:
        assert o["keys"].size > 20 * 2048
    dt = fg.DeviceTree(tree)
    fb = fg.FrameBuffers(dt, cam.width, cam.height, cap_sel, 1 << 20)
    fg.render_frame(dt, cam, fb, 3.0, 0.0)
    torch.cuda.synchronize()
    assert_frame_parity(read_frame(fb, tree.n_nodes), o)


def test_pair_overflow_with_a_full_slice_list():
    """Far more pairs than the capacity, so the slice list is full: the required
    size is reported, and every stored value is a splat of the frame."""
    tree, cam = scene(3000, 4.0)
    o = oracle.render_frame(tree, cam, 3.0, 0.0)
    dt = fg.DeviceTree(tree)
    for cap_pairs in (1000, 5000):
        fb = fg.FrameBuffers(dt, cam.width, cam.height, 4096, cap_pairs)
        fb.vals.fill_(-1)
        fg.filter_stage(dt, cam, fb, 3.0)
        fg.preprocess_stage(dt, cam, fb, 0.0)
        fg.sort_stage(cam, fb)
        torch.cuda.synchronize()
        n_sel, n_pairs, status = fg.read_counts(fb)
        assert n_pairs == o["keys"].size > 20 * cap_pairs and status & fg.FG_STATUS_PAIR_OVERFLOW
        v = fb.vals[:cap_pairs].cpu().numpy().view(np.uint32)
        assert v.max() < n_sel
        r = fb.ranges.cpu().numpy().view(np.uint32).reshape(-1, 2)
        assert (r[:, 0] <= r[:, 1]).all() and r.max() <= cap_pairs
