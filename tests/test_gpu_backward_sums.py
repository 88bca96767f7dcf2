"""Backward: a splat's sum over a tile does not round from block to block.

One splat of the capped opacity covers the only tile of a 16 x 16 image, so each
pixel's term of the colour gradient is dL/dimage times one and the same
weight. dL/dimage holds +-2^26 in one pixel of one 4 x 2 block of each wave's
four rows (two of each sign), 0 in the rest of those blocks and 0.4875 elsewhere: a float32 running sum over the blocks
loses the 28 other blocks' 3.9, which are below half a unit in the last place
of 2^26. The large terms cancel exactly, so what is left is held to ten float32
roundings: at most seven occur (three in the weight, one in the term, the sum's
tree of eight equal terms is exact, one in each of the conversion, the addition
to memory and the product with the basis)."""
import numpy as np
import pytest

import oracle
from paper_2603_23891_amd import synth
from tests.test_gpu_backward import gpu_fwd_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("place", [(0, 0), (5, 1), (15, 2), (10, 3)])
def test_block_sums_do_not_round(place):
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 16, 16)
    log_scale = np.full((3, 1), np.log(400.0 * 10.0 / cam.fx))
    prm = oracle.ParamsRef(np.array([[0.0], [0.0], [10.0]]), log_scale, np.array([[1.0], [0], [0], [0]]),
                           np.array([12.0]), np.full((1, 1, 3), 0.2), 0)
    fwd = oracle.forward32(prm, cam)
    assert np.all(fwd["n_contrib"] == 1) and np.unique(fwd["final_T"]).size == 1
    w = np.full((3, 16, 16), 0.4875)
    for wave in range(4):
        y, x = 4 * wave + place[1], place[0]
        w[:, y // 2 * 2:y // 2 * 2 + 2, x // 4 * 4:x // 4 * 4 + 4] = 0.0
        w[:, y, x] = 2.0**26 if wave % 2 else -2.0**26
    img, g, _ = gpu_fwd_bwd(prm, cam, w)
    assert np.array_equal(img, fwd["image"])
    _, g64 = oracle.replay64(prm, cam, fwd, dL_dimage=np.float32(w).astype(np.float64), want_image=False)
    assert np.all(np.abs(g64["sh"]) > 30.0)
    assert np.all(np.abs(g["sh"] - g64["sh"]) <= 10 * 2.0**-24 * np.abs(g64["sh"]))
