"""Blend of more tiles than one launch can hold a workgroup for (2^24 of 256
threads): a one-pixel column whose every tile lists the same splat, wide enough
to blend everywhere with the same alpha."""
import numpy as np
import pytest
import torch

from paper_2603_23891_amd import fg, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frag_stats", [False, True])
def test_tiles_past_one_launch(frag_stats):
    n_tiles = (1 << 24) + 10
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 1, 16 * n_tiles - 3)
    splats = fg.Splats(1)
    splats.xy.copy_(torch.tensor([[0.5, 0.5]]))
    splats.conic_o.copy_(torch.tensor([[1e-10, 0.0, 1e-26, 0.25]]))  # exp(power) rounds to 1 down the whole column
    splats.rgb_depth.copy_(torch.tensor([[0.5, 1.0, 2.0, 1.0]]))
    vals = torch.zeros(1, dtype=torch.int32, device="cuda")
    ranges = torch.tensor([0, 1], dtype=torch.int32, device="cuda").repeat(n_tiles, 1)
    image = torch.full((3, cam.height, 1), -1.0, device="cuda")
    final_T = torch.full((cam.height, 1), -1.0, device="cuda")
    n_contrib = torch.full((cam.height, 1), -1, dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda") if frag_stats else None
    ws = torch.empty(fg.fg_render_workspace_size(cam, 1), dtype=torch.uint8, device="cuda")
    fg.fg_render(splats, vals, ranges, cam, (0.0, 0.0, 4.0), image, final_T, n_contrib, 1, stats, status, ws)
    torch.cuda.synchronize()
    for plane, want in ((image[0], 0.125), (image[1], 0.25), (image[2], 3.5), (final_T, 0.75), (n_contrib, 1)):
        lo, hi = plane.aminmax()
        assert abs(float(lo) - want) <= 1e-6 and abs(float(hi) - want) <= 1e-6
    if frag_stats:
        assert int(stats[3]) == cam.height
