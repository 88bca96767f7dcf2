"""Multi-view filter where tiles lie inside some views' frustums only, at the pass
widths: 7 views (bit planes), 8 (one byte per node), 9 (a pass of 8 and one of 1);
the selections must equal the oracle's view by view, with the fixed scratch too."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_views", [7, 8, 9])
@pytest.mark.parametrize("tau_R", [3.0, 20.0])
def test_views_in_all_directions(n_views, tau_R):
    tree = synth.city_tree(synth.CitySpec(n_leaves=20_000, box=(30, 30, 8), n_blobs=12, blob_sigma=(5, 5, 2),
                                          leaf_log_scale_mu=-2.5, seed=3))
    cams = [synth.make_camera(synth.yaw_pitch_rotation(2 * np.pi * k / n_views, np.radians(-20)), (2.0 * k - 8, 3, 6),
                              320, 200) for k in range(n_views)]
    dt = fg.DeviceTree(tree)
    N = tree.n_nodes
    words = (N + 31) // 32
    ws = torch.empty(fg.fg_filter_workspace_size(N, dt.n_internal_span, n_views), dtype=torch.uint8, device="cuda")
    sizes = set()
    for noalloc in (False, True):
        sel_bits = torch.full((n_views * words,), -1, dtype=torch.int32, device="cuda")
        sel_idx = torch.full((n_views * N,), -1, dtype=torch.int32, device="cuda")
        n_sel = torch.zeros(n_views, dtype=torch.int32, device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        if noalloc:
            fg.fg_filter_noalloc(dt, cams, tau_R, sel_bits, sel_idx, N, n_sel, status)
        else:
            fg.fg_filter(dt, cams, tau_R, sel_bits, sel_idx, N, n_sel, status, ws)
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        for v, cam in enumerate(cams):
            _, sel = oracle.filter(tree, cam, tau_R)
            assert int(n_sel[v]) == sel.size
            assert np.array_equal(sel_idx[v * N:v * N + sel.size].cpu().numpy().view(np.uint32), sel)
            bits = np.unpackbits(sel_bits[v * words:(v + 1) * words].cpu().numpy().view(np.uint8), bitorder="little")
            assert np.array_equal(np.flatnonzero(bits[:N]), sel)
            sizes.add(sel.size)
    assert len(sizes) > 3
