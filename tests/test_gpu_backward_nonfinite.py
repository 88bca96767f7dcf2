"""Backward over splats whose opacity is not finite (a caller's own splat planes):
their alpha is the cap of 0.99, which passes no gradient to mean, conic and
opacity, so those gradients are exactly zero and no other gradient is lost."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth
from tests.test_gpu_backward import GROUPS, gpu_fwd_bwd, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_capped_splats_pass_no_gradient(value):
    m = 40
    rng = np.random.default_rng(m)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 48, 32)
    z = rng.uniform(8, 14, m)
    px, py = rng.uniform(2, 46, m), rng.uniform(2, 30, m)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    log_scale = rng.uniform(-0.5, 1.0, (m, 3)) + np.log(z / cam.fx)[:, None]
    prm = oracle.ParamsRef(mean.T, log_scale.T, rng.standard_normal((m, 4)).T, rng.normal(-2.0, 0.5, m),
                           rng.normal(0, 0.3, (m, 1, 3)), 0)
    w = rng.normal(0, 1, (3, cam.height, cam.width))
    _, _, r = gpu_fwd_bwd(prm, cam, w)
    args = to_dev(prm)
    n_sel = fg.read_counts(r.fb)[0]
    odd = torch.arange(0, n_sel, 7, device="cuda")
    r.fb.splats.conic_o[odd, 3] = value
    g = r.backward(*args, cam, torch.from_numpy(w.astype(np.float32)).cuda())
    torch.cuda.synchronize()
    g = {k: v.cpu().numpy() for k, v in zip(GROUPS, g)}
    at = r.fb.sel_idx[odd].cpu().numpy()
    for k in GROUPS:
        assert np.all(np.isfinite(g[k])), k
    for k in ("mean", "log_scale", "quat", "logit"):
        assert np.all(g[k][..., at] == 0), k
    assert np.any(g["sh"][at] != 0)
