"""The Python binding's host side, without a GPU: camera values in every form that
converts to float32, one by one."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_2603_23891_amd import fg, synth


def camera(shape=None, kind=np.asarray):
    cam = synth.make_camera(synth.yaw_pitch_rotation(0.3, -0.2), (1.0, -2.5, 3.25), 64, 48)
    if shape == "column":
        cam.R, cam.t, cam.campos = (np.asarray(a).reshape(-1, 1) for a in (cam.R, cam.t, cam.campos))
    cam.R, cam.t, cam.campos = kind(cam.R), kind(cam.t), kind(cam.campos)
    return cam


@pytest.mark.filterwarnings("ignore::DeprecationWarning")
@pytest.mark.parametrize("shape", [None, "column"])
@pytest.mark.parametrize("kind", [np.asarray, np.ndarray.tolist, torch.from_numpy, lambda a: np.asarray(a, np.float64)])
def test_camera_forms(shape, kind):
    want = camera()
    c = fg.camera_struct(camera(shape, kind))
    for name in ("R", "t", "campos"):
        assert list(getattr(c, name)) == np.asarray(getattr(want, name), np.float32).ravel().tolist()
    arr, n = fg.camera_array([want, camera(shape, kind)])
    assert n == 2 and bytes(arr[1]) == bytes(c) == bytes(arr[0])


def test_camera_of_the_wrong_size_is_refused():
    cam = camera()
    for name, value in (("R", np.eye(3, dtype=np.float32)), ("t", np.zeros(4, np.float32)), ("campos", np.zeros(2))):
        bad = camera()
        setattr(bad, name, value)
        with pytest.raises((TypeError, ValueError)):
            fg.camera_struct(bad)
    assert fg.camera_struct(cam).width == 64


def test_counts_may_be_replaced():
    """n_sel, n_pairs and status are those of the counts tensor in place."""
    tree = SimpleNamespace(n_nodes=100, n_internal_span=10)
    fb = fg.FrameBuffers(tree, 64, 48, 50, 200, device="cpu")
    for counts in (fb.counts, torch.tensor([7, 8, 9, 0], dtype=torch.int32), torch.zeros(8, dtype=torch.int32)[2:6]):
        fb.counts = counts
        for k, t in enumerate((fb.n_sel, fb.n_pairs, fb.status)):
            assert t.data_ptr() == counts.data_ptr() + 4 * k and t.shape == (1,)
    fb.counts[:3] = torch.tensor([3, 4, 2], dtype=torch.int32)
    assert fg.read_counts(fb) == (3, 4, 2) and int(fb.n_pairs) == 4
