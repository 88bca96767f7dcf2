"""Sort of more pairs than the capacity, where the slice list admits some blocks of
the emission and refuses others: the stored pairs are the first cap_pairs in
depth order, stably ordered by tile, every slot written, from workspaces that
hold stale words."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth
from tests.helpers import flat_tree

pytestmark = pytest.mark.gpu


def uneven_scene(n):
    """n splats whose sizes vary from block to block of 1024 in depth order."""
    rng = np.random.default_rng(n)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), 520, 260)
    z = np.sort(rng.uniform(5, 60, n))
    px, py = rng.uniform(0, 520, n), rng.uniform(0, 260, n)
    mean = np.stack([(px - cam.cx) * z / cam.fx, (py - cam.cy) * z / cam.fy, z], 1)
    size = rng.uniform(-3.0, 3.2, n // 1024 + 1)[np.arange(n) // 1024]
    scale = np.exp(size[:, None] + rng.uniform(-1.0, 0.5, (n, 3))) * z[:, None] / cam.fx
    q = rng.standard_normal((n, 4))
    op = 1 / (1 + np.exp(-rng.normal(-3.0, 1.0, n)))
    return flat_tree(mean, scale, q / np.linalg.norm(q, axis=1, keepdims=True), op, rng.normal(0, 0.3, (n, 1, 3))), cam


def emitted(sp, cam):
    """(tile, splat) of every pair in emission order, and each 1024-splat block's pair count."""
    vis = np.flatnonzero(sp["tiles"])
    order = vis[np.argsort(sp["depth"][vis].view(np.uint32), kind="stable")]
    s = sp[order]
    w = s["x1"] - s["x0"]
    count = s["tiles"].astype(np.int64)
    rep = np.repeat(np.arange(order.size), count)
    local = np.arange(rep.size) - np.repeat(np.cumsum(count) - count, count)
    tile = (s["y0"][rep] + local // w[rep]) * cam.tiles_x + s["x0"][rep] + local % w[rep]
    blocks = np.add.reduceat(count, np.arange(0, order.size, 1024))
    return tile.astype(np.uint32), order[rep].astype(np.uint32), blocks


@pytest.mark.parametrize("share", [0.02, 0.3, 0.7, 0.98, 1.0])
def test_stored_pairs_are_a_prefix(share):
    tree, cam = uneven_scene(40_000)
    _, sel = oracle.filter(tree, cam, 3.0)
    sp = oracle.preprocess(tree, cam, 0.0, sel)
    tile, splat, blocks = emitted(sp, cam)
    cap_pairs = int(share * tile.size)
    more = (blocks - 1) // 2048
    assert (more > 0).sum() > 10 and (more == 0).sum() > 3
    if share < 0.9:
        assert more.sum() > cap_pairs // 2048 + 1 > more.min()  # some blocks fit, not all
    order = np.argsort(tile[:cap_pairs], kind="stable")
    dt = fg.DeviceTree(tree)
    fb = fg.FrameBuffers(dt, cam.width, cam.height, tree.n_nodes, cap_pairs)
    for stale in (0, 0xFF, 0x01):
        fb.sort_ws.fill_(stale)
        fb.vals.fill_(-1)
        fb.tile_keys.fill_(-1)
        fg.filter_stage(dt, cam, fb, 3.0)
        fg.preprocess_stage(dt, cam, fb, 0.0)
        fg.sort_stage(cam, fb)
        torch.cuda.synchronize()
        n_sel, n_pairs, status = fg.read_counts(fb)
        assert n_sel == sel.size and n_pairs == tile.size
        assert status == (fg.FG_STATUS_PAIR_OVERFLOW if cap_pairs < tile.size else 0)
        assert np.array_equal(fb.tile_keys.cpu().numpy().view(np.uint32), tile[:cap_pairs][order])
        assert np.array_equal(fb.vals.cpu().numpy().view(np.uint32), splat[:cap_pairs][order])
