"""Blend of many heavy tiles, at the lines that tell long tiles from the others.

Tile lists are laid out by hand (every splat of a list belongs to its tile): heavy
tiles of two or three chunks and tiles around 11 to 13 chunks of 256 splats, which
are also 22 to 26 of 128 and 6 or 7 of 512. "alike" has enough equal tiles that
only the longest are walked from pass masks, "mixed" too few of them, "long" an average
of more than four chunks, so that all are. At every chunk size: image,
transmittance and contributor counts equal the oracle's bit for bit; the KPC
walked from the saved state is within its nine float32 roundings of the oracle's;
gradients walked from the saved state agree with those of whole tiles walked from
the final transmittance. Translucent lists, and lists that saturate within a
chunk."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_23891_amd import fg, synth

pytestmark = pytest.mark.gpu
W, H = 630, 470  # 40 x 30 tiles, the last column and row ragged
EDGES = [2560, 2561, 2816, 2817, 2944, 2945, 3072, 3073, 3328, 3329]


def lengths(kind, rng):
    n = np.zeros(40 * 30, np.int64)
    heavy = {"alike": 1150, "mixed": 560, "long": 140}[kind]
    n[:heavy] = rng.integers(*{"alike": (257, 768), "mixed": (257, 768), "long": (1025, 1792)}[kind], heavy)
    n[heavy:heavy + len(EDGES)] = EDGES
    n[heavy + len(EDGES):] = rng.integers(0, 257, n.size - heavy - len(EDGES))
    return rng.permutation(n)


def line(n, chunk):
    """Chunks from which a tile is long, as the blend's schedule chooses it."""
    c = -(-n // chunk)
    c = c[c > 1]
    equal = c.sum() ** 2 / (c ** 2).sum()
    if equal >= 900 and equal >= 0.75 * c.size:
        return "alike"
    return "long" if c.sum() >= 4 * c.size or c.sum() < 1024 else "mixed"


def scene(kind, mu):
    rng = np.random.default_rng(len(kind))
    n = lengths(kind, rng)
    cam = synth.make_camera(np.eye(3), (0, 0, 0), W, H)
    end = np.cumsum(n)
    ranges = np.stack([end - n, end], 1)
    ranges[n == 0] = 0
    P = int(end[-1])
    tile = np.repeat(np.arange(n.size), n)
    sp = np.zeros(P, oracle.SPLAT_DTYPE)
    sp["u"] = (tile % 40) * 16 + rng.uniform(-2, 18, P)
    sp["v"] = (tile // 40) * 16 + rng.uniform(-2, 18, P)
    s = np.exp(rng.uniform(-0.5, 1.5, P))
    sp["A"], sp["C"] = s**-2.0, s**-2.0 * rng.uniform(0.5, 2.0, P)
    sp["B"] = rng.uniform(-0.6, 0.6, P) * np.sqrt(sp["A"] * sp["C"])
    sp["opacity"] = 1 / (1 + np.exp(-rng.normal(mu, 1.0, P)))
    for f in "rgb":
        sp[f] = rng.uniform(0, 1, P)
    sp["depth"] = 1.0
    return n, cam, sp, np.arange(P, dtype=np.uint32), ranges.astype(np.uint32)


def cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("mu", [-5.0, 1.0])
@pytest.mark.parametrize("kind", ["alike", "mixed", "long"])
def test_lines(kind, mu):
    n, cam, sp, vals, ranges = scene(kind, mu)
    P = vals.size
    bg = (0.1, 0.2, 0.3)
    image, final_T, n_contrib = oracle.render(sp, vals, ranges, cam, bg)
    kpc = oracle.kpc(sp, vals, ranges, cam)
    splats = fg.Splats(P)
    splats.xy.copy_(cuda(np.stack([sp["u"], sp["v"]], 1)))
    splats.conic_o.copy_(cuda(np.stack([sp["A"], sp["B"], sp["C"], sp["opacity"]], 1)))
    splats.rgb_depth.copy_(cuda(np.stack([sp["r"], sp["g"], sp["b"], sp["depth"]], 1)))
    d_vals, d_ranges = cuda(vals.view(np.int32)), cuda(ranges.view(np.int32))
    counts = torch.tensor([P], dtype=torch.int32, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    # raw parameters for the chain behind the blend's gradients: the same in all walks
    raw = [torch.zeros(s, device="cuda") for s in ((3, P), (3, P), (4, P), (P,), (P, 1, 3))]
    raw[0][2], raw[2][0] = 10.0, 1.0
    prm = fg.params_struct(*raw, 0)
    dL = cuda(np.random.default_rng(1).normal(0, 1, (3, H, W)).astype(np.float32))
    bws = torch.empty(fg.fg_render_backward_workspace_size(P), dtype=torch.uint8, device="cuda")
    want = None
    assert line(n, 256) == kind
    for chunk in (256, 128, 512):
        for save in (False, True):
            tune = fg.tune_struct(chunk, save_state=save)
            ws = torch.full((fg.fg_render_workspace_size(cam, P, tune),), 0xFF, dtype=torch.uint8, device="cuda")
            out = [torch.full(s, -1, dtype=t, device="cuda") for s, t in
                   (((3, H, W), torch.float32), ((H, W), torch.float32), ((H, W), torch.int32))]
            fg.fg_render(splats, d_vals, d_ranges, cam, bg, *out, P, None, status, ws, tune)
            torch.cuda.synchronize()
            got = [t.cpu().numpy() for t in out]
            assert np.array_equal(got[2].view(np.uint32), n_contrib), (chunk, save)
            assert np.array_equal(got[0], image) and np.array_equal(got[1], final_T), (chunk, save)
            g = [torch.full_like(x, -1.0) for x in raw]
            fg.fg_render_backward(prm, cam, bg, d_vals, counts, P, splats, d_vals, d_ranges, out[1], out[2], out[0], ws,
                                  P, tune, dL, fg.FgGrads(*[x.data_ptr() for x in g]), bws)
            g = [x.double().cpu().numpy() for x in g]
            if want is None:
                want = g  # whole tiles, from the final transmittance
            for a, b in zip(g, want):
                assert np.linalg.norm(a - b) <= 1e-3 * np.linalg.norm(b), (chunk, save)
            if save:
                k = torch.full((P,), -1.0, device="cuda")
                tile_gtc = torch.empty(n.size, device="cuda")
                view = torch.zeros(2, dtype=torch.float64, device="cuda")
                fg.fg_gtc(splats, d_vals, d_ranges, cam, counts, P, k, tile_gtc, view, n_contrib=out[2], render_ws=ws,
                          tune=tune)
                torch.cuda.synchronize()
                k = k.double().cpu().numpy()
                assert np.all(np.abs(k - kpc) <= 9 * 2.0**-24 * kpc), chunk
                assert int(view[1]) == (n > 0).sum()
