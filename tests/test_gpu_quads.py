"""The rasterizers' lists per pixel quad (2x2 pixels), against the oracle at
the forward and the gradient bar: triangles from below a pixel (one quad) to
beyond a tile (every quad, so that a wave's lists outgrow their LDS space and
are walked in parts), batches of entries just before, at and after the 64 of a
mask word and the 256 of a batch, and images whose last tiles are cut."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2505_19175_amd import synth
from paper_2505_19175_amd.synth import WINDOW_LSE, WINDOW_PAPER, WINDOW_SIGMOID, Config

import gpu_util as G
from helpers import random_soup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("window", [WINDOW_PAPER, WINDOW_SIGMOID, WINDOW_LSE])
@pytest.mark.parametrize("n,size,W,H", [
    (64, 0.05, 16, 16), (65, 0.3, 16, 16), (256, 0.05, 16, 16), (257, 2.0, 16, 16),
    (700, 2.0, 17, 15), (900, 0.1, 33, 31), (400, 0.5, 31, 18)])
def test_quad_lists(window, n, size, W, H):
    sc, cam = random_soup(n + W, n, W=W, H=H, size=size, deg=1, sigma=(0.3, 2.0), o=(0.02, 0.08),
                          dtype=np.float32)
    cfg = Config(sh_degree=1, bg=(0.1, 0.2, 0.3), window=window)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    ref = O.render(sc, cam, cfg)
    G.assert_forward(G.to_np(out), ref, resolve=(sc, cam, cfg, True))
    dC, dA, dD = synth.upstream(n, cam.width, cam.height, True, True)
    keep = ref["flag"] == 0
    dC, dA, dD = dC * keep[None], dA * keep, dD * keep
    g = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    G.assert_grads(g, O.backward(sc, cam, cfg, dC, dA, dD))


# Triangles that cover many of an image's tiles, up to and beyond the entries
# of a batch that the backward sums per tile, and over several batches.
@pytest.mark.parametrize("window", [WINDOW_PAPER, WINDOW_LSE])
@pytest.mark.parametrize("n", [1, 10, 11, 300])
def test_wide_entries(n, window):
    wide, cam = random_soup(61, n, W=520, H=512, size=1.5, deg=1, sigma=(0.3, 2.0), o=(0.02, 0.1),
                            dtype=np.float32)
    small, _ = random_soup(62, 200, W=520, H=512, size=0.05, deg=1, sigma=(0.3, 2.0), o=(0.2, 0.9),
                           dtype=np.float32)
    sc = type(wide)(*(np.concatenate([a, b]) for a, b in
                      zip((wide.v, wide.o, wide.sigma, wide.sh),
                          (small.v, small.o, small.sigma, small.sh))))
    cfg = Config(sh_degree=1, bg=(0.1, 0.2, 0.3), window=window)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg, capacity=1 << 20)
    ref = O.render(sc, cam, cfg)
    G.assert_forward(G.to_np(out), ref, resolve=(sc, cam, cfg, True))
    dC, dA, dD = synth.upstream(n, cam.width, cam.height, True, True)
    keep = ref["flag"] == 0
    dC, dA, dD = dC * keep[None], dA * keep, dD * keep
    g = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    G.assert_grads(g, O.backward(sc, cam, cfg, dC, dA, dD))
