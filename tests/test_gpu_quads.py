"""The rasterizers' lists per pixel quad (2x2 pixels), against the oracle at
the forward and the gradient bar: triangles from below a pixel (one quad) to
beyond a tile (every quad, so that a wave's lists outgrow their LDS space and
are walked in parts), batches of entries just before, at and after the 64 of a
mask word and the 256 of a batch, and images whose last tiles are cut."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_19175_amd import binding as B
from paper_2505_19175_amd import synth
from paper_2505_19175_amd.render import PruneStats, StoredFragments
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


# The sigmoid window sums the wide entries of an image of 800 tiles or more,
# batches of 128 entries: narrow ones between them (sigma well below the pixel),
# and all of a batch wide.
@pytest.mark.parametrize("W,H", [(512, 400), (496, 400)])   # 800 tiles, and 775: without the sums
@pytest.mark.parametrize("n,narrow", [(1, 200), (127, 0), (128, 1), (300, 200)])
def test_wide_entries_of_the_sigmoid(n, narrow, W, H):
    wide, cam = random_soup(71, n, W=W, H=H, size=1.5, deg=1, sigma=(0.3, 2.0), o=(0.02, 0.1),
                            dtype=np.float32)
    small, _ = random_soup(72, max(narrow, 1), W=W, H=H, size=0.05, deg=1, sigma=(0.01, 0.05),
                           o=(0.2, 0.9), dtype=np.float32)
    sc = wide if narrow == 0 else type(wide)(*(np.concatenate([a, b]) for a, b in
                                               zip((small.v, small.o, small.sigma, small.sh),
                                                   (wide.v, wide.o, wide.sigma, wide.sh))))
    cfg = Config(sh_degree=1, bg=(0.1, 0.2, 0.3), window=WINDOW_SIGMOID)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg, capacity=1 << 20)
    ref = O.render(sc, cam, cfg)
    G.assert_forward(G.to_np(out), ref, resolve=(sc, cam, cfg, True))
    dC, dA, dD = synth.upstream(n, cam.width, cam.height, True, True)
    keep = ref["flag"] == 0
    dC, dA, dD = dC * keep[None], dA * keep, dD * keep
    g = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    G.assert_grads(g, O.backward(sc, cam, cfg, dC, dA, dD))


@pytest.mark.parametrize("window,sigma", [(WINDOW_PAPER, 1.0), (WINDOW_SIGMOID, 0.05),
                                          (WINDOW_LSE, 1.0)])
@pytest.mark.parametrize("W,H", [(16, 16), (528, 512)])   # the second sums wide entries
def test_opaque_neighbour_leaves_gradients_alone(window, sigma, W, H):
    """An opaque triangle (alpha 1, T_min 0: its own gradient is undefined)
    behind one that shares its 4x4 block of pixels but none of its pixels: the
    second one's gradients are those it has alone."""
    f = 16.0

    def tri(pts, z):
        return [[(x - W / 2) * z / f, (y - H / 2) * z / f, z] for x, y in pts]

    v = np.array([tri([(-6, -6), (2.2, -6), (-2, 30)], 4.0),
                  tri([(2.2, -40), (14, -40), (2.4, 60)], 2.0)], np.float32)
    o = np.array([1.0, 0.5], np.float32)
    s = np.array([1e-12, sigma], np.float32)
    sh = np.array([[[0.3, 0.2, 0.1]], [[0.5, 0.1, 0.4]]], np.float32)
    both = synth.Scene(v, o, s, sh)
    alone = synth.Scene(*(a[1:] for a in (v, o, s, sh)))
    cam = synth.Camera(np.eye(3, dtype=np.float32), np.zeros(3, np.float32), f, f, W / 2, H / 2,
                       W, H).astype32()
    cfg = Config(sh_degree=0, alpha_max=1.0, T_min=0.0, window=window)
    dC, dA, dD = synth.upstream(3, W, H, True, True)
    ras, st, sct, out = G.gpu_forward(both, cam, cfg)
    opaque = out.T_final.cpu().numpy() == 0.0
    assert opaque.any()
    g = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    ras, st, sct, out = G.gpu_forward(alone, cam, cfg)
    # no pixel of the two in common, some 4x4 block in common
    mine = out.last.cpu().numpy() > 0
    assert mine.any() and not (mine & opaque).any()
    blocks = lambda m: m[:H // 4 * 4, :W // 4 * 4].reshape(H // 4, 4, W // 4, 4).any((1, 3))
    assert (blocks(mine) & blocks(opaque)).any()
    a = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    for k in g:   # the same FP32 terms, summed in another order
        np.testing.assert_allclose(g[k][1], a[k][0], rtol=0,
                                   atol=G.GRAD_RTOL * np.abs(a[k]).max())


# The statistics forward packs its per-entry words into the lists' masks: batches
# of more than 256 entries, images of cut tiles, and lists that outgrow their LDS
# space (walked in parts) while the counters are live.
@pytest.mark.parametrize("window", [WINDOW_PAPER, WINDOW_SIGMOID, WINDOW_LSE])
@pytest.mark.parametrize("n,size,W,H", [(64, 2.0, 16, 16), (257, 2.0, 16, 16), (700, 2.0, 17, 15),
                                        (900, 0.5, 33, 31), (1500, 3.0, 16, 16)])
def test_statistics_of_quad_lists(window, n, size, W, H):
    """Largest weight and composited pixels of every triangle: those of the
    fragments that the storing forward lists, bit for bit, and the oracle's up to
    its flagged pixels; images and block records are the plain forward's."""
    sc, cam = random_soup(n + W, n, W=W, H=H, size=size, deg=0, sigma=(0.3, 2.0), o=(0.02, 0.08),
                          dtype=np.float32)
    cfg = Config(sh_degree=0, window=window)
    ras, st, sct, _ = G.gpu_forward(sc, cam, cfg, capacity=1 << 16)
    stream = torch.cuda.current_stream().cuda_stream

    def forward(call, *stats):
        out = st.outputs()
        st.blocks.zero_()
        call(st.proj, st.bins, st.ccam, ras.ccfg, out.rgb, out.alpha, out.depth, out.T_final,
             out.last, *stats, stream)
        torch.cuda.synchronize()
        return out, st.blocks[:st.M].clone()

    stats = PruneStats(n)
    plain, plain_blocks = forward(B.ts_render_forward)
    out, blocks = forward(B.ts_render_forward_stats, stats.c)
    assert torch.equal(blocks, plain_blocks)
    for k in ("rgb", "alpha", "depth", "T_final", "last"):
        assert torch.equal(getattr(out, k), getattr(plain, k))
    w, px = stats.max_weight.cpu().numpy(), stats.pixels.cpu().numpy()

    sf = StoredFragments(ras, st)
    sf.forward(sct, cam)
    torch.cuda.synchronize()
    count = sf.count.cpu().numpy().ravel()
    pixel = np.repeat(np.arange(W * H), count)          # offsets are in pixel order
    assert np.array_equal(sf.offset.cpu().numpy().ravel(), np.cumsum(count) - count)
    tile = (pixel // W // 16) * ((W + 15) // 16) + pixel % W // 16
    first = st.ranges.cpu().numpy()[tile, 0]
    tri = st.vals.cpu().numpy()[first + sf.entry[:sf.F].cpu().numpy()]
    np.testing.assert_array_equal(px[:n], np.bincount(tri, minlength=n))
    want = np.zeros(n, np.float32)
    np.maximum.at(want, tri, sf.T[:sf.F].cpu().numpy() * sc.o[tri])
    np.testing.assert_array_equal(w[:n], want)
    assert (px > 0).sum() > n // 8

    flag = O.render(sc, cam, cfg)["flag"].ravel() != 0
    ref = O.prune_stats(sc, cam, cfg, pix=np.flatnonzero(~flag))
    assert (px[:n] >= ref["pixels"]).all() and (px[:n] <= ref["pixels"] + flag.sum()).all()
    assert (w[:n] >= ref["max_weight"] - G.FWD_ATOL).all() and flag.sum() <= 0.1 * W * H
