"""GPU parity: the C-ABI HIP path against the FP64 oracle, per stage.

  projection   depth keys bit-exact, tight boxes / tile counts exact
  binning      sorted keys, values and tile ranges bit-exact
  forward      |delta| <= 1e-5 per channel on every unflagged pixel
  backward     per element 1e-3 relative (+1e-6 of the group's max) and
               1e-3 relative L2 per group, upstream zeroed on flagged pixels

Small workloads are compared on the full frame; the 300k and 3M triangle
workloads on a seeded sample of 4,096 pixels (the oracle's cost is
O(pixels x triangles))."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2505_19175_amd import synth
from paper_2505_19175_amd.synth import Config

import gpu_util as G
from helpers import random_soup as _soup64
from paper_2505_19175_amd import binding as B


def random_soup(*a, **k):
    """The GPU reads float32: give the oracle the very same float32 values."""
    return _soup64(*a, dtype=np.float32, **k)

pytestmark = pytest.mark.gpu


def _cases_small():
    wl = synth.workload_small()
    return wl.scene, wl.cameras[0], wl.config, wl.upstream_seed


@pytest.fixture(scope="module")
def small():
    return _cases_small()


def _check_projection(st, scene, cam, cfg):
    ref = O.setup(scene, cam, cfg)
    depth = st.depth_key.cpu().numpy()[: scene.n]
    assert np.array_equal(depth.view(np.uint32), ref["key"].view(np.uint32))
    nt = st.ntiles.cpu().numpy()[: scene.n].astype(np.int64)
    np.testing.assert_array_equal(nt, ref["ntiles"])
    vis = ref["ntiles"] > 0
    rect = st.rect.cpu().numpy()[: scene.n].astype(np.int64)
    np.testing.assert_array_equal(rect[vis], ref["rect"][vis])
    return int(vis.sum())


def _check_bins(st, scene, cam, cfg):
    ref = O.bin_instances(scene, cam, cfg)
    M = st.M
    assert M == ref["count"]
    vals = st.vals.cpu().numpy()[:M].view(np.uint32)
    keys = st.keys.cpu().numpy()[:M].view(np.uint64)
    np.testing.assert_array_equal(vals, ref["vals"])
    np.testing.assert_array_equal(keys, ref["keys"])
    ranges = st.ranges.cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(ranges, ref["ranges"])
    dc = st.d_count.cpu().numpy()
    assert dc[0] == M and dc[1] == int((ref["setup"]["ntiles"] > 0).sum()) and dc[2] == 0
    # raster order: a permutation of the tiles by non-increasing list length
    order = st.order.cpu().numpy()[: ref["n_tiles"]].astype(np.int64)
    assert np.array_equal(np.sort(order), np.arange(ref["n_tiles"]))
    lens = np.minimum((ref["ranges"][:, 1] - ref["ranges"][:, 0]).astype(np.int64), 2047)[order]
    assert np.all(np.diff(lens) <= 0)
    return M


# ---------------------------------------------------------------------------
# 1k triangles, 128x128, full frame
# ---------------------------------------------------------------------------

def test_small_projection_and_bins(small):
    scene, cam, cfg, _ = small
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    nvis = _check_projection(st, scene, cam, cfg)
    M = _check_bins(st, scene, cam, cfg)
    assert nvis > 500 and M >= nvis


def test_small_forward(small):
    scene, cam, cfg, _ = small
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    ref = O.render(scene, cam, cfg)
    n_ok, n_flag, worst = G.assert_forward(G.to_np(out), ref)
    assert n_ok > 0.95 * cam.width * cam.height
    print("small forward", n_ok, n_flag, worst)


def test_small_backward(small):
    scene, cam, cfg, seed = small
    dC, _, _ = synth.upstream(seed, cam.width, cam.height)
    ref_f = O.render(scene, cam, cfg)
    dC = dC * (ref_f["flag"] == 0)[None]
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    g = G.gpu_backward(ras, st, sct, out, dC)
    r = O.backward(scene, cam, cfg, dC)
    print("small backward", G.assert_grads(g, r))


# ---------------------------------------------------------------------------
# 20k triangles, 256x256, SH-1, sigma in {0.25, 1, 4}; rgb, alpha, depth
# upstream gradients
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("sigma", [0.25, 1.0, 4.0])
def test_grad_workload(sigma):
    wl = synth.workload_grad(sigma)
    scene, cam, cfg = wl.scene, wl.cameras[0], wl.config
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    _check_projection(st, scene, cam, cfg)
    _check_bins(st, scene, cam, cfg)
    ref_f = O.render(scene, cam, cfg)
    n_ok, n_flag, worst = G.assert_forward(G.to_np(out), ref_f)
    dC, dA, dD = synth.upstream(wl.upstream_seed, cam.width, cam.height, True, True)
    keep = (ref_f["flag"] == 0)
    dC, dA, dD = dC * keep[None], dA * keep, dD * keep
    g = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    r = O.backward(scene, cam, cfg, dC, dA, dD)
    print("grad workload", sigma, n_ok, n_flag, worst, G.assert_grads(g, r))


# ---------------------------------------------------------------------------
# 300k and 3M triangles at 1280x720 (and 1600x1040): sampled pixels
# ---------------------------------------------------------------------------

def _sampled(scene, cam, cfg, seed, n_pix=4096, max_flag_frac=0.01, resolve=False):
    pix = synth.pixel_sample(seed, cam.width, cam.height, n_pix)
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    if resolve:     # depth keys bit-exact: a depth tie orders alike on both sides
        _check_projection(st, scene, cam, cfg)
    ref = O.render(scene, cam, cfg, pix=pix)
    n_ok, n_flag, worst = G.assert_forward(G.to_np(out), ref, pix=pix, max_flag_frac=max_flag_frac,
                                           resolve=(scene, cam, cfg, True) if resolve else None)
    dC, _, _ = synth.upstream(seed + 1000, cam.width, cam.height)
    dCs = dC.reshape(3, -1)[:, pix] * (ref["flag"] == 0)[None]
    full = np.zeros_like(dC).reshape(3, -1)
    full[:, pix] = dCs
    g = G.gpu_backward(ras, st, sct, out, full.reshape(dC.shape))
    r = O.backward(scene, cam, cfg, dCs, pix=pix)
    s = G.assert_grads(g, r)
    return st, n_ok, n_flag, worst, s


def test_mid_workload_sampled():
    wl = synth.workload_mid()
    st, n_ok, n_flag, worst, s = _sampled(wl.scene, wl.cameras[0], wl.config, 7)
    print("mid", st.M, st.N_v, n_ok, n_flag, worst, s)


@pytest.mark.parametrize("view", [0, 1])
def test_large_workload_sampled(view):
    wl = synth.workload_large()
    cam = wl.cameras[view]
    st, n_ok, n_flag, worst, s = _sampled(wl.scene, cam, wl.config, 11 + view)
    print("large", view, cam.width, cam.height, st.M, st.N_v, n_ok, n_flag, worst, s)


@pytest.mark.parametrize("which", ["mid", "large"])
def test_partition_of_unity_full_frame(which):
    """With every colour 1 and a black background the image is sum_i w_i,
    which must equal alpha = 1 - T_final (the weights and the final
    transmittance telescope to 1) on every pixel of the full frame."""
    wl = synth.workload_mid() if which == "mid" else synth.workload_large()
    sc = wl.scene
    sh = np.zeros_like(sc.sh)
    sh[:, 0, :] = 0.5 * 2.0 * np.sqrt(np.pi)      # dc Y_0 = 1/2: colour 1
    white = synth.Scene(sc.v, sc.o, sc.sigma, sh.astype(np.float32))
    cfg = Config(sh_degree=wl.config.sh_degree)
    ras, st, st_scene, out = G.gpu_forward(white, wl.cameras[0], cfg)
    g = G.to_np(out)
    np.testing.assert_array_equal(g["alpha"], 1.0 - g["T_final"].astype(np.float32))
    err = np.abs(g["rgb"] - g["alpha"][None]).max()
    print(which, "max |sum w - (1 - T_final)|", err, "covered", (g["alpha"] > 0).mean())
    assert (g["alpha"] > 0).mean() > 0.2
    assert err <= 1e-6


def test_mid_bins_bit_exact():
    wl = synth.workload_mid()
    scene, cam, cfg = wl.scene, wl.cameras[0], wl.config
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    _check_projection(st, scene, cam, cfg)
    _check_bins(st, scene, cam, cfg)


def _one_tile_soup(seed, n, mode):
    """n small triangles whose tight boxes all fall in tile (1, 1) of a 64x64
    image, every triangle flat at depth z (so its depth key is exactly z).
    mode: 'equal' (one key), 'ulps' (keys 3.0 + 0..199 ulps: only the low
    byte differs), 'spread' (z in [2, 4) with repeats), 'wide' (z in [0.5, 40)),
    'clustered' ('ulps' with 2% of the triangles at z = 30: a wide key range
    whose entries nearly all share their leading bits), 'few' (five depths in
    [2, 25): long runs of equal keys over a wide range)."""
    rng = np.random.default_rng(seed)
    W = H = 64
    cam = synth.identity_camera(W, H)
    f, c = float(cam.fx), float(cam.cx)
    if mode == "equal":
        z = np.full(n, 3.0, np.float32)
    elif mode == "ulps":
        z = (np.float32(3.0).view(np.uint32) + rng.integers(0, 200, n).astype(np.uint32)).view(np.float32)
    elif mode == "spread":
        z = rng.uniform(2.0, 4.0, n).astype(np.float32)
        rep = rng.random(n) < 0.2
        z[rep] = z[rng.integers(0, n, int(rep.sum()))]
    elif mode == "clustered":
        z = (np.float32(3.0).view(np.uint32) + rng.integers(0, 200, n).astype(np.uint32)).view(np.float32)
        z[rng.random(n) < 0.02] = np.float32(30.0)
    elif mode == "few":
        z = rng.choice(rng.uniform(2.0, 25.0, 5), n).astype(np.float32)
    else:
        z = rng.uniform(0.5, 40.0, n).astype(np.float32)
    ctr = rng.uniform(21.0, 26.0, (n, 2))
    ang = rng.uniform(0, 2 * np.pi, n)[:, None] + np.array([0.0, 2.0944, 4.1888])[None, :]
    px = ctr[:, None, 0] + 2.5 * np.cos(ang)
    py = ctr[:, None, 1] + 2.5 * np.sin(ang)
    v = np.stack([(px - c) * z[:, None] / f, (py - c) * z[:, None] / f,
                  np.repeat(z[:, None], 3, 1)], -1).astype(np.float32)
    sc = synth.Scene(v, np.full(n, 0.9, np.float32), np.ones(n, np.float32),
                     rng.uniform(0, 1, (n, 1, 3)).astype(np.float32))
    return sc, cam


@pytest.mark.parametrize("n,mode", [(2, "spread"), (65, "wide"), (700, "equal"), (1024, "spread"),
                                    (1024, "ulps"), (1025, "ulps"), (1500, "equal"),
                                    (2048, "spread"), (2049, "spread"), (4096, "spread"),
                                    (4097, "ulps"), (5000, "equal"), (5000, "ulps"),
                                    (5000, "spread"), (4500, "wide"), (300, "clustered"),
                                    (1024, "clustered"), (3000, "clustered"), (900, "few"),
                                    (2500, "few")])
def test_bins_one_deep_tile(n, mode):
    """The per-tile depth sort in its three forms (one wave up to 1024
    entries, four waves and a merge up to 4096, global ping-pong beyond) and
    with 0, 1, 3 and 4 digit passes, over key sets with long runs of equal
    keys or of keys equal in all but the low byte ('clustered', 'few'); ties
    keep index order.  Bit-exact against the oracle's stable sort."""
    sc, cam = _one_tile_soup(61, n, mode)
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    ref = O.bin_instances(sc, cam, cfg)
    lens = ref["ranges"][:, 1] - ref["ranges"][:, 0]
    assert lens.max() == n == ref["count"]          # one tile holds every triangle
    _check_bins(st, sc, cam, cfg)


def test_bins_three_radix_passes():
    """A 4160x4160 view (260 x 260 = 67600 tiles, more than 2^16): the sort by
    tile id takes three passes of six bits instead of two; bins bit-exact
    against the oracle's stable sort."""
    sc, cam = random_soup(65, 3000, W=4160, H=4160, size=0.004, deg=0)
    # a third of the triangles moved down to the bottom rows of tiles (ids
    # above 2^16), at the same depth (the oracle gets the same float32 values)
    rng = np.random.default_rng(66)
    v = sc.v.astype(np.float64)
    z = v[2000:, :, 2].mean(1)
    dy = rng.uniform(4040.0, 4150.0, 1000) - (v[2000:, :, 1].mean(1) * cam.fy / z + cam.cy)
    v[2000:, :, 1] += (dy * z / cam.fy)[:, None]
    sc.v[...] = v.astype(np.float32)
    cfg = Config(sh_degree=0)
    assert ((cam.width + 15) // 16) * ((cam.height + 15) // 16) > 1 << 16
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    M = _check_bins(st, sc, cam, cfg)
    assert M > 2000
    assert int(st.keys.cpu().numpy()[:M].view(np.uint64).max() >> np.uint64(32)) >= 1 << 16


@pytest.mark.parametrize("n,mode", [(4097, "ulps"), (5000, "equal"), (20000, "spread"),
                                    (20000, "ulps"), (45000, "wide")])
def test_bins_segmented_sort(n, mode):
    """Tiles of more than 4096 entries under the segmented sort (many
    workgroups per tile): the sizing call reports the huge tile, the state
    switches to the segmented sort, and the next call is bit-exact against
    the oracle's stable sort."""
    sc, cam = _one_tile_soup(62, n, mode)
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    assert st.segmented and int(st.d_count[3].item()) == 1
    ras.forward(st, sct, cam, sync=True)
    torch.cuda.synchronize()
    _check_bins(st, sc, cam, cfg)


def test_segmented_sort_many_tiles():
    """A dense view where every tile holds thousands of entries: segmented
    bins bit-exact, and the forward through them within the bar."""
    sc, cam = random_soup(63, 40000, W=64, H=64, size=0.9, deg=0, sigma=(0.5, 2.0),
                          o=(0.05, 0.6), zrange=(3.0, 4.0))
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    assert st.segmented and int(st.d_count[3].item()) >= 4
    out = ras.forward(st, sct, cam, sync=True)
    torch.cuda.synchronize()
    _check_bins(st, sc, cam, cfg)
    pix = synth.pixel_sample(64, cam.width, cam.height, 512)
    ref = O.render(sc, cam, cfg, pix=pix)
    G.assert_forward(G.to_np(out), ref, pix=pix, max_flag_frac=0.05)


# ---------------------------------------------------------------------------
# edge cases
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("W,H", [(1, 1), (17, 33), (100, 7), (255, 129)])
def test_ragged_images(W, H):
    sc, cam = random_soup(41, 300, W=W, H=H, size=0.8, deg=2)
    cfg = Config(sh_degree=2, bg=(0.2, 0.1, 0.3))
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    _check_bins(st, sc, cam, cfg)
    ref = O.render(sc, cam, cfg)
    G.assert_forward(G.to_np(out), ref)
    rng = np.random.default_rng(3)
    dC = rng.normal(size=(3, H, W)) * (ref["flag"] == 0)[None]
    g = G.gpu_backward(ras, st, sct, out, dC)
    G.assert_grads(g, O.backward(sc, cam, cfg, dC))


def test_deep_lists_and_termination():
    """Thousands of large, overlapping triangles: tile lists longer than one
    LDS batch, early termination, clamped opacities."""
    sc, cam = random_soup(42, 3000, W=64, H=48, size=2.0, deg=0, sigma=(0.05, 2.0),
                          o=(0.5, 1.0), zrange=(2.5, 6.0))
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    _check_bins(st, sc, cam, cfg)
    r = st.ranges.cpu().numpy()
    assert (r[:, 1] - r[:, 0]).max() > 256
    ref = O.render(sc, cam, cfg)
    assert (ref["T_final"] < 2e-4).mean() > 0.3
    G.assert_forward(G.to_np(out), ref)
    rng = np.random.default_rng(4)
    dC = rng.normal(size=(3, 48, 64)) * (ref["flag"] == 0)[None]
    g = G.gpu_backward(ras, st, sct, out, dC)
    G.assert_grads(g, O.backward(sc, cam, cfg, dC))


def test_empty_and_fully_culled():
    cam = synth.identity_camera(40, 24)
    cfg = Config(sh_degree=0)
    empty = synth.Scene(np.zeros((0, 3, 3), np.float32), np.zeros(0, np.float32),
                        np.zeros(0, np.float32), np.zeros((0, 1, 3), np.float32))
    ras, st, sct, out = G.gpu_forward(empty, cam, cfg)
    o = G.to_np(out)
    assert st.M == 0 and np.all(o["alpha"] == 0) and np.all(o["T_final"] == 1)
    # the empty path still writes a valid raster order (regression: it used to
    # leave the order uninitialised and the raster read ranges out of bounds)
    assert np.array_equal(np.sort(st.order.cpu().numpy()), np.arange(st.num_tiles))
    behind = box = synth.box_soup(5, 50)
    behind.v[:, :, 2] = -1.0                                  # all behind the camera
    ras, st, sct, out = G.gpu_forward(behind, cam, cfg)
    o = G.to_np(out)
    assert st.M == 0 and st.N_v == 0 and np.all(o["rgb"] == 0)
    g = G.gpu_backward(ras, st, sct, out, np.ones((3, 24, 40), np.float32))
    assert all(np.all(x == 0) for x in g.values())


def test_capacity_growth_and_device_count_mode():
    """A too-small instance list is reported and grown (host-count mode);
    in device-count mode the overflow flag is set on the device."""
    sc, cam = random_soup(43, 400, W=64, H=64, size=1.5, deg=0)
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg, capacity=8)
    assert st.capacity >= st.M > 8
    _check_bins(st, sc, cam, cfg)
    ras2, st2, sct2, out2 = G.gpu_forward(sc, cam, cfg, capacity=8, sync=False)
    dc = st2.d_count.cpu().numpy()
    assert dc[0] == st.M and dc[2] == 1
    ras3, st3, sct3, out3 = G.gpu_forward(sc, cam, cfg, capacity=st.M, sync=False)
    dc = st3.d_count.cpu().numpy()
    assert dc[0] == st.M and dc[2] == 0
    a, b = G.to_np(out), G.to_np(out3)
    for k in ("rgb", "alpha", "depth", "T_final", "last"):
        np.testing.assert_array_equal(a[k], b[k])


def test_backward_without_block_masks():
    """With ts_bins.blocks NULL the forward keeps no masks and the backward
    finds each entry's blocks with the geometric test instead: same gradients
    (to the oracle bar)."""
    wl = synth.workload_grad(1.0)
    scene, cam, cfg = wl.scene, wl.cameras[0], wl.config
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    ref_f = O.render(scene, cam, cfg)
    dC, dA, dD = synth.upstream(wl.upstream_seed, cam.width, cam.height, True, True)
    keep = (ref_f["flag"] == 0)
    dC, dA, dD = dC * keep[None], dA * keep, dD * keep
    st.bins.blocks = None
    out = ras.forward(st, sct, cam, sync=True)
    assert not st.bins.blocks
    g = G.gpu_backward(ras, st, sct, out, dC, dA, dD)
    r = O.backward(scene, cam, cfg, dC, dA, dD)
    print("no block masks", G.assert_grads(g, r))


def _stats_gpu(ras, st, out, N):
    mw = torch.zeros(max(N, 1), dtype=torch.float32, device="cuda:0")
    px = torch.zeros(max(N, 1), dtype=torch.int32, device="cuda:0")
    stats = B.ts_prune_stats(mw.data_ptr(), px.data_ptr())
    B.ts_render_forward_stats(st.proj, st.bins, st.ccam, ras.ccfg, out.rgb, out.alpha, out.depth,
                              out.T_final, out.last, stats, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return mw.cpu().numpy()[:N].astype(np.float64), px.cpu().numpy()[:N].astype(np.int64)


def _near_flag(scene, cam, cfg):
    """Triangles whose tight box holds a pixel the oracle flags (a decision
    within rounding of alpha_min, T_min or a depth tie): their composited set
    may differ by one pixel."""
    flag = O.render(scene, cam, cfg)["flag"] != 0
    rect = O.setup(scene, cam, cfg)["rect"]
    sat = np.zeros((cam.height + 1, cam.width + 1), np.int64)
    sat[1:, 1:] = flag.cumsum(0).cumsum(1)
    x0, x1, y0, y1 = rect[:, 0], rect[:, 1], rect[:, 2], rect[:, 3]
    ok = x0 <= x1
    x0c, x1c, y0c, y1c = (np.where(ok, a, 0) for a in (x0, x1, y0, y1))
    cnt = sat[y1c + 1, x1c + 1] - sat[y0c, x1c + 1] - sat[y1c + 1, x0c] + sat[y0c, x0c]
    return ok & (cnt > 0)


@pytest.mark.parametrize("which", ["small", "grad"])
def test_prune_statistics(which):
    """Largest T*o and composited pixels per triangle (Sec. 3.2, Pruning)
    against the oracle: pixel counts exact, weights to 1e-5."""
    if which == "small":
        wl = synth.workload_small()
    else:
        wl = synth.workload_grad(1.0)
    scene, cam, cfg = wl.scene, wl.cameras[0], wl.config
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    mw, px = _stats_gpu(ras, st, out, scene.n)
    ref = O.prune_stats(scene, cam, cfg)
    skip = _near_flag(scene, cam, cfg)
    keep = ~skip
    np.testing.assert_array_equal(px[keep], ref["pixels"][keep])
    assert np.max(np.abs(mw[keep] - ref["max_weight"][keep])) <= 1e-5
    assert skip.sum() <= 0.02 * scene.n + 2 and (ref["pixels"] > 0).sum() > 100


def test_prune_statistics_over_views():
    """Two views through the autograd-free wrapper: weights combine by max,
    views count those that rendered a triangle with more than one pixel."""
    from paper_2505_19175_amd.render import PruneStats, Rasterizer, ViewState, scene_to_device
    wl = synth.workload_grad(1.0)
    scene, cfg = wl.scene, wl.config
    cams = [wl.cameras[0], synth.identity_camera(200, 160)]
    sct = scene_to_device(scene, "cuda:0")
    ras = Rasterizer(cfg, device="cuda:0")
    ps = PruneStats(scene.n, device="cuda:0")
    for cam in cams:
        st = ViewState(scene.n, cam.width, cam.height, 4 * scene.n + 4096, device="cuda:0")
        ras.forward(st, sct, cam, stats=ps)
    torch.cuda.synchronize()
    refs = [O.prune_stats(scene, cam, cfg) for cam in cams]
    skip = _near_flag(scene, cams[0], cfg) | _near_flag(scene, cams[1], cfg)
    keep = ~skip
    want_views = sum((r["pixels"] > 1).astype(np.int64) for r in refs)
    want_w = np.maximum(refs[0]["max_weight"], refs[1]["max_weight"])
    np.testing.assert_array_equal(ps.views.cpu().numpy()[: scene.n][keep], want_views[keep])
    assert np.max(np.abs(ps.max_weight.cpu().numpy()[: scene.n][keep] - want_w[keep])) <= 1e-5
    assert np.all(ps.pixels.cpu().numpy() == 0)
    assert (want_views == 2).sum() > 100


def test_forward_deterministic():
    wl = synth.workload_grad(1.0)
    outs = [G.to_np(G.gpu_forward(wl.scene, wl.cameras[0], wl.config)[3]) for _ in range(2)]
    for k in outs[0]:
        np.testing.assert_array_equal(outs[0][k], outs[1][k])


@pytest.mark.parametrize("which", ["grad", "mid"])
def test_permutation_invariance(which):
    """Reordering the triangles changes only how equal depth keys are
    ordered (ties go to the lower index): every tile whose list holds no
    equal keys renders bit for bit the same image, and the gradients, mapped
    back through the permutation, agree up to the order of FP32 atomics."""
    wl = synth.workload_grad(1.0) if which == "grad" else synth.workload_mid()
    sc, cam, cfg = wl.scene, wl.cameras[0], wl.config
    perm = np.random.default_rng(17).permutation(sc.n)
    scp = synth.Scene(sc.v[perm], sc.o[perm], sc.sigma[perm], sc.sh[perm])
    runs = [G.gpu_forward(x, cam, cfg) for x in (sc, scp)]
    outs = [G.to_np(r[3]) for r in runs]
    keys = runs[0][1].keys.cpu().numpy()[: runs[0][1].M].view(np.uint64)
    assert runs[1][1].M == keys.size
    tied = np.unique(keys[1:][keys[1:] == keys[:-1]] >> np.uint64(32)).astype(np.int64)
    tiles_x = (cam.width + 15) // 16
    mask = np.ones((cam.height, cam.width), bool)
    for t in tied:
        ty, tx = divmod(int(t), tiles_x)
        mask[16 * ty:16 * ty + 16, 16 * tx:16 * tx + 16] = False
    print(which, "tiles with tied keys", tied.size, "pixels compared", mask.mean())
    assert mask.mean() > 0.5
    for k in ("rgb", "alpha", "depth", "T_final"):
        a, b = outs[0][k], outs[1][k]
        np.testing.assert_array_equal(a[..., mask], b[..., mask])
    rng = np.random.default_rng(18)
    dC = rng.normal(size=(3, cam.height, cam.width)) * mask   # tied tiles blend differently
    g0 = G.gpu_backward(*runs[0], dC)
    g1 = G.gpu_backward(*runs[1], dC)
    inv = np.argsort(perm)
    for k in ("v", "o", "sigma", "sh"):
        a, b = g0[k], g1[k][inv]
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(a) + 1e-12


def test_abi_rejects_bad_arguments():
    from paper_2505_19175_amd import binding as B
    sc, cam = random_soup(44, 10, W=32, H=32)
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg)
    bad_cfg = B.make_config(Config(sh_degree=7))
    with pytest.raises(B.TSError) as e:
        B.ts_project(*sct, sc.n, B.make_camera(cam), bad_cfg, st.proj)
    assert e.value.code == B.TS_EINVAL
    with pytest.raises(B.TSError) as e:
        B.ts_bin_sort(st.proj, sc.n, B.make_camera(cam), st.ws, 16, st.bins)
    assert e.value.code == B.TS_EWORKSPACE
    big = synth.identity_camera(20000, 8)
    with pytest.raises(B.TSError) as e:
        B.ts_project(*sct, sc.n, B.make_camera(big), B.make_config(cfg), st.proj)
    assert e.value.code == B.TS_EINVAL


def test_raster_backward_twice_without_projection_is_rejected(small):
    """The 2D gradient accumulators of a raster backward must be consumed by
    a backward projection before the next raster backward: a second one is
    refused (TS_EINVAL) instead of summing into them, and the pair order
    then works again."""
    scene, cam, cfg, seed = small
    ras, st, sct, out = G.gpu_forward(scene, cam, cfg)
    dC, _, _ = synth.upstream(seed, cam.width, cam.height)
    dCt = torch.tensor(dC, device="cuda:0")
    args = (st.proj, st.bins, st.ccam, ras.ccfg, dCt, None, None, out.T_final, out.last)
    B.ts_raster_backward(*args)
    with pytest.raises(B.TSError) as e:
        B.ts_raster_backward(*args)
    assert e.value.code == B.TS_EINVAL
    grads = [torch.empty_like(t) for t in sct]
    with pytest.raises(B.TSError) as e:
        B.ts_render_backward(*sct, st.N, st.proj, st.bins, st.ccam, ras.ccfg, dCt, None, None,
                             out.T_final, out.last, *grads)
    assert e.value.code == B.TS_EINVAL
    B.ts_project_backward(sct[0], sct[3], st.N, st.proj, st.ccam, ras.ccfg, *grads)
    first = [g.clone() for g in grads]
    B.ts_raster_backward(*args)
    B.ts_project_backward(sct[0], sct[3], st.N, st.proj, st.ccam, ras.ccfg, *grads)
    torch.cuda.synchronize()
    G.assert_grads({k: g.cpu().numpy().astype(np.float64) for k, g in zip(("v", "o", "sigma", "sh"), grads)},
                   {k: g.cpu().numpy().astype(np.float64) for k, g in zip(("v", "o", "sigma", "sh"), first)})


def test_short_lists_and_a_huge_tile():
    """A first view whose lists are too short and one of whose tiles holds more
    than 4096 entries even in them: grown and sorted over many workgroups in the
    same call, bit-exact against the oracle's stable sort."""
    sc, cam = _one_tile_soup(64, 9000, "ulps")
    cfg = Config(sh_degree=0)
    ras, st, sct, out = G.gpu_forward(sc, cam, cfg, capacity=5000)
    assert st.segmented and st.capacity >= 9000 and int(st.d_count[3].item()) == 1
    _check_bins(st, sc, cam, cfg)
