"""GPU tests of the binning's launch forms (one workgroup; group counts with
the columns summed by the placing workgroups or scanned by a launch; a batch's
windows of tiles) against a numpy sort of the instances by (tile, depth key,
triangle index)."""
import ctypes
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2505_19175_amd import binding as B
from paper_2505_19175_amd import synth
from paper_2505_19175_amd.render import Rasterizer, ViewState, scene_to_device
from paper_2505_19175_amd.serve.executor import BatchedExecutor
from paper_2505_19175_amd.serve.scheduler import Request

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _entries(seed, N, W, H):
    """Random boxes (a third culled, most of a few pixels, some covering many
    tiles), depth keys with ties."""
    rng = np.random.default_rng(seed)
    side = np.where(rng.random(N) < 0.995, rng.integers(1, 20, N), rng.integers(20, 400, N))
    x0, y0 = rng.integers(0, W, N), rng.integers(0, H, N)
    x1, y1 = np.minimum(x0 + side, W - 1), np.minimum(y0 + side // 2, H - 1)
    nt = (x1 // 16 - x0 // 16 + 1) * (y1 // 16 - y0 // 16 + 1)
    gone = rng.random(N) < 0.33
    nt[gone] = 0
    rect = np.stack([x0, x1, y0, y1], 1).astype(np.int16)
    rect[gone] = (0, -1, 0, -1)
    depth = (rng.integers(0, max(2, N // 3), N) * np.float32(1e-3) + 1).astype(np.float32)
    return rect, nt.astype(np.int32), depth


def _reference(rect, nt, depth, tiles_x):
    e = np.repeat(np.arange(len(nt)), nt)
    k = np.arange(len(e)) - np.repeat(np.cumsum(nt) - nt, nt)
    r = rect.astype(np.int64)[e] // 16
    nx = r[:, 1] - r[:, 0] + 1
    tile = (r[:, 2] + k // nx) * tiles_x + r[:, 0] + k % nx
    order = np.lexsort((e, depth[e], tile))
    return tile[order], e[order]


def _bin(rect, nt, depth, W, H, capacity, sync=True):
    N = len(nt)
    st = ViewState(N, W, H, capacity, device=DEV, keys=True)
    st.rect[:N].copy_(torch.as_tensor(rect))
    st.ntiles[:N].copy_(torch.as_tensor(nt))
    st.depth_key[:N].copy_(torch.as_tensor(depth))
    cam = B.make_camera(synth.identity_camera(W, H))
    count = (ctypes.c_uint32 * 2)() if sync else None
    B.ts_bin_sort(st.proj, N, cam, st.ws, st.ws_bytes, st.bins, count,
                  torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return st, count


# one workgroup up to 4096 entries (4, 1023, 4096); groups with folded columns
# (4097: 5 groups of 920 tiles; 20011: 20 of 256) or a column scan (70001: 69 of
# 3600); runs of eight from 4096 entries per group (1200007: 4688); the last
# size also in a 1600x1040 view and in one of a single tile row
@pytest.mark.parametrize("N,W,H", [(1, 16, 16), (4, 130, 40), (1023, 640, 360), (4096, 640, 360),
                                   (4097, 640, 360), (20_011, 256, 256), (70_001, 1280, 720),
                                   (1_200_007, 1600, 1040), (1_200_007, 2047, 16)])
def test_instances_in_tile_depth_index_order(N, W, H):
    rect, nt, depth = _entries(N + W, N, W, H)
    tiles_x = (W + 15) // 16
    tile, vals = _reference(rect, nt, depth, tiles_x)
    M = len(vals)
    st, count = _bin(rect, nt, depth, W, H, max(M, 1))
    assert (count[0], count[1]) == (M, int((nt > 0).sum()))
    np.testing.assert_array_equal(st.vals[:M].cpu().numpy(), vals)
    want = (tile.astype(np.uint64) << np.uint64(32)) | depth[vals].view(np.uint32)
    np.testing.assert_array_equal(st.keys[:M].cpu().numpy().view(np.uint64), want)
    T = st.num_tiles
    lens = np.bincount(tile, minlength=T)
    ends = np.cumsum(lens)
    ranges = np.stack([ends - lens, ends], 1)
    ranges[lens == 0] = 0
    np.testing.assert_array_equal(st.ranges.cpu().numpy(), ranges)
    order = st.order.cpu().numpy()
    np.testing.assert_array_equal(np.sort(order), np.arange(T))
    # longest first, lengths of 2047 and more in any order
    assert (np.diff(np.minimum(lens[order], 2047)) <= 0).all()
    assert st.d_count.cpu().tolist() == [M, int((nt > 0).sum()), 0, int((lens > 4096).sum())]


@pytest.mark.parametrize("N,W,H", [(3000, 640, 360), (20_011, 256, 256), (70_001, 1280, 720)])
def test_overflow_keeps_sorted_runs(N, W, H):
    """With room for half the instances the flag is set, the ranges are
    clamped, and each run holds entries of its tile in order."""
    rect, nt, depth = _entries(N, N, W, H)
    tiles_x = (W + 15) // 16
    tile, vals = _reference(rect, nt, depth, tiles_x)
    cap = len(vals) // 2
    st, _ = _bin(rect, nt, depth, W, H, cap, sync=False)
    d = st.d_count.cpu().tolist()
    assert d[0] == len(vals) and d[2] == 1
    r, got = st.ranges.cpu().numpy(), st.vals.cpu().numpy()
    assert r[:, 1].max() == cap and (r[:, 1] - r[:, 0]).sum() == cap
    every = set(zip(tile.tolist(), vals.tolist()))
    for t in np.flatnonzero(r[:, 1] > r[:, 0])[:: max(1, len(r) // 200)]:
        run = got[r[t, 0]:r[t, 1]]
        assert all((int(t), int(v)) in every for v in run)
        assert (np.lexsort((run, depth[run])) == np.arange(len(run))).all()


# a batch's tiles in one window (two 360p views), in two (three 1080p views:
# 24480 of 16384 a window), a budget under 12288 tiles (32-bit counters), and
# more views than a group's share of a soup of 40
@pytest.mark.parametrize("n,sizes,budget", [
    (30_000, [(640, 360), (640, 360)], 65_280),
    (30_000, [(1920, 1080), (1920, 1079), (1919, 1080)], 65_280),
    (30_000, [(640, 360), (333, 200), (64, 48)], 4000),
    (40, [(64 + 16 * i, 48) for i in range(6)], 20_000)])
def test_batch_windows_equal_single_views(n, sizes, budget):
    rng = np.random.Generator(np.random.PCG64(5))
    sc = synth.cluster_soup(5, n, extent=3.0, std=0.4, edge_median=0.05, sh_degree=1, rng=rng)
    cfg = synth.Config(sh_degree=1)
    scene = scene_to_device(sc, DEV)
    cams = [synth.look_at(e, width=w, height=h)
            for e, (w, h) in zip(synth.hemisphere_eyes(rng, len(sizes)), sizes)]
    ex = BatchedExecutor(scene, cfg, time.perf_counter, max_views=len(sizes) + 1,
                         max_tiles=budget, max_pixels=sum(w * h for w, h in sizes),
                         capacity=1 << 21, slots=1)
    for views in (len(sizes), 1, len(sizes)):        # replays with other views
        batch = [Request(i, c, 0.0) for i, c in enumerate(cams[:views])]
        ex.submit(0, batch)
        while (res := ex.poll(0)) is None:
            pass
        assert not res.overflow
        total = 0
        for cam, (rgb, alpha, depth) in zip(cams, ex.outputs(0, batch)):
            st = ViewState(n, cam.width, cam.height, 1 << 20)
            out = Rasterizer(cfg).forward(st, scene, cam, sync=True)
            total += st.M
            for a, b in ((rgb, out.rgb), (alpha, out.alpha), (depth, out.depth)):
                assert torch.equal(a, b)
        assert res.instances == total


def _disjoint_runs(ranges, cap):
    r = ranges[ranges[:, 1] != ranges[:, 0]]
    r = r[np.argsort(r[:, 0])]
    assert (r[:, 0] < r[:, 1]).all() and r[0, 0] == 0 and r[-1, 1] == cap
    assert (r[1:, 0] == r[:-1, 1]).all()


# More than 2^32 instances: 2^21 boxes over all of 3600 tiles (in 32 bits every
# 2048th tile starts at 0), 1.25M over 3600.
@pytest.mark.parametrize("N", [1 << 21, 1_250_000])
@pytest.mark.parametrize("cap", [5000, 3_000_000])
def test_more_instances_than_32_bits(N, cap):
    W, H = 1280, 720
    rect = np.tile(np.array([0, W - 1, 0, H - 1], np.int16), (N, 1))
    nt = np.full(N, 3600, np.int32)
    depth = (np.random.default_rng(N).permutation(N) + 1).astype(np.float32)
    st, _ = _bin(rect, nt, depth, W, H, cap, sync=False)
    d = st.d_count.cpu().numpy().view(np.uint32)
    assert d[0] == 0xffffffff and d[1] == N and d[2] == 1
    r, got = st.ranges.cpu().numpy(), st.vals.cpu().numpy()
    _disjoint_runs(r, cap)
    for t in np.flatnonzero(r[:, 1] > r[:, 0]):
        run = got[r[t, 0]:r[t, 1]]
        assert (run >= 0).all() and (run < N).all() and len(set(run.tolist())) == len(run)
        assert (np.diff(depth[run]) > 0).all()


def _covering(n):
    """Triangles over the whole image of an identity camera."""
    rng = np.random.Generator(np.random.PCG64(n))
    z = rng.uniform(3.0, 4.0, n).astype(np.float32)
    v = np.empty((n, 3, 3), np.float32)
    v[:, :, :2] = np.array([[-400, -300], [400, -300], [0, 500]], np.float32)
    v[:, :, 2] = z[:, None]
    sh = rng.uniform(-1.0, 1.0, (n, 1, 3)).astype(np.float32)
    return synth.Scene(v, np.full(n, 0.3, np.float32), np.ones(n, np.float32), sh)


def test_view_of_more_instances_than_a_list_holds_is_refused():
    """The view is refused with the capacity error, before lists are allocated
    for what the 32-bit count says."""
    n, W, H = 540_000, 1920, 1080
    scene = scene_to_device(_covering(n), DEV)
    cfg = synth.Config(sh_degree=0)
    st, ras = ViewState(n, W, H, 4096), Rasterizer(cfg)
    cam = synth.identity_camera(W, H)
    for call in (lambda: ras.forward(st, scene, cam, sync=True),
                 lambda: ras.bin_sort(st, ras.project(st, scene, cam))):
        with pytest.raises(B.TSError) as e:
            call()
        assert e.value.code == B.TS_ECAPACITY
    assert st.capacity == 4096
    few = scene_to_device(_covering(20), DEV)   # each covers every tile
    st = ViewState(20, W, H, 4096)
    ras.forward(st, few, cam, sync=True)
    assert st.M == 20 * st.num_tiles


def test_batch_of_more_instances_than_32_bits():
    n, W, H, cap = 70_000, 1920, 1080, 100_000
    scene = scene_to_device(_covering(n), DEV)
    cam = synth.identity_camera(W, H)
    ex = BatchedExecutor(scene, synth.Config(sh_degree=0), time.perf_counter, max_views=8,
                         max_tiles=8 * 8160, max_pixels=8 * W * H, capacity=cap, slots=1)
    batch = [Request(i, cam, 0.0) for i in range(8)]
    ex.submit(0, batch)
    while (res := ex.poll(0)) is None:
        pass
    assert res.overflow and res.instances == 0xffffffff
    _disjoint_runs(ex._slots[0].ranges.cpu().numpy(), cap)
    for rgb, alpha, depth in ex.outputs(0, batch):
        assert all(bool(torch.isfinite(x).all()) for x in (rgb, alpha, depth))


def test_short_lists_on_another_stream():
    """A state whose lists are too short, rendered on a stream other than the one
    its buffers come from, while that one allocates blocks of the lists' size."""
    n, W, H = 200_000, 1280, 720
    rng = np.random.Generator(np.random.PCG64(8))
    scene = scene_to_device(synth.cluster_soup(8, n, sh_degree=0, edge_median=0.1, rng=rng), DEV)
    cfg = synth.Config(sh_degree=0)
    cam = synth.look_at(synth.hemisphere_eyes(rng, 1)[0], width=W, height=H)
    ref = ViewState(n, W, H, 1 << 22, device=DEV)
    want = Rasterizer(cfg).forward(ref, scene, cam, sync=True)
    side = torch.cuda.Stream()
    for cap in (1, 1000, ref.M - 1, ref.M):
        st = ViewState(n, W, H, cap, device=DEV)
        size = st._lists.raw.numel()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            out = Rasterizer(cfg).forward(st, scene, cam, sync=True)
        junk = [torch.full((size,), 255, dtype=torch.uint8, device=DEV) for _ in range(4)]
        torch.cuda.synchronize()
        assert st.M == ref.M and st.capacity >= ref.M and len(junk) == 4
        for a, b in ((out.rgb, want.rgb), (out.alpha, want.alpha), (out.depth, want.depth)):
            assert torch.equal(a, b)


# Views in windows of their own, across a window's edge and beyond it, small views
# that share one, and (the second set) more views than groups.
@pytest.mark.parametrize("n,sizes", [
    (30_000, [(2100, 2048), (64, 48), (1920, 1080), (333, 200), (2048, 2063), (16, 16)]),
    (40, [(2100, 2048), (64, 48), (1920, 1080), (333, 200), (2048, 2063), (16, 16)])])
def test_batch_of_many_windows(n, sizes):
    rng = np.random.Generator(np.random.PCG64(6))
    sc = synth.cluster_soup(6, n, extent=3.0, std=0.4, edge_median=0.05, sh_degree=0, rng=rng)
    cfg = synth.Config(sh_degree=0)
    scene = scene_to_device(sc, DEV)
    cams = [synth.look_at(e, width=w, height=h)
            for e, (w, h) in zip(synth.hemisphere_eyes(rng, len(sizes)), sizes)]
    ex = BatchedExecutor(scene, cfg, time.perf_counter, max_views=len(sizes), max_tiles=70_000,
                         max_pixels=sum(w * h for w, h in sizes), capacity=1 << 22, slots=1)
    for pick in ([0, 1, 2, 3, 4, 5], [4, 5], [5, 3, 0, 2], [1], [2, 0]):
        batch = [Request(i, cams[i], 0.0) for i in pick]
        ex.submit(0, batch)
        while (res := ex.poll(0)) is None:
            pass
        assert not res.overflow
        total = 0
        for i, got in zip(pick, ex.outputs(0, batch)):
            st = ViewState(n, cams[i].width, cams[i].height, 1 << 21)
            out = Rasterizer(cfg).forward(st, scene, cams[i], sync=True)
            total += st.M
            for a, b in zip(got, (out.rgb, out.alpha, out.depth)):
                assert torch.equal(a, b)
        assert res.instances == total


def test_batch_time_does_not_grow_with_its_windows():
    """What a soup adds to a batch's time (no triangle is visible, so walking it is
    all there is): over 16 windows of tiles no more than twice what it adds over
    one."""
    def ms(n, w, h):
        v = torch.zeros(n, 3, 3, device=DEV)
        v[:, :, 2] = -5.0
        one = torch.ones(n, device=DEV)
        ex = BatchedExecutor((v, one, one, torch.zeros(n, 1, 3, device=DEV)),
                             synth.Config(sh_degree=0), time.perf_counter, max_views=8,
                             max_tiles=8 * 32400, max_pixels=8 * w * h, capacity=1 << 16, slots=1)
        cam = synth.identity_camera(w, h)
        ex.submit(0, [Request(i, cam, 0.0) for i in range(8)])
        torch.cuda.synchronize()
        s, best = ex._slots[0], 1e9
        with torch.cuda.stream(s.stream):
            for _ in range(8):
                e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                e[0].record()
                s.graph.replay()
                e[1].record()
                torch.cuda.synchronize()
                best = min(best, e[0].elapsed_time(e[1]))
        return best

    big, few = 2_000_000, 40_000   # 256 groups either way: the same matrix of counts
    many = ms(big, 3840, 2160) - ms(few, 3840, 2160)
    one = ms(big, 640, 360) - ms(few, 640, 360)
    assert 0.0 < many < 2.0 * one, (many, one)


def _batch_against_single_views(scene, cfg, cams, n, **kw):
    """A batch's frames and instance count against the views rendered alone; returns
    the executor."""
    ex = BatchedExecutor(scene, cfg, time.perf_counter, slots=1, **kw)
    alone = {}
    for pick in (range(len(cams)), range(len(cams) // 2, len(cams))):   # replays
        batch = [Request(i, cams[i], 0.0) for i in pick]
        ex.submit(0, batch)
        while (res := ex.poll(0)) is None:
            pass
        assert not res.overflow
        total = 0
        for i, got in zip(pick, ex.outputs(0, batch)):
            key = id(cams[i])
            if key not in alone:
                st = ViewState(n, cams[i].width, cams[i].height, 1 << 20)
                out = Rasterizer(cfg).forward(st, scene, cams[i], sync=True)
                alone[key] = st.M, out
            total += alone[key][0]
            out = alone[key][1]
            for a, b in zip(got, (out.rgb, out.alpha, out.depth)):
                assert torch.equal(a, b)
        assert res.instances == total
    return ex


# 128 views of one tile that every triangle covers, so a group's 16-bit counter
# holds all of its entries: 65528 at most (the last size that is counted by
# groups), and one triangle more, which takes the radix chain.
@pytest.mark.parametrize("n", [131_042, 131_043])
def test_batch_at_the_most_entries_of_a_group(n):
    scene = scene_to_device(_covering(n), DEV)
    cams = [synth.identity_camera(16, 16), synth.identity_camera(16, 15)] * 64
    _batch_against_single_views(scene, synth.Config(sh_degree=0), cams, n, max_views=128,
                                max_tiles=20_000, max_pixels=128 * 256, capacity=17_000_000)


# The radix chain of a batch: more views than groups (257), and a soup too large for
# the groups' counters with the default eight views.
@pytest.mark.parametrize("n,views,sizes", [
    (300, 257, [(640, 360), (333, 200), (64, 48), (1920, 1080), (16, 16)]),
    (2_200_000, 8, [(640, 360), (1280, 720), (333, 200)])])
def test_batch_by_the_radix_chain(n, views, sizes):
    rng = np.random.Generator(np.random.PCG64(9))
    sc = synth.cluster_soup(9, n, extent=3.0, std=0.4, edge_median=0.05 if n < 1000 else 0.005,
                            sh_degree=0, rng=rng)
    scene = scene_to_device(sc, DEV)
    cams = [synth.look_at(e, width=w, height=h)
            for e, (w, h) in zip(synth.hemisphere_eyes(rng, len(sizes)), sizes)]
    kw = dict(max_views=views, max_tiles=20_000, max_pixels=sum(w * h for w, h in sizes))
    cfg = synth.Config(sh_degree=0)
    ex = _batch_against_single_views(scene, cfg, cams, n, capacity=1 << 23, **kw)
    # lists for half of the first batch's instances: flagged, runs inside the lists
    batch = [Request(i, c, 0.0) for i, c in enumerate(cams)]
    ex.submit(0, batch)
    while (res := ex.poll(0)) is None:
        pass
    cap = res.instances // 2
    ex = BatchedExecutor(scene, cfg, time.perf_counter, slots=1, capacity=cap, **kw)
    ex.submit(0, batch)
    while (short := ex.poll(0)) is None:
        pass
    assert short.overflow and short.instances == res.instances
    r = ex._slots[0].ranges.cpu().numpy()
    assert r.min() >= 0 and r.max() == cap and (r[:, 1] - r[:, 0]).sum() == cap


@pytest.mark.parametrize("mul", [1, 40])
def test_view_of_more_tiles_than_the_groups_count(mul):
    """A 3840x2160 view (32400 tiles: the radix chain), its counts read after the
    render and its launches sized by the lists: the same as with the counts read
    first, for lists that fit, are far too long, and are too short."""
    n, W, H = 30_000, 3840, 2160
    rng = np.random.Generator(np.random.PCG64(10))
    sc = synth.cluster_soup(10, n, extent=2.0, std=0.4, edge_median=0.05, sh_degree=0, rng=rng)
    scene, cfg = scene_to_device(sc, DEV), synth.Config(sh_degree=0)
    cam = synth.look_at(synth.hemisphere_eyes(rng, 1)[0], width=W, height=H)
    ras, ref = Rasterizer(cfg), ViewState(n, W, H, 1 << 20)
    cc = ras.project(ref, scene, cam)
    ras.bin_sort(ref, cc)                       # the counts first
    ref.ccam = cc
    want = ref.outputs()
    B.ts_render_forward(ref.proj, ref.bins, cc, ras.ccfg, want.rgb, want.alpha, want.depth,
                        want.T_final, want.last, torch.cuda.current_stream().cuda_stream)
    for cap in (ref.M * mul, ref.M // 3):
        st = ViewState(n, W, H, cap)
        out = ras.forward(st, scene, cam, sync=True)
        assert (st.M, st.N_v) == (ref.M, ref.N_v) and st.capacity >= ref.M
        assert torch.equal(st.vals[:st.M], ref.vals[:st.M]) and torch.equal(st.ranges, ref.ranges)
        for a, b in ((out.rgb, want.rgb), (out.alpha, want.alpha), (out.depth, want.depth)):
            assert torch.equal(a, b)


# The radix chain past 2^32 instances: a 4K view (32400 tiles), and a state that
# sorts huge tiles segment-wise.
@pytest.mark.parametrize("n,W,H,segmented", [(140_000, 3840, 2160, False),
                                             (540_000, 1920, 1080, True)])
def test_radix_chain_past_32_bits(n, W, H, segmented):
    scene = scene_to_device(_covering(n), DEV)
    cap = 100_000
    st, ras = ViewState(n, W, H, cap), Rasterizer(synth.Config(sh_degree=0))
    if segmented:
        Rasterizer._seen_huge(st, 1)
    cam = synth.identity_camera(W, H)
    with pytest.raises(B.TSError) as e:
        ras.forward(st, scene, cam, sync=True)
    assert e.value.code == B.TS_ECAPACITY and st.capacity == cap
    out = ras.forward(st, scene, cam, sync=False)
    torch.cuda.synchronize()
    d = st.d_count.cpu().numpy().view(np.uint32)
    assert d[0] == 0xffffffff and d[1] == n and d[2] == 1
    r = st.ranges.cpu().numpy()
    _disjoint_runs(r, cap)
    vals, depth = st.vals.cpu().numpy(), st.depth_key.cpu().numpy()
    assert (vals >= 0).all() and (vals < n).all()
    for t in np.flatnonzero(r[:, 1] > r[:, 0])[::500]:
        run = vals[r[t, 0]:r[t, 1]]
        assert (np.lexsort((run, depth[run])) == np.arange(len(run))).all()
    assert bool(torch.isfinite(out.rgb).all())
