"""GPU parity of the densification step (Sec. 3.2, "Densification") against
the oracle: Bernoulli selection bit-exact (decisions within 1e-12 of their
threshold are flagged and counted instead), midpoint subdivision bit-exact,
on a small soup, a soup that triggers the cap at one, and the 3M-triangle
soup; overflow leaves the soup untouched."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import densify as D
from paper_2505_19175_amd import binding as B
from paper_2505_19175_amd import synth

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def _select(o, s, mode, k, u):
    N = o.size
    ws_bytes = B.ts_densify_workspace_bytes(N)
    ws = torch.empty(max(ws_bytes, 1), dtype=torch.uint8, device=DEV)
    sel = torch.zeros(max(N, 1), dtype=torch.uint8, device=DEV)
    B.ts_densify_select(_t(o), _t(s), N, mode, k, _t(u), sel, ws, ws_bytes)
    torch.cuda.synchronize()
    return sel.cpu().numpy()[:N].astype(bool)


def _check_select(o, s, mode, k, u):
    got = _select(o, s, mode, k, u)
    p = D.probabilities(o, s, mode, k)
    want = D.select(o, s, mode, k, u)
    near = np.abs(u.astype(np.float64) - p) <= 1e-12 * np.maximum(p, 1e-300)
    assert near.sum() <= 2
    np.testing.assert_array_equal(got[~near], want[~near])
    return int(want.sum())


@pytest.mark.parametrize("mode", [B.TS_DENSIFY_OPACITY, B.TS_DENSIFY_INV_SIGMA])
def test_select_small(mode):
    rng = np.random.default_rng(5 + mode)
    N = 10000
    o = rng.uniform(0.0, 1.0, N).astype(np.float32)
    s = rng.uniform(0.2, 5.0, N).astype(np.float32)
    u = rng.random(N).astype(np.float32)
    n = _check_select(o, s, mode, 1000.0, u)
    assert 850 < n < 1150


def test_select_cap_and_degenerate():
    rng = np.random.default_rng(9)
    N = 3000
    o = rng.uniform(0.0, 0.01, N).astype(np.float32)
    o[:5] = 1.0                                     # p = 1 for these at k = 200
    s = np.ones(N, np.float32)
    u = rng.random(N).astype(np.float32)
    assert _check_select(o, s, B.TS_DENSIFY_OPACITY, 200.0, u) >= 5
    assert not _select(np.zeros(N, np.float32), s, B.TS_DENSIFY_OPACITY, 50.0, u).any()
    assert not _select(o, s, B.TS_DENSIFY_OPACITY, 0.0, u).any()
    # ragged sizes around the workgroup and the partial-sum chunk
    for N in (1, 255, 257, 4095, 4097):
        _check_select(o[:N] + 0.5, s[:N], B.TS_DENSIFY_INV_SIGMA, N / 7.0, u[:N])


def _subdivide(v, o, s, sh, deg, sel, capacity, host=True):
    N = o.size
    K = (deg + 1) ** 2
    tv = torch.zeros((capacity, 3, 3), dtype=torch.float32, device=DEV)
    to = torch.zeros(capacity, dtype=torch.float32, device=DEV)
    ts_ = torch.zeros(capacity, dtype=torch.float32, device=DEV)
    tsh = torch.zeros((capacity, K, 3), dtype=torch.float32, device=DEV)
    tv[:N], to[:N], ts_[:N], tsh[:N] = _t(v), _t(o), _t(s), _t(sh)
    ws_bytes = B.ts_densify_workspace_bytes(N)
    ws = torch.empty(max(ws_bytes, 1), dtype=torch.uint8, device=DEV)
    d = torch.zeros(2, dtype=torch.int32, device=DEV)
    hc = (ctypes.c_uint32 * 2)() if host else None
    B.ts_densify_subdivide(tv, to, ts_, tsh, deg, N, capacity, _t(sel.astype(np.uint8)), ws,
                           ws_bytes, d, hc)
    torch.cuda.synchronize()
    return (tv.cpu().numpy(), to.cpu().numpy(), ts_.cpu().numpy(), tsh.cpu().numpy(),
            d.cpu().numpy().view(np.uint32))


def _soup(seed, N, deg):
    rng = np.random.default_rng(seed)
    v = rng.normal(0, 2, (N, 3, 3)).astype(np.float32)
    o = rng.uniform(0.01, 1, N).astype(np.float32)
    s = rng.uniform(0.3, 3, N).astype(np.float32)
    sh = rng.normal(0, 1, (N, (deg + 1) ** 2, 3)).astype(np.float32)
    return v, o, s, sh


@pytest.mark.parametrize("N,deg", [(1, 0), (300, 1), (777, 2), (5000, 3)])
def test_subdivide_bit_exact(N, deg):
    v, o, s, sh = _soup(11, N, deg)
    sel = np.random.default_rng(12).random(N) < 0.3
    sel[0] = True
    n = int(sel.sum())
    gv, go, gs, gsh, d = _subdivide(v, o, s, sh, deg, sel, N + 3 * n + 7)
    wv, wo, ws_, wsh = D.subdivide(v, o, s, sh, sel)
    M = N + 3 * n
    assert d[0] == M and d[1] == 0
    assert np.array_equal(gv[:M], wv) and np.array_equal(go[:M], wo)
    assert np.array_equal(gs[:M], ws_) and np.array_equal(gsh[:M], wsh)
    assert not gv[M:].any()                    # nothing past the new count


def test_subdivide_overflow_leaves_soup():
    v, o, s, sh = _soup(13, 400, 1)
    sel = np.random.default_rng(14).random(400) < 0.5
    cap = 400 + 3 * int(sel.sum()) - 1
    gv, go, gs, gsh, d = _subdivide(v, o, s, sh, 1, sel, cap, host=False)
    assert d[1] == 1 and np.array_equal(gv[:400], v) and not gv[400:].any()
    with pytest.raises(B.TSError) as e:
        _subdivide(v, o, s, sh, 1, sel, cap, host=True)
    assert e.value.code == B.TS_ECAPACITY


def test_densify_3m_soup():
    """The 3M-triangle, SH-3 soup: select 10% by inverse sigma (30% more
    triangles after the split), then subdivide; everything bit-exact."""
    sc = synth.workload_large().scene
    N = sc.n
    u = np.random.default_rng(21).random(N).astype(np.float32)
    n = _check_select(sc.o, sc.sigma, B.TS_DENSIFY_INV_SIGMA, 0.1 * N, u)
    sel = _select(sc.o, sc.sigma, B.TS_DENSIFY_INV_SIGMA, 0.1 * N, u)
    gv, go, gs, gsh, d = _subdivide(sc.v, sc.o, sc.sigma, sc.sh, 3, sel, N + 3 * n + 16)
    wv, wo, ws_, wsh = D.subdivide(sc.v, sc.o, sc.sigma, sc.sh, sel)
    M = N + 3 * int(sel.sum())
    assert d[0] == M
    assert np.array_equal(gv[:M], wv) and np.array_equal(go[:M], wo)
    assert np.array_equal(gs[:M], ws_) and np.array_equal(gsh[:M], wsh)


# Around the subdivision's chunk (512 triangles, 2048 above 2^18) and its
# batches of 256 selected ones, with every triangle, none, or some selected;
# degrees whose SH rows are (1, 3) and are not (0, 2) whole 16-byte vectors.
@pytest.mark.parametrize("N,deg,share", [(511, 3, 1.0), (512, 2, 1.0), (513, 1, 1.0),
                                         (4097, 0, 0.3), (6150, 3, 0.0), (257, 3, 1.0),
                                         (1 << 18, 1, 0.1), ((1 << 18) + 1, 1, 1.0),
                                         ((1 << 18) + 2047, 0, 0.3), ((1 << 18) + 2048, 2, 0.1)])
def test_subdivide_chunk_edges(N, deg, share):
    v, o, s, sh = _soup(31, N, deg)
    sel = np.random.default_rng(32).random(N) < share
    n = int(sel.sum())
    gv, go, gs, gsh, d = _subdivide(v, o, s, sh, deg, sel, N + 3 * n)
    wv, wo, ws_, wsh = D.subdivide(v, o, s, sh, sel)
    assert d[0] == N + 3 * n and d[1] == 0
    for got, want in ((gv, wv), (go, wo), (gs, ws_), (gsh, wsh)):
        assert np.array_equal(got, want)


def test_select_from_unaligned_arrays():
    """Slices that start 4 (and 1) bytes into an array: element-wise loads."""
    rng = np.random.default_rng(33)
    N = 5001
    o, u = (rng.random(N + 1).astype(np.float32) for _ in range(2))
    ws_bytes = B.ts_densify_workspace_bytes(N)
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
    sel = torch.zeros(N + 1, dtype=torch.uint8, device=DEV)
    B.ts_densify_select(_t(o)[1:], _t(o)[1:], N, B.TS_DENSIFY_OPACITY, 700.0, _t(u)[1:], sel[1:],
                        ws, ws_bytes)
    torch.cuda.synchronize()
    got = sel.cpu().numpy()
    assert got[0] == 0
    assert np.array_equal(got[1:].astype(bool), _select(o[1:], o[1:], B.TS_DENSIFY_OPACITY, 700.0,
                                                        u[1:]))


# Around the size from which the sums get launches of their own: the same
# decisions and children on both sides.
@pytest.mark.parametrize("N", [1 << 22, (1 << 22) + 1, 9_000_001])
def test_select_of_large_soups(N):
    rng = np.random.default_rng(34)
    o, u = (rng.random(N).astype(np.float32) for _ in range(2))
    assert _check_select(o, o, B.TS_DENSIFY_OPACITY, 0.1 * N, u) > 0


@pytest.mark.parametrize("N,share", [(1 << 22, 0.1), ((1 << 22) + 1, 0.1), ((1 << 22) + 2049, 0.0),
                                     (2305 * 2048 + 7, 0.01), (5_000_003, 0.3)])
def test_subdivide_of_large_soups(N, share):
    v, o, s, sh = _soup(35, N, 0)
    sel = np.random.default_rng(36).random(N) < share
    n = int(sel.sum())
    gv, go, gs, gsh, d = _subdivide(v, o, s, sh, 0, sel, N + 3 * n)
    wv, wo, ws_, wsh = D.subdivide(v, o, s, sh, sel)
    assert d[0] == N + 3 * n and d[1] == 0
    for got, want in ((gv, wv), (go, wo), (gs, ws_), (gsh, wsh)):
        assert np.array_equal(got, want)
    if n:   # one slot too few
        with pytest.raises(B.TSError) as e:
            _subdivide(v, o, s, sh, 0, sel, N + 3 * n - 1)
        assert e.value.code == B.TS_ECAPACITY


def test_densify_time_grows_with_the_soup():
    """Ten times the triangles take less than twenty times as long: no work that
    grows with the square of the soup."""
    def passes(n):
        cap = n + n // 8
        o, s, u = torch.rand(cap, device=DEV), torch.rand(cap, device=DEV), torch.rand(n, device=DEV)
        v, sh = torch.zeros(cap, 3, 3, device=DEV), torch.zeros(cap, 1, 3, device=DEV)
        sel = torch.empty(n, dtype=torch.uint8, device=DEV)
        nb = B.ts_densify_workspace_bytes(n)
        ws = torch.empty(nb, dtype=torch.uint8, device=DEV)
        d = torch.zeros(2, dtype=torch.int32, device=DEV)
        best = [1e9, 1e9]
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
            e[0].record()
            B.ts_densify_select(o, s, n, B.TS_DENSIFY_OPACITY, 0.03 * n, u, sel, ws, nb)
            e[1].record()
            B.ts_densify_subdivide(v, o, s, sh, 0, n, cap, sel, ws, nb, d)
            e[2].record()
            torch.cuda.synchronize()
            best = [min(best[k], e[k].elapsed_time(e[k + 1])) for k in range(2)]
        assert d.tolist()[1] == 0
        return best

    small, large = passes(10_000_000), passes(100_000_000)
    assert all(b < 20 * a for a, b in zip(small, large)), (small, large)
