"""Device buffers and the four-call pipeline for one view.

`ViewState` owns every buffer the C ABI needs for N triangles and one
camera (torch tensors are only storage); `Rasterizer` runs
ts_project -> ts_bin_sort -> ts_render_forward and ts_render_backward on the
current torch stream.
"""
from __future__ import annotations

import ctypes
import dataclasses
from typing import Optional

import torch

from . import binding as B


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


@dataclasses.dataclass
class Outputs:
    rgb: torch.Tensor      # [3,H,W]
    alpha: torch.Tensor    # [H,W]
    depth: torch.Tensor    # [H,W]
    T_final: torch.Tensor  # [H,W]
    last: torch.Tensor     # [H,W] int32 (uint32 bits)


class _Arena:
    """Named buffers in one allocation, each 256-byte aligned: a buffer's
    pointer is arithmetic, its tensor is made when somebody asks for it (with
    a view made per call, as by the autograd function, fifteen allocations
    took 0.1 ms of host time)."""

    def __init__(self, device, specs):
        self.specs, off = {}, 0
        for name, shape, dtype in specs:
            n = dtype.itemsize
            for x in shape:
                n *= x
            self.specs[name] = (off, n, shape, dtype)
            off += (n + 255) & ~255
        self.raw = torch.empty(off, dtype=torch.uint8, device=device)
        self.base = self.raw.data_ptr()

    def ptr(self, name) -> int:
        return self.base + self.specs[name][0]

    def tensor(self, name):
        off, n, shape, dtype = self.specs[name]
        return self.raw[off:off + n].view(dtype).view(shape)


class ViewState:
    """Projection state, tile lists and workspace of one view."""

    def __init__(self, N: int, width: int, height: int, capacity: int, device="cuda",
                 keys: bool = False):
        self.N, self.W, self.H = int(N), int(width), int(height)
        self.device = torch.device(device)
        self.num_tiles = B.ts_num_tiles(self.W, self.H)
        n = max(self.N, 1)
        f32, i32 = torch.float32, torch.int32
        self._state = _Arena(self.device, [
            ("g2d", (n, B.TS_G2D_STRIDE), f32), ("d_count", (4,), i32),
            ("rec", (n * B.ts_proj_record_bytes(),), torch.uint8), ("rect", (n, 4), torch.int16),
            ("depth_key", (n,), f32), ("ntiles", (n,), i32),
            ("cgrad", (n, B.TS_CGRAD_STRIDE), f32), ("ranges", (self.num_tiles, 2), i32),
            ("order", (max(self.num_tiles, 1),), i32)])
        # g2d zero once (every backward consumes its accumulations and clears
        # them), and the counters behind it
        st = self._state
        st.raw[:st.specs["rec"][0]].zero_()
        self.want_keys = keys
        self.segmented = False   # tiles of more than 4096 instances seen: segmented sort
        self._alloc_lists(capacity)
        self.proj = B.ts_proj(st.ptr("rec"), st.ptr("rect"), st.ptr("depth_key"),
                              st.ptr("ntiles"), st.ptr("g2d"), st.ptr("cgrad"))
        self.count = (ctypes.c_uint32 * 2)()
        self.M = None
        self.N_v = None

    def _alloc_lists(self, capacity: int):
        capacity = int(max(capacity, 1))
        for name in ("vals", "keys", "blocks", "ws"):
            self.__dict__.pop(name, None)
        if not self.want_keys:
            self.keys = None
        # the old lists go before the new ones come; should that allocation fail,
        # the library refuses the null pointers and the next call allocates again
        self._lists, self.bins, self.ws_ptr, self.ws_bytes = None, B.ts_bins(), None, 0
        ws_bytes = B.ts_bin_sort_workspace_bytes(self.N, capacity, self.num_tiles)
        specs = [("vals", (capacity,), torch.int32), ("blocks", (capacity,), torch.int16),
                 ("ws", (ws_bytes,), torch.uint8)]
        if self.want_keys:
            specs.append(("keys", (capacity,), torch.int64))
        ls = self._lists = _Arena(self.device, specs)
        self.capacity, self.ws_ptr, self.ws_bytes = capacity, ls.ptr("ws"), ws_bytes
        self.bins = B.ts_bins(ls.ptr("keys") if self.want_keys else None, ls.ptr("vals"),
                              self._state.ptr("ranges"), self._state.ptr("d_count"),
                              self.capacity, self._state.ptr("order"), ls.ptr("blocks"),
                              B.TS_BINS_SEGMENTED_SORT if self.segmented else 0)

    def _need_lists(self):
        if self._lists is None:
            self._alloc_lists(self.capacity)

    def _grow(self, M: int):
        """Lists for a view of M instances, which the present ones do not hold."""
        if M > 0xffffffff - 1024:   # the count saturates; the binning keeps 1024 slots free
            raise B.TSError(B.TS_ECAPACITY, "ViewState",
                            "the view has more instances than a list can hold")
        self._alloc_lists(min(int(M * 1.25) + 1024, 0xffffffff))

    def __getattr__(self, name):
        # a buffer's tensor (rec, rect, vals, ranges, ...), kept once made
        for part in ("_state", "_lists"):
            arena = self.__dict__.get(part)
            if arena is not None and name in arena.specs:
                t = arena.tensor(name)
                setattr(self, name, t)
                return t
        raise AttributeError(name)

    def outputs(self) -> Outputs:
        dev, H, W = self.device, self.H, self.W
        return Outputs(torch.empty((3, H, W), dtype=torch.float32, device=dev),
                       torch.empty((H, W), dtype=torch.float32, device=dev),
                       torch.empty((H, W), dtype=torch.float32, device=dev),
                       torch.empty((H, W), dtype=torch.float32, device=dev),
                       torch.empty((H, W), dtype=torch.int32, device=dev))


class PruneStats:
    """Pruning statistics over the views rendered with them (Sec. 3.2,
    "Pruning"): per triangle the largest blending weight T*o and the number
    of views that rendered it with more than one pixel."""

    def __init__(self, N: int, device="cuda"):
        n = max(N, 1)
        self.max_weight = torch.zeros(n, dtype=torch.float32, device=device)
        self.pixels = torch.zeros(n, dtype=torch.int32, device=device)   # per view, cleared
        self.views = torch.zeros(n, dtype=torch.int32, device=device)
        self.c = B.ts_prune_stats(self.max_weight.data_ptr(), self.pixels.data_ptr())

    def prune_mask(self, tau_prune: float, min_views: int = 2):
        """Triangles to prune: largest weight below tau_prune, or rendered with
        more than one pixel in fewer than min_views views."""
        return (self.max_weight < tau_prune) | (self.views < min_views)


class Rasterizer:
    """Runs the four library calls for one camera."""

    def __init__(self, cfg, device="cuda"):
        self.cfg = cfg
        self.ccfg = B.make_config(cfg)
        self.device = torch.device(device)

    def project(self, st: ViewState, scene_t, cam):
        return self._project(st, scene_t, cam, _stream())

    def _project(self, st: ViewState, scene_t, cam, stream: int):
        v, o, sigma, sh = scene_t
        ccam = B.make_camera(cam)
        B.ts_project(v, o, sigma, sh, st.N, ccam, self.ccfg, st.proj, stream)
        return ccam

    def bin_sort(self, st: ViewState, ccam, sync: bool = True):
        """With sync, read back (M, N_v) and grow the lists until they fit."""
        st._need_lists()
        while True:
            try:
                B.ts_bin_sort(st.proj, st.N, ccam, st.ws_ptr, st.ws_bytes, st.bins,
                              st.count if sync else None, _stream())
            except B.TSError as e:
                if e.code != B.TS_ECAPACITY:
                    raise
                st._grow(int(st.count[0]))
                continue
            break
        if sync:
            st.M, st.N_v = int(st.count[0]), int(st.count[1])
            if not st.segmented:   # one more read of the device
                self._seen_huge(st, int(st.d_count[3].item()))

    @staticmethod
    def _seen_huge(st: ViewState, huge: int):
        # a view with tiles of more than 4096 instances: later calls on the
        # same state sort those tiles with the segmented sort
        if not st.segmented and huge > 0:
            st.segmented = True
            st.bins.flags = B.TS_BINS_SEGMENTED_SORT

    def forward(self, st: ViewState, scene_t, cam, out: Optional[Outputs] = None,
                sync: bool = True, stats: Optional["PruneStats"] = None) -> Outputs:
        stream = _stream()
        ccam = self._project(st, scene_t, cam, stream)
        if out is None:
            out = st.outputs()
        st.ccam = ccam
        if stats is not None:
            # the statistics accumulate: only lists known to fit are rendered
            self.bin_sort(st, ccam, sync=sync)
            B.ts_render_forward_stats(st.proj, st.bins, ccam, self.ccfg, out.rgb, out.alpha,
                                      out.depth, out.T_final, out.last, stats.c, stream)
            B.ts_prune_count_views(stats.pixels, stats.views, st.N, stream)
            return out
        st._need_lists()
        while True:
            late = sync and not st.segmented
            if late:
                # the counts' copy is waited for after the render is enqueued,
                # so the GPU does not wait for the host in between; lists that
                # turn out too short (their clamped runs render safely) are
                # grown and the view rendered again (a 3M-triangle view
                # 0.457 -> 0.408 ms, reading the counts after the render 0.419;
                # small views 0.10 -> 0.05 ms)
                B.ts_bin_sort(st.proj, st.N, ccam, st.ws_ptr, st.ws_bytes, st.bins, None, stream)
                counts = torch.empty(4, dtype=torch.int32, pin_memory=True)
                counts.copy_(st.d_count, non_blocking=True)
                binned = torch.cuda.Event()
                binned.record()
            else:
                self.bin_sort(st, ccam, sync=sync)
            B.ts_render_forward(st.proj, st.bins, ccam, self.ccfg, out.rgb, out.alpha, out.depth,
                                out.T_final, out.last, stream)
            if not late:
                return out
            binned.synchronize()
            M, N_v, over, huge = (x & 0xffffffff for x in counts.tolist())
            if not over:
                st.M, st.N_v = M, N_v
                self._seen_huge(st, huge)
                return out
            # the render reads the lists, and this stream need not be theirs
            torch.cuda.current_stream().synchronize()
            self._seen_huge(st, huge)   # clamped runs: at least as long in the new lists
            st._grow(M)

    def backward(self, st: ViewState, scene_t, out: Outputs, dC, dA=None, dD=None, grads=None):
        v, o, sigma, sh = scene_t
        if grads is None:
            grads = (torch.empty_like(v), torch.empty_like(o), torch.empty_like(sigma),
                     torch.empty_like(sh))
        gv, go, gs, gsh = grads
        B.ts_render_backward(v, o, sigma, sh, st.N, st.proj, st.bins, st.ccam, self.ccfg, dC, dA,
                             dD, out.T_final, out.last, gv, go, gs, gsh, _stream())
        return grads


class StoredFragments:
    """The stored-fragment variant of one view (kept to measure the memory
    the recompute backward saves): a counting forward, then a forward that
    keeps every composited fragment (tile-list entry, alpha, transmittance
    in front of it: 12 bytes each), and a backward that reads them."""

    def __init__(self, ras: "Rasterizer", st: ViewState):
        self.ras, self.st = ras, st
        dev, H, W = st.device, st.H, st.W
        self.count = torch.empty((H, W), dtype=torch.int32, device=dev)
        self.offset = torch.empty((H, W), dtype=torch.int32, device=dev)
        self.total = torch.zeros(1, dtype=torch.int32, device=dev)
        self.ws_bytes = B.ts_fragment_workspace_bytes(W, H)
        self.ws = torch.empty(self.ws_bytes, dtype=torch.uint8, device=dev)
        self.entry = self.alpha = self.T = None
        self.F = 0

    def forward(self, scene_t, cam, out: Optional[Outputs] = None) -> Outputs:
        """Project, bin, count, size the fragment arrays (one host read of
        F), then the storing forward."""
        st, ras = self.st, self.ras
        ccam = ras.project(st, scene_t, cam)
        ras.bin_sort(st, ccam, sync=True)
        st.ccam = ccam
        if out is None:
            out = st.outputs()
        B.ts_render_forward_count(st.proj, st.bins, ccam, ras.ccfg, out.rgb, out.alpha, out.depth,
                                  out.T_final, out.last, self.count, self.offset, self.total,
                                  self.ws, self.ws_bytes, _stream())
        F = int(self.total.item())
        if self.entry is None or self.entry.numel() < max(F, 1):
            n = max(F, 1)
            self.entry = torch.empty(n, dtype=torch.int32, device=st.device)
            self.alpha = torch.empty(n, dtype=torch.float32, device=st.device)
            self.T = torch.empty(n, dtype=torch.float32, device=st.device)
        self.F = F
        B.ts_render_forward_store(st.proj, st.bins, ccam, ras.ccfg, out.rgb, out.alpha, out.depth,
                                  out.T_final, out.last, self.offset, self.entry, self.alpha,
                                  self.T, _stream())
        return out

    def backward(self, scene_t, out: Outputs, dC, dA=None, dD=None, grads=None):
        st, ras = self.st, self.ras
        v, o, sigma, sh = scene_t
        if grads is None:
            grads = (torch.empty_like(v), torch.empty_like(o), torch.empty_like(sigma),
                     torch.empty_like(sh))
        gv, go, gs, gsh = grads
        B.ts_raster_backward_stored(st.proj, st.bins, st.ccam, ras.ccfg, dC, dA, dD, out.T_final,
                                    out.last, self.count, self.offset, self.entry, self.alpha,
                                    self.T, _stream())
        B.ts_project_backward(v, sh, st.N, st.proj, st.ccam, ras.ccfg, gv, go, gs, gsh, _stream())
        return grads


def scene_to_device(scene, device="cuda"):
    """Float32 contiguous device copies (v, o, sigma, sh) of a synth.Scene."""
    return tuple(torch.as_tensor(a).to(device=device, dtype=torch.float32).contiguous()
                 for a in (scene.v, scene.o, scene.sigma, scene.sh))
