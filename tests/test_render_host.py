"""The host side of a view's forward, without a GPU: the library calls are
stand-ins that record their order, on CPU tensors."""
import pytest

torch = pytest.importorskip("torch")

from paper_2505_19175_amd import binding as B
from paper_2505_19175_amd import render, synth
from paper_2505_19175_amd.render import Rasterizer, ViewState


class _Host:
    """Stands in for the library and torch.cuda; `views` are the counts (M, N_v,
    huge tiles) of the binning calls to come, the last one repeated."""

    def __init__(self, monkeypatch, st, views):
        self.st, self.views, self.log, self.flags = st, list(views), [], []
        host = self

        class Event:
            def record(self):
                host.log.append("event")

            def synchronize(self):
                host.log.append("wait event")

        class Stream:
            cuda_stream = 0

            def synchronize(self):
                host.log.append("wait stream")

        class Cuda:
            @staticmethod
            def current_stream(*a):
                return Stream()

        Cuda.Event = Event

        class Torch:
            cuda = Cuda

            def __getattr__(self, name):
                return getattr(torch, name)

            @staticmethod
            def empty(*a, pin_memory=False, **k):
                return torch.empty(*a, **k)

        monkeypatch.setattr(render, "torch", Torch())
        monkeypatch.setattr(render, "_stream", lambda: 0)
        monkeypatch.setattr(B, "ts_project", lambda *a: None)
        monkeypatch.setattr(B, "ts_bin_sort", self._bin_sort)
        monkeypatch.setattr(B, "ts_render_forward", lambda *a: host.log.append("render"))
        alloc = st._alloc_lists
        monkeypatch.setattr(st, "_alloc_lists",
                            lambda c: (host.log.append("lists"), alloc(c))[1])

    def _bin_sort(self, proj, N, cam, ws, ws_bytes, bins, count, stream):
        assert bins.vals and ws   # the library refuses null lists
        self.log.append("bin")
        self.flags.append(bins.flags)
        M, nv, huge = self.views.pop(0) if len(self.views) > 1 else self.views[0]
        self.st.d_count.copy_(torch.tensor([M, nv, int(M > bins.capacity), huge]))
        if count is not None:
            count[0], count[1] = M, nv
            if M > bins.capacity:
                raise B.TSError(B.TS_ECAPACITY, "ts_bin_sort", "instances exceed capacity")


def _view(monkeypatch, capacity, views):
    st = ViewState(10, 64, 48, capacity, device="cpu")
    host = _Host(monkeypatch, st, views)
    ras, cam = Rasterizer(synth.Config(sh_degree=0), device="cpu"), synth.identity_camera(64, 48)
    return st, host, lambda **k: ras.forward(st, (None,) * 4, cam, **k)


def test_counts_are_waited_for_after_the_render(monkeypatch):
    st, host, forward = _view(monkeypatch, 100, [(70, 9, 0)])
    forward()
    assert host.log == ["bin", "event", "render", "wait event"]
    assert (st.M, st.N_v, st.capacity, st.segmented) == (70, 9, 100, False)


def test_lists_are_freed_after_the_render_that_reads_them(monkeypatch):
    """Lists too short: the render already enqueued reads them, on a stream that
    need not be the one they were allocated on, so it is waited for before they
    are freed."""
    st, host, forward = _view(monkeypatch, 100, [(400, 9, 0)])
    forward()
    first = host.log[:host.log.index("lists")]
    assert first[-1] == "wait stream" and first.index("render") < len(first) - 1
    assert host.log[len(first) + 1:] == ["bin", "event", "render", "wait event"]
    assert (st.M, st.N_v) == (400, 9) and st.capacity >= 400


@pytest.mark.parametrize("sync", [True, False])
def test_failed_growth_leaves_no_pointer_to_freed_lists(monkeypatch, sync):
    """Out of memory while the lists grow: the state holds null pointers (which
    the library refuses) until the next call has allocated its lists again."""
    st, host, forward = _view(monkeypatch, 100, [(400, 9, 0), (70, 9, 0)])
    arena = render._Arena

    def fail(*a):
        raise torch.OutOfMemoryError("out of memory")

    monkeypatch.setattr(render, "_Arena", fail)
    with pytest.raises(torch.OutOfMemoryError):
        forward()
    assert st.bins.vals is None and st.bins.blocks is None and st.bins.capacity == 0
    assert st.ws_ptr is None and st.ws_bytes == 0 and not hasattr(st, "vals")
    monkeypatch.setattr(render, "_Arena", arena)
    forward(sync=sync)
    assert st.capacity == st.bins.capacity == 100 and st.vals.numel() == 100
    assert st.bins.vals == st.vals.data_ptr() and st.ws_ptr == st.ws.data_ptr()


def test_huge_tiles_seen_in_short_lists(monkeypatch):
    """Lists too short and a tile already beyond one workgroup's sort in them:
    the repeated binning sorts such tiles over many workgroups."""
    st, host, forward = _view(monkeypatch, 5000, [(9000, 9, 1)])
    forward()
    assert host.flags == [0, B.TS_BINS_SEGMENTED_SORT]
    assert st.segmented and st.bins.flags == B.TS_BINS_SEGMENTED_SORT and st.M == 9000


def test_segmented_view_reads_the_counts_once(monkeypatch):
    """A state that sorts its huge tiles segment-wise has nothing to learn from
    their count: the binning's own read is the only one."""
    st, host, forward = _view(monkeypatch, 5000, [(4500, 9, 1)])
    forward()
    assert st.segmented
    counts = st.d_count

    class Counts:
        def copy_(self, t):
            counts.copy_(t)

        def __getitem__(self, i):
            raise AssertionError("read back")

    monkeypatch.setattr(st, "d_count", Counts())
    host.log.clear()
    forward()
    assert host.log == ["bin", "render"] and st.M == 4500
