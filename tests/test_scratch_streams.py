"""Memory that a call on a stream of its own writes, scratch and outputs: it comes
from that stream's pool, so that the allocator orders it against the work before
and after the call. Taken from the current stream's pool it may be memory that work
still queued there writes (the scratch of the call before, say), and scratch may be
handed out again while the call still runs."""
import contextlib

import pytest
import torch

import paper_2402_18008_amd as hg
from tests.gpu_util import announce, require_gpu


class _Handle:
    """A stream of another library: a raw handle and nothing else."""

    def __init__(self, raw):
        self.cuda_stream = raw


class _Noted(torch.Tensor):
    def record_stream(self, stream):
        self.recorded = getattr(self, "recorded", ()) + (stream.cuda_stream,)


class _Host:
    """Stands for torch's streams and allocator, and notes which stream was
    current at every allocation; library calls are noted and not made."""

    def __init__(self, monkeypatch):
        self.current, self.allocated, self.calls, self.waits = 1, [], [], []
        empty = torch.empty

        class Stream(_Handle):
            def record_event(this):
                return ("event", this.cuda_stream)

            def wait_event(this, event):
                self.waits.append((this.cuda_stream, event))

        def noted(*size, device=None, **kw):
            t = empty(*size, **kw).as_subclass(_Noted)
            self.allocated.append((t, self.current))
            return t

        @contextlib.contextmanager
        def use(stream):
            before, self.current = self.current, stream.cuda_stream
            yield
            self.current = before

        monkeypatch.setattr(torch, "empty", noted)
        monkeypatch.setattr(torch.cuda, "stream", use)
        monkeypatch.setattr(torch.cuda, "ExternalStream", lambda raw, device=None: _Handle(raw))
        monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: Stream(self.current))
        monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
        monkeypatch.setattr(hg, "_native", None)
        monkeypatch.setattr(hg, "_dev", lambda t, name, dtype=torch.float32: t)
        monkeypatch.setattr(hg._abi, "call", lambda name, *a: self.calls.append((name, a)))

    def of(self, ptr):
        """The allocation at an address, and the stream it is from."""
        (found,) = [x for x in self.allocated if x[0].data_ptr() == ptr]
        return found


@pytest.mark.parametrize("stream", [None, _Handle(7)])
def test_memory_is_from_the_pool_of_the_call(monkeypatch, stream):
    if hg._native is None:
        pytest.skip("libhomog.so not built")
    host = _Host(monkeypatch)
    want = 1 if stream is None else 7
    img, off, gl = torch.zeros((4, 128, 128)), torch.zeros((4, 4, 2)), torch.zeros(4)
    H, gu = torch.zeros((4, 9), dtype=torch.float64), torch.zeros((4, 4, 2))
    p, c = torch.zeros((8, 5)), torch.zeros((4, 50))
    o = torch.tensor([0, 50])
    for fn, args, scratch in (
            (hg.hg_photometric_fwd, (off, img, img), True),
            (hg.hg_photometric_bwd, (off, img, img, gl), True),
            (hg.hg_photometric_fwd_grad, (off, img, img), True),
            (hg.hg_warp_l1_fwd, (H, img, img), True), (hg.hg_warp_l1_bwd, (H, img, img, gl), True),
            (hg.hg_ransac, (c, 64, 3.0, 1), True), (hg.hg_ransac_plain, (c, 64, 3.0, 1), True),
            (hg.hg_ransac_noalloc, (c, 64, 3.0, 1), False), (hg.hg_solve4, (p, p), False),
            (hg.hg_solve_sk, ([0.0] * 8, p), False), (hg.hg_solve3_affine, (p[:6], p[:6]), False),
            (hg.hg_refit_ho, (c, o), False), (hg.hg_stream_copy, (img,), False),
            (hg.hg_stream_planes, (p, 9), False), (hg.hg_aca_fwd, (off, off), False),
            (hg.hg_aca_bwd, (off, off, H), False), (hg.hg_scale_grad, (gu, gl), False),
            (hg.hg_aca_rect_fwd, (off, 0.0, 0.0, 9.0, 1.0), False),
            (hg.hg_aca_rect_bwd, (off, H, 0.0, 0.0, 9.0, 1.0), False),
            (hg.hg_warp_store_fwd, (H, img), False), (hg.hg_l1_fwd, (img, img), False),
            (hg.hg_l1_bwd, (img, img, gl), False), (hg.hg_warp_bwd_from_grad, (H, img, img), False)):
        first = len(host.allocated)
        fn(*args, stream=stream)
        made = host.allocated[first:]
        assert made and all(s == want for _, s in made), fn.__name__
        if scratch:   # where it is passed: ahead of its size and the stream
            assert host.of(host.calls[-1][1][-3])[1] == want
            made = made[1:] if "ransac" in fn.__name__ else made[:-1]
        if stream is not None:   # outputs are used on the current stream
            assert all(t.recorded == (1,) for t, _ in made), fn.__name__


def test_refinement_waits_for_the_stream_that_made_its_buffers(monkeypatch):
    if hg._native is None:
        pytest.skip("libhomog.so not built")
    host = _Host(monkeypatch)
    img, off = torch.zeros((4, 128, 128)), torch.zeros((4, 4, 2))
    R = hg.Refine(img, img, off)
    R.run()
    assert not host.waits
    for _ in range(3):
        R.run(stream=_Handle(9))
    R.graph(stream=_Handle(7))
    graph = hg.Graph(0, R)
    graph.launch(_Handle(5))
    assert host.waits == [(s, ("event", 1)) for s in (9, 7, 5)]
    assert R.ws.recorded == R.loss.recorded == (9, 7, 5)
    graph.launch()
    assert len(host.waits) == 3


@pytest.mark.gpu
def test_calls_in_flight_on_two_streams():
    """Work queued on the current stream, one call behind it and one on another
    stream at once, of other inputs and the same shapes: each gives what it gives
    alone."""
    require_gpu()
    B, h, w = 8, 128, 128
    g = torch.Generator(device="cuda").manual_seed(3)
    sets = [[torch.randn((B, h, w), generator=g, device="cuda") for _ in range(2)]
            + [torch.rand((B, 4, 2), generator=g, device="cuda") * 8] for _ in range(2)]
    corr = [torch.rand((4, 700), generator=g, device="cuda") * 500 for _ in range(2)]
    gl = torch.rand(B, generator=g, device="cuda")
    load = torch.randn(1 << 28, generator=g, device="cuda")
    sink = torch.empty_like(load)
    side = torch.cuda.Stream()

    def refine(i, stream):
        img, tgt, off = sets[i]
        o = offs[i]
        r = hg.Refine(img, tgt, o, iters=3, step=5.0)
        r.run(stream=stream)
        return o, r.loss

    def refine_graph(i, stream):
        img, tgt, off = sets[i]
        r = hg.Refine(img, tgt, offs[i], iters=3, step=5.0)
        graph = r.graph(side)
        graph.launch(stream)
        return offs[i], r.loss, graph

    def ransac(i, stream):
        r = hg.hg_ransac(corr[i], 512, 3.0, 5, stream=stream)
        return r["best_H"], r["hyp_counts"], r["mask"]

    forms = {
        "fwd": lambda i, s: (hg.hg_photometric_fwd(sets[i][2], *sets[i][:2], stream=s),),
        "fwd_grad": lambda i, s: hg.hg_photometric_fwd_grad(sets[i][2], *sets[i][:2], stream=s),
        "bwd": lambda i, s: (hg.hg_photometric_bwd(sets[i][2], *sets[i][:2], gl, stream=s),),
        "refine": refine, "refine graph": refine_graph, "ransac": ransac,
    }
    for name, fn in forms.items():
        ref = []
        for i in range(2):
            offs = [s[2].clone() for s in sets]
            torch.cuda.synchronize()
            got = fn(i, None)
            torch.cuda.synchronize()
            ref.append([t.clone() for t in got if isinstance(t, torch.Tensor)])
        for _ in range(3):
            offs = [s[2].clone() for s in sets]
            torch.cuda.synchronize()
            announce(f"two streams: {name}")
            if name != "refine graph":   # making a graph waits for a stream
                sink.copy_(load)
            a = fn(0, None)
            b = fn(1, side)
            torch.cuda.synchronize()
            for got, want in ((a, ref[0]), (b, ref[1])):
                got = [t for t in got if isinstance(t, torch.Tensor)]
                assert all(torch.equal(x, y) for x, y in zip(got, want)), name


@pytest.mark.gpu
def test_streams_known_by_their_handle_alone():
    """An object with a cuda_stream handle and nothing else is a stream, for a
    batch that is cut and for one that is not; 0 is the default stream."""
    require_gpu()
    side = torch.cuda.Stream()
    for B in (8, 1024):
        g = torch.Generator(device="cuda").manual_seed(B)
        img, tgt = (torch.randn((B, 64, 128), generator=g, device="cuda") for _ in range(2))
        off = torch.rand((B, 4, 2), generator=g, device="cuda")
        ref = hg.hg_photometric_fwd(off, img, tgt)
        torch.cuda.synchronize()
        for raw in (side.cuda_stream, 0):
            announce(f"stream handle {raw != 0}, {B} patches")
            out = hg.hg_photometric_fwd(off, img, tgt, stream=_Handle(raw))
            o = off.clone()
            torch.cuda.synchronize()
            r = hg.Refine(img, tgt, o, iters=1)
            r.run(stream=_Handle(raw))
            graph = r.graph(stream=_Handle(raw))
            graph.launch(_Handle(raw))
            torch.cuda.synchronize()
            assert torch.equal(out, ref) and torch.isfinite(r.loss).all()


@pytest.mark.gpu
def test_native_path_takes_streams(monkeypatch):
    """Calls with a stream go through the native path, allocate from that stream's
    pool, leave the current stream as it was, and give what the Python path gives."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(12)
    B, h, w = 8, 96, 128
    img, tgt = (torch.randn((B, h, w), generator=g, device="cuda") for _ in range(2))
    off = torch.rand((B, 4, 2), generator=g, device="cuda") * 4
    gl = torch.rand(B, generator=g, device="cuda")
    q = torch.rand((8, 99), generator=g, device="cuda") * 500
    r = (0.0, 0.0, float(w - 1), 1.25)
    H = hg.hg_aca_rect_fwd(off, *r)
    gH = torch.randn((B, 9), generator=g, device="cuda", dtype=torch.float64)
    po = torch.tensor([0, 40, 99], device="cuda")
    side, here = torch.cuda.Stream(), torch.cuda.current_stream()
    torch.cuda.synchronize()
    pattern = [0.0, 0.0, 90.0, 0.0, 0.0, 80.0, 99.0, 95.0]
    calls = {
        "solve4": lambda **k: hg.hg_solve4(q, q + 1, "sks", **k),
        "solve4 kept": lambda **k: hg.hg_solve4(q, q + 1, H=torch.zeros((9, 99), device="cuda"), **k),
        "sk": lambda **k: hg.hg_solve_sk(pattern, q, **k)[:2],
        "affine": lambda **k: hg.hg_solve3_affine(q[:6], q[:6] + 1, **k),
        "ransac": lambda **k: tuple(hg.hg_ransac(q[:4], 64, 3.0, 1, **k).values()),
        "refit": lambda **k: hg.hg_refit_ho(q[:4], po, off_host=[0, 40, 99], **k),
        "refit native": lambda **k: hg.hg_refit_ho(q[:4], po, off_host=po.cpu(), **k),
        "aca": lambda **k: (hg.hg_aca_fwd(off, off + 1, **k),),
        "aca bwd": lambda **k: hg.hg_aca_bwd(off, off + 1, gH, **k),
        "fwd": lambda **k: (hg.hg_photometric_fwd(off, img, tgt, **k),),
        "bwd": lambda **k: (hg.hg_photometric_bwd(off, img, tgt, gl, **k),),
        "both": lambda **k: hg.hg_photometric_fwd_grad(off, img, tgt, **k),
        "scale": lambda **k: (hg.hg_scale_grad(off, gl, **k),),
        "warp": lambda **k: (hg.hg_warp_l1_fwd(H, img, tgt, **k),),
        "warp bwd": lambda **k: (hg.hg_warp_l1_bwd(H, img, tgt, gl, **k),),
        "rect": lambda **k: (hg.hg_aca_rect_fwd(off, *r, **k),),
        "rect bwd": lambda **k: (hg.hg_aca_rect_bwd(off, gH, *r, **k),),
    }
    for name, fn in calls.items():
        want = fn()
        torch.cuda.synchronize()
        for stream in (side, here, _Handle(side.cuda_stream), _Handle(0)):
            for native in (hg._native, None):
                monkeypatch.setattr(hg, "_native", native)
                announce(f"{name} on a stream, native {native is not None}")
                if native is not None and name != "refit":   # a list of offsets is not its own
                    monkeypatch.setattr(hg._abi, "call", lambda n, *a: pytest.fail(n))
                torch.cuda.synchronize()
                got = fn(stream=stream)
                monkeypatch.undo()
                assert torch.cuda.current_stream() == here
                torch.cuda.synchronize()
                assert all(torch.equal(x, y) for x, y in zip(got, want)), name
    # a block that the call used is handed out again to its own stream only
    blocks = torch.cuda.memory_snapshot
    n = 3 << 20
    out = hg.hg_solve4(torch.rand((8, n), device="cuda"), torch.rand((8, n), device="cuda"),
                       stream=side)[0]
    torch.cuda.synchronize()
    seg = [s for s in blocks() if s["address"] <= out.data_ptr() < s["address"] + s["total_size"]]
    assert [s["stream"] for s in seg] == [side.cuda_stream]
    assert hg._native.solve4(q, q, 0, None, None, object()) is None
    with pytest.raises(AttributeError):
        hg.hg_solve4(q, q, stream=object())
