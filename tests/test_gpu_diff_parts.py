"""Batches whose patches are cut into parts over several workgroups against the
same calls without a workspace (one workgroup per patch).

Both forms take the same float terms per pixel and differ in the order of their
float partial sums (at most 16 terms each) and of the double sums above them: the
loss, a mean of non-negative terms, within 1e-6 relative, and the gradient, a
sum with cancellation, within 1e-5 norm-wise per patch, the bounds between any
two launch shapes of these kernels. A refinement of n steps moves its offsets by
n gradients of that accuracy."""
import ctypes as C

import numpy as np
import pytest
import torch

from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu
EINVAL, EWORKSPACE = -1, -3

# (patches, height, width): widths that divide 256 and that do not; the smallest
# patch that is cut and its neighbours; a last part of one row, of one pixel and
# of a whole number of iterations; one patch over many parts; the largest batch
# of a first round, and the batches of a part-filled first or second round
SHAPES = [(1, 64, 113), (1, 57, 128), (3, 99, 83), (2, 113, 145), (1, 512, 512), (128, 128, 128),
          (127, 97, 131), (5, 8193, 1), (7, 2, 4099), (129, 145, 160), (257, 101, 239)]


def _inputs(B, h, w, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    img = torch.randn((B, h, w), generator=g, device="cuda")
    tgt = torch.randn((B, h, w), generator=g, device="cuda")
    o = 0.1 * min(h, w)
    off = (torch.rand((B, 4, 2), generator=g, device="cuda") * 2 - 1) * o
    gl = torch.rand(B, generator=g, device="cuda") + 0.5
    return img, tgt, off, gl


def _rel(a, b):
    a, b = (t.double().reshape(t.shape[0], -1) for t in (a, b))
    return float(((a - b).norm(dim=1) / b.norm(dim=1).clamp(min=1e-300)).max())


@pytest.mark.parametrize("B,h,w", SHAPES)
def test_parts_equal_whole_patches(B, h, w):
    require_gpu()
    from paper_2402_18008_amd import _abi
    L = _abi.lib()
    img, tgt, off, gl = _inputs(B, h, w, h * w + B)
    st = torch.cuda.current_stream().cuda_stream
    n = L.hg_photometric_ws_bytes(B, h, w)
    assert n > 0, "this shape is meant to be cut"
    ws = torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN parts
    H = torch.randn((B, 9), dtype=torch.float64, device="cuda") * 1e-3
    H += torch.eye(3, dtype=torch.float64, device="cuda").reshape(1, 9)
    res = []
    for p, nb in ((None, 0), (ws.data_ptr(), n)):
        announce(f"photometric {B} x {h} x {w} {'cut' if p else 'whole'}")
        out = [torch.full((B,), -1.0, device="cuda") for _ in range(3)]
        g = [torch.full((B, 4, 2), 9.0, device="cuda") for _ in range(2)]
        gH = torch.full((B, 9), 9.0, dtype=torch.float64, device="cuda")
        i, t = img.data_ptr(), tgt.data_ptr()
        calls = []
        if h >= 2 and w >= 2:
            calls += [L.hg_photometric_fwd_ws(off.data_ptr(), i, t, B, h, w, out[0].data_ptr(), p,
                                              nb, st),
                      L.hg_photometric_bwd_ws(off.data_ptr(), i, t, gl.data_ptr(), B, h, w,
                                              g[0].data_ptr(), p, nb, st),
                      L.hg_photometric_fwd_grad_ws(off.data_ptr(), i, t, B, h, w,
                                                   out[1].data_ptr(), g[1].data_ptr(), p, nb, st)]
        calls += [L.hg_warp_l1_fwd_ws(H.data_ptr(), i, t, B, h, w, out[2].data_ptr(), p, nb, st),
                  L.hg_warp_l1_bwd_ws(H.data_ptr(), i, t, gl.data_ptr(), B, h, w, gH.data_ptr(),
                                      p, nb, st)]
        torch.cuda.synchronize()
        assert not any(calls), calls
        res.append((out, g, gH))
    (lw, gw, hw), (lp, gp, hp) = res
    for a, b in zip(lp, lw):
        assert torch.allclose(a, b, rtol=1e-6, atol=0)
    for a, b in zip(gp, gw):
        assert _rel(a, b) < 1e-5
    assert _rel(hp, hw) < 1e-5


@pytest.mark.parametrize("iters,with_loss", [(0, True), (1, True), (2, True), (5, True), (1, False),
                                             (4, False)])
def test_refine_parts(iters, with_loss):
    """The cut refinement against the whole one, eager and replayed from a graph
    (the offsets reset by eager work between replays)."""
    require_gpu()
    from paper_2402_18008_amd import _abi
    import paper_2402_18008_amd as hg
    B, h, w = 6, 96, 112
    img, tgt, off, _ = _inputs(B, h, w, 11)
    announce(f"refine {B} x {h} x {w} iters={iters} loss={with_loss}")
    a, b = off.clone(), off.clone()
    R = hg.Refine(img, tgt, a, iters=iters, step=5.0, with_loss=with_loss)
    assert R.ws is not None
    R.ws.fill_(0xFF)
    R.run()
    loss = torch.empty(B, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    assert _abi.lib().hg_refine(img.data_ptr(), tgt.data_ptr(), B, h, w, iters, 5.0, b.data_ptr(),
                                loss.data_ptr() if with_loss else None, st) == 0
    torch.cuda.synchronize()
    moved = (b - off).abs().max()
    assert (a - b).abs().max() <= 1e-5 * moved * max(iters, 1)
    if with_loss:
        assert torch.allclose(R.loss, loss, rtol=1e-5, atol=0)
    ref, ref_loss = a.clone(), None if R.loss is None else R.loss.clone()
    G = R.graph()
    for _ in range(3):
        a.copy_(off)
        R.ws.fill_(0xFF)
        torch.cuda.synchronize()
        G.launch()
        torch.cuda.synchronize()
        assert torch.equal(a, ref)
        if with_loss:
            assert torch.equal(R.loss, ref_loss)
    G.close()


def test_workspace_limits():
    """A workspace one byte short is refused; exactly enough is accepted (the bytes
    past it stay untouched); misaligned is refused; shapes that are not cut ask for
    nothing and ignore what they are given."""
    require_gpu()
    from paper_2402_18008_amd import _abi
    L = _abi.lib()
    B, h, w = 4, 128, 128
    img, tgt, off, _ = _inputs(B, h, w, 3)
    loss = torch.empty(B, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    n = L.hg_photometric_ws_bytes(B, h, w)
    ws = torch.full((n + 64,), 0x5A, dtype=torch.uint8, device="cuda")

    def call(p, nb):
        return L.hg_photometric_fwd_ws(off.data_ptr(), img.data_ptr(), tgt.data_ptr(), B, h, w,
                                       loss.data_ptr(), p, nb, st)
    assert call(ws.data_ptr(), n - 1) == EWORKSPACE
    assert call(ws.data_ptr() + 8, n + 16) == EINVAL
    assert call(ws.data_ptr(), n) == 0
    torch.cuda.synchronize()
    assert bool((ws[n:] == 0x5A).all())
    assert L.hg_photometric_ws_bytes(4, 16, 16) == 0 and L.hg_refine_ws_bytes(4, 16, 16) == 0
    assert L.hg_photometric_ws_bytes(4096, 128, 128) == 0
    # 10 idle iterations (of 11), a full round, a third round
    for b, hh, ww in ((192, 200, 200), (256, 256, 256), (513, 320, 320)):
        assert L.hg_photometric_ws_bytes(b, hh, ww) == 0
    assert L.hg_photometric_ws_bytes(0, 128, 128) == 0
    assert L.hg_photometric_ws_bytes(1, 1 << 20, 1 << 20) == 0
    nr = L.hg_refine_ws_bytes(B, h, w)
    assert L.hg_refine_ws(img.data_ptr(), tgt.data_ptr(), B, h, w, 2, 1.0, off.data_ptr(), None,
                          ws.data_ptr(), nr - 1, st) == EWORKSPACE
    out = C.c_void_p()
    assert L.hg_refine_graph_create_ws(img.data_ptr(), tgt.data_ptr(), B, h, w, 2, 1.0,
                                       off.data_ptr(), None, ws.data_ptr(), nr - 1, st,
                                       C.byref(out)) == EWORKSPACE and not out.value


def test_python_calls_on_another_stream():
    """The binding's workspace under a stream argument: the result equals the
    current stream's, with the workspace's memory wanted again at once."""
    require_gpu()
    import paper_2402_18008_amd as hg
    B, h, w = 8, 128, 128
    img, tgt, off, _ = _inputs(B, h, w, 5)
    ref = hg.hg_photometric_fwd(off, img, tgt)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    announce("photometric on a side stream")
    outs = []
    for _ in range(20):
        outs.append(hg.hg_photometric_fwd(off, img, tgt, stream=side))
        torch.full((B * 80 * 16,), 0xFF, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    assert all(torch.equal(o, ref) for o in outs)
    assert np.isfinite(ref.cpu().numpy()).all()
