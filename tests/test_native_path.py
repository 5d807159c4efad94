"""The native call path against the Python checks and ctypes, over the forms the
calls accept and refuse: the same results bit for bit (the same kernels run), and
the same errors."""
import numpy as np
import pytest
import torch

import paper_2402_18008_amd as hg
from tests.gpu_util import announce, require_gpu


def _both(fn, monkeypatch):
    """What fn gives with the native path and without it: a value or an error."""
    got = []
    for native in (hg._native, None):
        monkeypatch.setattr(hg, "_native", native)
        try:
            got.append(("value", fn()))
        except Exception as e:   # noqa: BLE001 - the error itself is compared
            got.append(("error", (type(e), str(e))))
        monkeypatch.undo()
    return got


def _equal(a, b):
    if isinstance(a, torch.Tensor):
        return (isinstance(b, torch.Tensor) and a.dtype == b.dtype and a.shape == b.shape
                and a.stride() == b.stride() and a.device == b.device
                and a.requires_grad == b.requires_grad and torch.equal(a, b))
    if isinstance(a, np.ndarray):
        return a.dtype == b.dtype and np.array_equal(a, b)
    if isinstance(a, dict):
        return list(a) == list(b) and all(_equal(a[k], b[k]) for k in a)
    if isinstance(a, tuple):
        return len(a) == len(b) and all(_equal(x, y) for x, y in zip(a, b))
    return a is b or a == b


def _same(name, fn, monkeypatch):
    announce(f"native path: {name}")
    (k1, v1), (k2, v2) = _both(fn, monkeypatch)
    if torch.cuda.is_available():
        torch.cuda.synchronize()
    assert k1 == k2, (name, v1, v2)
    assert v1 == v2 if k1 == "error" else _equal(v1, v2), (name, v1, v2)
    return k1


def test_native_is_built_and_declines_cpu_tensors(monkeypatch):
    if hg._native is None:
        pytest.skip("_native.so not built")
    x = torch.zeros((8, 4))
    assert hg._native.solve4(x, x, 0, None, None, None) is None
    c = torch.zeros((4, 9))
    img, off = torch.zeros((2, 8, 8)), torch.zeros((2, 4, 2))
    for name, fn in {
        "solve4": lambda: hg.hg_solve4(x, x),
        "sk": lambda: hg.hg_solve_sk([0.0] * 8, x),
        "affine": lambda: hg.hg_solve3_affine(x[:6], x[:6]),
        "ransac": lambda: hg.hg_ransac(c, 8, 3.0, 1),
        "refit": lambda: hg.hg_refit_ho(c, torch.zeros(2, dtype=torch.int64), off_host=[0, 9]),
        "aca_fwd": lambda: hg.hg_aca_fwd(x, x),
        "photometric": lambda: hg.hg_photometric_fwd(off, img, img),
        "scale_grad": lambda: hg.hg_scale_grad(off, torch.zeros(2)),
        "rect": lambda: hg.hg_aca_rect_fwd(off, 0.0, 0.0, 7.0, 1.0),
    }.items():
        assert _same(name, fn, monkeypatch) == "error"
    with pytest.raises(TypeError):
        hg._native.solve4(x, x)


@pytest.mark.gpu
def test_solvers(monkeypatch):
    require_gpu()
    assert hg._native is not None
    g = torch.Generator(device="cuda").manual_seed(2)

    def planes(k, n, ld=None):
        t = torch.rand((k, ld or n), generator=g, device="cuda") * 600
        return t[:, :n]
    for n, ld in ((1, 1), (5, 5), (1000, 1000), (777, 1024), (64, 67)):
        s, d = planes(8, n, ld), planes(8, n, ld)
        H, f = torch.empty((9, ld), device="cuda")[:, :n], torch.empty(n, dtype=torch.uint8,
                                                                       device="cuda")
        for m in ("aca", "SKS", hg.HG_ACA, hg.HG_SKS, 7, "lu"):
            _same(f"solve4 {n} {m}", lambda: hg.hg_solve4(s, d, m), monkeypatch)
        _same("solve4 kept", lambda: hg.hg_solve4(s, d, "aca", H, f), monkeypatch)
        _same("affine", lambda: hg.hg_solve3_affine(s[:6], d[:6]), monkeypatch)
        for obj in ((0.0, 0.0, 90.0, 0.0, 0.0, 80.0, 99.0, 95.0), np.arange(8.0) ** 2,
                    [1, 2, 3], (float("nan"),) * 8):
            _same("sk", lambda: hg.hg_solve_sk(obj, d), monkeypatch)
        _same("other stride", lambda: hg.hg_solve4(s, planes(8, n, ld + 3)), monkeypatch)
    s, d = planes(8, 50), planes(8, 50)
    for a, b in ((s.double(), d.double()), (s[:7], d[:7]), (s.T, d.T), (s[:, ::2], d[:, ::2]),
                 (s[:, :0], d[:, :0]), (s.cpu(), d), (s.numpy if False else 3, d)):
        _same("refused or empty", lambda: hg.hg_solve4(a, b), monkeypatch)
    H, f = hg.hg_solve4(s, d, H=(h := torch.empty((9, 50), device="cuda")))
    assert H is h
    side = torch.cuda.Stream()
    _same("stream", lambda: hg.hg_solve4(s, d, stream=side), monkeypatch)


@pytest.mark.gpu
def test_ransac_and_refit(monkeypatch):
    require_gpu()
    import synth
    cb = synth.correspondence_batch(5, 7, n_min=40, n_max=300)
    corr, off = torch.from_numpy(cb.corr).cuda(), torch.from_numpy(cb.off).cuda()
    one = corr[:, :200]
    for nh in (1, 100, 3000, 0, -1, 1 << 40):
        for hc in (True, False):
            _same(f"ransac {nh}", lambda: hg.hg_ransac(one, nh, 3.0, 5, hc), monkeypatch)
    _same("plain", lambda: hg.hg_ransac_plain(one, 64, 3.0, 5), monkeypatch)
    for seed in (0, -1, (1 << 64) + 3, 1 << 63):
        _same("seed", lambda: hg.hg_ransac(one, 64, 3, seed), monkeypatch)
    for th in (0.0, float("nan"), 1e-40, "x"):
        _same("threshold", lambda: hg.hg_ransac(one, 64, th, 5), monkeypatch)
    _same("3 points", lambda: hg.hg_ransac(corr[:, :3], 64, 3.0, 5), monkeypatch)
    small = torch.empty(16, dtype=torch.uint8, device="cuda")
    _same("workspace", lambda: hg.hg_ransac(one, 64, 3.0, 5, ws=small), monkeypatch)
    mask = torch.from_numpy(cb.inlier.astype(np.uint8)).cuda()
    host = torch.from_numpy(cb.off)
    for oh in (cb.off, host, list(cb.off), cb.off.astype(np.int32), cb.off[:-1], cb.off[::-1],
               cb.off + 1, -cb.off, None):
        _same("refit offsets", lambda: hg.hg_refit_ho(corr, off, mask, off_host=oh), monkeypatch)
    _same("refit all", lambda: hg.hg_refit_ho(corr, off, off_host=cb.off), monkeypatch)
    _same("refit mask", lambda: hg.hg_refit_ho(corr, off, mask[:9], off_host=cb.off), monkeypatch)
    _same("refit mask type", lambda: hg.hg_refit_ho(corr, off, mask.bool(), off_host=cb.off),
          monkeypatch)
    H = torch.empty((5, 9), device="cuda")
    _same("refit kept", lambda: hg.hg_refit_ho(corr, off, mask, H, off_host=cb.off), monkeypatch)
    _same("refit short", lambda: hg.hg_refit_ho(corr, off, mask, H[:2], off_host=cb.off),
          monkeypatch)


@pytest.mark.gpu
def test_differentiable(monkeypatch):
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(4)
    for B, h, w in ((1, 2, 2), (3, 37, 53), (2, 128, 128), (0, 8, 8)):
        img, tgt = (torch.randn((B, h, w), generator=g, device="cuda") for _ in range(2))
        off = torch.rand((B, 4, 2), generator=g, device="cuda")
        gl = torch.rand(B, generator=g, device="cuda")
        args = (off, img, tgt)
        _same("fwd", lambda: hg.hg_photometric_fwd(*args), monkeypatch)
        _same("bwd", lambda: hg.hg_photometric_bwd(*args, gl), monkeypatch)
        _same("both", lambda: hg.hg_photometric_fwd_grad(*args), monkeypatch)
        _same("scale", lambda: hg.hg_scale_grad(off, gl), monkeypatch)
        _same("scale rows", lambda: hg.hg_scale_grad(off.reshape(B, 8), gl), monkeypatch)
        r = (0.0, 0.0, float(w - 1), 1.25)
        H = hg.hg_aca_rect_fwd(off, *r)
        gH = torch.randn((B, 9), generator=g, device="cuda", dtype=torch.float64)
        _same("rect", lambda: hg.hg_aca_rect_fwd(off, *r), monkeypatch)
        _same("rect int", lambda: hg.hg_aca_rect_fwd(off, 0, 0, w - 1, 1), monkeypatch)
        _same("rect bad", lambda: hg.hg_aca_rect_fwd(off, 0.0, 0.0, -1.0, 1.0), monkeypatch)
        _same("rect bwd", lambda: hg.hg_aca_rect_bwd(off, gH, *r), monkeypatch)
        _same("warp", lambda: hg.hg_warp_l1_fwd(H, img, tgt), monkeypatch)
        _same("warp bwd", lambda: hg.hg_warp_l1_bwd(H, img, tgt, gl), monkeypatch)
        for s, d in ((off, off + 1), (off.reshape(B, 8), off.reshape(B, 8) + 2)):
            _same("aca", lambda: hg.hg_aca_fwd(s, d), monkeypatch)
            for want in ((True, True), (True, False), (False, True), (False, False)):
                _same("aca bwd", lambda: hg.hg_aca_bwd(s, d, gH, *want), monkeypatch)
        _same("strided", lambda: hg.hg_photometric_fwd(off, img.transpose(1, 2), tgt), monkeypatch)
        _same("double", lambda: hg.hg_photometric_fwd(off.double(), img, tgt), monkeypatch)
        o = off.clone().requires_grad_(True)
        for form in (True, False, "recompute"):
            def step():
                loss = hg.photometric_loss(o, img, tgt, fused=form)
                return loss.detach(), *torch.autograd.grad(loss, o, gl)
            if h > 2:
                _same(f"autograd {form}", step, monkeypatch)
        _same("needs grad", lambda: hg.hg_photometric_fwd(o, img, tgt), monkeypatch)
