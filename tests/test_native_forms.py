"""Forms of the arguments that the native call path leaves to the Python code, and
calls that it must not change: the same results and errors with it and without."""
import numpy as np
import pytest
import torch

import paper_2402_18008_amd as hg
from tests.gpu_util import announce, require_gpu
from tests.test_native_path import _same


@pytest.mark.gpu
def test_truthy_flags(monkeypatch):
    """Any truthy want_src / want_dst asks for the gradient."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(6)
    s, d = (torch.rand((5, 8), generator=g, device="cuda") * 100 for _ in range(2))
    gH = torch.randn((5, 9), generator=g, device="cuda", dtype=torch.float64)
    for want in ((1, True), (True, 1), (np.True_, True), (0, "yes"), (None, 2.0), (False, 1)):
        assert _same(f"aca bwd {want}", lambda: hg.hg_aca_bwd(s, d, gH, *want),
                     monkeypatch) == "value"
        got = hg.hg_aca_bwd(s, d, gH, *want)
        assert [x is not None for x in got] == [bool(w) for w in want]
    for src in (s, s.clone().requires_grad_(True)):
        H = hg.ACAGeneral.apply(src, d.clone().requires_grad_(True))
        assert torch.isfinite(H).all()


def test_pattern_from_an_iterator(monkeypatch):
    """The pattern reaches the library whole when it can be read only once and the
    native path leaves the call to the Python code."""
    obj = [0.0, 0.0, 90.0, 0.0, 0.0, 80.0, 99.0, 95.0]
    seen = []
    monkeypatch.setattr(hg, "_dev", lambda t, name, dtype=torch.float32: t)
    monkeypatch.setattr(hg, "_stream", lambda stream=None: 0)
    monkeypatch.setattr(hg._abi, "call", lambda name, o, *a: seen.append(list(o)))
    for form in (obj, iter(obj), (v for v in obj), np.array(obj)):
        hg.hg_solve_sk(form, torch.zeros((8, 3)))
    assert seen == [obj] * 4
    with pytest.raises(IndexError):
        hg.hg_solve_sk(obj + [1.0], torch.zeros((8, 3)))


@pytest.mark.gpu
def test_pattern_from_an_iterator_on_a_stream():
    require_gpu()
    obj = [0.0, 0.0, 90.0, 0.0, 0.0, 80.0, 99.0, 95.0]
    g = torch.Generator(device="cuda").manual_seed(7)
    dst = torch.rand((8, 50), generator=g, device="cuda") * 500
    H, flags, frame = hg.hg_solve_sk(obj, dst)
    torch.cuda.synchronize()
    announce("pattern from an iterator, on a stream")
    H2, flags2, frame2 = hg.hg_solve_sk(iter(obj), dst, stream=torch.cuda.Stream())
    torch.cuda.synchronize()
    assert torch.equal(H, H2) and torch.equal(flags, flags2) and np.array_equal(frame, frame2)


@pytest.mark.gpu
def test_tensors_without_storage(monkeypatch):
    """A sparse tensor where a buffer is expected has no pointer: an error, raised
    with the interpreter's lock held."""
    require_gpu()
    g = torch.Generator(device="cuda").manual_seed(8)
    s, d = (torch.rand((8, 50), generator=g, device="cuda") * 100 for _ in range(2))
    flags = torch.zeros(50, dtype=torch.uint8, device="cuda").to_sparse()
    ws = torch.ones(1 << 16, dtype=torch.uint8, device="cuda").to_sparse()
    for name, fn in {
        "solve4": lambda: hg.hg_solve4(s, d, flags=flags),
        "affine": lambda: hg.hg_solve3_affine(s[:6], d[:6], flags=flags),
        "sk": lambda: hg.hg_solve_sk([0.0, 0.0, 9.0, 0.0, 0.0, 8.0, 9.0, 9.0], d, flags=flags),
        "ransac": lambda: hg.hg_ransac(s[:4], 64, 3.0, 1, ws=ws),
        "sparse planes": lambda: hg.hg_solve4(s.to_sparse(), d),
    }.items():
        assert _same(name, fn, monkeypatch) == "error", name


@pytest.mark.parametrize("method", [2**70, -2**70, 2**63, -2**63, 2**31, -1, 2, True])
def test_any_integer_as_method(monkeypatch, method):
    """A number that is no method, or fits no machine integer, is left to the Python
    code without an error of the native path's own."""
    x = torch.zeros((8, 4))
    if hg._native is None:
        pytest.skip("_native.so not built")
    assert hg._native.solve4(x, x, method, None, None, None) is None
    assert _same("method", lambda: hg.hg_solve4(x, x, method), monkeypatch) == "error"


@pytest.mark.gpu
def test_number_of_hypotheses(monkeypatch):
    """A fraction is no size of a counts tensor; without counts it is cut to an
    integer, and integers of other types are taken."""
    require_gpu()
    corr = torch.rand((4, 50), generator=torch.Generator(device="cuda").manual_seed(9),
                      device="cuda") * 500
    for n, counts, kind in ((10.5, True, "error"), (10.0, True, "error"), ("10", True, "error"),
                            (10.5, False, "value"), (np.int64(10), True, "value"),
                            (10, True, "value")):
        for fn in (hg.hg_ransac, hg.hg_ransac_plain):
            assert _same(f"{n!r} hypotheses", lambda: fn(corr, n, 3.0, 1, counts),
                         monkeypatch) == kind, n
