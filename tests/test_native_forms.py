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
