"""Sign of grad_loss in the L1 gradient: of either sign, in every form against
float64 autograd. Bars as for other patches: gradient within 1e-4 norm-wise of the
oracle's, and 1e-5 between forms."""
import numpy as np
import pytest
import torch

import paper_2402_18008_amd as hgpu
import synth
from oracle import warp as ow
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu
GRAD_TOL = 1e-4


def rel(a, b):
    a, b = (np.asarray(v, np.float64).reshape(len(v), -1) for v in (a, b))
    return np.linalg.norm(a - b, axis=1) / np.maximum(np.linalg.norm(b, axis=1), 1e-300)


@pytest.mark.parametrize("size", [48, 128])   # one workgroup a patch, and cut into parts
def test_gradient_signs(size):
    require_gpu()
    B = 6
    pb = synth.patches(B, 42, size=size, sigma=3.0, max_shift=4, max_offset=6.0)
    off, img, tgt = pb.offsets, pb.img, pb.tgt
    gl = np.array([1.0, -1.0, 0.5, -2.0, -0.25, 3.0], np.float32)
    Lr, gr = ow.loss_and_grad(off, img, tgt)
    want = gr.numpy() * gl[:, None, None]
    o, i, t, g = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (off, img, tgt, gl))
    got = {}
    for form in (True, "recompute", False):
        announce(f"gradient signs {size} form={form}")
        x = o.clone().requires_grad_(True)
        loss = hgpu.photometric_loss(x, i, t, fused=form)
        (got[form],) = torch.autograd.grad(loss, x, g)
        assert np.allclose(loss.detach().cpu().numpy(), Lr.numpy(), rtol=1e-6, atol=0)
    # dL/dH of the fused kernel and of the stored-intermediate kernels
    rect = (0.0, 0.0, float(size - 1), 1.0)
    H = hgpu.hg_aca_rect_fwd(o, *rect)
    warped = hgpu.hg_warp_store_fwd(H, i)
    stored = hgpu.hg_warp_bwd_from_grad(H, i, hgpu.hg_l1_bwd(warped, t, g))
    got["stored"] = hgpu.hg_aca_rect_bwd(o, stored, *rect)
    for form, v in got.items():
        assert rel(v.cpu().numpy(), want).max() < GRAD_TOL, form
        assert rel(v.cpu().numpy(), got[True].cpu().numpy()).max() < 1e-5, form
