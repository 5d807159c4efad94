"""Large batches whose planes do not start on cache lines take ordinary instead
of non-temporal accesses, and these and planes a multiple of 4 MB apart another
order of workgroups: the arithmetic is the same, so every plane and flag has the
bits of the same batch laid out on whole lines."""
import pytest
import torch

import synth
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def layout(planes, ld, offset):
    t = torch.full((planes.shape[0] * ld + offset,), float("nan"), device="cuda")
    t = t[offset:].view(planes.shape[0], ld)[:, :planes.shape[1]]
    t.copy_(planes)
    return t


@pytest.mark.parametrize("solver", ["aca", "sks", "sk", "affine"])
@pytest.mark.parametrize("n,pad,offset", [(2**18, 1, 0),       # the largest that stays non-temporal
                                          (2**18 + 1, 0, 0),   # the smallest that does not
                                          (2**18 + 511, 1, 8),  # planes on a half sector
                                          (300003, 13, 3),
                                          (2**18, 2**20 - 2**18, 0),       # 4 MB apart
                                          (2**18 + 1, 2**20 - 2**18 - 1, 0),
                                          (400000, 2**20 - 400000, 0),
                                          (2**20 + 5, 2**20 - 5, 0)])      # large groups
def test_misaligned_planes(solver, n, pad, offset):
    require_gpu()
    import paper_2402_18008_amd as hgpu
    src, dst = (torch.from_numpy(p).cuda() for p in synth.quadruples(n, 7)[:2])
    announce(f"{solver} n={n} pad={pad} offset={offset}")

    def solve(ld, off):
        guard = torch.full((9 * ld + off + 64,), 7.5, device="cuda")
        k = 6 if solver == "affine" else 9
        out = guard[off:off + k * ld].view(k, ld)[:, :n]
        d = layout(dst[:6] if solver == "affine" else dst, ld, off)
        if solver == "sk":
            H, f, _ = hgpu.hg_solve_sk(synth.PATTERN, d, H=out)
        elif solver == "affine":
            H, f = hgpu.hg_solve3_affine(layout(src[:6], ld, off), d, A=out)
        else:
            H, f = hgpu.hg_solve4(layout(src, ld, off), d, solver, H=out)
        H, f = H.clone(), f.clone()
        out.fill_(7.5)
        assert bool((guard == 7.5).all())   # nothing outside the planes was written
        return H, f

    H0, f0 = solve((n + 63) // 64 * 64, 0)
    H1, f1 = solve(n + pad, offset)
    assert torch.equal(H0.view(torch.int32), H1.view(torch.int32)) and torch.equal(f0, f1)
