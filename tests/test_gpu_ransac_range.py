"""Many-pair scoring at the ends of float's range against the plain single-pair
form: the tile form splits coordinates and rows into bfloat16 pieces, which run out
of range before a float does, and then has to leave a pair to the float64 test."""
import numpy as np
import pytest
import torch

import paper_2402_18008_amd as hg
import synth
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s1,s2", [(5.2e35, 1.0), (1e35, 1.0), (1e33, 1.0), (1e24, 1.0), (1e17, 1.0),
                                   (1e15, 1.0), (1e-9, 1.0), (1e-15, 1.0), (1.0, 1e15), (1.0, 1e30),
                                   (1.0, 1e-12), (1e18, 1e18), (1e30, 1e-5), (1e-12, 1e12)])
def test_scales(s1, s2):
    """Source and target coordinates, and the threshold, scaled apart."""
    require_gpu()
    corr = synth.correspondences(900, 0.7, 21).corr.astype(np.float64)
    corr[:2] *= s1
    corr[2:] *= s2
    corr = corr.astype(np.float32)
    assert np.isfinite(corr).all()
    tau = float(np.float32(3.0 * s2))
    c = torch.from_numpy(corr).cuda()
    announce(f"scales {s1:g} {s2:g}")
    ref = hg.hg_ransac_plain(c, 200, tau, 5)
    off = torch.tensor([0, 900], device="cuda")
    br = hg.BatchedRansac(c, off, 200, tau, 5, hyp_counts=True).run()
    torch.cuda.synchronize()
    assert torch.equal(br.hyp_counts[0], ref["hyp_counts"])
    assert torch.equal(br.best_H[0], ref["best_H"]) and torch.equal(br.mask, ref["mask"])
    ad = hg.AdaptiveRansac(c, off, 200, tau, 5, confidence=1.0 - 1e-15).run()
    torch.cuda.synchronize()
    if int(ad.n_evaluated) == 200:
        assert int(ad.best_count) == int(ref["best_count"])


def test_extreme_points_among_ordinary_ones():
    """The largest and smallest floats as single coordinates of a pair."""
    require_gpu()
    base = synth.correspondences(600, 0.7, 22).corr
    top, low = np.finfo(np.float32).max, np.float32(1e-45)
    for name, values in (("largest", (top, -top)), ("smallest", (low, -low)), ("zero", (0.0, -0.0)),
                         ("both", (top, low))):
        for row in range(4):
            corr = base.copy()
            corr[row, 40], corr[row, 333] = values
            c = torch.from_numpy(corr).cuda()
            announce(f"{name} coordinates in row {row}")
            ref = hg.hg_ransac_plain(c, 130, 3.0, 6)
            off = torch.tensor([0, 600], device="cuda")
            br = hg.BatchedRansac(c, off, 130, 3.0, 6, hyp_counts=True).run()
            torch.cuda.synchronize()
            assert torch.equal(br.hyp_counts[0], ref["hyp_counts"]), (name, row)
            assert torch.equal(br.mask, ref["mask"])
