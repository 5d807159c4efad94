"""The refit's launch shapes against the oracle: 512-thread workgroups (large
pairs), 256 threads, and 256 threads held to 128 registers (many pairs), with
pairs around the points one batch of a workgroup covers (8 per thread: 2048 and
4096), a far reference point (moments summed twice) and pairs without enough
points. Bar as for every refit: 1e-6 after normalisation, counts exact."""
import numpy as np
import pytest

import synth
from tests.gpu_util import announce, require_gpu
from tests.test_gpu_refit import check, gpu_refit

pytestmark = pytest.mark.gpu

EDGES = [4095, 4096, 4097, 8193, 3, 2047, 2048, 2049, 1, 255, 257, 5000]


@pytest.mark.parametrize("pairs,sizes", [(12, EDGES), (512, [1536]), (768, [40, 513, 2048, 2049]),
                                         (769, [40, 257, 2048, 2049]), (513, [1600])])
def test_launch_shapes(pairs, sizes):
    require_gpu()
    n = [sizes[k % len(sizes)] for k in range(pairs)]
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    src = synth.correspondence_batch(8, 17, n_min=int(max(n)), n_max=int(max(n)))
    corr = np.empty((4, off[-1]), np.float32)
    mask = np.empty(off[-1], np.uint8)
    for p in range(pairs):
        q, a, b = p % 8, off[p], off[p + 1]
        s = src.off[q]
        corr[:, a:b] = src.corr[:, s:s + b - a]
        mask[a:b] = src.inlier[s:s + b - a]
        if p % 5 == 2:   # a first point far from the rest, not selected
            corr[:, a] = 3.0e4
            mask[a] = 0
    announce(f"refit_ho {pairs} pairs, {off[-1] / pairs:.0f} points on average")
    Hg, ug, fg = gpu_refit(corr, off, mask)
    check(corr, off, mask, Hg, ug, fg, pairs=range(0, pairs, max(1, pairs // 24)), label=f"{pairs}")
