"""The tile form of the scoring (many pairs) against the plain single-pair form.

A batch of one pair draws the samples of the plain call with the same seed, and
both give the float64 test's decision for every (hypothesis, point): counts, best
hypothesis and mask are equal, whatever the inputs."""
import numpy as np
import pytest
import torch

import paper_2402_18008_amd as hg
import synth
from tests.gpu_util import announce, require_gpu

pytestmark = pytest.mark.gpu


def _same(corr, n_hyp, tau, seed, label, tunes=(None,)):
    c = torch.from_numpy(np.ascontiguousarray(corr, np.float32)).cuda()
    n = c.shape[1]
    announce(f"tiles against plain: {label}, {n} points x {n_hyp}")
    ref = hg.hg_ransac_plain(c, n_hyp, tau, seed)
    off = torch.tensor([0, n], dtype=torch.int64, device="cuda")
    br = hg.BatchedRansac(c, off, n_hyp, tau, seed, hyp_counts=True)
    for tune in tunes:
        br.ws.fill_(0xFF)
        br.run(tune)
        torch.cuda.synchronize()
        assert torch.equal(br.hyp_counts[0], ref["hyp_counts"]), label
        assert torch.equal(br.best_H[0], ref["best_H"]) and torch.equal(br.mask, ref["mask"])
        assert int(br.best_count) == int(ref["best_count"])
        assert int(br.best_hyp) == int(ref["best_hyp"])
    return ref


# points: around one tile, one wave's share of tiles, a block of tiles between checks
# and of all waves; hypotheses: around a tile's height and an item
@pytest.mark.parametrize("n", [4, 31, 32, 33, 127, 128, 129, 511, 513, 2047, 2048, 2049, 4097])
@pytest.mark.parametrize("n_hyp", [1, 31, 33, 64, 65, 200])
def test_sizes(n, n_hyp):
    require_gpu()
    cs = synth.correspondences(n, 0.6, n + n_hyp)
    _same(cs.corr, n_hyp, 3.0, n, "sizes", (None, (8, 16, 1), (8, 32, 4), (16, 32, 2), (8, 64, 1),
                                            (16, 64, 8)))


@pytest.mark.parametrize("kind", ["far", "wide", "tiny", "huge", "one axis", "non-finite", "equal"])
def test_coordinates(kind):
    """Inputs that test the centring, the bound and what happens without one."""
    require_gpu()
    corr = synth.correspondences(900, 0.7, 21).corr.copy()
    tau = 3.0
    if kind == "far":            # a centre 10^6 px away: float keeps 1/16 px there
        corr += np.float32(1e6)
    elif kind == "wide":         # a few points far outside the frame
        corr[:, ::97] *= np.float32(1e4)
    elif kind == "tiny":
        corr *= np.float32(1e-6)
        tau = 3e-6
    elif kind == "huge":         # past the range of the bound: float64 throughout
        corr *= np.float32(2.0 ** 66)
        tau = float(3.0 * 2.0 ** 66)
    elif kind == "one axis":
        corr[1] = 0.0
    elif kind == "non-finite":
        corr[0, 5], corr[1, 77], corr[2, 300], corr[3, 850] = np.inf, np.nan, -np.inf, np.nan
        corr[:, 600:610] = np.nan
    elif kind == "equal":
        corr[:] = corr[:, :1]
    for n_hyp in (64, 300):
        _same(corr, n_hyp, tau, 5, kind, (None, (16, 32, 4), (8, 64, 4)))


def test_open_points_and_a_lost_list():
    """Points whose transfer error is exactly the threshold under every good
    hypothesis are open everywhere; there are more of them than an item's list
    holds, and the float64 test counts them (inclusive)."""
    require_gpu()
    rng = np.random.default_rng(8)
    for n, part in ((700, 0.02), (6000, 0.5)):
        x = rng.integers(0, 512, (2, n)).astype(np.float32)
        corr = np.concatenate([x, x])
        at = rng.random(n) < part
        corr[2, at] += 4.0
        ref = _same(corr, 96, 4.0, 3, f"open {part}", (None, (8, 32, 4), (16, 64, 2)))
        assert int(ref["best_count"]) == n


@pytest.mark.parametrize("sizes", [(4, 5, 40), (9000, 4, 700), (64,) * 70])
def test_pairs_of_many_sizes(sizes):
    """Batches whose launch shape the rules choose, sampled pairs against the
    oracle (counts outside its 1e-4 px band around the threshold)."""
    require_gpu()
    from oracle import ransac as oref
    sets = [synth.correspondences(n, 0.6, 40 + i).corr for i, n in enumerate(sizes)]
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    corr = torch.from_numpy(np.concatenate(sets, axis=1)).cuda()
    br = hg.BatchedRansac(corr, off, 130, 3.0, 9, hyp_counts=True)
    announce(f"pairs of sizes {sizes[:4]}")
    br.run()
    torch.cuda.synchronize()
    for i in range(0, len(sizes), max(1, len(sizes) // 4)):
        r = oref.ransac_ref(sets[i], 130, 3.0, 9, pair=i)
        got = br.hyp_counts[i].cpu().numpy()
        assert (got >= r["count_lo"]).all() and (got <= r["count_hi"]).all()
        assert int(br.best_count[i]) == int(got.max())
