"""The work that a program has this library do, as cases that can be timed and compared.

The families are the library's public calls, over the sizes of its own workloads (`bench.py`,
`synth/`, `tests/`) and the sizes around them:

* solve4, sk, affine: batches of minimal problems, from a few (one RANSAC iteration on the host, one
  marker) to 2^26, with plane strides that are whole cache lines and ones that are not;
* ransac, batched, adaptive, refit: hypothesise-and-verify on one pair and on many uneven pairs, and
  the least-squares homography of the inliers found;
* aca_general, photometric, refine: the differentiable path, forward and backward.

`exact` evaluates the same quantities in float64 with torch and numpy alone."""
import math

import numpy as np
import torch

import paper_2402_18008_amd as hg

FRAME_W, FRAME_H = 640.0, 480.0
TAU = 3.0                     # inlier threshold, px
CONFIDENCE = 0.99
THIN = 1e-2                   # a triangle thinner than this (px) is flagged near-degenerate
PATTERN = (20.0, 30.0, 180.0, 25.0, 35.0, 140.0, 170.0, 150.0)   # M N P Q of a planar target
DEVICE = "cuda"


def listed():
    return [
        # one small batch, outputs allocated by the call: launch latency and the binding's own time
        dict(name="aca 4096", family="solve4", method="aca", n=4096, keep=False),
        # the headline batch, buffers kept: streaming at the largest size
        dict(name="aca 2^26", family="solve4", method="aca", n=1 << 26, keep=True),
        # a ragged batch: a contiguous (8, n) tensor with odd n has planes that start anywhere
        dict(name="sks 1000003", family="solve4", method="sks", n=1000003, keep=False),
        # many images of one calibration pattern
        dict(name="pattern 2^22", family="sk", n=1 << 22, keep=True),
        # one image pair, as a tracker or a matcher calls it per frame
        dict(name="ransac 2000x4096", family="ransac", points=2000, hyps=4096, ratio=0.3,
             counts=True),
        # every pair of an image collection in one launch
        dict(name="batched 512x1024", family="batched", pairs=512, points=8000, hyps=1024),
        # the same with the loop rule at 99 % confidence
        dict(name="adaptive 512x1024", family="adaptive", pairs=512, points=8000, hyps=1024),
        # least squares on the inliers of every pair
        dict(name="refit 512", family="refit", pairs=512, points=8000),
        # the tensorised general solver in a training step, through autograd, both directions
        dict(name="general 2^20", family="aca_general", batch=1 << 20),
        # a training batch of 128 x 128 patches: loss and gradient in one pass over the images
        dict(name="photo 1024x128x128", family="photometric", batch=1024, height=128, width=128,
             form="single"),
        # a small batch of larger images of no special size, recomputing backward
        dict(name="photo 24x211x317", family="photometric", batch=24, height=211, width=317,
             form="recompute"),
        # iterative refinement at inference: six steps replayed from a graph
        dict(name="refine 64x128x128", family="refine", batch=64, height=128, width=128, iters=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["solve4", "solve4", "sk", "affine", "ransac", "batched", "adaptive", "refit",
                         "aca_general", "photometric", "photometric", "refine"])
    if family == "solve4":
        return dict(family=family, method=rng.choice(["aca", "sks"]), n=_log_int(rng, 1, 1 << 25),
                    keep=rng.random() < 0.5)
    if family in ("sk", "affine"):
        return dict(family=family, n=_log_int(rng, 1, 1 << 25), keep=rng.random() < 0.5)
    if family == "ransac":
        return dict(family=family, points=_log_int(rng, 16, 8000), hyps=_log_int(rng, 64, 16384),
                    ratio=round(rng.uniform(0.1, 0.9), 2), counts=rng.random() < 0.5)
    if family in ("batched", "adaptive"):
        return dict(family=family, pairs=_log_int(rng, 2, 512), points=_log_int(rng, 200, 8000),
                    hyps=_log_int(rng, 64, 1024))
    if family == "refit":
        return dict(family=family, pairs=_log_int(rng, 1, 512), points=_log_int(rng, 200, 8000))
    if family == "aca_general":
        return dict(family=family, batch=_log_int(rng, 1, 1 << 20))
    batch, height, width = _log_int(rng, 1, 1024), rng.randint(48, 320), rng.randint(48, 320)
    if rng.random() < 0.4:
        height = width = rng.choice([64, 128, 256])
    batch = max(1, min(batch, (1 << 24) // (height * width)))
    if family == "photometric":
        return dict(family=family, batch=batch, height=height, width=width,
                    form=rng.choice(["single", "recompute", "autograd", "separate"]))
    return dict(family=family, batch=min(batch, 256), height=height, width=width,
                iters=rng.randint(1, 6))


# ---- inputs ------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEVICE, dtype=torch.float32) * (hi - lo) + lo


def _maps(g, n):
    """n maps of the plane: a similarity (scale U[0.5, 2], any rotation, translation U[-100, 100]^2)
    and a perspective row U[-1e-3, 1e-3]^2; columns h11 .. h32 as (8, n)."""
    s, th = _uniform(g, (n,), 0.5, 2.0), _uniform(g, (n,), -math.pi, math.pi)
    t, p = _uniform(g, (2, n), -100.0, 100.0), _uniform(g, (2, n), -1e-3, 1e-3)
    c, d = s * torch.cos(th), s * torch.sin(th)
    return torch.stack([c, -d, t[0], d, c, t[1], p[0], p[1]])


def _apply(m, x, y):
    w = m[6] * x + m[7] * y + 1.0
    return (m[0] * x + m[1] * y + m[2]) / w, (m[3] * x + m[4] * y + m[5]) / w, w


def _images(g, x, y):
    """Images of the points x, y ((k, n) each) of n problems under n maps with w >= 0.1 at every
    point (perspective rows shrunk where needed), plus N(0, 0.5^2) px noise: (2 k, n) planes."""
    k, n = x.shape
    m = _maps(g, n)
    low = torch.clamp(-(m[6] * x + m[7] * y).amin(0), min=1e-9)      # 1 - low is the least w
    shrink = torch.clamp(0.9 / low, max=1.0)
    m[6] *= shrink
    m[7] *= shrink
    u, v, _ = _apply(m, x, y)
    out = torch.empty((2 * k, n), device=DEVICE)
    out[0::2], out[1::2] = u, v
    return out.add_(torch.randn((2 * k, n), generator=g, device=DEVICE), alpha=0.5)


def _quads(g, n, k=4):
    """n problems of k source points uniform in the frame and their images; in one of a hundred
    quadruples the last source point lies within 1e-3 px of the line through the first two."""
    x, y = _uniform(g, (k, n), 0.0, FRAME_W), _uniform(g, (k, n), 0.0, FRAME_H)
    if k == 4:
        a = _uniform(g, (n,), -0.5, 1.5)[::100]
        e = _uniform(g, (n,), -1e-3, 1e-3)[::100]
        x[3, ::100] = x[0, ::100] + a * (x[1, ::100] - x[0, ::100])
        y[3, ::100] = y[0, ::100] + a * (y[1, ::100] - y[0, ::100]) + e
    src = torch.empty((2 * k, n), device=DEVICE)
    src[0::2], src[1::2] = x, y
    return src, _images(g, x, y)


def _pair_sizes(case):
    """Points per pair and inlier ratios of a collection, fixed by the case: N ~ U{100 .. points},
    ratio ~ U[0.1, 0.9]. The offsets come back as int64, one more than there are pairs."""
    rng = np.random.default_rng([case["pairs"], case["points"]])
    sizes = rng.integers(100, case["points"] + 1, case["pairs"])
    ratios = rng.uniform(0.1, 0.9, case["pairs"])
    off = np.zeros(case["pairs"] + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    return off, ratios


def _correspondences(g, off, ratios):
    """(4, total) planes x1 y1 x2 y2 and the (total,) inlier labels: per pair one map about the
    frame's centre, inliers with N(0, 1) px noise, outliers uniform in both frames."""
    sizes = torch.as_tensor(np.diff(off), device=DEVICE)
    total, pairs = int(off[-1]), len(off) - 1
    pair = torch.repeat_interleave(torch.arange(pairs, device=DEVICE), sizes, output_size=total)
    x, y = _uniform(g, (total,), 0.0, FRAME_W), _uniform(g, (total,), 0.0, FRAME_H)
    u, v = _uniform(g, (total,), 0.0, FRAME_W), _uniform(g, (total,), 0.0, FRAME_H)
    m = _maps(g, pairs)[:, pair]
    a, b, w = _apply(m, x - FRAME_W / 2, y - FRAME_H / 2)
    noise = torch.randn((2, total), generator=g, device=DEVICE)
    ratio = torch.as_tensor(ratios, dtype=torch.float32, device=DEVICE)[pair]
    inlier = (_uniform(g, (total,), 0.0, 1.0) < ratio) & (w > 0.1)
    u = torch.where(inlier, a + FRAME_W / 2 + noise[0], u)
    v = torch.where(inlier, b + FRAME_H / 2 + noise[1], v)
    return torch.stack([x, y, u, v]).contiguous(), inlier.to(torch.uint8)


def _patches(g, batch, height, width):
    """Two views of smooth random scenes (noise blurred with sigma = 4 px; the second view shifted by
    up to 16 px), standardised, and corner offsets U[-32, 32] px."""
    radius, reach = 12, 16
    a = torch.randn((batch, height + 2 * (reach + radius), width + 2 * (reach + radius)),
                    generator=g, device=DEVICE)
    taps = [math.exp(-0.5 * (i / 4.0) ** 2) for i in range(-radius, radius + 1)]
    for dim in (1, 2):
        size = a.shape[dim] - 2 * radius
        b = torch.zeros_like(a.narrow(dim, 0, size))
        for i, t in enumerate(taps):
            b.add_(a.narrow(dim, i, size), alpha=t)
        a = b
    shift = torch.randint(0, 2 * reach + 1, (2, batch), generator=g, device=DEVICE)
    rows = shift[0][:, None, None] + torch.arange(height, device=DEVICE)[None, :, None]
    cols = shift[1][:, None, None] + torch.arange(width, device=DEVICE)[None, None, :]
    img = a[:, reach:reach + height, reach:reach + width]
    tgt = a[torch.arange(batch, device=DEVICE)[:, None, None], rows, cols]

    def standard(t):
        return ((t - t.mean((1, 2), keepdim=True)) / t.std((1, 2), keepdim=True)).contiguous()
    return standard(img), standard(tgt), _uniform(g, (batch, 4, 2), -32.0, 32.0)


def prepare(case, seed):
    g, f = _generator(seed), case["family"]
    if f in ("solve4", "affine"):
        src, dst = _quads(g, case["n"], 4 if f == "solve4" else 3)
        s = dict(src=src, dst=dst)
    elif f == "sk":
        p = torch.tensor(PATTERN, device=DEVICE).reshape(4, 2)
        p = p - p.mean(0)
        x, y = (p[:, k:k + 1].expand(4, case["n"]) for k in (0, 1))
        dst = _images(g, x, y)
        dst[0::2] += FRAME_W / 2
        dst[1::2] += FRAME_H / 2
        s = dict(dst=dst)
    elif f == "ransac":
        off = np.array([0, case["points"]], np.int64)
        s = dict(corr=_correspondences(g, off, [case["ratio"]])[0])
    elif f in ("batched", "adaptive", "refit"):
        off, ratios = _pair_sizes(case)
        corr, inlier = _correspondences(g, off, ratios)
        s = dict(corr=corr, off=torch.from_numpy(off).to(DEVICE), off_host=off, inlier=inlier)
        if f == "batched":
            s["plan"] = hg.BatchedRansac(corr, s["off"], case["hyps"], TAU, seed)
        elif f == "adaptive":
            s["plan"] = hg.AdaptiveRansac(corr, s["off"], case["hyps"], TAU, seed, CONFIDENCE)
    elif f == "aca_general":
        src, dst = _quads(g, case["batch"])
        s = dict(src=src.T.contiguous(), dst=dst.T.contiguous(),
                 grad_H=torch.randn((case["batch"], 9), generator=g, device=DEVICE,
                                    dtype=torch.float64))
        s["src"].requires_grad_(True)
        s["dst"].requires_grad_(True)
    else:
        img, tgt, offsets = _patches(g, case["batch"], case["height"], case["width"])
        s = dict(img=img, tgt=tgt, offsets=offsets)
        if f == "photometric":
            s["offsets"].requires_grad_(case["form"] in ("autograd", "separate"))
            s["grad_loss"] = _uniform(g, (case["batch"],), 0.5, 1.5)
        else:
            s["plan"] = hg.Refine(img, tgt, torch.empty_like(offsets), case["iters"], step=20.0)
            s["plan"].offsets.copy_(offsets)
            s["graph"] = s["plan"].graph()
    if case.get("keep"):
        n, rows = case["n"], 6 if f == "affine" else 9
        s["out"] = torch.empty((rows, n), device=DEVICE)
        s["flags"] = torch.empty(n, dtype=torch.uint8, device=DEVICE)
    return dict(s, case=case, seed=int(seed))


def run(s):
    case = s["case"]
    f = case["family"]
    if f == "solve4":
        return hg.hg_solve4(s["src"], s["dst"], case["method"], s.get("out"), s.get("flags"))
    if f == "sk":
        return hg.hg_solve_sk(PATTERN, s["dst"], s.get("out"), s.get("flags"))
    if f == "affine":
        return hg.hg_solve3_affine(s["src"], s["dst"], s.get("out"), s.get("flags"))
    if f == "ransac":
        return hg.hg_ransac(s["corr"], case["hyps"], TAU, s["seed"], hyp_counts=case["counts"])
    if f in ("batched", "adaptive"):
        r = s["plan"].run()
        out = dict(best_H=r.best_H, best_count=r.best_count, best_hyp=r.best_hyp, mask=r.mask)
        return dict(out, n_evaluated=r.n_evaluated) if f == "adaptive" else out
    if f == "refit":
        return hg.hg_refit_ho(s["corr"], s["off"], s["inlier"], off_host=s["off_host"])
    if f == "aca_general":
        H = hg.ACAGeneral.apply(s["src"], s["dst"])
        return (H, *torch.autograd.grad(H, (s["src"], s["dst"]), s["grad_H"]))
    if f == "photometric":
        a = (s["offsets"], s["img"], s["tgt"])
        if case["form"] == "single":
            loss, unit = hg.hg_photometric_fwd_grad(*a)
            return loss, hg.hg_scale_grad(unit, s["grad_loss"])
        if case["form"] == "recompute":
            return hg.hg_photometric_fwd(*a), hg.hg_photometric_bwd(*a, s["grad_loss"])
        loss = hg.photometric_loss(*a, fused=case["form"] == "autograd")
        return (loss, *torch.autograd.grad(loss, s["offsets"], s["grad_loss"]))
    s["plan"].offsets.copy_(s["offsets"])     # the starting offsets of these images
    s["graph"].launch()
    return s["plan"].offsets, s["plan"].loss


def work(case):
    f = case["family"]
    if f in ("solve4", "sk", "affine"):
        planes = {"solve4": 25, "sk": 17, "affine": 18}[f]
        flops = {"solve4": 85 if case.get("method") == "aca" else 161, "sk": 75, "affine": 43}[f]
        return dict(bytes=(4 * planes + 1) * case["n"], flops=flops * case["n"])
    if f == "ransac":
        n, m = case["points"], case["hyps"]
        # 21 operations per (hypothesis, point): the division-free test, an FMA counted as two
        return dict(bytes=17 * n + (4 * m if case["counts"] else 0) + 44, flops=m * (21 * n + 85))
    if f in ("batched", "adaptive", "refit"):
        off, ratios = _pair_sizes(case)
        n = np.diff(off).astype(float)
        if f == "refit":
            return dict(bytes=17 * n.sum() + 41 * len(n), flops=70 * (n * ratios).sum())
        m = np.full(len(n), case["hyps"], float)
        if f == "adaptive":       # what the rule asks for at the true ratios, in rounds of 64
            need = np.log(1 - CONFIDENCE) / np.log1p(-ratios ** 4)
            m = np.minimum(m, 64 * np.ceil(need / 64))
        return dict(bytes=17 * n.sum() + 48 * len(n), flops=(m * (21 * n + 85)).sum())
    if f == "aca_general":
        # points in and H out; points and dL/dH in and both gradients out
        return dict(bytes=(64 + 72 + 64 + 72 + 64) * case["batch"], flops=400 * case["batch"])
    pixels = case["batch"] * case["height"] * case["width"]
    passes = {"single": 1, "autograd": 1, "recompute": 2, "separate": 2}.get(case.get("form"), 0) \
        or case["iters"] + 1
    return dict(bytes=8 * pixels * passes + 100 * case["batch"], flops=60 * pixels * passes)


# ---- the same in 64 bits, with torch and numpy alone ---------------------------

def _aca(s, d):
    """H (9 columns) of the affine-core-affine decomposition from the 8 coordinates of either side
    (M N P Q), at the decomposition's own scale."""
    def side(q):
        mn, mp, mq = ((q[k] - q[0], q[k + 1] - q[1]) for k in (2, 4, 6))
        f = mn[0] * mp[1] - mn[1] * mp[0]
        qx = mq[0] * mp[1] - mq[1] * mp[0]
        qy = mn[0] * mq[1] - mn[1] * mq[0]
        return mn, mp, f, qx, qy, f - qx - qy
    mn, mp, f1, ax, ay, t1 = side(s)
    _, _, _, bx, by, t2 = side(d)
    c1, c2, c3 = t1 * ay * bx, t1 * ax * by, t2 * ax * ay
    H = []
    for m, n, p in ((d[0], d[2], d[4]), (d[1], d[3], d[5]), (1.0, 1.0, 1.0)):
        l0, l1, l2 = n * c1 - m * c3, p * c2 - m * c3, m * c3
        h0, h1 = l0 * mp[1] - l1 * mn[1], l1 * mn[0] - l0 * mp[0]
        H += [h0, h1, l2 * f1 - (h0 * s[0] + h1 * s[1])]
    return H


def _unit(H, dim=0):
    """H times the power of two that brings its largest entry into [0.5, 1)."""
    e = torch.frexp(H.abs().amax(dim, keepdim=True))[1]
    return torch.ldexp(H, -e)


def _sks(s, d):
    """H at the scale of the similarity-kernel-similarity decomposition, whose kernel
    [[a, u, b], [0, 1, 0], [b, v, a]] takes the source anchor M, at (-1, 0) in its frame, to weight
    f1 (a - b): ACA's H, rescaled to that weight at M."""
    H = torch.stack(_aca(s, d))
    on = ((s[2] - s[0]) * 0.5, (s[3] - s[1]) * 0.5)
    f1 = on[0] ** 2 + on[1] ** 2

    def kernel_points(q):
        nx, ny = (q[2] - q[0]) * 0.5, (q[3] - q[1]) * 0.5
        ox, oy, f = q[0] + nx, q[1] + ny, nx * nx + ny * ny
        pts = []
        for k in (4, 6):
            dx, dy = q[k] - ox, q[k + 1] - oy
            cy = nx * dy - ny * dx
            pts.append(((nx * dx + ny * dy) / cy, f / cy))
        return pts
    (px, py), (qx, qy) = kernel_points(s)
    (rx, ry), (tx, ty) = kernel_points(d)
    minus = ((tx - rx) - (ty - ry)) / ((qx - px) - (qy - py))       # a - b
    w = H[6] * s[0] + H[7] * s[1] + H[8]
    return H * (f1 * minus / w)


def _thin(q):
    """Whether one of the four triangles of a side has a height of at most THIN."""
    x, y = q[0::2], q[1::2]
    bad = torch.zeros_like(q[0], dtype=torch.bool)
    for tri in ((0, 1, 2), (0, 3, 2), (0, 1, 3), (1, 2, 3)):
        e = [(x[b] - x[a], y[b] - y[a]) for a, b in ((tri[0], tri[1]), (tri[0], tri[2]),
                                                      (tri[1], tri[2]))]
        area = e[0][0] * e[1][1] - e[0][1] * e[1][0]
        longest = torch.stack([u * u + v * v for u, v in e]).amax(0)
        bad |= area * area <= THIN ** 2 * longest
    return bad


def _samples(n, hyps, seed, pair):
    """Philox4x32-10 (key: the seed's words; counter: hypothesis, pair) and Floyd's choice of 4 of n."""
    u64, low = np.uint64, np.uint64(0xFFFFFFFF)
    k = [u64(seed & 0xFFFFFFFF), u64(seed >> 32)]
    c = [np.arange(hyps, dtype=u64), np.full(hyps, pair, u64), np.zeros(hyps, u64),
         np.zeros(hyps, u64)]
    for _ in range(10):
        a, b = c[0] * u64(0xD2511F53), c[2] * u64(0xCD9E8D57)
        c = [(b >> u64(32)) ^ c[1] ^ k[0], b & low, (a >> u64(32)) ^ c[3] ^ k[1], a & low]
        k = [(k[0] + u64(0x9E3779B9)) & low, (k[1] + u64(0xBB67AE85)) & low]
    got = []
    for i, r in enumerate(c):
        j = n - 4 + i
        t = (r * u64(j + 1)) >> u64(32)
        taken = np.zeros(hyps, bool)
        for p in got:
            taken |= p == t
        got.append(np.where(taken, u64(j), t))
    return torch.from_numpy(np.stack(got).astype(np.int64)).to(DEVICE)


def _best_H(corr, hyps, seed, pair, adaptive):
    """The winning hypothesis's H (9,) in float64: most points with a transfer error of at most TAU
    under the float H, the first of them, over all hypotheses or until the loop rule holds."""
    n = corr.shape[1]
    p = corr.double()[:, _samples(n, hyps, seed, pair)]               # (4, 4 points, hyps)
    s = p[:2].transpose(0, 1).reshape(8, hyps)
    d = p[2:].transpose(0, 1).reshape(8, hyps)
    H = _unit(torch.stack(_aca(s, d)))
    h = H.float().double()
    x, y, u, v = corr.double()[:, None]
    h = h[:, :, None]
    W = h[6] * x + h[7] * y + h[8]
    inlier = torch.hypot((h[0] * x + h[1] * y + h[2]) / W - u,
                         (h[3] * x + h[4] * y + h[5]) / W - v) <= TAU
    count = inlier.sum(1).masked_fill_(_thin(s) | _thin(d), -1)
    if adaptive:
        best = torch.cummax(count, 0)[0].cpu().numpy()
        for m in range(64, hyps + 64, 64):
            m = min(m, hyps)
            if (1.0 - (max(int(best[m - 1]), 0) / n) ** 4) ** m <= 1.0 - CONFIDENCE:
                break
        count = count[:m]
    most = int(count.max())
    if most < 0:
        return torch.zeros(9, dtype=torch.float64, device=DEVICE)
    return H[:, int((count == most).nonzero()[0])]


def _refit_H(c):
    """HO-SVD of the points c (4, n) in float64: rows 1 and 2 of H eliminated by least squares."""
    if c.shape[1] < 4:
        return torch.zeros(9, dtype=torch.float64, device=DEVICE)

    def normal(z):
        m = z.mean(1)
        k = torch.sqrt(2.0 / ((z - m[:, None]) ** 2).sum(0).mean())
        return (z - m[:, None]) * k, k, m
    z1, k1, m1 = normal(c[:2])
    z2, k2, m2 = normal(c[2:])
    X = torch.cat([z1, torch.ones_like(z1[:1])]).T
    Q, R = torch.linalg.qr(X)
    Y = [z2[k][:, None] * X for k in (0, 1)]
    h3 = torch.linalg.svd(torch.cat([y - Q @ (Q.T @ y) for y in Y]), full_matrices=False)[2][-1]
    h3 = h3 * torch.sign(h3[h3.abs().argmax()])
    Hn = torch.stack([torch.linalg.solve(R, Q.T @ (y @ h3)) for y in Y] + [h3])
    T1 = torch.eye(3, dtype=torch.float64, device=DEVICE)
    T1[0, 0] = T1[1, 1] = k1
    T1[:2, 2] = -k1 * m1
    T2 = torch.eye(3, dtype=torch.float64, device=DEVICE)
    T2[0, 0] = T2[1, 1] = 1.0 / k2
    T2[:2, 2] = m2
    return _unit((T2 @ Hn @ T1).reshape(9))


def _photometric(offsets, img, tgt):
    """Per-patch mean |img warped by H(offsets) - tgt|, all float64, bilinear with zeros outside."""
    B, h, w = img.shape
    kw = dict(dtype=torch.float64, device=DEVICE)
    # the patch's rectangle: width w - 1 and the aspect ratio as a float argument holds it
    x1, y1 = float(w - 1), float(w - 1) / float(np.float32((w - 1) / (h - 1)))
    s = [torch.full((B,), v, **kw) for v in (0.0, 0.0, x1, 0.0, 0.0, y1, x1, y1)]
    corner = offsets[:, (0, 1, 3, 2)].reshape(B, 8).T                 # TL TR BL BR
    H = torch.stack(_aca(s, [a + b for a, b in zip(s, corner)]), 1).reshape(B, 3, 3)
    G = torch.linalg.inv(H / H.abs().amax((1, 2), keepdim=True))
    y, x = torch.meshgrid(torch.arange(h, **kw), torch.arange(w, **kw), indexing="ij")
    q = [G[:, k, 0, None] * x.reshape(-1) + G[:, k, 1, None] * y.reshape(-1) + G[:, k, 2, None]
         for k in range(3)]
    sx, sy = q[0] / q[2], q[1] / q[2]
    fx, fy = sx.detach().floor(), sy.detach().floor()
    ax, ay, flat, value = sx - fx, sy - fy, img.reshape(B, -1), 0.0
    for dy, wy in ((0, 1 - ay), (1, ay)):
        for dx, wx in ((0, 1 - ax), (1, ax)):
            cx, cy = fx + dx, fy + dy
            inside = (cx >= 0) & (cx < w) & (cy >= 0) & (cy < h)
            at = torch.where(inside, cy * w + cx, torch.zeros_like(cx)).long()
            value = value + wx * wy * torch.where(inside, flat.gather(1, at),
                                                  torch.zeros_like(ax))
    return (value - tgt.reshape(B, -1)).abs().mean(1)


def _photometric_grad(offsets, img, tgt):
    """Loss (B,) and its gradient (B, 4, 2), a few patches at a time."""
    step = max(1, (1 << 21) // (img.shape[1] * img.shape[2]))
    L, G = [], []
    for a in range(0, img.shape[0], step):
        o = offsets[a:a + step].double().requires_grad_(True)
        loss = _photometric(o, img[a:a + step].double(), tgt[a:a + step].double())
        G.append(torch.autograd.grad(loss.sum(), o)[0])
        L.append(loss.detach())
    return torch.cat(L), torch.cat(G)


def exact(case, seed):
    s, f = prepare(dict(case, keep=False), seed), case["family"]
    if f in ("solve4", "sk", "affine"):
        n, step = case["n"], 1 << 21
        out = torch.empty((6 if f == "affine" else 9, n), dtype=torch.float64, device=DEVICE)
        for a in range(0, n, step):
            d = s["dst"][:, a:a + step].double()
            if f == "sk":
                # the pattern in its canonical frame: anchors at (-1, 0) and (1, 0)
                p = np.array(PATTERN).reshape(4, 2)
                o, e = (p[0] + p[1]) / 2, (p[1] - p[0]) / 2
                r = np.array([[e[0], e[1]], [-e[1], e[0]]]) / (e @ e)
                c = torch.as_tensor(((p - o) @ r.T).reshape(8, 1), device=DEVICE)
                out[:, a:a + step] = _unit(_sks(list(c.expand(8, d.shape[1])), d))
                continue
            q = s["src"][:, a:a + step].double()
            if f == "solve4":
                H = torch.stack(_aca(q, d)) if case["method"] == "aca" else _sks(q, d)
                out[:, a:a + step] = _unit(H)
                continue
            mn, mp = (q[2] - q[0], q[3] - q[1]), (q[4] - q[0], q[5] - q[1])
            area = mn[0] * mp[1] - mn[1] * mp[0]
            for k in (0, 1):
                en, ep = d[2 + k] - d[k], d[4 + k] - d[k]
                a1, a2 = (en * mp[1] - ep * mn[1]) / area, (ep * mn[0] - en * mp[0]) / area
                out[3 * k:3 * k + 3, a:a + step] = torch.stack([a1, a2, d[k] - a1 * q[0]
                                                               - a2 * q[1]])
        return (out, None, None) if f == "sk" else (out, None)
    none = dict(best_count=None, best_hyp=None, mask=None)
    if f == "ransac":
        return dict(none, hyp_counts=None,
                    best_H=_best_H(s["corr"], case["hyps"], s["seed"], 0, False))
    if f in ("batched", "adaptive"):
        off = s["off_host"]
        H = [_best_H(s["corr"][:, off[p]:off[p + 1]], case["hyps"], s["seed"], p, f == "adaptive")
             for p in range(len(off) - 1)]
        return dict(none, best_H=torch.stack(H))
    if f == "refit":
        off, sel = s["off_host"], s["inlier"].bool()
        H = [_refit_H(s["corr"][:, off[p]:off[p + 1]].double()[:, sel[off[p]:off[p + 1]]])
             for p in range(len(off) - 1)]
        return torch.stack(H), None, None
    if f == "aca_general":
        q, d = (s[k].detach().double().requires_grad_(True) for k in ("src", "dst"))
        H = torch.stack(_aca(q.T, d.T), 1)
        return (H.detach(), *torch.autograd.grad(H, (q, d), s["grad_H"]))
    if f == "photometric":
        loss, grad = _photometric_grad(s["offsets"].detach(), s["img"], s["tgt"])
        return loss, grad * s["grad_loss"].double()[:, None, None]
    offsets = s["offsets"].double()
    for _ in range(case["iters"]):
        offsets = offsets - 20.0 * _photometric_grad(offsets, s["img"], s["tgt"])[1]
    return offsets, _photometric_grad(offsets, s["img"], s["tgt"])[0]
