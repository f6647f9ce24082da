"""Performance cases: the calls a user of this library makes, over the sizes they make them at.

listed() names the cases, draw(rng) makes one more of the same ranges; a case
is a dict of plain values.  Kinds and what they stand for:

  prox      one t-SVT call: the proximal step on its own, in a caller's loop or
            as a denoiser (the SVDs start cold)
  complete  a completion solve with a fixed number of ADMM iterations
  rpca      a tensor robust PCA solve, entrywise (l1) or tube (l112) shrink
  unfold    the vectorised matrix nuclear-norm baseline: a completion of the
            (n1 n2) x n3 unfolding, one very tall slice
  compress  compression by truncated t-SVD, Method 1 or 2
  batch     uneven completion problems solved together

Inputs follow the library's workloads: low-tubal-rank tensors A * B, smoothed
translated textures for the video shapes, Bernoulli masks, sparse or
tube-sparse corruption.  Penalties, growth factors and caps are the library's
defaults.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1407_1785_amd as lib

RHO, GROWTH, RHO_MAX = 1e-2, 1.1, 1e3          # completion schedule
MU, MU_GROWTH, MU_MAX = 1e-3, 1.2, 1e10        # RPCA schedule


def listed():
    return [
        # the smallest call: the plain test tensor, where launches and latency count
        dict(name="prox_small_f64", kind="prox", n1=32, n2=32, n3=16, n4=0, dtype="f64", data="lowrank"),
        # the video-shaped tensor of the completion experiments, one cold prox
        dict(name="prox_video_f32", kind="prox", n1=128, n2=160, n3=64, n4=0, dtype="f32", data="video"),
        # a 4-D colour video (two transformed modes, 75 slices)
        dict(name="prox_color_f64", kind="prox", n1=96, n2=128, n3=3, n4=48, dtype="f64", data="video"),
        # plain completion, tubal rank 2, half the entries seen
        dict(name="complete_small_f64", kind="complete", n1=32, n2=32, n3=16, n4=0, dtype="f64", data="lowrank",
             rank=2, frac=0.5, iters=100),
        # the headline solve: 200 iterations of the video completion, 20% seen
        dict(name="complete_video_f32", kind="complete", n1=128, n2=160, n3=64, n4=0, dtype="f32", data="video",
             rank=0, frac=0.2, iters=200),
        # the same in plain FP64, its first 60 iterations
        dict(name="complete_video_f64", kind="complete", n1=128, n2=160, n3=64, n4=0, dtype="f64", data="video",
             rank=0, frac=0.2, iters=60),
        # a ragged low-rank completion with an odd, prime tube
        dict(name="complete_ragged_f32", kind="complete", n1=201, n2=87, n3=37, n4=0, dtype="f32", data="lowrank",
             rank=5, frac=0.4, iters=60),
        # the robust-PCA workload, the widest slices a single solve meets
        dict(name="rpca_wide_f32", kind="rpca", n1=256, n2=256, n3=64, n4=0, dtype="f32", shrink="l1", rank=5,
             iters=30),
        # tube-block robust PCA of a small video
        dict(name="rpca_tube_f64", kind="rpca", n1=72, n2=128, n3=80, n4=0, dtype="f64", shrink="l112", rank=0,
             iters=40),
        # the vectorised baseline of the same video: a 20480 x 64 matrix
        dict(name="unfold_video_f32", kind="unfold", n1=20480, n2=64, n3=1, n4=0, dtype="f32", frac=0.3, rank=4,
             iters=30),
        # compression of the video at ratio about ten (Method 1)
        dict(name="compress_video_f64", kind="compress", n1=128, n2=160, n3=64, n4=0, dtype="f64", method=1, k=454),
        # twelve uneven problems together
        dict(name="batch_uneven_f32", kind="batch", dtype="f32", count=12, lo=48, hi=320, lo3=8, hi3=128, shapes=7,
             iters=30),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    cap = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["prox", "prox", "complete", "complete", "rpca", "rpca", "unfold", "compress", "batch"])
        dtype = rng.choice(["f32", "f64"])
        n1, n2, n3 = _logint(rng, 16, 320), _logint(rng, 16, 320), _logint(rng, 4, 128)
        if kind == "prox":
            n4 = rng.choice([0, 0, 0, rng.randint(2, 24)])
            c = dict(kind=kind, n1=n1, n2=n2, n3=rng.randint(2, 5) if n4 else n3, n4=n4, dtype=dtype,
                     data=rng.choice(["lowrank", "video"]))
        elif kind == "complete":
            c = dict(kind=kind, n1=n1, n2=n2, n3=n3, n4=0, dtype=dtype, data=rng.choice(["lowrank", "video"]),
                     rank=rng.randint(2, 8), frac=rng.uniform(0.2, 0.6), iters=rng.randint(20, 120))
        elif kind == "rpca":
            c = dict(kind=kind, n1=n1, n2=n2, n3=n3, n4=0, dtype=dtype, shrink=rng.choice(["l1", "l112"]), rank=5,
                     iters=rng.randint(15, 40))
        elif kind == "unfold":
            c = dict(kind=kind, n1=_logint(rng, 2000, 20480), n2=rng.randint(24, 80), n3=1, n4=0, dtype=dtype,
                     frac=rng.uniform(0.2, 0.6), rank=4, iters=rng.randint(10, 30))
        elif kind == "compress":
            n0 = min(n1, n2)
            method = rng.choice([1, 2])
            k = max(1, int(rng.uniform(0.03, 0.2) * n0 * (n3 if method == 1 else 1)))
            c = dict(kind=kind, n1=n1, n2=n2, n3=n3, n4=0, dtype=dtype, method=method, k=k)
        else:
            c = dict(kind=kind, dtype=dtype, count=rng.randint(3, 10), lo=24, hi=rng.randint(64, 256), lo3=4,
                     hi3=rng.randint(8, 64), shapes=rng.randint(0, 1 << 20), iters=rng.randint(10, 30))
        # FP64 costs about twice the FP32 form
        if work(c)["flops"] * (2 if dtype == "f64" else 1) <= cap:
            return c


# ------------------------------------------------------------------ inputs

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed, stream):
    g = torch.Generator()
    g.manual_seed(int(seed) * 1000003 + stream)
    return g


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, dtype=torch.float64).to(_device())


def _lowrank(gen, n1, n2, n3, rank, std=1.0):
    """A * B with N(0, std^2) factors: the t-product, slice by slice in the Fourier domain."""
    a = torch.fft.rfft(std * _randn(gen, n3, n1, rank), dim=0)
    b = torch.fft.rfft(std * _randn(gen, n3, rank, n2), dim=0)
    x = torch.empty(a.shape[0], n1, n2, dtype=torch.complex128, device=a.device)
    for k in range(a.shape[0]):
        x[k] = a[k] @ b[k]
    return torch.fft.irfft(x, n=n3, dim=0).permute(1, 2, 0).contiguous()


def _texture(gen, rows, cols, sigma=4.0):
    """Uniform noise smoothed by a Gaussian, scaled to [0, 1]."""
    t = torch.rand(1, 1, rows, cols, generator=gen, dtype=torch.float64).to(_device())
    r = int(4 * sigma)
    k = torch.exp(-0.5 * (torch.arange(-r, r + 1, dtype=torch.float64, device=t.device) / sigma) ** 2)
    k = k / k.sum()
    t = torch.cat([t.flip(2), t, t.flip(2)], 2)[:, :, rows - r:2 * rows + r] if rows > r else t.repeat(1, 1, 40, 1)[:, :, :rows + 2 * r]
    t = torch.cat([t.flip(3), t, t.flip(3)], 3)[:, :, :, cols - r:2 * cols + r] if cols > r else t.repeat(1, 1, 1, 40)[:, :, :, :cols + 2 * r]
    t = sum(k[i] * t[:, :, i:i + rows] for i in range(2 * r + 1))
    t = sum(k[i] * t[:, :, :, i:i + cols] for i in range(2 * r + 1))[0, 0]
    t = t - t.min()
    return t / t.max()


def _video(gen, n1, n2, frames, vy=0.4, vx=0.7):
    """A texture drifting (vy, vx) pixels a frame, sampled bilinearly."""
    rows, cols = n1 + int(math.ceil(vy * frames)) + 6, n2 + int(math.ceil(vx * frames)) + 6
    tex = _texture(gen, rows, cols)
    out = torch.empty(n1, n2, frames, dtype=torch.float64, device=tex.device)
    for t in range(frames):
        y, x = 2.0 + vy * t, 2.0 + vx * t
        y0, x0 = int(y), int(x)
        fy, fx = y - y0, x - x0
        p = tex[y0:y0 + n1 + 1, x0:x0 + n2 + 1]
        p = (1 - fy) * p[:-1] + fy * p[1:]
        out[:, :, t] = (1 - fx) * p[:, :-1] + fx * p[:, 1:]
    return out


def _tensor(case, seed):
    """The data tensor of a case in FP64 (before rounding to its dtype)."""
    gen = _gen(seed, 1)
    n1, n2, n3, n4 = case["n1"], case["n2"], case["n3"], case["n4"]
    if case.get("data", "video") == "lowrank":
        rank = max(1, min(case.get("rank") or 3, n1, n2))
        x = _lowrank(gen, n1, n2, n3 * (n4 or 1), rank)
        if case["kind"] == "prox":
            x = x + 0.1 * _randn(gen, *x.shape)   # a noisy low-rank tensor to denoise
        return x.reshape(n1, n2, n3, n4) if n4 else x
    if n4:
        return torch.stack([_video(gen, n1, n2, n4) for _ in range(n3)], 2).contiguous()
    x = _video(gen, n1, n2, n3)
    if case["kind"] == "prox":
        x = x + 0.05 * _randn(gen, *x.shape)
    return x


def _tau(case, x):
    """A threshold that keeps the signal and drops the noise: the noise
    level of a Fourier slice's largest singular value."""
    tubes = x[0, 0].numel()
    noise = 0.1 if case["data"] == "lowrank" else 0.05
    return noise * math.sqrt(tubes) * (math.sqrt(case["n1"]) + math.sqrt(case["n2"]))


def _mask(gen, shape, frac):
    return (torch.rand(*shape, generator=gen) < frac).to(torch.uint8).to(_device())


def _shapes(case):
    """Shapes, ranks and sampling ratios of a batch."""
    g = np.random.default_rng(case["shapes"])
    lo, hi = case["lo"], case["hi"]
    return [(int(g.integers(lo, hi + 1)), int(g.integers(lo, hi + 1)), int(g.integers(case["lo3"], case["hi3"] + 1)),
             int(g.integers(2, 11)), float(g.uniform(0.2, 0.6))) for _ in range(case["count"])]


def _inputs(case, seed):
    dt, kind = _dtype(case), case["kind"]
    if kind == "prox":
        x = _tensor(case, seed).to(dt)
        return dict(x=x, tau=_tau(case, x))
    if kind == "compress":
        return dict(x=_tensor(case, seed).to(dt))
    if kind == "complete":
        x = _tensor(case, seed).to(dt)
        m = _mask(_gen(seed, 2), x.shape, case["frac"])
        return dict(x=x * m, mask=m)
    if kind == "unfold":
        # a matrix of that rank with a decaying tail, as an unfolded video has
        g = _gen(seed, 1)
        n1, n2 = case["n1"], case["n2"]
        w = (1.0 / (1.0 + torch.arange(n2, dtype=torch.float64)) ** 2).to(_device())
        x = (_randn(g, n1, n2) * w) @ _randn(g, n2, n2) / math.sqrt(n2)
        x = x.reshape(n1, n2, 1).to(dt)
        m = _mask(_gen(seed, 2), x.shape, case["frac"])
        return dict(x=x * m, mask=m)
    if kind == "rpca":
        n1, n2, n3 = case["n1"], case["n2"], case["n3"]
        g, gs = _gen(seed, 1), _gen(seed, 2)
        if case["shrink"] == "l1":
            lo = _lowrank(g, n1, n2, n3, case["rank"], 1.0 / math.sqrt(n1))
            sp = (2 * torch.rand(n1, n2, n3, generator=gs, dtype=torch.float64) - 1).to(_device())
            sp = sp * _mask(gs, (n1, n2, n3), 0.1)
            lam = 1.0 / math.sqrt(max(n1, n2) * n3)
        else:
            lo = _video(g, n1, n2, n3)
            sp = torch.zeros_like(lo)
            for t in range(0, n3, 10):   # the same corrupted pixels within a block of frames
                f = min(10, n3 - t)
                sp[:, :, t:t + f] = 0.5 * _randn(gs, n1, n2, f) * _mask(gs, (n1, n2, 1), 0.02)
            lam = 1.0 / math.sqrt(max(n1, n2))
        return dict(x=(lo + sp).to(dt), lam=lam)
    xs, ms = [], []
    for i, (n1, n2, n3, rank, p) in enumerate(_shapes(case)):
        x = _lowrank(_gen(seed, 10 + 2 * i), n1, n2, n3, min(rank, n1, n2)).to(dt)
        m = _mask(_gen(seed, 11 + 2 * i), x.shape, p)
        xs.append(x * m)
        ms.append(m)
    return dict(xs=xs, ms=ms)


def _precision(case):
    return lib.PREC_FP64 if case["dtype"] == "f64" else lib.PREC_FP32


def prepare(case, seed):
    st = dict(case=case, **_inputs(case, seed))
    if case["kind"] == "batch":
        st["handle"] = lib.Handle(0, 16 << 30)
        st["probs"] = [lib.complete_problem(x, m, RHO, 0.0, GROWTH, RHO_MAX, case["iters"])
                       for x, m in zip(st["xs"], st["ms"])]
    else:
        st["handle"] = lib.Handle(0)
    return st


def run(st):
    case, h = st["case"], st["handle"]
    kind, prec = case["kind"], _precision(case)
    if kind == "prox":
        z, ranks = lib.tsvt(st["x"], st["tau"], prec, handle=h)
        return [z, np.asarray(ranks, dtype=np.int64)]
    if kind == "compress":
        return lib.compress(st["x"], case["method"], case["k"], prec, handle=h)[0]
    if kind == "rpca":
        sh = lib.SHRINK_L1 if case["shrink"] == "l1" else lib.SHRINK_L112
        lo, sp, _ = lib.trpca(st["x"], st["lam"], MU, 0.0, sh, MU_GROWTH, MU_MAX, case["iters"], prec, handle=h)
        return [lo, sp]
    if kind == "batch":
        for status, _ in lib.batch_run(st["probs"], handle=h):
            if status:
                raise RuntimeError(f"batch problem status {status}")
        return [p.out for p in st["probs"]]
    return lib.tsvd_complete(st["x"], st["mask"], RHO, 0.0, GROWTH, RHO_MAX, case["iters"], prec, handle=h)[0]


# ------------------------------------------------------------ work and exactness

def _work(n1, n2, n3, n4, esize, proxes, planes):
    """One solve.  A slice's SVD with both factors and the thresholded product
    takes about 14 m n^2 + 8 n^3 multiply-adds' worth of real flops for real
    data (QR, bidiagonalisation, both factors, rebuild), four times that for
    complex; the real DFT of a tube of length L about 5/2 L log2 L each way.
    planes: tensors read and written once by the call."""
    tube = n3 * (n4 or 1)
    slices = n3 * (n4 // 2 + 1) if n4 else n3 // 2 + 1
    m, n = max(n1, n2), min(n1, n2)
    svd = (4 if tube > 2 else 1) * slices * (14.0 * m * n * n + 8.0 * n ** 3)
    dft = 5.0 * n1 * n2 * tube * math.log2(tube) if tube > 1 else 0.0
    return float(n1 * n2 * tube * planes(esize)), proxes * (svd + dft)


def work(case):
    es = 8 if case["dtype"] == "f64" else 4
    planes = {"prox": lambda e: 2 * e, "compress": lambda e: 2 * e, "complete": lambda e: 2 * e + 1,
              "unfold": lambda e: 2 * e + 1, "rpca": lambda e: 3 * e, "batch": lambda e: 2 * e + 1}[case["kind"]]
    proxes = case.get("iters", 1)
    if case["kind"] == "batch":
        w = [_work(n1, n2, n3, 0, es, proxes, planes) for n1, n2, n3, _, _ in _shapes(case)]
    else:
        w = [_work(case["n1"], case["n2"], case["n3"], case["n4"], es, proxes, planes)]
    return {"bytes": sum(b for b, _ in w), "flops": sum(f for _, f in w)}


def tolerance(case):
    f64 = case["dtype"] == "f64"
    # About four times the largest distance from FP64 LAPACK measured over some
    # 70 cases of these ranges.  FP64 is rounding of the transforms and
    # rotations (6e-14 for one prox, 3e-13 after 100 iterations).  FP32 is its
    # 2e-6 for one prox; iterated solves carry the level its rotations stop at
    # (3e-5 for completions, 7e-5 for an RPCA whose threshold is crossing the
    # corruption's size, 1.6e-4 for the clustered spectrum of an unfolding).
    rel = {"prox": (3e-13, 1e-5), "compress": (5e-13, 1e-5), "complete": (4e-12, 1.2e-4), "unfold": (4e-12, 6e-4),
           "rpca": (4e-12, 3e-4), "batch": (4e-12, 1.2e-4)}[case["kind"]][0 if f64 else 1]
    out = {"rel": rel}
    if case["kind"] == "prox":
        out["differ"] = 0.02   # ranks: a singular value at the threshold may fall either way
    return out


def _svt_all(x, tau, keep=None):
    """SVT of every Fourier slice in FP64 (NumPy).  keep: instead of the
    threshold, a function of the slices' singular values that says which stay."""
    tr = x.shape[2:]
    xh = np.fft.rfftn(x, axes=tuple(range(2, x.ndim))) if np.prod(tr) > 1 else x.astype(np.complex128)
    hs = xh.shape
    a = np.ascontiguousarray(np.moveaxis(xh.reshape(hs[0], hs[1], -1), 2, 0))
    u, s, vh = np.linalg.svd(a, full_matrices=False)
    w = np.maximum(s - tau, 0.0) if keep is None else s * keep(s)
    z = np.moveaxis((u * w[:, None, :]) @ vh, 0, 2).reshape(hs)
    ranks = (s > tau).sum(1).astype(np.int64)
    z = np.fft.irfftn(z, s=tr, axes=tuple(range(2, x.ndim))) if np.prod(tr) > 1 else z.real
    return z, ranks


def _keep(case):
    """Method 1: the k largest values of the full spectrum, conjugate pairs
    together; Method 2: the first k of every slice."""
    n3, k = case["n3"], case["k"]

    def one(s):
        mult = np.full(s.shape, 2)
        mult[0] = 1
        if n3 % 2 == 0:
            mult[n3 // 2] = 1
        order = np.argsort(-s, axis=None)
        kept = np.zeros(s.size, dtype=bool)
        kept[order[np.cumsum(mult.ravel()[order]) <= k]] = True
        return kept.reshape(s.shape)

    def two(s):
        return np.broadcast_to(np.arange(s.shape[1]) < k, s.shape)

    return one if case["method"] == 1 else two


def _exact_complete(y, mask, iters):
    z, q, rho, x = np.zeros_like(y), np.zeros_like(y), RHO, y
    for _ in range(iters):
        x = np.where(mask, y, z - q)
        z, _ = _svt_all(x + q, 1.0 / rho)
        q = q + x - z
        nxt = min(GROWTH * rho, RHO_MAX)
        q *= rho / nxt
        rho = nxt
    return x


def _exact_rpca(m, lam, shrink, iters):
    s, w, mu, lo = np.zeros_like(m), np.zeros_like(m), MU, m
    for _ in range(iters):
        lo, _ = _svt_all(m - s - w, 1.0 / mu)
        d, t = m - w - lo, lam / mu
        if shrink == "l1":
            s = np.sign(d) * np.maximum(np.abs(d) - t, 0.0)
        else:
            nrm = np.sqrt((d * d).sum(2, keepdims=True))
            s = d * np.maximum(1.0 - t / np.maximum(nrm, 1e-300), 0.0)
        w = w + lo + s - m
        nxt = min(MU_GROWTH * mu, MU_MAX)
        w *= mu / nxt
        mu = nxt
    return lo, s


def exact(case, seed):
    if work(case)["flops"] > 2.5e11:   # about 15 s of LAPACK on one thread
        return None
    inp = _inputs(case, seed)
    host = lambda t: t.cpu().numpy().astype(np.float64)   # noqa: E731
    kind = case["kind"]
    if kind == "batch":
        return [_exact_complete(host(x), m.cpu().numpy() != 0, case["iters"]) for x, m in zip(inp["xs"], inp["ms"])]
    x = host(inp["x"])
    if kind == "prox":
        return list(_svt_all(x, inp["tau"]))
    if kind == "compress":
        return _svt_all(x, 0.0, _keep(case))[0]
    if kind == "rpca":
        return list(_exact_rpca(x, inp["lam"], case["shrink"], case["iters"]))
    return _exact_complete(x, inp["mask"].cpu().numpy() != 0, case["iters"])
