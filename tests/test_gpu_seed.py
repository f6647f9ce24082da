"""The QR start of a cold FP64 SVD (csrc/seed.hip) at the edges of its tiles
and of the sizes it serves, against the FP64 oracle."""

import numpy as np
import pytest

import paper_1407_1785_amd as lib
from oracle.tsvt import tsvt as tsvt_oracle
from tests.gpu_util import announce, rel_fro, to_gpu, torch_cuda

pytestmark = pytest.mark.gpu

# 100 n eps at n = 128: a few hundred rotations and reflections per column,
# each adding about eps of the slice's norm
TOL = 3e-12

# (longer, shorter) matrix mode around the 16-row lane groups, the column
# slots per lane row and the largest sizes served (the last of each group is
# one past them and starts from V = I)
SIZES = [(2, 2), (17, 16), (33, 31), (256, 32), (257, 32), (65, 33), (64, 64), (256, 50), (97, 65), (192, 96),
         (193, 96), (128, 97), (160, 128), (161, 128), (131, 129)]


def smooth(rng, m, n, n3):
    """Slices with singular values over the whole FP64 range, plus one zero
    column and one repeated column."""
    i, j = np.linspace(0, 1, m)[:, None], np.linspace(0, 1, n)[None, :]
    x = np.stack([np.exp(-8 * (i - j - 0.1 * rng.random()) ** 2) * (1 + rng.random()) for _ in range(n3)], axis=2)
    if n > 4:
        x[:, 1] = 0.0
        x[:, 3] = x[:, 2]
    return x


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("kind", ["noise", "smooth", "one slice"])
def test_seeded_prox_matches_oracle(size, kind):
    torch = torch_cuda()
    m, n = size
    rng = np.random.default_rng(m * 1000 + n)
    x = smooth(rng, m, n, 4) if kind == "smooth" else rng.normal(size=(m, n, 4))
    if kind == "one slice":   # noise that takes the QR for one slice's sake
        x += 10.0 * np.outer(rng.normal(size=m), rng.normal(size=n))[:, :, None]
    sv = np.linalg.svd(x.sum(axis=2), compute_uv=False)
    k = min(4, len(sv) - 1) if kind == "smooth" else len(sv) // 2
    tau = float(0.5 * (sv[k - 1] + sv[k])) + 1e-9 * sv[0]
    z_ref, _ = tsvt_oracle(x, tau)
    for data, ref in ((x, z_ref), (x.transpose(1, 0, 2), z_ref.transpose(1, 0, 2))):
        announce("seed", size, kind, data.shape)
        z, _ = lib.tsvt(to_gpu(torch, data), tau)
        assert rel_fro(z.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("scale", [1e-200, 1e-60, 1e60])
def test_seeded_prox_scales(scale):
    """Data whose squared norms leave the FP64 range (the QR then keeps what
    it has, down to V = I; the rotations, which multiply squared norms, need
    data within about 1e-70 to 1e70) and data inside it."""
    torch = torch_cuda()
    x = smooth(np.random.default_rng(3), 40, 36, 3) * scale
    tau = 0.01 * np.linalg.svd(x.sum(axis=2) / scale, compute_uv=False)[0] * scale
    announce("seed scale", scale)
    z, _ = lib.tsvt(to_gpu(torch, x), tau)
    assert torch.isfinite(z).all()
    if scale >= 1e-60:
        z_ref, _ = tsvt_oracle(x, tau)
        assert rel_fro(z.cpu().numpy() / scale, z_ref / scale) <= TOL


def test_seed_saves_sweeps(monkeypatch):
    """Smooth slices: under half of the sweeps, the same result."""
    torch = torch_cuda()
    x = to_gpu(torch, smooth(np.random.default_rng(9), 96, 80, 6))
    out, sweeps = [], []
    for on in ("1", "0"):
        monkeypatch.setenv("TSVD_SEED", on)
        h = lib.Handle(0)
        h.profile(True)
        announce("seed sweeps", on)
        out.append(lib.tsvt(x, 0.5, handle=h)[0].cpu().numpy())
        sweeps.append(h.profile_read()["jacobi_persistent"]["slice_sweeps"])
        h.close()
    assert rel_fro(out[0], out[1]) <= TOL
    assert sweeps[0] < 0.5 * sweeps[1], sweeps


@pytest.mark.parametrize("power", [-100, 83])
def test_seed_at_every_scale(power):
    """Data scaled by a power of two take the same steps and sweeps, also where
    their squared norms leave the FP32 range."""
    torch = torch_cuda()
    x = smooth(np.random.default_rng(9), 96, 80, 6)
    out, sweeps = [], []
    for scale in (1.0, 2.0 ** power):
        h = lib.Handle(0)
        h.profile(True)
        announce("seed scale sweeps", scale)
        out.append(lib.tsvt(to_gpu(torch, x * scale), 0.5 * scale, handle=h)[0].cpu().numpy() / scale)
        sweeps.append(h.profile_read()["jacobi_persistent"]["slice_sweeps"])
        h.close()
    assert sweeps[0] == sweeps[1]
    np.testing.assert_array_equal(out[0], out[1])


def test_seed_where_columns_are_alike():
    """Noise, scaled noise and orthogonal columns keep V = I; smooth data, and
    noise around one smooth Fourier slice, take the QR.  It shows in the time of
    the launches besides transforms, products and sweeps: the QR of 160 x 100
    slices is some 300 us, the question and V = I under 20."""
    torch = torch_cuda()
    rng = np.random.default_rng(5)
    m, n, n3 = 160, 100, 4
    noise = rng.normal(size=(m, n, n3))
    plain = {"noise": noise, "scaled": noise * np.geomspace(1, 1e-6, n)[None, :, None],
             "orthogonal": np.stack([np.linalg.qr(noise[:, :, t])[0] for t in range(n3)], axis=2)}
    alike = {"smooth": smooth(rng, m, n, n3), "one slice": 1e-3 * noise + smooth(rng, m, n, 1)}
    other = {}
    for name, x in {**plain, **alike}.items():
        tau = float(0.1 * np.linalg.svd(x.sum(axis=2), compute_uv=False)[0])
        announce("columns alike", name)
        best = []
        for _ in range(3):
            h = lib.Handle(0)
            h.profile(True)
            z, _ = lib.tsvt(to_gpu(torch, x), tau, handle=h)
            best.append(h.profile_read()["other"]["total_ms"])
            h.close()
        other[name] = min(best)
        assert rel_fro(z.cpu().numpy(), tsvt_oracle(x, tau)[0]) <= TOL
    assert max(other[k] for k in plain) < 0.5 * min(other[k] for k in alike), other
