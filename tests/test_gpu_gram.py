"""Tall FP32 slices through the FP64 Gram matrix (csrc/tall.hip) and the
matrix form of the transforms (tubes of length 1), at the edges of their tiles
and of the sizes the Gram path serves, against the FP64 oracle."""

import numpy as np
import pytest

import paper_1407_1785_amd as lib
from oracle import admm
from oracle.tsvt import tsvt as tsvt_oracle
from tests.gpu_util import announce, assert_close_fp32, rel_fro, slice_rel_max, to_gpu, torch_cuda

pytestmark = pytest.mark.gpu

# one product with V diag(d) V^H and the roundings of A, V and the result:
# about ten FP32 units (6e-8) of the slice's norm over the result's
TOL_GRAM = 2e-6


def graded(rng, m, n, tail=1e-9):
    """Singular values from 1 down to `tail`, then exact zeros."""
    u, _ = np.linalg.qr(rng.normal(size=(m, n)))
    v, _ = np.linalg.qr(rng.normal(size=(n, n)))
    s = np.geomspace(1.0, tail, n)
    s[-max(1, n // 8):] = 0.0
    return (u * s) @ v.T


# (rows, columns, tube): the 16-column tiles of the Gram kernel, the 64-column
# and 96-column edges, one past 96 and fewer rows than 12 n (global-memory
# Jacobi), rows that are no multiple of a chunk, complex slices
SIZES = [(1500, 2, 1), (1201, 15, 1), (1100, 17, 1), (2003, 63, 1), (1300, 64, 1), (1999, 65, 1), (1152, 96, 1),
         (1151, 96, 1), (1500, 97, 1), (1100, 33, 4), (1031, 16, 5)]


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("wide", [False, True])
def test_gram_prox(size, wide):
    torch = torch_cuda()
    m, n, tube = size
    rng = np.random.default_rng(m + n)
    x = np.stack([graded(rng, m, n) * (1 + t) for t in range(tube)], axis=2).astype(np.float32)
    if wide:
        x = np.ascontiguousarray(x.transpose(1, 0, 2))
    sv = np.linalg.svd(x.astype(np.float64).sum(axis=2), compute_uv=False)
    tau = float(0.9 * sv[min(n // 3, n - 1)])
    z_ref, r_ref = tsvt_oracle(x, tau)
    announce("gram", size, wide)
    z, ranks = lib.tsvt(to_gpu(torch, x), tau, lib.PREC_FP32)
    gram = n <= 96 and m >= 12 * n
    assert rel_fro(z.cpu().numpy(), z_ref) <= (TOL_GRAM if gram else 1e-4)
    if gram:
        assert ranks == list(r_ref)


def test_gram_completion_warm_and_cold(monkeypatch):
    """Warm-started iterations, with and without the Gram path, a resumed solve
    bit for bit, and a persistent Jacobi that gives up."""
    torch = torch_cuda()
    rng = np.random.default_rng(4)
    x = graded(rng, 1400, 40, 1e-4)[:, :, None].astype(np.float32)
    mask = (rng.random(x.shape) < 0.5).astype(np.uint8)
    ref = admm.complete(x * mask, mask, max_iter=12, tol=0.0)["X"]
    xg, mg = to_gpu(torch, x * mask), to_gpu(torch, mask)
    solve = lambda **k: lib.tsvd_complete(xg, mg, 1e-2, 0.0, precision=lib.PREC_FP32, **k)[0].cpu().numpy()  # noqa: E731
    announce("gram completion")
    whole = solve(max_iter=12)
    assert_close_fp32(whole, ref, 1e-5, "gram completion")
    state = lib.SolverState(xg)
    solve(max_iter=5, state=state)
    np.testing.assert_array_equal(solve(max_iter=7, state=state, load=True), whole)
    monkeypatch.setenv("TSVD_PERSIST_SPIN", "0")
    announce("gram fallback")
    assert_close_fp32(solve(max_iter=12), ref, 1e-5, "gram fallback")
    monkeypatch.delenv("TSVD_PERSIST_SPIN")
    monkeypatch.setenv("TSVD_GRAM", "0")
    announce("global-memory Jacobi")
    assert_close_fp32(solve(max_iter=12), ref, 1e-4, "global-memory Jacobi")


@pytest.mark.parametrize("size", [(1400, 40, 1), (1100, 33, 3), (48, 40, 6)])
def test_refused_persistent_launch(monkeypatch, size):
    """A card that does not hold the persistent Jacobi's grid: the SVDs of the
    Gram path and of the ordinary one finish by another kernel."""
    torch = torch_cuda()
    m, n, tube = size
    rng = np.random.default_rng(m)
    x = np.stack([graded(rng, m, n, 1e-4) * (1 + t) for t in range(tube)], axis=2).astype(np.float32)
    tau = float(0.5 * np.linalg.svd(x.sum(axis=2), compute_uv=False)[n // 4])
    mask = (rng.random(x.shape) < 0.5).astype(np.uint8)
    monkeypatch.setenv("TSVD_PERSIST_CUS", "0")
    announce("refused launch", size)
    h = lib.Handle(0)
    for prof in (False, True):
        h.profile(prof)
        z, _ = lib.tsvt(to_gpu(torch, x), tau, lib.PREC_FP32, handle=h)
        err = rel_fro(z.cpu().numpy(), tsvt_oracle(x, tau)[0])
        assert err <= (TOL_GRAM if m > 1000 else 1e-4)   # or the FP32 rotations' own bar
    out = lib.tsvd_complete(to_gpu(torch, x * mask), to_gpu(torch, mask), 1e-2, 0.0, max_iter=6,
                            precision=lib.PREC_FP32, handle=h)[0]
    h.close()
    assert_close_fp32(out.cpu().numpy(), admm.complete(x * mask, mask, max_iter=6, tol=0.0)["X"], 1e-4,
                      "refused launch")


def test_gram_profile_counts_rotations():
    """The profile of a Gram-path call has its rotations, and leaves none to the
    next call's."""
    torch = torch_cuda()
    rng = np.random.default_rng(2)
    h = lib.Handle(0)
    h.profile(True)
    announce("gram profile")
    lib.tsvt(to_gpu(torch, graded(rng, 1200, 24)[:, :, None].astype(np.float32)), 1e-3, lib.PREC_FP32, handle=h)
    k = h.profile_read()["jacobi_persistent"]
    assert 0 < k["rotations"] <= k["pairs_visited"]
    before = k["rotations"]
    lib.tsvt(to_gpu(torch, np.zeros((32, 32, 1))), 0.5, handle=h)   # rotates nothing
    assert h.profile_read()["jacobi_persistent"]["rotations"] == before
    h.close()


@pytest.mark.parametrize("shape", [(65, 63, 1), (63, 130, 1), (64, 64, 1), (3, 200, 1)])
@pytest.mark.parametrize("fp32", [False, True])
def test_matrix_transforms(shape, fp32):
    """Every prologue and epilogue of the matrix form: prox, completion, both
    RPCA shrinks, ragged 64 x 64 tiles in either orientation."""
    torch = torch_cuda()
    rng = np.random.default_rng(shape[1])
    r = min(3, min(shape[:2]))
    low = (rng.normal(size=(shape[0], r)) @ rng.normal(size=(r, shape[1])))[:, :, None]
    mask = (rng.random(shape) < 0.6).astype(np.uint8)
    noisy = low + (rng.random(shape) < 0.05) * rng.normal(size=shape)
    dt, prec, bar = (np.float32, lib.PREC_FP32, 1e-4) if fp32 else (np.float64, lib.PREC_FP64, 1e-10)
    lam = 1.0 / np.sqrt(max(shape))
    announce("matrix", shape, fp32)
    got = [lib.tsvt(to_gpu(torch, low.astype(dt)), 1.0, prec)[0]]
    want = [tsvt_oracle(low.astype(dt), 1.0)[0]]
    got.append(lib.tsvd_complete(to_gpu(torch, (low * mask).astype(dt)), to_gpu(torch, mask), 1e-2, 0.0, max_iter=8,
                                 precision=prec)[0])
    want.append(admm.complete((low * mask).astype(dt), mask, max_iter=8, tol=0.0)["X"])
    for code, name in ((lib.SHRINK_L1, "l1"), (lib.SHRINK_L112, "l112")):
        lo, sp, _ = lib.trpca(to_gpu(torch, noisy.astype(dt)), lam, 1e-3, 0.0, code, max_iter=14, precision=prec)
        ref = admm.trpca(noisy.astype(dt), lam, max_iter=14, tol=0.0, shrink=name)
        got += [lo, sp]
        want += [ref["L"], ref["S"]]
    for k, (a, b) in enumerate(zip(got, want)):
        assert slice_rel_max(a.cpu().numpy(), b) <= bar, k
