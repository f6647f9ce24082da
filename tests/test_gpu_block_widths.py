"""Jacobi block pairs narrower than the pair groups of a workgroup: the ring of
cross steps closes over the columns there are.  Widths of 1 to 16, equal and
one apart, odd and even, two to twelve blocks (one block of a pair moves between
rounds), in the single-problem and both batched schedules, against the FP64
oracle; the batched schedules meet the same pairs in the same order and agree
bit for bit."""

import numpy as np
import pytest

import paper_1407_1785_amd as lib
from oracle import admm
from oracle.tsvt import tsvt as tsvt_oracle
from tests.gpu_util import announce, rel_fro, to_gpu, torch_cuda

pytestmark = pytest.mark.gpu

# block widths: 1; 1, 2; 2, 3; 8, 9; 9; 15, 16; 16; 8, 9 in four blocks; 12, 14 and 15, 16 in
# six; 14 in eight; 14 in ten; 14 and 15 in twelve
WIDTHS = [2, 3, 5, 17, 18, 31, 32, 33, 72, 87, 96, 112, 140, 170]


@pytest.mark.parametrize("n", WIDTHS)
@pytest.mark.parametrize("batch", [False, True])
def test_narrow_blocks(monkeypatch, n, batch):
    torch = torch_cuda()
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n + 5, n, 2))
    mask = (rng.random(x.shape) < 0.6).astype(np.uint8)
    ref = admm.complete(x * mask, mask, max_iter=3, tol=0.0)["X"]
    announce("block widths", n, batch)
    if not batch:
        out, _ = lib.tsvd_complete(to_gpu(torch, x * mask), to_gpu(torch, mask), 1e-2, 0.0, max_iter=3)
        assert rel_fro(out.cpu().numpy(), ref) <= 1e-10
        return
    monkeypatch.setenv("TSVD_TUNE", "0")
    monkeypatch.setenv("TSVD_BATCH_BW", "16")
    out = []
    for pairs_min in ("1", "99"):
        monkeypatch.setenv("TSVD_PAIRS_MIN", pairs_min)
        h = lib.Handle(0, 1 << 28)
        p = lib.complete_problem(to_gpu(torch, x * mask), to_gpu(torch, mask), 1e-2, 0.0, max_iter=3)
        (status, _), = lib.batch_run([p], handle=h)
        h.close()
        assert status == 0
        out.append(p.out.cpu().numpy())
        assert rel_fro(out[-1], ref) <= 1e-10
    np.testing.assert_array_equal(out[0], out[1])


@pytest.mark.parametrize("size", [(500, 20, 2), (560, 32, 2), (600, 12, 2), (545, 9, 2), (600, 17, 2)])
def test_few_columns_many_rows(size):
    """One block pair of 16 columns a slice, too many rows for the persistent
    kernel (17 to 20 row groups in FP64): narrower blocks, in one launch."""
    torch = torch_cuda()
    x = np.random.default_rng(size[0]).normal(size=size)
    tau = 0.7 * np.sqrt(size[0])
    h = lib.Handle(0)
    h.profile(True)
    announce("few columns", size)
    z, ranks = lib.tsvt(to_gpu(torch, x), tau, handle=h)
    kinds = h.profile_read()
    h.close()
    ref, rank_ref = tsvt_oracle(x, tau)
    assert rel_fro(z.cpu().numpy(), ref) <= 1e-12 and ranks == list(rank_ref)
    assert "jacobi_persistent" in kinds and "jacobi_cross" not in kinds


@pytest.mark.parametrize("size", [(613, 27, 1), (540, 100, 2), (320, 320, 2)])
def test_blocks_as_large_as_the_lds(size):
    """Stacked columns of 640 rows in FP64: 16 of them are the whole LDS, which
    leaves none for the kernels' own words, so narrower blocks run."""
    torch = torch_cuda()
    x = np.random.default_rng(size[0]).normal(size=size)
    tau = 0.7 * np.sqrt(size[0])
    announce("largest blocks", size)
    z, ranks = lib.tsvt(to_gpu(torch, x), tau)
    ref, rank_ref = tsvt_oracle(x, tau)
    assert rel_fro(z.cpu().numpy(), ref) <= 1e-12 and ranks == list(rank_ref)
