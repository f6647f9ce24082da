"""Jacobi block pairs with one block in registers and one in LDS: the sizes at
which a block only just fits the LDS, in the single-problem and the batched
schedules, against the FP64 oracle."""

import numpy as np
import pytest

import paper_1407_1785_amd as lib
from oracle import admm
from oracle.tsvt import tsvt as tsvt_oracle
from tests.gpu_util import announce, assert_close_fp32, rel_fro, to_gpu, torch_cuda

pytestmark = pytest.mark.gpu


def tau_between(x):
    sv = np.linalg.svd(x.sum(axis=2), compute_uv=False)
    k = len(sv) // 3
    return float(0.5 * (sv[k - 1] + sv[k]))


# stacked columns of 18, 19 and 20 groups of 32 rows: 16-column FP64 blocks end
# at 19 groups, where an 8-column block takes over
@pytest.mark.parametrize("size", [(300, 250), (300, 260), (310, 300)])
@pytest.mark.parametrize("fp32", [False, True])
def test_prox_at_the_lds_edge(size, fp32):
    torch = torch_cuda()
    rng = np.random.default_rng(size[1])
    x = rng.normal(size=size + (2,))
    tau = tau_between(x)
    if fp32:
        # the threshold in a spectral gap: inside a band of n values the FP32
        # form leaves couplings of 32 sqrt(m) eps = 7e-5 per pair, together up
        # to 7e-5 sqrt(n) = 1e-3 of the result, over the bar
        low = np.einsum("ikt,kjt->ijt", rng.normal(size=(size[0], 6, 2)), rng.normal(size=(6, size[1], 2)))
        x = (low + 0.01 * x).astype(np.float32)
        tau = 2.0
    z_ref, _ = tsvt_oracle(x, tau)
    announce("lds edge", size, fp32)
    z, _ = lib.tsvt(to_gpu(torch, x), tau, lib.PREC_FP32 if fp32 else lib.PREC_FP64)
    if fp32:
        assert_close_fp32(z.cpu().numpy(), z_ref, 1e-4, f"lds edge {size}")
    else:
        assert rel_fro(z.cpu().numpy(), z_ref) <= 1e-10


@pytest.mark.parametrize("bw", ["4", "8", "16"])
@pytest.mark.parametrize("pairs_min", ["1", "99"])
def test_batch_schedules_at_every_width(monkeypatch, bw, pairs_min):
    """Both batched schedules at each block width, ragged last blocks."""
    torch = torch_cuda()
    monkeypatch.setenv("TSVD_TUNE", "0")
    monkeypatch.setenv("TSVD_BATCH_BW", bw)
    monkeypatch.setenv("TSVD_PAIRS_MIN", pairs_min)
    rng = np.random.default_rng(int(bw))
    x = rng.normal(size=(45, 37, 3))
    mask = (rng.random(x.shape) < 0.6).astype(np.uint8)
    announce("batch", bw, pairs_min)
    h = lib.Handle(0, 1 << 28)
    p = lib.complete_problem(to_gpu(torch, x * mask), to_gpu(torch, mask), 1e-2, 0.0, max_iter=4)
    (status, _), = lib.batch_run([p], handle=h)
    h.close()
    assert status == 0
    ref = admm.complete(x * mask, mask, max_iter=4, tol=0.0)
    assert rel_fro(p.out.cpu().numpy(), ref["X"]) <= 1e-10
