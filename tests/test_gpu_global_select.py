"""Compression Method 1 at the edges of its selection: the first and the last
value, the whole spectrum and more, several slice multiplicities, more values
than threads, and an all-zero spectrum, against the FP64 oracle."""

import numpy as np
import pytest

import paper_1407_1785_amd as lib
from oracle import compress as C
from tests.gpu_util import announce, rel_fro, to_gpu, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(7, 5, 1), (12, 9, 2), (9, 12, 7), (40, 36, 60), (18, 16, 128)])
def test_global_selection(shape):
    torch = torch_cuda()
    rng = np.random.default_rng(len(shape) + shape[0])
    m = rng.normal(size=shape) * np.exp(-rng.uniform(0, 3, size=shape[:2] + (1,)))
    total = min(shape[:2]) * shape[2]
    mg = to_gpu(torch, m)
    announce("global selection", shape)
    for k in sorted({1, 2, 3, total // 3, total - 2, total - 1, total}):
        if not 1 <= k <= total:
            continue
        out, _ = lib.compress(mg, lib.COMPRESS_TSVD, k)
        ref = C.method1(m, k)
        # the bar of the other compression tests
        assert rel_fro(out.cpu().numpy(), ref) <= 1e-10 if np.any(ref) else not np.any(out.cpu().numpy())
    out, _ = lib.compress(torch.zeros_like(mg), lib.COMPRESS_TSVD, max(total // 2, 1))
    assert not out.any()
