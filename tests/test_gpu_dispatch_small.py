"""Edges of the one-workgroup sort (up to 4096 entries): the largest key of one 10-bit pass and the first
past it, the largest entry count, one entry, ids outside [0, M)."""
import numpy as np
import pytest

import oracle
from gpu_util import announce, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,M", [(1, 1, 1), (512, 8, 1023), (512, 8, 1024), (1025, 1, 1022), (64, 3, 255),
                                   (333, 7, 70000)])
def test_small_sort_edges(T, k, M):
    torch = require_gpu()
    from paper_2609_36301_amd import router
    rng = np.random.default_rng(T + M)
    idx = rng.integers(-1, M + 1, size=(T, k)).astype(np.int32)
    idx[rng.random((T, k)) < 0.3] = M - 1
    announce("dispatch_sort T=%d k=%d M=%d" % (T, k, M))
    offsets, srt = router.dispatch_sort(to_dev(idx), M)
    torch.cuda.synchronize()
    want_o, want_s = oracle.dispatch_sort(idx, M)
    assert np.array_equal(offsets.cpu().numpy().astype(np.int64), want_o)
    assert np.array_equal(srt.cpu().numpy().astype(np.int64), want_s)
