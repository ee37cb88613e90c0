"""Edges of the histogram's slices and ranges: one slice and two, experts that do not divide into the
ranges, ids outside [0, M), an id buffer that is not 16-byte aligned, no ids left for a slice."""
import numpy as np
import pytest

from gpu_util import announce, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,shift", [(1, 5, 0), (255, 65536, 0), (257, 65537, 1), (16385, 131075, 2),
                                       (70001, 200001, 3), (300000, 7, 0)])
def test_histogram_slices_and_ranges(M, n, shift):
    torch = require_gpu()
    from paper_2609_36301_amd import router
    rng = np.random.default_rng(M + n)
    ids = rng.integers(-3, M + 3, size=(n + shift, 1)).astype(np.int32)
    ids[rng.random(n + shift) < 0.2] = M - 1
    dev = to_dev(ids)[shift:]  # contiguous, 4 * shift bytes past an aligned address
    announce("expert_histogram M=%d n=%d shift=%d" % (M, n, shift))
    got = router.expert_histogram(dev, M)
    torch.cuda.synchronize()
    valid = ids[shift:][(ids[shift:] >= 0) & (ids[shift:] < M)]
    assert np.array_equal(got.cpu().numpy(), np.bincount(valid, minlength=M).astype(np.int32))
