"""Edges of the histogram's slices and ranges: one slice and two, experts that do not divide into the
ranges, ids outside [0, M), an id buffer that is not 16-byte aligned, no ids left for a slice; the
hash table of the largest expert sets; a hot expert must not stall a call."""
import numpy as np
import pytest

from gpu_util import announce, call_us, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n,shift", [(1, 5, 0), (255, 65536, 0), (257, 65537, 1), (16385, 131075, 2),
                                       (70001, 200001, 3), (300000, 7, 0), (600, 16384, 1),
                                       (1 << 20, 300000, 0), ((1 << 20) + 20000, 600001, 1),
                                       (70000000, 1030, 2)])
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


def test_histogram_of_the_largest_expert_set():
    """2^30 experts: more ranges than a grid has rows."""
    torch = require_gpu()
    from paper_2609_36301_amd import router
    M = 1 << 30
    ids = np.array([[0], [M - 1], [5], [M - 1], [-1], [M // 2]], dtype=np.int32)
    announce("expert_histogram M=2^30")
    got = router.expert_histogram(to_dev(ids), M)
    where = torch.nonzero(got).flatten().cpu().numpy()
    assert where.tolist() == [0, 5, M // 2, M - 1]
    assert got[torch.from_numpy(where).cuda()].tolist() == [1, 1, 1, 2]


@pytest.mark.parametrize("M,n", [(64, 65536), (256, 262144), (1024, 65536), (4096, 262144)])
def test_histogram_hot_experts(M, n):
    """A few experts with most of the ids cost little more than an even spread (one workgroup's atomics on
    one address took three times as long)."""
    torch = require_gpu()
    from paper_2609_36301_amd import router
    rng = np.random.default_rng(M)
    even = to_dev(rng.integers(0, M, size=(n // 8, 8)).astype(np.int32))
    ids = (rng.random((n // 8, 8)) ** 6 * M).astype(np.int32)
    hot = to_dev(ids)
    announce("timing expert_histogram M=%d n=%d" % (M, n))
    a, b = call_us(lambda: router.expert_histogram(even, M)), call_us(lambda: router.expert_histogram(hot, M))
    print("[time] even %.1f us, skewed %.1f us" % (a, b), flush=True)
    assert b < 1.4 * a + 1.0
    assert np.array_equal(router.expert_histogram(hot, M).cpu().numpy(), np.bincount(ids.ravel(), minlength=M))
