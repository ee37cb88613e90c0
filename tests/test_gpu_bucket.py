"""GPU tests of the bucket route (the library's choice with m_chunks = 0 where no fused route
applies): bitwise agreement with the expert-resident route's kernels (m_chunks = 8: another screening,
the same z and the same exact sum) and oracle parity.

Shapes sit at the edges of the route's tiles: expert counts at, one past and just short of a
super-group of 256 and of a tile of 32; token counts at the edges of a wave's groups and on both sides
of the size where a workgroup takes one token; every rank and list size; more than one slab of
tokens; expert offsets that make the screening bounds loose; ties that overflow the lists."""
import numpy as np
import pytest

from oracle import parity
from gpu_util import route_lowrank
from paper_2609_36301_amd import router
from paper_2609_36301_amd.inputs import make_inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    # T, h, r, M, k, expert_bias_var
    (1, 64, 64, 4097, 1, 0.0),
    (31, 32, 64, 4352, 16, 0.0),         # whole super-groups
    (33, 48, 32, 8193, 8, 0.0),          # one expert in the last super-group
    (127, 64, 16, 16479, 9, 0.5),        # one short of a tile
    (129, 64, 64, 70000, 16, 0.5),       # several rounds of coarse values
    (1024, 96, 64, 5000, 8, 0.0),        # a workgroup per token
    (1025, 96, 64, 5000, 8, 0.0),        # two tokens per wave, one past the last pair
    (1100, 64, 32, 9000, 3, 0.5),
    (2050, 32, 16, 20001, 16, 0.25),
    (3000, 16, 64, 40000, 12, 0.5),
    (2048, 16, 32, 270000, 4, 0.0),      # a workgroup per token up to 2048 of them
    (2049, 16, 32, 270000, 4, 0.0),
    (3500, 16, 16, 33030, 8, 0.0),       # chunks of whole fours of super-groups, the last four not whole
    (3500, 16, 64, 21000, 8, 0.5),       # the same with one four per chunk
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_h%d_r%d_M%d_k%d_b%g" % s)
def test_bucket_route_matches_resident_kernels_and_oracle(shape):
    T, h, r, M, k, var = shape
    assert router.lowrank_route(T, h, r, M, k) == "expert-resident"
    inp = make_inputs(T, h, r, M, seed=T + M, expert_bias_var=var)
    got = route_lowrank(inp, k, histogram=True, tag="bucket")
    ref = route_lowrank(inp, k, histogram=True, m_chunks=8, tag="resident kernels")
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    rep = parity.evaluate(inp.x, inp.R1, inp.R2, k, got[0], got[1], got[2])
    assert rep.ok(), "%s: %s" % (shape, rep)


@pytest.mark.parametrize("T,h,r,M,k", [
    # the maxima of a slab take up to 208 MB
    (2900, 16, 16, 1300000, 8),    # about 1000 tokens: three even slabs, a workgroup per token
    (11000, 16, 16, 200000, 8),    # 5120: two whole rounds of the sweep and 760, two tokens per wave and one each
    (10300, 16, 32, 200003, 16),   # the same with a partial super-group
])
def test_bucket_route_more_than_one_slab(T, h, r, M, k):
    inp = make_inputs(T, h, r, M, seed=3)
    got = route_lowrank(inp, k, histogram=True, tag="bucket slabs")
    ref = route_lowrank(inp, k, histogram=True, m_chunks=8, tag="resident kernels")
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("T", [40, 1500])
def test_bucket_route_ties_take_the_exact_sweep(T):
    """Zero tokens tie every expert at 0 and overflow the lists; tokens beside them are unaffected.
    Repeated expert rows give equal logits and maxima: the lower id wins."""
    h, r, M, k = 64, 64, 6000, 8
    inp = make_inputs(T, h, r, M, seed=T, dup_expert_frac=0.3)
    inp.x[[0, 7, T - 1]] = 0
    idx, gate, topval, _ = route_lowrank(inp, k, tag="bucket ties")
    for t in (0, 7, T - 1):
        assert np.array_equal(idx[t], np.arange(k, dtype=np.int32))
        assert np.allclose(gate[t], 1.0 / k, atol=1e-7)
        assert np.all(topval[t] == 0.0)
    ref = route_lowrank(inp, k, m_chunks=8, tag="resident kernels")
    for a, b in zip((idx, gate, topval), ref[:3]):
        assert np.array_equal(a, b)
    rep = parity.evaluate(inp.x, inp.R1, inp.R2, k, idx, gate, topval)
    assert rep.ok(), str(rep)


WIDE = [
    # T, h, r, M, k, expert_bias_var: every rank the sweep is compiled for, padded and exact, and k > 16
    (70, 64, 48, 2048, 4, 0.0),
    (33, 64, 80, 2049, 9, 0.5),
    (1100, 32, 96, 2303, 17, 0.0),
    (300, 128, 112, 4111, 32, 0.0),
    (1300, 64, 128, 9000, 8, 0.5),
    (200, 48, 144, 5000, 20, 0.0),
    (1025, 32, 192, 3000, 16, 0.0),
    (129, 96, 240, 2600, 7, 0.25),
    (1050, 32, 256, 2304, 32, 0.0),
    (1030, 64, 16, 20000, 24, 0.0),
    (90, 64, 32, 7000, 32, 0.5),
    (1030, 64, 192, 3000, 16, 0.5),
    (1026, 32, 256, 2304, 32, 0.5),
    (33, 64, 256, 5000, 32, 0.5),
    (1030, 64, 128, 6000, 17, 0.5),
]


@pytest.mark.parametrize("shape", WIDE, ids=lambda s: "T%d_h%d_r%d_M%d_k%d_b%g" % s)
def test_bucket_route_at_wide_ranks_and_long_lists(shape):
    T, h, r, M, k, var = shape
    assert router.lowrank_route(T, h, r, M, k) == "wide"
    inp = make_inputs(T, h, r, M, seed=T + M, expert_bias_var=var)
    idx, gate, topval, counts = route_lowrank(inp, k, histogram=True, tag="wide bucket")
    rep = parity.evaluate(inp.x, inp.R1, inp.R2, k, idx, gate, topval)
    assert rep.ok(), "%s: %s" % (shape, rep)
    assert np.array_equal(counts, np.bincount(idx.ravel(), minlength=M).astype(np.int32))
