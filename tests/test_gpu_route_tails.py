"""Inputs that make the bucket route's lists long: padding tokens, experts that tie, expert offsets, values
that are not finite; and expert sets too large for its slabs.
Results stay exact, and a call does not stall: times are compared with the same shape on plain
inputs, with bounds several times what is measured and a fraction of what sweeping all experts for
such tokens takes."""
import numpy as np
import pytest

from oracle import parity
from gpu_util import announce, call_us, require_gpu, route_lowrank, to_dev
from paper_2609_36301_amd import router
from paper_2609_36301_amd.inputs import make_inputs, transposed_factors

pytestmark = pytest.mark.gpu


def _f64(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def _us(inp, k):
    require_gpu()
    T, h, r, M = inp.shape
    R1t, R2t = transposed_factors(inp)
    args = [to_dev(a) for a in (inp.x, R1t, R2t)]
    handle = router.LowrankRouter(T, h, r, M, k)
    announce("timing route_lowrank T=%d h=%d r=%d M=%d k=%d" % (T, h, r, M, k))
    return call_us(lambda: handle(*args))


@pytest.mark.parametrize("T,h,r,M,k", [(4096, 128, 128, 8192, 8), (2000, 64, 256, 2304, 32), (512, 64, 64, 20000, 16)])
def test_padding_tokens_cost_no_more_than_others(T, h, r, M, k):
    inp = make_inputs(T, h, r, M, seed=T + M)
    plain = _us(inp, k)
    zero = np.random.default_rng(M).random(T) < 0.3
    zero[[0, T - 1]] = True
    inp.x[zero] = 0
    padded = _us(inp, k)
    print("[time] plain %.1f us, 30%% zero tokens %.1f us" % (plain, padded), flush=True)
    assert padded < 1.5 * plain + 5.0  # 30% of the tokens do less; they were 6 to 40 times slower
    idx, gate, topval, _ = route_lowrank(inp, k, tag="padding")
    assert np.array_equal(idx[zero], np.broadcast_to(np.arange(k, dtype=np.int32), (zero.sum(), k)))
    assert np.allclose(gate[zero], 1.0 / k, atol=1e-7)
    assert np.all(topval[zero] == 0.0)
    rep = parity.evaluate(inp.x, inp.R1, inp.R2, k, idx, gate, topval)
    assert rep.ok(), str(rep)


# every form of the selection: rank (padded and exact), list length, one token per workgroup and packed
TIES = [(T, r, M, k) for T in (37, 1041) for r, M, k in (
    (16, 16500, 8), (16, 16500, 16), (32, 9000, 3), (64, 6000, 16), (48, 2048, 8), (80, 2300, 9), (128, 2049, 8),
    (128, 4100, 32), (112, 4111, 17), (256, 2100, 32), (240, 5000, 16), (32, 2600, 24))]


@pytest.mark.parametrize("shape", TIES, ids=lambda s: "T%d_r%d_M%d_k%d" % s)
def test_tying_experts(shape):
    """All experts are copies of six: each token ties M / 6 or so of them at its largest logit, and the
    smallest ids win.  Then all experts are equal, and all zero."""
    T, r, M, k = shape
    h = 64
    inp = make_inputs(T, h, r, M, seed=T + M + r)
    which = np.random.default_rng(M).integers(0, 6, M)
    inp.R2[:] = inp.R2[:, which]
    idx, gate, topval, counts = route_lowrank(inp, k, histogram=True, tag="copies of six")
    z = _f64(inp.x) @ _f64(inp.R1)
    logits = z @ _f64(inp.R2[:, [int(np.nonzero(which == i)[0][0]) for i in range(6)]])
    top2 = np.sort(logits, axis=1)[:, -2:]
    clear = top2[:, 1] - top2[:, 0] > 1e-4
    assert clear.mean() > 0.9
    first = np.stack([np.nonzero(which == i)[0][:k] for i in range(6)]).astype(np.int32)
    assert np.array_equal(idx[clear], first[logits.argmax(axis=1)][clear])
    assert np.allclose(gate, 1.0 / k, atol=1e-6)
    assert np.allclose(topval[clear], top2[clear, 1:], rtol=1e-4, atol=1e-4)
    assert np.array_equal(counts, np.bincount(idx.ravel(), minlength=M))
    if r in (16, 32, 64) and k <= 16:
        for a, b in zip((idx, gate, topval), route_lowrank(inp, k, m_chunks=8, tag="resident kernels")):
            assert np.array_equal(a, b)
    for value in (inp.R2[:, :1].copy(), 0):
        inp.R2[:] = value
        idx, gate, _, _ = route_lowrank(inp, k, tag="equal experts")
        assert np.array_equal(idx, np.broadcast_to(np.arange(k, dtype=np.int32), (T, k)))
        assert np.allclose(gate, 1.0 / k, atol=1e-6)
@pytest.mark.parametrize("T,r,M,k", [(1500, 256, 16384, 32), (1500, 128, 40000, 32), (700, 256, 40000, 16),
                                     (2100, 256, 9000, 8)])
def test_expert_offsets_at_long_ranks(T, r, M, k):
    """Offsets of the experts' rows (a skewed load) give them large norms, so that for tokens whose offsets
    cancel many buckets lie within the screening bounds of the threshold."""
    h = 128
    plain = _us(make_inputs(T, h, r, M, seed=1), k)
    inp = make_inputs(T, h, r, M, seed=2, expert_bias_var=0.5)
    skewed = _us(inp, k)
    print("[time] plain %.1f us, offsets %.1f us" % (plain, skewed), flush=True)
    assert skewed < 5.0 * plain  # 10 to 40 times slower with a sweep of all experts for such tokens
    idx, gate, topval, _ = route_lowrank(inp, k, tag="offsets")
    rep = parity.evaluate(inp.x, inp.R1, inp.R2, k, idx, gate, topval,
                          rows=np.arange(0, T, 3, dtype=np.int64))
    assert rep.ok(), str(rep)


@pytest.mark.parametrize("T,r,M,k", [(60, 64, 6000, 8), (1500, 64, 6000, 16), (1300, 128, 2100, 32), (40, 240, 3000, 8)])
def test_tokens_that_are_not_finite(T, r, M, k):
    """An infinite, a NaN and an overflowing token get k distinct experts (which, is not specified) and leave the
    others as they are."""
    inp = make_inputs(T, 64, r, M, seed=r)
    want = route_lowrank(inp, k, tag="finite")
    inp.x[3, 5] = 0x7F80           # +inf
    inp.x[T - 1, 0] = 0x7FC0       # NaN
    inp.x[8] = 0x7F00              # 1.7e38 in every entry
    bad = np.zeros(T, dtype=bool)
    bad[[3, 8, T - 1]] = True
    got = route_lowrank(inp, k, histogram=True, tag="not finite")
    for a, b in zip(got[:3], want[:3]):
        assert np.array_equal(a[~bad], b[~bad])
    ids = np.sort(got[0][bad], axis=1)
    assert ids.min() >= 0 and ids.max() < M and np.all(ids[:, 1:] != ids[:, :-1])
    assert got[3].sum() == T * k


def test_millions_of_experts():
    """Where the maxima of few tokens fill a slab, the call takes the resident route's kernels: the
    same result and no slower than asked for by a chunk count."""
    torch = require_gpu()
    T, h, r, M, k = 512, 64, 16, 1 << 23, 8
    gen = torch.Generator(device="cuda").manual_seed(1)
    x, R1t, R2t = (torch.randn(s, device="cuda", generator=gen).mul_(f).bfloat16()
                   for s, f in (((T, h), 1.0), ((r, h), h ** -0.5), ((M, r), r ** -0.5)))
    own = router.LowrankRouter(T, h, r, M, k, topval=True)
    asked = router.LowrankRouter(T, h, r, M, k, topval=True, m_chunks=1024)
    announce("route_lowrank T=%d h=%d r=%d M=%d k=%d" % (T, h, r, M, k))
    a, b = own(x, R1t, R2t), asked(x, R1t, R2t)
    assert torch.equal(a.idx, b.idx) and torch.equal(a.gate, b.gate) and torch.equal(a.topval, b.topval)
    a, b = call_us(lambda: own(x, R1t, R2t)), call_us(lambda: asked(x, R1t, R2t))
    print("[time] own choice %.1f us, resident kernels %.1f us" % (a, b), flush=True)
    assert a < 1.25 * b
