"""Inputs that make the bucket route's lists long must not stall a call: padding tokens.  Times are
compared with the same shape on plain inputs; the bounds are several times what is measured and
a fraction of what sweeping all experts for such tokens takes."""
import numpy as np
import pytest

from oracle import parity
from gpu_util import announce, call_us, require_gpu, route_lowrank, to_dev
from paper_2609_36301_amd import router
from paper_2609_36301_amd.inputs import make_inputs, transposed_factors

pytestmark = pytest.mark.gpu


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
