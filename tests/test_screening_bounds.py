"""The bucket route's screening bounds, emulated in float32 on the CPU: |z_hi.u - z.u| <= c N + d m with c and d of
a token (screen_scale, mean_scale) and N, m of a row (row_bounds), whatever offset the rows carry."""
import numpy as np
import pytest

F = np.float32


def _bf16(a):
    u = a.astype(F).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(F)


@pytest.mark.parametrize("offset", [0.0, 0.5, 4.0, 100.0, 1e4])
@pytest.mark.parametrize("r", [16, 48, 64, 256])
def test_bounds_hold(r, offset):
    rng = np.random.default_rng(r)
    for scale in (1.0, 1e-3, 1e6):
        z = (rng.standard_normal((200, r)) * scale).astype(F)
        z[:50] += F(5 * scale)  # tokens whose own mean is large
        u = _bf16(rng.standard_normal((1000, r)) * r ** -0.5 + rng.standard_normal((1000, 1)) * offset)
        hi = _bf16(z)
        lo = z - hi
        hi2 = (hi ** 2).sum(1, dtype=F)
        c = (np.sqrt((lo ** 2).sum(1, dtype=F)) + F(r * 2.0 ** -23) * np.sqrt(hi2)) * F(1 + 2.0 ** -10)
        d = (np.abs(lo.sum(1, dtype=F)) + F(r) * np.sqrt(F(r) * hi2) * F(2.0 ** -22)) * F(1 + 2.0 ** -10)
        ss, su = (u ** 2).sum(1, dtype=F), u.sum(1, dtype=F)
        mu = su * F(1.0 / r)
        n = np.sqrt(ss * F(2.0 ** -13) + np.maximum(ss - su * mu, F(0))) * F(1 + 2.0 ** -20)
        m = np.abs(mu) * F(1 + 2.0 ** -20)
        err = np.abs((hi @ u.T).astype(np.float64) - z.astype(np.float64) @ u.T.astype(np.float64))
        width = c[:, None].astype(np.float64) * n + d[:, None].astype(np.float64) * m
        assert (err <= width).all(), (err / width).max()
