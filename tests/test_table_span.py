"""The span of the weight table (largest score difference that can carry a weight), enumerated against
Algorithm 2 and Eq. 10 in Python integers."""
import numpy as np
import pytest

import oracle


def weight(x, p):
    xs = x << p.x_shift
    q = (xs * p.exp_mul) >> 32
    r = xs + q * p.s_inv
    y = np.where(q > 31, 0, ((r >> 1) + p.s_inv) >> np.minimum(q, 31))
    return np.minimum(127, (y * p.p_mul) >> p.p_shift)


def table_span(p):
    y1 = -(-(1 << p.p_shift) // p.p_mul)
    assert 1274 * y1 >= 10 * p.s_inv and 128 * y1 <= 2 * p.s_inv      # holds for constants from real scales
    return ((8 * p.s_inv - 128 * y1) >> p.x_shift) + 1


@pytest.mark.parametrize("seed", range(6))
def test_span_is_exact(seed):
    rng = np.random.default_rng(seed)
    for _ in range(60):
        s_real = float(10 ** rng.uniform(-2.2, 0.9))
        try:
            p = oracle.derive_params(s_real, float(10 ** rng.uniform(-2.2, 0.9)), 64)
        except ValueError:
            continue
        x_p = table_span(p)
        x = -np.arange(0, 21 * p.s_inv // (1 << p.x_shift) + 2, dtype=np.int64)
        w = weight(x, p)
        assert w[x_p:].max() == 0 and w[x_p - 1] > 0, p
        assert x_p <= -(-8 * p.s_inv >> p.x_shift)
