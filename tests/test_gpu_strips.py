"""Strips of the Lorenz-96 integrations at the sizes where their layout changes (one, four and
eight waves, halos longer than the state, a short last strip; beyond 4207 elements the lane
layout), windows longer and shorter than the steps between two halo refreshes, strips with no,
few and all positions observed, and the kernel of two members per workgroup with an odd block,
against the oracle."""

import numpy as np
import pytest

from oracle import bcov, fourdvar, l96
from tests._problems import rel, riot_for, to_np

pytestmark = pytest.mark.gpu


def _problem(n, T, seed):
    """Steps 0 and T, one dense step, one step observed in the first 130 elements only, scattered
    single observations and duplicates."""
    rng = np.random.default_rng(seed)
    x = 8.0 + rng.standard_normal(n)
    t = [np.full(n, max(T - 1, 0)), np.full(min(n, 130), T // 2), [0, 0, T, T, T]]
    i = [np.arange(n), np.arange(min(n, 130)), [0, n - 1, n // 2, n // 2, n // 3]]
    k = rng.integers(5, 40)
    t.append(rng.integers(0, T + 1, size=k))
    i.append(rng.integers(0, n, size=k))
    t, i = np.concatenate(t), np.concatenate(i)
    y = 8.0 + rng.standard_normal(t.size)
    return fourdvar.Problem(n, T, 0.01, 8.0, t, i, y, rng.uniform(0.5, 2.0, t.size), x,
                            bcov.gaussian_taps(2.0, 1.0))


@pytest.mark.parametrize("n,T,m", [
    (4, 3, 2), (5, 20, 3), (61, 9, 2), (62, 9, 2), (77, 17, 1), (78, 17, 1), (93, 6, 2),
    (94, 6, 2), (141, 7, 2), (142, 17, 2), (211, 9, 2), (212, 4, 2), (213, 13, 1), (308, 7, 2),
    (309, 9, 3), (564, 5, 2), (565, 9, 2), (1001, 9, 3), (1076, 18, 2), (1080, 15, 2),
    (2152, 8, 2), (2160, 9, 257), (4096, 17, 2), (4192, 4, 2), (4208, 9, 3), (8192, 9, 2),
])
def test_strips_match_oracle(n, T, m):
    p = _problem(n, T, 10 * n + T)
    lin = fourdvar.linearize(p, p.xb)
    r = riot_for(p, m_max=m)
    # each value is a sum of products of at most 20 steps' rounding errors (T e^(T dt 2) eps)
    assert rel(to_np(r.forecast(p.xb, T)), l96.forecast(p.xb, T, p.h, p.F)) < 1e-13
    d, g, J = r.linearize(p.xb)
    assert rel(to_np(d), lin.d) < 1e-12
    assert rel(to_np(g), lin.g) < 1e-11
    W = np.random.default_rng(n).standard_normal((n, m))
    assert rel(to_np(r.hess_apply(W)), fourdvar.hvp(p, lin, W)) < 1e-11


@pytest.mark.parametrize("n,T,m", [(4208, 9, 3), (4320, 7, 2), (4336, 5, 3), (4432, 4, 257), (4448, 4, 2)])
def test_last_strips_match_oracle(n, T, m):
    """The largest strips, whose halos last two steps (n = 4208 .. 4320) and one (.. 4432), and the
    first size of the lane layout (4448)."""
    test_strips_match_oracle(n, T, m)


@pytest.mark.parametrize("n,T", [(40, 2), (212, 1), (309, 2), (1001, 3), (1080, 5), (2160, 1), (4096, 2), (4208, 1)])
def test_forecast_in_place(n, T):
    """x0 and xout the same buffer, fewer steps than between two halo refreshes."""
    import ctypes
    import torch
    from paper_1906_01413_amd.riot import load_library
    p = _problem(n, 4, n)
    r = riot_for(p, m_max=1)
    x = torch.as_tensor(p.xb, device="cuda")
    ref = to_np(r.forecast(x, T))
    assert rel(ref, l96.forecast(p.xb, T, p.h, p.F)) < 1e-13
    for _ in range(20):
        y = x.clone()
        ptr = ctypes.c_void_p(y.data_ptr())
        assert load_library().riot_forecast(r.h, ptr, T, ptr) == 0
        assert np.array_equal(to_np(y), ref)


@pytest.mark.parametrize("n,T,m", [
    (129, 9, 2), (130, 4, 1), (141, 17, 3), (142, 9, 3), (143, 17, 1), (211, 6, 2), (213, 12, 2), (217, 7, 2),
])
def test_two_strips_match_oracle(n, T, m):
    """Two waves: what is too long for one and too short for four."""
    test_strips_match_oracle(n, T, m)
