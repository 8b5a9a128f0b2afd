"""The lane layout, which FP32 handles have: every elements-per-lane choice, odd sizes among them,
against the FP64 oracle within ten times what the oracle's own sweeps rounded to FP32 are off."""

import numpy as np
import pytest

from oracle import fourdvar, precise
from tests._problems import rel, riot_for, to_np
from tests.test_gpu_strips import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,E", [
    (13, 0), (77, 1), (1001, 0), (40, 1), (40, 2), (40, 4), (40, 8), (48, 16), (1024, 1), (2048, 2),
    (4096, 4), (1024, 8), (4096, 8), (8192, 16),
])
def test_fp32_layouts_match_oracle(n, E):
    p = _problem(n, 9, n + E)
    lin = fourdvar.linearize(p, p.xb)
    r = riot_for(p, m_max=3, prec=1, elems_per_lane=E)
    d, g, J = r.linearize(p.xb)
    assert rel(to_np(d), lin.d) < 1e-12  # the trajectory stays FP64
    assert rel(to_np(g), lin.g) < 10.0 * rel(precise.grad_lowprec(p, lin), lin.g)
    W = np.random.default_rng(n).standard_normal((n, 3))
    Y, Yo, Y32 = to_np(r.hess_apply(W)), fourdvar.hvp(p, lin, W), precise.hvp_lowprec(p, lin, W)
    for c in range(3):
        assert rel(Y[:, c], Yo[:, c]) < 10.0 * rel(Y32[:, c], Yo[:, c]), c
