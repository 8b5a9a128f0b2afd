"""Tall sketches: the products over n on one wave per 64 x 64 tile and the triangular solves on one
wave per 32 rows, at ragged rows, columns, tiles and splits, on a diagonal operator against the
oracle."""

import numpy as np
import pytest

from oracle import fourdvar
from tests._problems import rel, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(16384, 289), (16401, 300), (24579, 353), (33000, 321), (40000, 176)])
def test_tall_sketch_matches_oracle(n, m):
    from paper_1906_01413_amd import Sketch
    rng = np.random.default_rng(n + m)
    d = 1e3 * 10.0 ** (-4.0 * rng.random(n))
    Om = rng.standard_normal((n, m))
    ro = fourdvar.rsvd(lambda X: d[:, None] * X, Om, q=0)
    lam, V, info = Sketch(n, m).eig(Om, d[:, None] * Om)
    lam, V = to_np(lam), to_np(V)
    assert info.orth_err < 1e-11
    assert np.max(np.abs(V.T @ V - np.eye(m))) < 1e-11
    assert np.max(np.abs(lam - ro.lam)) <= 1e-10 * ro.lam[0]
    X = rng.standard_normal((n, 3))
    assert rel((V * lam) @ (V.T @ X), (ro.V * ro.lam) @ (ro.V.T @ X)) < 1e-10


@pytest.mark.parametrize("n,m", [(16385, 470), (24601, 401), (33001, 449)])
def test_wide_tall_sketch_matches_oracle(n, m):
    """Wide enough (22 tiles of the lower half and more, 16 or 24 splits of 1024 rows) that the
    Gram matrices themselves go to the wave kernel, at ragged rows, columns and splits."""
    test_tall_sketch_matches_oracle(n, m)
