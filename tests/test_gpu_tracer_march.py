"""Marching tracer sweeps: every group size (1 to 8 steps per launch, ragged groups), strips that
wrap the whole period, several strips and chunks, control blocks of 1, 2 and 4 cells, and rows
with more observations than a wave has lanes, against the oracle."""

import numpy as np
import pytest

from oracle import advdiff
from tests._problems import rel, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,spb,ntb,block,m", [
    (64, 1, 3, 4, 2), (64, 2, 2, 1, 1), (64, 3, 2, 2, 3), (64, 4, 1, 4, 1), (128, 5, 2, 4, 2),
    (192, 6, 1, 2, 8), (64, 7, 2, 1, 2), (256, 8, 1, 4, 1), (64, 9, 2, 4, 3), (64, 17, 1, 2, 2),
])
def test_marching_sweeps_match_oracle(N, spb, ntb, block, m):
    from paper_1906_01413_amd import Tracer
    rng = np.random.default_rng(1000 * N + 10 * spb + block)
    g = advdiff.Grid(N=N, T=spb * ntb, dt=0.1, u0=5.0, u1=2.0, v=1.0, K=0.1, block=block, ntb=ntb)
    E = rng.uniform(0.1, 1.0, size=(N, N))
    # scattered observations, duplicates, and 80 in one row at one step
    t = np.concatenate([rng.integers(1, g.T + 1, size=60), np.full(80, g.T), [1, 1]])
    y = np.concatenate([rng.integers(0, N, size=60), np.full(80, 3), [0, 0]])
    x = np.concatenate([rng.integers(0, N, size=60), rng.integers(0, N, size=80), [N - 1, N - 1]])
    L1 = advdiff.sqrt_corr_1d(g.Nb, 3.0)
    ones = np.ones(t.size)
    tr = Tracer(dict(N=N, T=g.T, dt=g.dt, u0=g.u0, u1=g.u1, v=g.v, K=g.K, block=block, ntb=ntb),
                E, t, y, x, ones, ones, L1, 0.5, m)
    obs = advdiff.Obs(t, y, x)
    s0 = 0.3 * rng.standard_normal(g.ncontrol)
    ref, _ = advdiff.forward(g, E, s0, obs)
    # sums of non-negative terms, at most 6 T roundings each
    assert rel(to_np(tr.forward(s0)), ref) < 1e-13
    dS = rng.standard_normal((g.ncontrol, m))
    assert rel(to_np(tr.tangent(dS)), advdiff.tangent(g, E, s0, obs, dS)) < 1e-12
    f = rng.standard_normal((t.size, m))
    assert rel(to_np(tr.adjoint(f)), advdiff.adjoint(g, E, s0, obs, f)) < 1e-12


@pytest.mark.parametrize("N,ntb,block,m", [
    (64, 1, 4, 1), (64, 2, 1, 2), (128, 4, 2, 3), (192, 5, 4, 2), (256, 6, 4, 5),
])
def test_time_blocks_of_one_step(N, ntb, block, m):
    """A launch takes the steps of two time blocks (and an odd last one alone)."""
    test_marching_sweeps_match_oracle(N, 1, ntb, block, m)
