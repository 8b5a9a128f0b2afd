"""CholeskyQR of a batch (triangular solves through the inverses of the factor's 32 x 32 blocks) on
graded blocks: Hessians of eight decades, so that the products' columns are nearly dependent,
against the problems' own handles."""

import numpy as np
import pytest

from oracle import bcov
from tests._problems import rel, to_np

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("ns,ms", [([256, 40], [96, 20]), ([512, 1032, 264], [130, 31, 33]), ([2048], [256])])
def test_graded_blocks(ns, ms):
    from paper_1906_01413_amd import RiotBatch
    specs, xs = [], []
    for j, n in enumerate(ns):
        rng = np.random.default_rng(n + j)
        step, idx = np.repeat([2, 4], n), np.tile(np.arange(n), 2)
        specs.append(dict(n=n, nsteps=4, dt=0.01, forcing=8.0, obs_step=step, obs_idx=idx,
                          y=8.0 + rng.standard_normal(2 * n),
                          rinv=10.0 ** np.tile(rng.uniform(-4.0, 4.0, size=n), 2),
                          taps=bcov.gaussian_taps(1.0, 1.0), m=ms[j]))
        xs.append(8.0 + rng.standard_normal(n))
    b = RiotBatch(specs)
    b.set_x(xs)
    b.run(5)
    torch.cuda.synchronize()
    for j, (n, m) in enumerate(zip(ns, ms)):
        r = b.problem(j)
        with torch.cuda.stream(b.stream):
            Om = r.philox_normal(n, m, seed=5, stream=j)
            lam1, V1, _ = r.rsvd(m, 0, q=0, Omega=Om)
        torch.cuda.synchronize()
        lam, V, lam1, V1 = to_np(b.lam_of(j)), to_np(b.V_of(j)), to_np(lam1), to_np(V1)
        assert np.max(np.abs(V.T @ V - np.eye(m))) < 1e-11
        assert np.max(np.abs(lam - lam1)) <= 1e-10 * lam1[0]
        X = np.random.default_rng(j).standard_normal((n, 3))
        assert rel((V * lam) @ (V.T @ X), (V1 * lam1) @ (V1.T @ X)) < 1e-10
