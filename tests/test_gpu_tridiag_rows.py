"""Row-wise tridiagonalisation at the edges of its variants (one workgroup of four or eight waves,
grids of 2 to 17 columns per lane, ragged last workgroups), on a matrix whose columns need no
reflector, against the oracle or NumPy; and in a batch of
small problems, against their own handles."""

import numpy as np
import pytest

from oracle import fourdvar
from synthetic import batch_workloads
from tests._problems import rel, to_np
from tests.test_gpu_eig_sizes import _spd

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [1, 4, 31, 32, 63, 65, 66, 127, 128, 129, 192, 193, 320, 321, 513, 769])
def test_sizes_match_oracle(m):
    from paper_1906_01413_amd import Sketch
    n = m + 16
    A = _spd(n, 300 + m)
    Om = np.random.default_rng(400 + m).standard_normal((n, m))
    Y = A @ Om
    ro = fourdvar.rsvd(lambda X: A @ X, Om, q=0)
    lam, V, _ = Sketch(n, m).eig(Om, Y)
    lam, V = to_np(lam), to_np(V)
    assert np.max(np.abs(lam - ro.lam)) <= 1e-10 * ro.lam[0]
    assert rel((V * lam) @ V.T, (ro.V * ro.lam) @ ro.V.T) < 1e-10
    assert np.max(np.abs(V.T @ V - np.eye(m))) < 1e-11


@pytest.mark.parametrize("m", [9, 40, 150])
def test_diagonal_matrix(m):
    """Probes that are unit vectors of a diagonal matrix: K is diagonal, every reflector empty."""
    from paper_1906_01413_amd import Sketch
    n = m + 16
    d = np.random.default_rng(m).uniform(1.0, 5.0, size=n)
    Om = np.eye(n)[:, :m]
    lam, V, _ = Sketch(n, m).eig(Om, d[:, None] * Om)
    lam, V = to_np(lam), to_np(V)
    assert np.max(np.abs(lam - np.sort(d[:m])[::-1])) < 1e-13 * 5.0
    assert rel((V * lam) @ V.T, np.diag(np.concatenate([d[:m], np.zeros(16)]))) < 1e-12


@pytest.mark.parametrize("m", [12, 48])
def test_batch_of_small_problems(m):
    from paper_1906_01413_amd import RiotBatch
    probs = [p for p in (fourdvar.realize_l96(w, d)[0] for w, d in batch_workloads(6, 3))
             if p.n >= 2 * m][:4]
    specs = [dict(n=p.n, nsteps=p.nsteps, dt=p.h, forcing=p.F, obs_step=p.obs_step,
                  obs_idx=p.obs_idx, y=p.y, rinv=p.rinv, taps=p.taps, m=m + q)
             for q, p in enumerate(probs)]  # a block of another size each
    b = RiotBatch(specs)
    b.set_x([p.xb for p in probs])
    b.run(77)
    torch.cuda.synchronize()
    for j in range(len(probs)):
        r = b.problem(j)
        with torch.cuda.stream(b.stream):
            Om = r.philox_normal(probs[j].n, m + j, seed=77, stream=j)
            one, _, _ = r.rsvd(m + j - 4, 4, q=0, Omega=Om)
        torch.cuda.synchronize()
        one = to_np(one)
        assert np.max(np.abs(to_np(b.lam_of(j)) - one)) <= 1e-12 * one[0], j
