"""A batch in a workspace of stale values: what earlier work left in device memory (NaN, Inf, large
values) must not reach a result."""

import numpy as np
import pytest

from oracle import bcov

pytestmark = pytest.mark.gpu


def _problem(n, seed):
    rng = np.random.default_rng(seed)
    step = np.repeat([2, 5, 8], n // 2)
    idx = np.tile(np.arange(0, n - n % 2, 2), 3)
    return dict(n=n, nsteps=8, dt=0.01, forcing=8.0, obs_step=step, obs_idx=idx,
                y=8.0 + rng.standard_normal(step.size), rinv=np.ones(step.size),
                taps=bcov.gaussian_taps(2.0, 1.0)), 8.0 + rng.standard_normal(n)


def _run(fill, prec, monkeypatch):
    import torch
    from paper_1906_01413_amd import RiotBatch
    empty = torch.empty

    def filled(*a, **k):
        t = empty(*a, **k)
        if t.is_cuda and t.dtype == torch.uint8:
            t[: t.numel() // 8 * 8].view(torch.float64).fill_(fill)
        return t

    probs = [_problem(n, n) for n in (40, 512, 1040)]
    with monkeypatch.context() as mp:
        mp.setattr(torch, "empty", filled)
        b = RiotBatch([dict(p, m=m) for (p, _), m in zip(probs, (17, 70, 33))], prec=prec)
    b.set_x([x for _, x in probs])
    torch.cuda.synchronize()
    b.run(1)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (b.d, b.grad, b.lam, b.V, b.dz, b.dx)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("fill", [float("nan"), float("inf"), 1e300])
def test_stale_workspace_changes_nothing(fill, prec, monkeypatch):
    for clean, stale in zip(_run(0.0, prec, monkeypatch), _run(fill, prec, monkeypatch)):
        assert np.array_equal(clean, stale) and np.isfinite(stale).all()
