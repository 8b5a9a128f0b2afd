"""The tracer's workspace query for very long windows (no GPU needed): a size, without tables of the
window's length."""

import ctypes
import resource

import numpy as np
import pytest


@pytest.mark.parametrize("nsteps,ntb", [((1 << 31) - 1, 1), (1 << 30, 1 << 30), ((1 << 30) + 1, (1 << 30) + 1)])
def test_size_of_a_long_window(nsteps, ntb):
    from paper_1906_01413_amd.riot import _TracerDesc, load_library
    lib = load_library()
    N = 64
    E, L1 = np.ones((N, N)), np.eye(N // 4)
    d = _TracerDesc()
    d.N, d.nsteps, d.block, d.ntb, d.nobs, d.m_max = N, nsteps, 4, ntb, 0, 1
    d.dt, d.u0, d.u1, d.v, d.K, d.sigma = 0.1, 2.0, 1.0, 1.0, 0.1, 0.5
    d.E = E.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    d.L1 = L1.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
    nb = lib.riot_tracer_workspace_bytes(ctypes.byref(d))
    grown = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before
    launches = (ntb + 1) // 2 if nsteps == ntb else ntb * -(-(nsteps // ntb) // 8)
    # the weights of every block and two pointer tables per launch; the controls are less
    least = 8 * N * N * ntb + 8 * launches * (N + 1)
    assert least < nb < 1.5 * least + (1 << 20)
    assert grown < 1 << 16  # KiB
