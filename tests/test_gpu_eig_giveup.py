"""The eigen-solve where the tridiagonalisation's grid gives up waiting for its workgroups (they did
not all get onto the chip): with no polls allowed the reduction must come from one workgroup, at
sizes of the register tiles and beyond, against NumPy."""

import ctypes

import numpy as np
import pytest

from tests._problems import rel
from tests.test_gpu_eig_sizes import _spd

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("m", [65, 128, 279, 280, 400, 1088])
@pytest.mark.parametrize("polls", [0, 1 << 22])
def test_no_polls_left(m, polls):
    from paper_1906_01413_amd.riot import load_library
    lib = load_library()
    work_doubles = lib["_ZN4riot16eig_work_doublesEi"]  # the library's internal entry
    work_doubles.restype = ctypes.c_size_t
    launch = lib["_ZN4riot10launch_eigEiPKdPdS2_S2_PiP12ihipStream_ti"]
    A = _spd(m, 700 + m)
    A = 0.5 * (A + A.T)
    K = torch.as_tensor(A, device="cuda")
    lam = torch.empty(m, dtype=torch.float64, device="cuda")
    Z = torch.empty(m, m, dtype=torch.float64, device="cuda")
    work = torch.zeros(work_doubles(m), dtype=torch.float64, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    p = [ctypes.c_void_p(t.data_ptr()) for t in (K, lam, Z, work, flag)]
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert launch(m, *p, stream, polls) == 0
    torch.cuda.synchronize()
    lam, V = lam.cpu().numpy(), Z.cpu().numpy().T
    assert flag.item() == 0
    ref = np.linalg.eigvalsh(A)[::-1]
    assert np.max(np.abs(lam - ref)) <= 1e-10 * ref[0]
    assert rel((V * lam) @ V.T, A) < 1e-10
    assert np.max(np.abs(V.T @ V - np.eye(m))) < 1e-11
