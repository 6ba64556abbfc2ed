"""mg_solve_noalloc's limit on the grid: the last grid below it is solved as by
mg_solve, the first above is refused, with the two numbers that were compared."""
import ctypes as C
import re

import pytest
import torch

from gpu_util import log

from paper_2307_04528_amd import Solver, _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nlat,fits", [(1026, True), (1028, True), (1030, False)])
def test_limit_of_noalloc(nlat, fits):
    # blocks of 256 columns: 32,832, 32,888 and 32,960 of 32,895
    nlon = 8192 if nlat != 1028 else 8190
    a = torch.full((1, nlat, nlon), 100.0, dtype=torch.float64, device="cuda")
    b = torch.empty_like(a).uniform_(-1, 1)
    S = Solver(nlon, nlat, 1, a, levels=2, coarse_sweeps=1, max_iters=2)
    u = torch.zeros_like(b)
    st = L.mg_stats()
    status = L.lib().mg_solve_noalloc(S.handle, b.data_ptr(), u.data_ptr(), 1e-13, C.byref(st))
    if fits:
        assert status == L.MG_ERR_NOT_CONVERGED
        v, sv = S.solve(b, tol=1e-13, u0=torch.zeros_like(b))
        assert torch.equal(u, v) and st.relres == sv.relres
    else:
        assert status == L.MG_ERR_ARG
        message = L.lib().mg_last_error(S.handle).decode()
        log(message)
        needed, available = map(int, re.findall(r"\d+", message))
        assert needed == nlon * nlat // 256 and needed > available
