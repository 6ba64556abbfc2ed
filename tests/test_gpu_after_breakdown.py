"""A solve that ends in MG_ERR_BREAKDOWN leaves nothing behind: the next ones on the
handle, on the same and on another stream, have the bits and the history of a fresh
handle's (the block counters of the refinement step are cleared again)."""
import pytest
import torch

import shellgen
from gpu_util import log, t, solver_for

from paper_2307_04528_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["mixed", "fp64", "fp32"])
def test_solves_after_a_breakdown(prec):
    sh = shellgen.Shell("after", 64, 64, 32, stretch=1.05)
    a, b = shellgen.alpha(sh), t(shellgen.rhs(sh))
    tol = 1e-3 if prec == "fp32" else 1e-8
    u, st = solver_for(sh, a, precision=prec).solve(b, tol=tol)
    S = solver_for(sh, a, precision=prec)
    bad = b.clone()
    bad[3, 4, 5] = float("nan")
    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            with pytest.raises(L.MGError) as e:
                S.solve(bad, tol=tol)
            assert e.value.status == L.MG_ERR_BREAKDOWN
            for _ in range(2):
                v, sv = S.solve(b, tol=tol)
                assert torch.equal(u, v) and st.res_hist == sv.res_hist
    log(f"after a breakdown {prec}: {st.iters} iterations each time")
