"""GPU parity of the refinement step's norms at the edges of the groups in which
its blocks count themselves done: 1, 64, 65, 72, 128, 300 and 2880 blocks. The
first residual of a solve from a random iterate against the oracle's operator,
in FP64 to 1e-12 (sums of up to 6M squares of values without cancellation:
about 1e-14); a second solve on the same handle gives the same history to the
bit, so the counts are back at zero.
"""
import numpy as np
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for

pytestmark = pytest.mark.gpu

SHELLS = [(8, 4, 4), (64, 32, 32), (64, 52, 20), (64, 32, 33), (64, 64, 32), (128, 100, 41),
          (320, 256, 72)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("size", SHELLS, ids=lambda s: "x".join(map(str, s)))
def test_norms_of_a_refinement_step(size, prec):
    sh = shellgen.Shell("norms", *size, stretch=1.02)
    a, b = shellgen.alpha(sh), shellgen.rhs(sh)
    u0 = np.random.default_rng(23).standard_normal(sh.shape)
    L = oracle.build_hierarchy(sh, a, levels=1)
    ref = np.linalg.norm((b - oracle.apply(L[0], u0)).ravel())
    S = solver_for(sh, a, precision=prec)
    hists = [S.solve(t(b), tol=1e-3, u0=t(u0))[1].res_hist
             for _ in range(2)]
    log(f"norms {size} {prec}: {hists[0][0] / ref - 1:.1e}, {len(hists[0])} norms")
    assert abs(hists[0][0] - ref) <= 1e-12 * ref
    assert list(hists[0]) == list(hists[1])
