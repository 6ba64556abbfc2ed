"""Diffusivities far below the mass term: the coarsest level's explicit matrix,
whose unknowns are scaled by factors proportional to K, equals the oracle's sweeps
also where the product of two such factors (K < 1e-150) or a factor itself
(K < 1e-300, the sweeps instead) underflows. FP64 to 1e-12 of the largest value,
FP32 to 1e-4 in the 2-norm, as for any coarsest solve."""
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel_inf, rel2, opts_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("K", [1e-20, 1e-170, 1e-305, 1e-320])
def test_coarsest_matrix_of_a_small_diffusivity(K, prec):
    sh = shellgen.Shell("smallK", 6, 12, 20, stretch=1.05, K=K)
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    S = solver_for(sh, a, precision=prec, levels=1, coarse_sweeps=5)
    ref = oracle.vcycle(oracle.build_hierarchy(sh, a, levels=1), f, opts_of(sh, coarse_sweeps=5))
    err = (rel_inf if prec == "fp64" else rel2)(n(S.vcycle(t(f))), ref)
    log(f"K {K:g} {prec}: {err:.2e}")
    assert err < (1e-12 if prec == "fp64" else 1e-4)
