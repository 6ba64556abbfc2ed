"""GPU parity of the coarsest-level solve with a single-level hierarchy, whose
V-cycle is that solve alone: the explicit matrix (up to 128 columns and 6144
cells), all sweeps in one block's LDS (up to 256 columns) and one launch per
sweep beyond. Sizes lie at the edges of the compiled half-column lengths (4,
8, 20, 36, 44, 64 layers per half), of the lanes (64, 128, 252, 256 columns)
and of the unit vectors per block (cell counts that they do not divide).

FP64 to 1e-12 of the largest value: a chain of a few convex combinations per
sweep. FP32 to 1e-4 in the 2-norm, as for a whole cycle.
"""
import numpy as np
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel_inf, rel2, opts_of

pytestmark = pytest.mark.gpu

SIZES = [(4, 2, 1), (4, 4, 2), (16, 8, 8), (8, 8, 9), (6, 12, 40), (6, 12, 41), (10, 8, 71),
         (6, 12, 72), (6, 10, 73), (4, 10, 88), (4, 10, 89), (4, 10, 128), (18, 14, 7),
         (16, 16, 24), (16, 16, 73), (22, 12, 16)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_single_level_solve(size, prec):
    sh = shellgen.Shell("one", *size, stretch=1.02)
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    S = solver_for(sh, a, precision=prec, levels=1, coarse_sweeps=6)
    L = oracle.build_hierarchy(sh, a, levels=1)
    opt = opts_of(sh, coarse_sweeps=6)
    got, gotT = n(S.vcycle(t(f))), n(S.vcycle(t(f), transposed=True))
    ref, refT = oracle.vcycle(L, f, opt), oracle.vcycle_T(L, f, opt)
    err = rel_inf if prec == "fp64" else rel2
    log(f"coarse {size} {prec}: {err(got, ref):.2e} transposed {err(gotT, refT):.2e}")
    bar = 1e-12 if prec == "fp64" else 1e-4
    assert err(got, ref) < bar and err(gotT, refT) < bar
