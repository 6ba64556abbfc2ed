"""GPU parity on levels whose route differs for more than 72 layers: the walking
restriction (at least 2^15 columns; whole coarse segments and ragged ones), and the
FP32 refinement step on 16-row tiles, in one range of layers and in two.

The restriction against the oracle: FP64 to 1e-12 of the largest restricted
magnitude, FP32 to 2e-5, as for every single kernel. The FP32 residual's norm to 1e-5 of the FP64 one:
each residual is a sum of about eight terms, some ten times larger, of relative
error 6e-8, and the errors of 9M cells average out."""
import numpy as np
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for
from test_gpu_operator import table_operator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("size", [(256, 130, 73), (250, 134, 128), (256, 130, 81)],
                         ids=lambda s: "x".join(map(str, s)))
def test_restriction_of_deep_levels(size, prec):
    sh = shellgen.Shell("deep", *size, stretch=1.02)
    a = shellgen.alpha(sh)
    rng = np.random.default_rng(37)
    f, x = rng.standard_normal(sh.shape), rng.standard_normal(sh.shape)
    L = oracle.build_hierarchy(sh, a, levels=2)
    S = solver_for(sh, a, precision=prec, levels=2, coarse_sweeps=1)
    got = n(S.level_residual_restrict(0, t(f), t(x)))
    Hx = oracle.apply(L[0], x)
    scale = np.abs(oracle.restrict(L[0], L[1], np.abs(f) + np.abs(Hx))).max()
    e = np.abs(got - oracle.restrict(L[0], L[1], f - Hx)).max() / scale
    log(f"deep restriction {size} {prec}: {e:.2e}")
    assert e < (1e-12 if prec == "fp64" else 2e-5)


@pytest.mark.parametrize("nz", [17, 71])
@pytest.mark.parametrize("plane", [(1024, 514), (1030, 482)], ids=["whole", "ragged"])
def test_fp32_refinement_of_large_levels(plane, nz):
    sh = shellgen.Shell("walk", *plane, nz, stretch=1.02)
    a, b = shellgen.alpha(sh), shellgen.rhs(sh)
    u0 = np.random.default_rng(41).standard_normal(sh.shape)
    want = np.linalg.norm((b - table_operator(sh, a, u0)).ravel())
    S = solver_for(sh, a, precision="fp32", levels=2, coarse_sweeps=1, max_iters=1)
    u, st = S.solve(t(b), tol=1e-13, u0=t(u0))
    want1 = np.linalg.norm((b - table_operator(sh, a, n(u))).ravel())
    log(f"fp32 {plane}x{nz}: {st.res_hist[0] / want - 1:.1e} {st.res_hist[1] / want1 - 1:.1e}")
    assert abs(st.res_hist[0] - want) <= 1e-5 * want
    assert abs(st.res_hist[1] - want1) <= 1e-5 * want1
