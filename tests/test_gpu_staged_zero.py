"""GPU parity of the staged sweep at the half columns that test_gpu_staged.py leaves
out (28 steps; the ends of 16, 20, 32 and 36), whose sweeps from zero hold other
values in registers than those from an iterate: FP64 to 1e-12 of the largest value,
FP32 to 2e-5, as for every single kernel."""
import numpy as np
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nz", [32, 33, 49, 56, 57, 72])
def test_staged_sweep_of_other_lengths(nz, prec):
    rng = np.random.default_rng(43)
    sh = shellgen.Shell("staged", 70, 8, nz, stretch=1.02)
    a = shellgen.alpha(sh)
    S = solver_for(sh, a, precision=prec, levels=1, staged_columns=1 << 30)
    L = oracle.build_hierarchy(sh, a, levels=1)
    f, x = rng.standard_normal(sh.shape), rng.standard_normal(sh.shape)
    e0 = rel_inf(n(S.level_sweep(0, t(f))), oracle.sweep_from_zero(L[0], f, 0.8))
    e1 = rel_inf(n(S.level_sweep(0, t(f), t(x))), oracle.sweep(L[0], x, f, 0.8))
    log(f"staged 70x8x{nz} {prec}: {e0:.2e} {e1:.2e}")
    assert max(e0, e1) < (1e-12 if prec == "fp64" else 2e-5)
