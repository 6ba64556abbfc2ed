"""GPU parity of the staged sweep of small levels at the edges of its compiled
half-column lengths (4, 8, 12, 20, 32, 36, 44, 54 and 64 layers per half) on
ragged rows (one segment of 20 columns, and 64 + 6): the sweep from zero and a
sweep from an iterate against the oracle. FP64 to 1e-12 of the largest value,
FP32 to 2e-5, as for every single kernel.
"""
import numpy as np
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel_inf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nz", [1, 2, 8, 9, 16, 17, 24, 25, 40, 41, 64, 65, 73, 88, 89, 108, 109,
                                127])
def test_staged_sweep(nz, prec):
    rng = np.random.default_rng(17)
    for nlon in (20, 70):
        sh = shellgen.Shell("staged", nlon, 6, nz, stretch=1.02)
        a = shellgen.alpha(sh)
        S = solver_for(sh, a, precision=prec, levels=1, staged_columns=1 << 30)
        L = oracle.build_hierarchy(sh, a, levels=1)
        f, x = rng.standard_normal(sh.shape), rng.standard_normal(sh.shape)
        got0, got1 = n(S.level_sweep(0, t(f))), n(S.level_sweep(0, t(f), t(x)))
        e0 = rel_inf(got0, oracle.sweep_from_zero(L[0], f, 0.8))
        e1 = rel_inf(got1, oracle.sweep(L[0], x, f, 0.8))
        log(f"staged {nlon}x6x{nz} {prec}: {e0:.2e} {e1:.2e}")
        assert max(e0, e1) < (1e-12 if prec == "fp64" else 2e-5)
