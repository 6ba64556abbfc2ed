"""GPU parity of the staged sweep that adds the prolonged correction itself
(small levels, up to 40 layers in FP32 and 16 in FP64): V-cycles of two levels
against the oracle, and against the same cycles with a prolongation of its own
and unstaged sweeps (staged_columns = 0). Shells at the edges of the compiled
half-column lengths (4, 8, 20 layers per half) and one layer beyond each rule;
rows of one ragged segment, one whole one, one and 6 columns, two; merged rows
and rows coarsened in longitude only, both poles. V(1,1) has the fused sweep
alone, V(2,3) more after it.

FP64 to 1e-12 of the largest value and FP32 to 1e-4 in the 2-norm, as for any
cycle; the two routes do the same operations up to the order of the sweeps'
sums: 1e-12 and 2e-5.
"""
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel_inf, rel2, opts_of

pytestmark = pytest.mark.gpu

SHELLS = [(20, 12, 1), (64, 32, 2), (70, 34, 8), (128, 60, 9), (20, 12, 16), (70, 40, 17),
          (134, 64, 16), (64, 32, 40), (70, 34, 41)]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nu", [(1, 1), (2, 3)])
@pytest.mark.parametrize("size", SHELLS, ids=lambda s: "x".join(map(str, s)))
def test_sweep_with_prolongation(size, nu, prec):
    sh = shellgen.Shell("staged-prolong", *size, stretch=1.02, nu_pre=nu[0], nu_post=nu[1])
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    kw = dict(precision=prec, nu_pre=nu[0], nu_post=nu[1], levels=2, coarse_sweeps=4)
    L = oracle.build_hierarchy(sh, a, levels=2)
    ref = oracle.vcycle(L, f, opts_of(sh, coarse_sweeps=4))
    got = n(solver_for(sh, a, **kw).vcycle(t(f)))
    one = n(solver_for(sh, a, staged_columns=0, **kw).vcycle(t(f)))
    err = rel_inf if prec == "fp64" else rel2
    log(f"staged prolong {size} V{nu} {prec}: oracle {err(got, ref):.2e} apart {err(got, one):.2e}")
    assert err(got, ref) < (1e-12 if prec == "fp64" else 1e-4)
    assert err(got, one) < (1e-12 if prec == "fp64" else 2e-5)
