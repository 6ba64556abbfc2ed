"""GPU parity where a wavefront has few lanes with a column of their own: pairs of
sweeps whose last strip is 2 columns wide (3722 and 3784 columns: 60 and 61 strips
of 62 before it), and the coarsest level's solve with a last wavefront of 4 lanes
(132 columns, swept in LDS) and of 8, 12 and 24 (unit vectors side by side: 2 of 100
columns, 3 of 68 and of 72, the iterate at a fixed stride and, with 80 layers, by
layer). The other lanes still hold the steps' vertical couplings, which all lanes
read.

Tolerances as for any FP32 cycle (1e-4 in the 2-norm) and, in FP64, 1e-12 of the
largest value.
"""
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel2, rel_inf, opts_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(3722, 28, 20), (3784, 26, 38), (3722, 28, 70)],
                         ids=lambda s: "x".join(map(str, s)))
def test_pairs_on_a_narrow_last_strip(size):
    sh = shellgen.Shell("narrow", *size, stretch=1.04, nu_pre=2, nu_post=2)
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    L = oracle.build_hierarchy(sh, a, levels=2)
    opt = opts_of(sh, coarse_sweeps=2)
    kw = dict(levels=2, coarse_sweeps=2, staged_columns=0)
    S = solver_for(sh, a, **kw)
    for tr in (False, True):
        got = n(S.vcycle(t(f), transposed=tr))
        ref = (oracle.vcycle_T if tr else oracle.vcycle)(L, f, opt)
        log(f"narrow {size} transposed={tr}: {rel2(got, ref):.2e}")
        assert rel2(got, ref) < 1e-4


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("size", [(6, 12, 40), (22, 6, 20), (34, 2, 30), (10, 10, 61), (34, 2, 80)],
                         ids=lambda s: "x".join(map(str, s)))
def test_coarsest_solve_with_a_narrow_last_wavefront(size, prec):
    sh = shellgen.Shell("narrow", *size, stretch=1.02)
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    S = solver_for(sh, a, precision=prec, levels=1, coarse_sweeps=7)
    ref = oracle.vcycle(oracle.build_hierarchy(sh, a, levels=1), f, opts_of(sh, coarse_sweeps=7))
    got = n(S.vcycle(t(f)))
    err = rel_inf if prec == "fp64" else rel2
    log(f"narrow coarsest {size} {prec}: {err(got, ref):.2e}")
    assert err(got, ref) < (1e-12 if prec == "fp64" else 1e-4)
