"""GPU parity of two sweeps in one pass over memory (FP32 levels of at least
98,304 columns and 17 to 72 layers): V-cycles whose finest level does its
sweeps in pairs against the same cycles with single staged sweeps, element by
element, and against the oracle. The shells lie where the pair kernel can go
wrong: strips that divide a row evenly, raggedly and with one strip more than
whole segments need; rows narrower than a strip; few rows per band; a last
band with few rows; odd layer counts and the edges of the compiled half
columns (17, 24, 25, 40, 41, 72) and below the first (14, 15, 16: single
sweeps). V(2,2) runs pairs from zero and from an
iterate, V(3,3) pairs and a single sweep, and the transposed cycle the factors
reversed.

The two routes do the same FP32 operations per cell up to the order of the
sums: a difference of a few eps32 = 6e-8 per sweep in the 2-norm, amplified by
at most the sweeps' condition; 2e-5 as for any single FP32 kernel here. The
oracle: 1e-4 as for any FP32 cycle.
"""
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel2, rel_inf, opts_of

pytestmark = pytest.mark.gpu

SHELLS = [(512, 256, 14), (512, 258, 16), (496, 268, 17), (620, 216, 40), (1024, 130, 41),
          (1100, 120, 24), (62, 1600, 15), (8, 12288, 16), (480, 208, 72),
          (62, 1600, 19), (8, 12288, 18), (512, 258, 25)]


@pytest.mark.parametrize("nu", [(2, 2), (3, 3)])
@pytest.mark.parametrize("size", SHELLS, ids=lambda s: "x".join(map(str, s)))
def test_pairs_of_sweeps(size, nu):
    sh = shellgen.Shell("pair", *size, stretch=1.04, nu_pre=nu[0], nu_post=nu[1])
    assert sh.nlon * sh.nlat >= 3 << 15
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    kw = dict(nu_pre=nu[0], nu_post=nu[1], levels=2, coarse_sweeps=2)
    L = oracle.build_hierarchy(sh, a, levels=2)
    opt = opts_of(sh, coarse_sweeps=2)
    pairs = solver_for(sh, a, staged_columns=0, **kw)
    single = solver_for(sh, a, staged_columns=1 << 30, **kw)
    for tr in (False, True):
        got, one = n(pairs.vcycle(t(f), transposed=tr)), n(single.vcycle(t(f), transposed=tr))
        ref = (oracle.vcycle_T if tr else oracle.vcycle)(L, f, opt)
        log(f"pairs {size} V{nu} transposed={tr}: single {rel2(got, one):.2e} "
            f"{rel_inf(got, one):.2e} oracle {rel2(got, ref):.2e}")
        assert rel2(got, one) < 2e-5 and rel_inf(got, one) < 2e-5
        assert rel2(got, ref) < 1e-4
