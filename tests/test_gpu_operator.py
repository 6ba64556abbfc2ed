"""The FP64 operator against the oracle on levels that walk ranges of layers
(at least 2^18 columns: rows of whole segments and ragged ones, layer counts
below, at and past a range of 25) and on smaller ones, and the residual step of
columns of more than 72 layers (zero, one and several ranges). 1e-13 of the
largest value: seven products per row, summed in another order. The reference takes the
library's own FP64 tables (whose agreement with the oracle's is tested by
itself), so that it measures the kernel and not the geometry near the poles."""
import numpy as np
import pytest

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel_inf

pytestmark = pytest.mark.gpu

def table_operator(sh, a, x):
    """H x in difference form from the host tables of level 0."""
    from paper_2307_04528_amd import mg_plan_tables
    V, Tl, Tt, Tr = mg_plan_tables(0, sh.nlon, sh.nlat, sh.nlev, sh.radius, sh.thickness,
                                   sh.stretch, sh.K, levels=2)
    y = a * V[:, :, None] * x
    y += Tl[:, :, None] * ((x - np.roll(x, 1, 2)) + (x - np.roll(x, -1, 2)))
    d = Tt[:, 1:-1, None] * (x[:, 1:] - x[:, :-1])
    y[:, 1:] += d
    y[:, :-1] -= d
    d = Tr[1:-1, :, None] * (x[1:] - x[:-1])
    y[1:] += d
    y[:-1] -= d
    return y


SIZES = [(512, 512, 3), (512, 514, 25), (516, 512, 26), (1024, 258, 51), (640, 400, 4)]


@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_operator_by_size(size):
    sh = shellgen.Shell("op", *size, stretch=1.03)
    a = shellgen.alpha(sh)
    S = solver_for(sh, a, levels=2, coarse_sweeps=1)
    x = np.random.default_rng(5).standard_normal(sh.shape)
    e = rel_inf(n(S.apply(t(x))), table_operator(sh, a, x))
    log(f"operator {size}: {e:.2e}")
    assert e < 1e-13


@pytest.mark.parametrize("nz", [73, 96, 97, 128])
def test_residual_of_deep_columns(nz):
    """One refinement step from a given iterate: the reported residual norm is
    the oracle's, to 1e-11 (a cancelling sum of terms about 1e3 larger)."""
    sh = shellgen.Shell("deep", 72, 40, nz, stretch=1.02)
    a, b = shellgen.alpha(sh), shellgen.rhs(sh)
    L = oracle.build_hierarchy(sh, a)
    S = solver_for(sh, a)
    u, _ = S.solve(t(b), tol=1e-3)
    _, st = S.solve(t(b), tol=1e-2, u0=u.clone())
    r = b - oracle.apply(L[0], n(u))
    want = np.linalg.norm(r) / np.linalg.norm(b)
    log(f"deep residual {nz}: {st.relres:.12e} {want:.12e}")
    assert st.iters == 0
    assert abs(st.relres - want) < 1e-11 * max(1.0, np.abs(oracle.apply(L[0], n(u))).max())
