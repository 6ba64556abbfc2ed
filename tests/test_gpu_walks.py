"""The walks of the refinement step and the FP64 operator on large levels (16-row
tiles; rows of whole segments and ragged ones) at the edges of their ranges of
layers: one range (16, 17, 70 layers), two of unequal and equal length (71, 72,
73, 128). The norms of a first residual from a random iterate and of the residual
after one update, and the operator, against the library's own FP64 tables.

Norms to 1e-12 and 1e-10 (sums of squares without cancellation, about 1e-14;
after the update each residual cancels to about a tenth of its terms), the
operator to 1e-13 of the largest value (seven products in another order): a cell
that is missed or counted twice would move a norm by 1e-8.

And that a walk's time goes with the layers there are. The bars lie between the
measured ratio of a walk that ends with its layers and of one that runs steps
for layers that are not there: operator 26 to 25 layers 1.1 and 1.5, 4 to 25
layers (a chunk instead of a walk) 0.3 and 0.65; refinement step 17 to 70 layers
0.29 and 0.56, 71 to 70 layers 1.1 and 1.5.
"""
import statistics

import numpy as np
import pytest
import torch

import shellgen
from gpu_util import log, t, n, solver_for, rel_inf
from test_gpu_operator import table_operator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [16, 17, 70, 71, 72, 73, 128])
@pytest.mark.parametrize("plane", [(1024, 514), (1030, 482)], ids=["whole", "ragged"])
def test_residual_norms_of_large_levels(plane, nz):
    sh = shellgen.Shell("walk", *plane, nz, stretch=1.02)
    a, b = shellgen.alpha(sh), shellgen.rhs(sh)
    u0 = np.random.default_rng(29).standard_normal(sh.shape)
    want0 = np.linalg.norm((b - table_operator(sh, a, u0)).ravel())
    for prec in ("mixed", "fp64"):
        S = solver_for(sh, a, precision=prec, levels=2, coarse_sweeps=1, max_iters=1)
        u, st = S.solve(t(b), tol=1e-13, u0=t(u0))
        want1 = np.linalg.norm((b - table_operator(sh, a, n(u))).ravel())
        S.close()
        log(f"walk {plane}x{nz} {prec}: {st.res_hist[0] / want0 - 1:.1e} "
            f"{st.res_hist[1] / want1 - 1:.1e}")
        assert abs(st.res_hist[0] - want0) <= 1e-12 * want0
        assert abs(st.res_hist[1] - want1) <= 1e-10 * want1


# the walk from 12,582,912 cells and 9 layers on, one chunk short of either too
SIZES = [(1024, 770, 16), (1024, 514, 25), (1028, 480, 26), (516, 512, 51), (512, 514, 100),
         (512, 512, 48), (512, 512, 47), (1664, 842, 9), (1664, 946, 8)]


@pytest.mark.parametrize("size", SIZES, ids=lambda s: "x".join(map(str, s)))
def test_operator_of_large_levels(size):
    sh = shellgen.Shell("walk", *size, stretch=1.02)
    a = shellgen.alpha(sh)
    S = solver_for(sh, a, levels=2, coarse_sweeps=1)
    x = np.random.default_rng(31).standard_normal(sh.shape)
    e = rel_inf(n(S.apply(t(x))), table_operator(sh, a, x))
    log(f"operator {size}: {e:.2e}")
    assert e < 1e-13


def test_operator_of_zero_is_zero():
    """Plain zeros, no negative ones, on a level that walks."""
    S, f = handle((512, 512), 48)
    assert not torch.signbit(S.apply(torch.zeros_like(f))).any()
    S.close()


def handle(plane, nz, **opts):
    from paper_2307_04528_amd import Solver
    a = torch.full((nz, plane[1], plane[0]), 100.0, dtype=torch.float64, device="cuda")
    f = torch.empty_like(a).uniform_(-1, 1)
    return Solver(*plane, nz, a, levels=2, coarse_sweeps=1, **opts), f


@pytest.mark.parametrize("plane,layers,bar", [((1536, 1024), 26, 1.3), ((1152, 576), 4, 0.48)],
                         ids=["26", "4"])
def test_operator_time_goes_with_the_layers(plane, layers, bar):
    ms = {}
    for nz in (25, layers):
        S, f = handle(plane, nz)
        times = []
        for _ in range(12):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(8):
                S.apply(f)
            ev[1].record()
            torch.cuda.synchronize()
            times.append(ev[0].elapsed_time(ev[1]))
        S.close()
        ms[nz] = statistics.median(times[2:])
    log(f"operator {layers} to 25 layers: {ms[layers] / ms[25]:.2f}")
    assert ms[layers] < bar * ms[25]


def test_refinement_time_goes_with_the_layers():
    ms = {}
    for nz in (17, 70, 71):
        S, f = handle((1024, 768), nz, precision="fp64", max_iters=3, profile=1)
        ms[nz] = statistics.median(S.solve(f, tol=1e-30)[1].ms_residual for _ in range(10))
        S.close()
    log(f"refinement 17 to 70 layers {ms[17] / ms[70]:.2f}, 71 to 70 {ms[71] / ms[70]:.2f}")
    assert ms[17] < 0.42 * ms[70]
    assert ms[71] < 1.3 * ms[70]
