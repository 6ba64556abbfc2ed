"""Which levels do their sweeps in pairs, read from the bytes that the profile counts
per sweep (8 per cell and sweep in a pair of FP32 sweeps, 16 in a single one), on
both sides of every line of the rule; and pairs at the compiled half columns of 28
and 32 layers (49, 56, 57 and 64 layers) against single sweeps and the oracle, with
the tolerances of any FP32 cycle (2e-5 and 1e-4)."""
import pytest
import torch

import shellgen
import oracle
from gpu_util import log, t, n, solver_for, rel2, rel_inf, opts_of

pytestmark = pytest.mark.gpu

PAIRS = [((512, 192, 17), True), ((512, 190, 17), False), ((512, 192, 16), False),
         ((512, 192, 72), True), ((512, 192, 73), False), ((8, 12288, 18), True),
         ((62, 1600, 17), True), ((66, 1500, 17), True), ((128, 768, 70), False), ((128, 1024, 70), True),
         ((64, 1536, 17), False), ((64, 2048, 32), False), ((64, 1536, 70), False),
         ((64, 1536, 33), True), ((64, 1536, 69), True)]


@pytest.mark.parametrize("size,pairs", PAIRS, ids=lambda s: "x".join(map(str, s))
                         if isinstance(s, tuple) else str(s))
def test_route_of_the_finest_sweeps(size, pairs):
    from paper_2307_04528_amd import Solver
    a = torch.full((size[2], size[1], size[0]), 100.0, dtype=torch.float64, device="cuda")
    S = Solver(*size, a, levels=2, coarse_sweeps=1, max_iters=1, profile=1)
    k = S.solve(torch.rand_like(a), tol=1e-13)[1].kernels["smooth"]
    bytes_per_cell = k["fine_bytes"] / k["fine_launches"] / a.numel()
    log(f"route {size}: {bytes_per_cell} B per cell and sweep")
    assert bytes_per_cell == pytest.approx(8 if pairs else 16)


@pytest.mark.parametrize("nz", [49, 56, 57, 64])
def test_pairs_of_middle_layer_counts(nz):
    sh = shellgen.Shell("pair", 500, 204, nz, stretch=1.04, nu_pre=2, nu_post=3)
    a, f = shellgen.alpha(sh), shellgen.rhs(sh)
    kw = dict(nu_pre=2, nu_post=3, levels=2, coarse_sweeps=2)
    L = oracle.build_hierarchy(sh, a, levels=2)
    opt = opts_of(sh, coarse_sweeps=2)
    pairs = solver_for(sh, a, staged_columns=0, **kw)
    single = solver_for(sh, a, staged_columns=1 << 30, **kw)
    for tr in (False, True):
        got, one = n(pairs.vcycle(t(f), transposed=tr)), n(single.vcycle(t(f), transposed=tr))
        ref = (oracle.vcycle_T if tr else oracle.vcycle)(L, f, opt)
        log(f"pairs 500x204x{nz} transposed={tr}: single {rel2(got, one):.2e} "
            f"oracle {rel2(got, ref):.2e}")
        assert rel2(got, one) < 2e-5 and rel_inf(got, one) < 2e-5
        assert rel2(got, ref) < 1e-4
