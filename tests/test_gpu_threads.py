"""Two threads, each with a handle, a stream and fields of its own, on grids whose
levels run the same kernels with LDS of different sizes above 64 KB: what a kernel
may use is a setting of the process, so it must not depend on the call that set it
last. Every result has the bits of the same solve alone."""
import threading

import pytest
import torch

from gpu_util import log
from paper_2307_04528_amd import Solver

pytestmark = pytest.mark.gpu


def test_two_threads_with_different_layer_counts():
    # FP64 levels below 65,536 columns: staged sweeps with 69 to 77 KB of LDS, a
    # coarsest level of 98 to 112 columns in the sweeps' kernel (no graphs: each
    # cycle launches anew)
    grids, fields, alone, out, errors = [(96, 48, 72), (96, 48, 66)], [], [], {}, []
    for g in grids:
        a = torch.full((g[2], g[1], g[0]), 100.0, dtype=torch.float64, device="cuda")
        b = torch.empty_like(a).uniform_(-1, 1)
        S = Solver(*g, a, precision="fp64", graphs=False)
        fields.append((a, b))
        alone.append(S.solve(b, tol=1e-6)[0])
        S.close()
    torch.cuda.synchronize()
    start = threading.Barrier(2)

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                S = Solver(*grids[i], fields[i][0], precision="fp64", graphs=False)
                start.wait(60)
                out[i] = [S.solve(fields[i][1], tol=1e-6)[0] for _ in range(60)]
                torch.cuda.current_stream().synchronize()
                S.close()
        except Exception as e:   # reported by the main thread
            errors.append((grids[i], e))
            start.abort()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for th in threads:
        th.start()
    for th in threads:
        th.join(100)
    log(f"two threads: {len(out)} done, errors {errors}")
    assert not errors and len(out) == 2
    for i in range(2):
        assert all(torch.equal(u, alone[i]) for u in out[i])
