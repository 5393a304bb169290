"""LB-ADMM with a workspace (and outputs) full of NaN gives the bits it gives with one of zeros: ranks whose number of 64-wide blocks
is and is not a power of two (the matrices of the factorisation are padded to one)."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,r", [(96, 80, 24), (200, 150, 128), (300, 200, 130), (321, 499, 171), (500, 700, 320), (900, 800, 450)])
def test_the_workspace_needs_no_initial_values(nqopt, n, m, r):
    import torch
    w, u0, v0 = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in synth.gen_admm_problem(n, m, r, seed=r))
    nbytes = nq.nq_lb_admm_workspace_bytes(n, m, r)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    for fused in (True, False):
        nqopt.set("admm_no_fused_step", 0 if fused else 1)
        results = []
        for fill in (0, 255):
            ws.fill_(fill)
            outs = [torch.full((rows, r), float("nan") if fill else 0.0, dtype=torch.float64, device="cuda") for rows in (n, m, n, m, n, m)]
            nq.nq_lb_admm(w, n, m, r, u0, v0, 2, 0.05, 0.2, 1e-3, 4, *outs, ws, nbytes)
            torch.cuda.synchronize()
            assert all(torch.isfinite(o).all() for o in outs)
            results.append(outs)
        assert all(torch.equal(a, b) for a, b in zip(*results))
