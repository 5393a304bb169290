"""The diagonal blocks of LB-ADMM's factorisation at the edges of their 16-wide tiles and of the 64-wide blocks, in one launch per block column and in
several; and the tiles of its lower matrices where there are one, two and many of them (the Gram product of 128-wide tiles needs 256 columns and 1536 rows)."""
import pytest

from oracle import lb_admm as O
from paper_2602_06694_amd import synth
from test_gpu_lb_admm import compare, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("r", [1, 15, 16, 17, 31, 48, 63, 64, 65, 80, 127, 129, 191, 257])
def test_ranks_around_tiles_and_blocks(nqopt, r, fused):
    n, m = r + 37, 2 * r + 5
    w, u0, v0 = synth.gen_admm_problem(n, m, r, seed=14000 + r)
    ref = O.lb_admm(w, u0, v0, 3, 0.05, 0.3, 1e-3, 3)
    nqopt.set("admm_no_fused_step", 0 if fused else 1)
    outs, _, _ = run_gpu(w, u0, v0, 3, 0.05, 0.3, 1e-3, 3)
    compare(outs, ref)


@pytest.mark.parametrize("n,m,r", [(1540, 1600, 256), (1600, 1700, 257), (1537, 1540, 520)])
def test_lower_tiles_of_the_gram_product(n, m, r):
    w, u0, v0 = synth.gen_admm_problem(n, m, r, seed=14500 + r)
    ref = O.lb_admm(w, u0, v0, 2, 0.5, 2.0, 1e-3, 3)
    outs, _, _ = run_gpu(w, u0, v0, 2, 0.5, 2.0, 1e-3, 3)
    compare(outs, ref)
