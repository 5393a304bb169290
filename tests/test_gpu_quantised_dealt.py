"""The stage kernel of few row blocks on an input that a launch of its own has quantised (too long to quantise along), in the forms that its rule takes: groups of tokens and bit
planes dealt out, whole row blocks of six to eight tokens, groups on one XCD or on all, several layers of unequal lengths in a launch (test_gpu_lone_forms.py has every compiled
form).  Outputs against lone calls by the launches that deal nothing out, bit for bit (the arithmetic is exact up to the same roundings), and against the oracle."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu
TOL = 1e-5          # of the largest output: two fixed-point steps of at least 21 bits and three roundings to fp32, as for all streaming paths


def plain(nqopt, L, x, batch):
    y = new_output(batch, L.d_out)
    for o in ("no_selfq", "no_fuse"):
        nqopt.set(o, 1)
    nq.nq_binlr_forward_exact(L.h, x, y, batch)
    for o in ("no_selfq", "no_fuse"):
        nqopt.unset(o)
    return y.cpu().numpy()


@pytest.mark.parametrize("shapes,batches", [
    ([(130, 17000, 100)], (2, 4, 5, 6, 8)), ([(260, 33000, 1025)], (1, 3, 4, 7, 8)),                    # one and nine row blocks of a long reduction
    ([(300, 12000, 4200)], (3, 4, 5, 8)), ([(200, 20000, 8300), (64, 300, 20)], (2, 5, 6)),             # 33 and 66
    ([(500, 9088, 480), (129, 64, 3), (640, 5000, 1000)], (4, 7, 8)),                                   # unequal lengths
    ([(60, 16400, 129 * 128 + 5)], (6, 8)),                                                             # 130: whole row blocks, eight waves on two column groups
])
def test_plans(nqopt, shapes, batches):
    hs = [Layer(*s, "f16", seed=12700 + i) for i, s in enumerate(shapes)]
    for batch in batches:
        xn = [synth.gen_x(batch, s[1], 12710 + i, "f16") for i, s in enumerate(shapes)]
        xs = [to_device(x, "f16") for x in xn]
        ys = [new_output(batch, s[0]) for s in shapes]
        plan = nq.nq_plan_create([L.h for L in hs], xs, ys, batch)
        nq.nq_plan_forward(plan)
        for L, x, xd, y in zip(hs, xn, xs, ys):
            got = y.cpu().numpy()
            assert np.array_equal(got, plain(nqopt, L, xd, batch)), (shapes, batch)
            assert rel_err(got, L.oracle(x)) <= TOL, (shapes, batch)
        nq.nq_plan_destroy(plan)
    for L in hs:
        L.close()


@pytest.mark.parametrize("shape,batches", [((260, 40000, 130), (9, 17, 24, 65)), ((140, 16000, 700), (10, 33, 40)), ((100, 9000, 2040), (9, 15, 16)),
                                           ((90, 2555, 79 * 128 + 7), (12, 13, 16))])       # ragged rows, 80 row blocks: whole ones on all XCDs, eight waves
def test_more_than_eight_tokens(nqopt, shape, batches):
    L = Layer(*shape, "bf16", seed=12800 + shape[1])
    nq.nq_binlr_reserve(L.h, max(batches))
    for batch in batches:
        x = synth.gen_x(batch, shape[1], 12810 + batch, "bf16")
        xd, y = to_device(x, "bf16"), new_output(batch, shape[0])
        nq.nq_binlr_forward_exact(L.h, xd, y, batch)
        got = y.cpu().numpy()
        assert np.array_equal(got, plain(nqopt, L, xd, batch)), (shape, batch)
        assert rel_err(got, L.oracle(x)) <= TOL, (shape, batch)
    L.close()


@pytest.mark.parametrize("shape,batch,exact_pays", [((1220, 389, 149), 108, True), ((942, 477, 213), 221, True), ((3341, 388, 258), 75, True), ((8712, 1167, 837), 60, True),
                                                    ((2503, 702, 188), 229, False), ((256, 250, 250), 330, False)])
def test_forward_on_the_faster_path(nqopt, shape, batch, exact_pays):
    """More pairs of row block and group than are shared in one stage, not in the other: the bits of the path that was measured to be the faster one."""
    L = Layer(*shape, "bf16", seed=12900 + shape[0])
    nq.nq_binlr_reserve(L.h, batch)
    xd = to_device(synth.gen_x(batch, shape[1], 12901, "bf16"), "bf16")
    y, exact = new_output(batch, shape[0]), new_output(batch, shape[0])
    nq.nq_binlr_forward(L.h, xd, y, batch)
    nq.nq_binlr_forward_exact(L.h, xd, exact, batch)
    assert np.array_equal(y.cpu().numpy(), exact.cpu().numpy()) == exact_pays
    L.close()
