"""The stage kernel that quantises along, at the edges of its forms: tokens dealt out in groups of one to eight, one to eight bit planes per workgroup, four or
16 elements of a lane at a time, eight or 16 waves, groups on one XCD or on all.  Every output and the intermediate against the launches that quantise separately, bit
for bit (the arithmetic is exact up to the same roundings, so there is nothing to tolerate), and y against the oracle."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu
TOL = 1e-5          # of the largest output: two fixed-point steps of at least 21 bits and three roundings to fp32, as for all streaming paths


@pytest.mark.parametrize("shape,x_dtype,batches", [
    ((130, 3, 5), "f32", (1, 2, 8, 9, 17)), ((1025, 5, 130), "f16", (3, 7, 8, 23)),             # rows shorter than a lane's elements, odd groups
    ((2000, 1023, 900), "bf16", (2, 5, 7, 24)), ((700, 4095, 260), "f16", (4, 6, 8, 13)),       # four and 16 elements at a time
    ((9000, 640, 2100), "bf16", (2, 3, 5, 8)), ((16300, 700, 520), "f32", (1, 4, 6, 8)),        # 17 and 128 row blocks: few planes to deal, few groups
    ((16600, 300, 1000), "bf16", (1, 2, 3, 6)), ((260, 28600, 200), "bf16", (1, 2, 5, 8)),      # whole row blocks on eight waves; one token as long as LDS takes
    ((128, 512, 128), "f32", (40, 100)), ((400, 260, 300), "f16", (64, 129)),                   # more groups than an XCD has CUs for a row block
])
def test_forms_agree(nqopt, shape, x_dtype, batches):
    L = Layer(*shape, x_dtype, seed=12000 + shape[1])
    nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(shape[2], 12001))
    nq.nq_binlr_reserve(L.h, max(batches))
    for batch in batches:
        x = to_device(synth.gen_x(batch, shape[1], 12010 + batch, x_dtype), x_dtype)
        y, apart = new_output(batch, shape[0]), new_output(batch, shape[0])
        nq.nq_binlr_forward_exact(L.h, x, y, batch)
        t = nq.nq_binlr_read_intermediate(L.h, L.r, batch) if batch <= 8 else None
        for o in ("no_selfq", "no_fuse"):
            nqopt.set(o, 1)
        nq.nq_binlr_forward_exact(L.h, x, apart, batch)
        for o in ("no_selfq", "no_fuse"):
            nqopt.unset(o)
        y, apart = y.cpu().numpy(), apart.cpu().numpy()
        assert np.array_equal(y, apart), (shape, batch)
        if t is not None:
            assert np.array_equal(t, nq.nq_binlr_read_intermediate(L.h, L.r, batch)), (shape, batch)
        assert np.isfinite(y).all()
    L.close()


@pytest.mark.parametrize("layers,batch", [(1, 3), (2, 8), (3, 5), (5, 7), (6, 6)])
def test_plans_of_mixed_lengths(layers, batch):
    """Row blocks of several layers in one launch, whose groups of tokens share the items: against calls on each layer alone and the oracle."""
    shapes = [(1000, 2300, 520), (520, 260, 130), (300, 4090, 700), (1300, 64, 60), (2048, 1024, 512), (129, 3, 2)][:layers]
    hs = [Layer(*s, "f16", seed=12100 + i) for i, s in enumerate(shapes)]
    xn = [synth.gen_x(batch, s[1], 12200 + i, "f16") for i, s in enumerate(shapes)]
    xs = [to_device(x, "f16") for x in xn]
    ys, alone = [new_output(batch, s[0]) for s in shapes], [new_output(batch, s[0]) for s in shapes]
    plan = nq.nq_plan_create([L.h for L in hs], xs, ys, batch)
    nq.nq_plan_forward(plan)
    for L, x, y in zip(hs, xs, alone):
        nq.nq_binlr_forward(L.h, x, y, batch)
    for L, x, a, b in zip(hs, xn, ys, alone):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
        assert rel_err(a.cpu().numpy(), L.oracle(x)) <= TOL
    nq.nq_plan_destroy(plan)
    for L in hs:
        L.close()
