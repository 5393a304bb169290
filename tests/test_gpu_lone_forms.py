"""Every form that the launches of few row blocks are compiled in, asked for by name: groups of one to eight tokens, one to eight bit planes of a workgroup, input quantised along
by 16 waves (16 or four elements of a lane at a time) or by eight, or quantised by a launch of its own.  Outputs and t against the launches that deal nothing out, bit for bit
(the arithmetic is exact up to the same roundings), and a form that no launch has is refused."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu
TOL = 1e-5          # of the largest output: two fixed-point steps of at least 21 bits and three roundings to fp32, as for all streaming paths
FORMS = [(kind, pl) for kind in (0, 1, 3) for pl in (1, 2, 4, 8)] + [(2, 8), (4, 8)]


def has(kind, per, pl, steps):
    """What the compiled forms hold: columns of five tokens (eight on eight waves), a wave's share of the input in registers, sums and fixed point in LDS."""
    if kind >= 3:
        return per <= 5 if kind == 3 else 5 < per <= 8
    waves = 8 if kind == 2 else 16
    if (per > 5 and kind < 2) or per * -(-steps // 16) > 32 or (kind == 1 and per * -(-steps // 4) > 64):
        return False
    ints = pl * 4 * (12 * per + 4 + 4 * (per & 1))
    return waves * ((ints + 15) // 32 * 32 + 16) * 4 + 96 + per * (steps * 192 + 48) <= 160 * 1024


def plain(nqopt, L, x, batch):
    y = new_output(batch, L.d_out)
    for o in ("no_selfq", "no_fuse"):
        nqopt.set(o, 1)
    nq.nq_binlr_forward_exact(L.h, x, y, batch)
    for o in ("no_selfq", "no_fuse"):
        nqopt.unset(o)
    return y.cpu().numpy(), nq.nq_binlr_read_intermediate(L.h, L.r, batch) if batch <= 8 else None


@pytest.mark.parametrize("shape,x_dtype,batches", [
    ((1530, 1003, 600), "bf16", (1, 2, 3, 4, 5, 6, 7, 8)),         # every instance: five and twelve row blocks of 16 and 12 steps
    ((1100, 8189, 260), "f16", (2, 4, 6, 8)),                      # shares of 32 elements in every lane, and past them
    ((260, 40, 1290), "f32", (9, 17, 24)),                         # groups on one XCD and on all
])
@pytest.mark.parametrize("kind,pl", FORMS)
def test_forms(nqopt, shape, x_dtype, batches, kind, pl):
    L = Layer(*shape, x_dtype, seed=15000 + shape[1])
    nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(shape[2], 15001))
    nq.nq_binlr_reserve(L.h, max(batches))
    ran = 0
    steps = [-(-n // 256) * 4 for n in shape[1:]]
    for batch in batches:
        x = to_device(synth.gen_x(batch, shape[1], 15010 + batch, x_dtype), x_dtype)
        ref, t_ref = plain(nqopt, L, x, batch)
        for groups in range(1, batch + 1):
            per = -(-batch // groups)
            if per > 8 or -(-batch // per) != groups:
                continue
            y = new_output(batch, shape[0])
            nqopt.set("lone_form", 100 * per + 10 * pl + kind)
            if all(has(kind, per, pl, s) for s in steps):
                nq.nq_binlr_forward_exact(L.h, x, y, batch)
                assert np.array_equal(y.cpu().numpy(), ref), (batch, per)
                if t_ref is not None:
                    assert np.array_equal(nq.nq_binlr_read_intermediate(L.h, L.r, batch), t_ref), (batch, per)
                ran += 1
            else:
                with pytest.raises(nq.NQError):
                    nq.nq_binlr_forward_exact(L.h, x, y, batch)
            nqopt.unset("lone_form")
    assert ran or shape[1] > 4096
    L.close()


@pytest.mark.parametrize("kind,pl", FORMS)
def test_forms_on_the_row_blocks_of_several_layers(nqopt, kind, pl):
    """Layers of unequal lengths in one launch, against calls on each alone."""
    shapes, batch = [(300, 1000, 200), (129, 3, 64), (520, 1020, 300)], 7
    hs = [Layer(*s, "f16", seed=15100 + i) for i, s in enumerate(shapes)]
    xn = [synth.gen_x(batch, s[1], 15110 + i, "f16") for i, s in enumerate(shapes)]
    xs = [to_device(x, "f16") for x in xn]
    refs = [plain(nqopt, L, x, batch)[0] for L, x in zip(hs, xs)]
    for groups in (1, 2, 3, 4, 7):
        per = -(-batch // groups)
        if not has(kind, per, pl, 16):
            continue
        ys = [new_output(batch, s[0]) for s in shapes]
        nqopt.set("lone_form", 100 * per + 10 * pl + kind)
        plan = nq.nq_plan_create([L.h for L in hs], xs, ys, batch)
        ms = nq.nq_plan_forward_timed(plan)
        assert (ms[0] == 0) == (ms[2] == 0) == (kind < 3), ms
        for y, ref, L, x in zip(ys, refs, hs, xn):
            assert np.array_equal(y.cpu().numpy(), ref), per
            assert rel_err(y.cpu().numpy(), L.oracle(x)) <= TOL
        nq.nq_plan_destroy(plan)
        nqopt.unset("lone_form")
    for L in hs:
        L.close()
