"""Few row blocks at batch 1 to 8: the stage kernels that deal bit planes out to workgroups and quantise their input themselves, and the one-launch kernel of
small layers, at the edges of their shares.  Every output and t against the launches that quantise separately, bit for bit
(the arithmetic is exact up to the same roundings), and y against the oracle."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu
TOL = 1e-5          # of the largest output: two fixed-point steps of at least 21 bits and three roundings to fp32, as for all streaming paths


def both(L, nqopt, x, y_dtype="f32"):
    """y and t of the default route, and of separate launches with four waves per row block."""
    batch = x.shape[0]
    y, t = L.forward(x), nq.nq_binlr_read_intermediate(L.h, L.r, batch)
    for o in ("no_selfq", "no_fuse"):
        nqopt.set(o, 1)
    y4, t4 = L.forward(x), nq.nq_binlr_read_intermediate(L.h, L.r, batch)
    for o in ("no_selfq", "no_fuse"):
        nqopt.unset(o)
    return (y, t), (y4, t4)


@pytest.mark.parametrize("shape,x_dtype", [
    ((1, 1, 1), "f32"), ((5, 3, 2), "bf16"), ((130, 15, 17), "f16"), ((129, 16, 33), "f32"), ((300, 17, 40), "bf16"),   # rows around a lane's 4 and 16
    ((256, 255, 130), "f16"), ((100, 1023, 90), "bf16"), ((128, 1025, 128), "f32"), ((260, 1537, 129), "f16"),          # around a wave's unit
    ((4100, 500, 300), "bf16"), ((8300, 520, 300), "f16"), ((16500, 300, 200), "f32"), ((33000, 260, 140), "bf16"),     # 1, 2, 4 and 8 planes, and more row blocks than CUs
    ((700, 8192, 600), "bf16"), ((640, 8193, 600), "f16"), ((300, 16384, 260), "bf16"), ((200, 30000, 150), "f32"),     # inputs around what workgroups quantise
    ((4200, 3000, 4096), "f32"),                                                                                        # t as long as an LDS takes, two planes
])
def test_routes_agree(nqopt, shape, x_dtype):
    L = Layer(*shape, x_dtype, seed=11000 + shape[1])
    for batch in (1, 2, 3, 4, 5, 6, 8):
        x = synth.gen_x(batch, shape[1], 11100 + batch, x_dtype)
        (y, t), (y4, t4) = both(L, nqopt, x)
        assert np.array_equal(t, t4), (shape, batch)
        assert np.array_equal(y, y4), (shape, batch)
        assert rel_err(y, L.oracle(x)) <= TOL, (shape, batch)
    L.close()


@pytest.mark.parametrize("shape", [(640, 512, 256), (5003, 3001, 777)])
def test_token_values(nqopt, shape):
    """A token of zeros, the smallest normal and denormal magnitudes, the largest finite ones and non-finite values, beside ordinary tokens; a rank-wise scale."""
    L = Layer(*shape, "f32", seed=11500)
    nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(shape[2], 11501))
    for batch in (2, 7):
        x = synth.gen_x(batch, shape[1], 11510 + batch, "f32")
        for value in (0.0, 1e-38, 1e-42, 1e30):
            x[1, :] = value * np.sign(x[1])
            (y, t), (y4, t4) = both(L, nqopt, x)
            assert np.array_equal(y, y4) and np.array_equal(t, t4) and np.isfinite(y).all(), value
        for value in (np.inf, -np.inf, np.nan):
            x[1] = synth.gen_x(1, shape[1], 11520, "f32")[0]
            x[1, shape[1] - 1] = value
            (y, _), (y4, _) = both(L, nqopt, x)
            assert np.isnan(y[1]).all() and np.isnan(y4[1]).all(), value
            keep = [i for i in range(batch) if i != 1]
            assert np.array_equal(y[keep], y4[keep]) and np.isfinite(y[keep]).all(), value
    L.close()


@pytest.mark.parametrize("layers,batch,codes", [(3, 2, [35, 35]), (4, 4, [35, 35]), (7, 3, [35, 4]), (4, 8, [35, 35]), (12, 8, [16, 4]), (7, 5, [35, 4]), (7, 8, [16, 4]), (1, 1, [34, 33])])
def test_plans(nqopt, layers, batch, codes):
    """Levels of decoder blocks: 4096- and 7B-shaped layers of unequal reductions and ranks as one plan, against lone calls."""
    import torch
    shapes = [(4096, 4096, 1024)] * layers if layers != 7 else [(4096, 4096, 1024)] * 4 + [(11008, 4096, 1664)] * 2 + [(4096, 3000, 1664)]
    hs, xs, ys, lone = [], [], [], []
    for i, s in enumerate(shapes):
        hs.append(Layer(*s, "bf16", seed=11600 + 10 * (i % 7)))
        xs.append(to_device(synth.gen_x(batch, s[1], 11601 + i, "bf16"), "bf16"))
        ys.append(new_output(batch, s[0]))
        lone.append(new_output(batch, s[0]))
    plan = nq.nq_plan_create([L.h for L in hs], xs, ys, batch)
    print(layers, batch, nq.nq_plan_schedules(plan))
    assert nq.nq_plan_schedules(plan) == codes
    nq.nq_plan_forward(plan)
    for L, x, y in zip(hs, xs, lone):
        nq.nq_binlr_forward(L.h, x, y, batch)
    torch.cuda.synchronize()
    for i, (a, b) in enumerate(zip(ys, lone)):
        assert torch.equal(a, b) and not torch.isnan(a).any(), i
    nq.nq_plan_destroy(plan)
    for L in hs:
        L.close()


@pytest.mark.parametrize("batch,steps,own", [(1, 192, False), (2, 96, False), (2, 97, True), (3, 32, False), (3, 33, True), (4, 16, False), (4, 17, True), (5, 32, True), (8, 16, False), (8, 17, True)])
def test_inputs_quantised_along_by_workgroups_of_whole_row_blocks(nqopt, batch, steps, own):
    """132 row blocks, each with a workgroup of its own: where the stage quantises its input along (no launch and no time for it) and where a launch does."""
    import torch
    L = Layer(132 * 128 - 5, 70, 64 * steps - 3, "f32", seed=11700 + steps)
    x = to_device(synth.gen_x(batch, 70, 11701, "f32"), "f32")
    y, lone, narrow = (new_output(batch, L.d_out) for _ in range(3))
    plan = nq.nq_plan_create([L.h], [x], [y], batch)
    ms = nq.nq_plan_forward_timed(plan)
    nq.nq_binlr_forward(L.h, x, lone, batch)
    for o in ("no_selfq", "no_fuse"):
        nqopt.set(o, 1)
    nqopt.set("force_w", 4)
    nq.nq_binlr_forward(L.h, x, narrow, batch)
    torch.cuda.synchronize()
    assert torch.equal(y, lone) and torch.equal(y, narrow) and not torch.isnan(y).any()
    if batch > 1:
        assert (ms[2] > 0) == own, ms
    nq.nq_plan_destroy(plan)
    L.close()


@pytest.mark.parametrize("row_blocks,steps,layers,batch,along", [
    (28, 188, 1, 2, True), (28, 192, 1, 2, True), (64, 256, 1, 2, True), (128, 240, 1, 2, True), (128, 256, 1, 2, False), (28, 257, 1, 2, False),      # past 7B-shaped reductions, to what fits
    (3, 160, 1, 3, True), (12, 216, 1, 3, False), (28, 320, 1, 4, False), (128, 512, 1, 5, False), (8, 252, 1, 6, False), (8, 256, 1, 8, False),
    (45, 64, 5, 2, True), (116, 172, 12, 2, True), (128, 216, 6, 3, False), (6, 300, 6, 8, False)])
def test_plans_of_any_length(nqopt, row_blocks, steps, layers, batch, along):
    """Few row blocks of long reductions and of many layers: dealt out whatever the length, the input quantised along (no launch, no time for it) where it fits; the bits
    of four waves per row block."""
    import torch
    per = [row_blocks // layers + (i < row_blocks % layers) for i in range(layers)]
    hs = [Layer(70, 64 * steps - (5 if i == 0 else 64 * i), 128 * k - (3 if i == 0 else 0), "bf16", seed=11800 + i) for i, k in enumerate(per)]
    xs = [to_device(synth.gen_x(batch, L.d_in, 11801 + i, "bf16"), "bf16") for i, L in enumerate(hs)]
    ys, narrow = [new_output(batch, 70) for _ in hs], [new_output(batch, 70) for _ in hs]
    plan = nq.nq_plan_create([L.h for L in hs], xs, ys, batch)
    ms = nq.nq_plan_forward_timed(plan)
    assert (ms[0] == 0) == along, ms
    nqopt.set("force_w", 4)
    for L, x, y in zip(hs, xs, narrow):
        nq.nq_binlr_forward(L.h, x, y, batch)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) and not torch.isnan(a).any() for a, b in zip(ys, narrow))
    nq.nq_plan_destroy(plan)
    for L in hs:
        L.close()
