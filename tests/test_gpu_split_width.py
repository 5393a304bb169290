"""How many waves share a row block in launches that do not fill the chip, at the lines between them; the bits do not depend on it."""
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,row_blocks,steps,waves", [
    (2, 28, 188, 4), (2, 28, 192, 16), (2, 16, 256, 4), (2, 16, 320, 16), (2, 1, 192, 16), (2, 112, 192, 16), (2, 257, 192, 4),
    (3, 3, 368, 4), (3, 3, 448, 16), (3, 28, 316, 4), (3, 56, 256, 16),
    (4, 112, 252, 4), (4, 112, 256, 16), (4, 28, 320, 4), (5, 112, 448, 4),
    (6, 8, 252, 4), (6, 8, 256, 12), (8, 224, 256, 12),
])
def test_waves_per_row_block(nqopt, batch, row_blocks, steps, waves):
    import torch
    d_out, d_in, r = 128, 64 * steps, 128 * row_blocks
    L = Layer(d_out, d_in, r, "f32", seed=9700 + steps)
    x = to_device(synth.gen_x(batch, d_in, 9701, "f32"), "f32")
    y, narrow = new_output(batch, d_out), new_output(batch, d_out)
    plan = nq.nq_plan_create([L.h], [x], [y], batch)
    assert nq.nq_plan_schedules(plan)[0] == waves
    nq.nq_plan_forward(plan)
    nqopt.set("force_w", 4)
    nq.nq_binlr_forward(L.h, x, narrow, batch)
    torch.cuda.synchronize()
    assert torch.equal(y, narrow) and not torch.isnan(y).any()
    nq.nq_plan_destroy(plan)
    L.close()


@pytest.mark.parametrize("layers,waves", [(5, 4), (12, 16), (35, 16), (40, 4)])
def test_waves_of_launches_with_reductions_of_different_lengths(layers, waves):
    """Layers of 7B-shaped blocks (64 and 172 steps) as one plan at batch 2."""
    import torch
    shapes = [synth.llama2_7b_block()[i % 7] for i in range(layers)]
    hs, xs, ys, lone = [], [], [], []
    for i, s in enumerate(shapes):
        hs.append(Layer(s.d_out, s.d_in, s.r, "bf16", seed=9800 + 10 * (i % 7)))
        xs.append(to_device(synth.gen_x(2, s.d_in, 9801 + i, "bf16"), "bf16"))
        ys.append(new_output(2, s.d_out))
        lone.append(new_output(2, s.d_out))
    plan = nq.nq_plan_create([L.h for L in hs], xs, ys, 2)
    assert nq.nq_plan_schedules(plan)[0] == waves
    nq.nq_plan_forward(plan)
    for L, x, y in zip(hs, xs, lone):
        nq.nq_binlr_forward(L.h, x, y, 2)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(ys, lone))
    nq.nq_plan_destroy(plan)
    for L in hs:
        L.close()
