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
