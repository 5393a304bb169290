"""More than eight tokens of a small layer: dealt out in groups of up to eight, and nq_binlr_forward's choice between the exact and
the dense path, at the edges of groups, rows and inputs that workgroups quantise themselves."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import DECODE_TOL, Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu
DENSE_TOL = 7e-4        # fp16 operands: of the largest output, as for the dense path elsewhere


@pytest.mark.parametrize("shape,x_dtype,y_dtype,batches", [
    ((1, 1, 1), "f32", "f32", (9, 17, 512)),
    ((130, 15, 17), "f16", "bf16", (9, 16, 25, 200)),
    ((129, 1023, 90), "bf16", "f32", (10, 23, 64, 127)),          # groups of 5, 8 and fewer in the last
    ((4096, 260, 140), "f32", "f16", (9, 24, 32, 33)),            # 32 row blocks: 2, 4 and 8 planes, and past what is dealt out
    ((300, 8192, 600), "bf16", "bf16", (9, 20, 40)),              # inputs around what workgroups quantise
    ((200, 30000, 150), "f16", "f32", (9, 13, 31)),
    ((260, 300, 3001), "bf16", "f32", (11, 37)),
])
def test_groups_of_eight_give_the_bits_of_groups_of_16(nqopt, shape, x_dtype, y_dtype, batches):
    import torch
    L = Layer(*shape, x_dtype, seed=12000 + shape[1], y_dtype=y_dtype)
    nq.nq_binlr_reserve(L.h, max(batches))
    nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(shape[2], 12001))
    for batch in batches:
        x_np = synth.gen_x(batch, shape[1], 12100 + batch, x_dtype)
        x_np[batch - 1, 0] = np.float32(np.nan).astype(x_np.dtype) if x_np.dtype.kind == "f" else 0x7FC0     # the last token's own
        xd = to_device(x_np, x_dtype)
        for call in (nq.nq_binlr_forward_exact, nq.nq_binlr_forward_unscaled):
            a, b = new_output(batch, shape[0], y_dtype), new_output(batch, shape[0], y_dtype)
            call(L.h, xd, a, batch)
            nqopt.set("no_selfq", 1)
            call(L.h, xd, b, batch)
            nqopt.unset("no_selfq")
            torch.cuda.synchronize()
            assert torch.isnan(a[batch - 1]).all() and not torch.isnan(a[: batch - 1].float()).any(), batch
            assert torch.equal(a[: batch - 1], b[: batch - 1]) and torch.isnan(b[batch - 1]).all(), batch
    L.close()


@pytest.mark.parametrize("shape,x_dtype", [((5003, 301, 77), "f16"), ((256, 256, 64), "bf16"), ((384, 2500, 700), "f32")])
def test_forward_on_either_path(nqopt, shape, x_dtype):
    """Few tokens take the exact path and give its bits, reserved or not; the dense path when asked for, within its own tolerance."""
    import torch
    for batch in (9, 24, 65, 300):
        L = Layer(*shape, x_dtype, seed=12200 + batch)
        x_np = synth.gen_x(batch, shape[1], 12210 + batch, x_dtype)
        xd = to_device(x_np, x_dtype)
        ref = L.oracle(x_np)
        y, again, exact, dense = (new_output(batch, shape[0]) for _ in range(4))
        nq.nq_binlr_forward(L.h, xd, y, batch)
        nq.nq_binlr_reserve(L.h, 2 * batch)
        nq.nq_binlr_forward(L.h, xd, again, batch)
        nq.nq_binlr_forward_exact(L.h, xd, exact, batch)
        nqopt.set("dense_only", 1)
        nq.nq_binlr_forward(L.h, xd, dense, batch)
        nqopt.unset("dense_only")
        torch.cuda.synchronize()
        assert torch.equal(y, again)
        assert torch.equal(y, exact) or torch.equal(y, dense)
        if batch <= 24:
            assert torch.equal(y, exact) and not torch.equal(y, dense)
        assert rel_err(exact.cpu().numpy(), ref) <= DECODE_TOL
        assert rel_err(dense.cpu().numpy(), ref) <= DENSE_TOL
        L.close()


@pytest.mark.parametrize("shape,x_dtype,batches", [
    ((1536, 1536, 1536), "bf16", (41, 48, 80)),                   # two workgroups per pair: groups of 16 in both stages
    ((2000, 3000, 1900), "f16", (33, 64)),                        # of eight in both
    ((1280, 8200, 1280), "bf16", (56, 96)), ((1030, 700, 1024), "f32", (72, 120)),      # of eight in the first only
    ((2048, 512, 1800), "bf16", (40, 64)),                        # in the second only
    ((250, 640, 256), "f16", (257, 320, 512)),
])
def test_each_stage_has_a_form_of_its_own(nqopt, shape, x_dtype, batches):
    import torch
    L = Layer(*shape, x_dtype, seed=12300 + shape[1])
    nq.nq_binlr_reserve(L.h, max(batches))
    nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(shape[2], 12301))
    for batch in batches:
        xd = to_device(synth.gen_x(batch, shape[1], 12310 + batch, x_dtype), x_dtype)
        a, b = new_output(batch, shape[0]), new_output(batch, shape[0])
        nq.nq_binlr_forward_exact(L.h, xd, a, batch)
        nqopt.set("no_selfq", 1)
        nq.nq_binlr_forward_exact(L.h, xd, b, batch)
        nqopt.unset("no_selfq")
        torch.cuda.synchronize()
        assert torch.equal(a, b) and not torch.isnan(a).any(), batch
    L.close()


@pytest.mark.parametrize("shape,batch,takes_exact", [
    ((256, 32768, 100), 24, True), ((256, 65536, 100), 9, True), ((256, 65536, 100), 16, False), ((130, 50000, 64), 64, False),
    ((128, 128, 128), 512, True), ((256, 256, 250), 256, True), ((256, 256, 250), 320, False), ((256, 512, 250), 320, True),
])
def test_forward_takes_the_faster_path_of_small_layers(nqopt, shape, batch, takes_exact):
    """Many tokens of a few row blocks and reductions longer than 32768: the bits of the path that was measured to be the faster one."""
    import torch
    L = Layer(*shape, "bf16", seed=12400 + shape[1])
    nq.nq_binlr_reserve(L.h, batch)
    xd = to_device(synth.gen_x(batch, shape[1], 12410 + batch, "bf16"), "bf16")
    y, exact, dense = (new_output(batch, shape[0]) for _ in range(3))
    nq.nq_binlr_forward(L.h, xd, y, batch)
    nq.nq_binlr_forward_exact(L.h, xd, exact, batch)
    nqopt.set("dense_only", 1)
    nq.nq_binlr_forward(L.h, xd, dense, batch)
    torch.cuda.synchronize()
    assert not torch.equal(exact, dense)
    assert torch.equal(y, exact if takes_exact else dense)
    L.close()
