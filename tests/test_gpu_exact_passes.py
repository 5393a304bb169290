"""The exact path above eight tokens: wide passes (after nq_binlr_reserve) give the bits of passes of eight, at the edges of
groups of 16 tokens, of eight waves per reduction and of row blocks; the values themselves against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import DECODE_TOL, Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_out,d_in,r,batch,reserve,x,y,mid", [
    (1, 1, 1, 9, 9, "f32", "f32", False),
    (128, 256, 128, 16, 16, "bf16", "f32", False),
    (129, 257, 65, 17, 17, "f16", "bf16", True),
    (300, 2049, 300, 40, 24, "bf16", "f16", False),       # passes of 32 tokens, the last of 8 through the decode kernels
    (1003, 515, 1025, 73, 64, "f32", "f32", True),        # passes of 64, nine left
    (260, 70, 33, 525, 600, "bf16", "f32", False),        # more than the widest pass of 512
])
def test_wide_passes_give_the_bits_of_passes_of_eight(d_out, d_in, r, batch, reserve, x, y, mid):
    import torch
    L = Layer(d_out, d_in, r, x, seed=6100 + r, y_dtype=y)
    d = L.data
    if mid:
        nq.nq_binlr_set_mid_scale(L.h, (np.random.default_rng(6101).standard_normal(r) * 0.5 + 1.0).astype(np.float16))
    x_np = synth.gen_x(batch, d_in, 6200 + batch, x)
    xd = to_device(x_np, x)
    narrow = [new_output(batch, d_out, y) for _ in range(2)]
    nq.nq_binlr_forward_exact(L.h, xd, narrow[0], batch)
    nq.nq_binlr_forward_unscaled(L.h, xd, narrow[1], batch)
    nq.nq_binlr_reserve(L.h, reserve)
    wide = [new_output(batch, d_out, y) for _ in range(2)]
    nq.nq_binlr_forward_exact(L.h, xd, wide[0], batch)
    nq.nq_binlr_forward_unscaled(L.h, xd, wide[1], batch)
    torch.cuda.synchronize()
    for a, b in zip(narrow, wide):
        assert not torch.isnan(b.float()).any()
        assert torch.equal(a, b)
    if y == "f32" and not mid:
        ref = oracle.forward_factored(d.U_words, d.V_words, d.s_out, d.s_in, d_out, d_in, r, synth.x_as_f64(x_np, x))
        assert rel_err(wide[0].cpu().numpy(), ref) <= DECODE_TOL
    L.close()


def test_layers_without_the_dense_path_take_the_wide_passes_too():
    import torch
    L = Layer(260, 520, 130, "bf16", seed=6300, flags=nq.NQ_FLAG_NO_PREFILL)
    x_np = synth.gen_x(50, 520, 6301, "bf16")
    x_np[5, 3] = 0x7F80                                   # +inf: that token only
    xd = to_device(x_np, "bf16")
    a, b = new_output(50, 260), new_output(50, 260)
    nq.nq_binlr_forward(L.h, xd, a, 50)
    nq.nq_binlr_reserve(L.h, 50)
    nq.nq_binlr_forward(L.h, xd, b, 50)
    torch.cuda.synchronize()
    assert torch.isnan(b[5]).all() and not torch.isnan(b[[4, 6]]).any()
    assert torch.equal(torch.nan_to_num(a, nan=7.0), torch.nan_to_num(b, nan=7.0))
    L.close()


@pytest.mark.parametrize("d_out,d_in,r,batch,x", [
    (200, 9000, 130, 20, "bf16"),                         # 512 threads hold the row, 1024, and rows that are read twice
    (130, 20000, 70, 18, "f32"),
    (70, 65536, 33, 17, "bf16"),
    (130, 20001, 65, 21, "f16"),                          # rows of odd lengths
    (70, 40001, 33, 17, "f32"),
    (64, 300, 9000, 20, "bf16"),                          # the same for the intermediate
    (64, 70, 40000, 17, "bf16"),
])
def test_long_rows_in_wide_passes(d_out, d_in, r, batch, x):
    import torch
    L = Layer(d_out, d_in, r, x, seed=6400 + d_in)
    xd = to_device(synth.gen_x(batch, d_in, 6401, x), x)
    narrow, wide = new_output(batch, d_out), new_output(batch, d_out)
    nq.nq_binlr_forward_exact(L.h, xd, narrow, batch)
    nq.nq_binlr_reserve(L.h, batch)
    nq.nq_binlr_forward_exact(L.h, xd, wide, batch)
    torch.cuda.synchronize()
    assert torch.equal(narrow, wide) and not torch.isnan(wide).any()
    L.close()


def test_accumulators_at_their_extreme_values_in_wide_passes():
    """Every sign +1, 65535 low bytes at -128, 127 or 127 (of -129) in 17 tokens: the largest int32 sums the format produces."""
    import torch
    d_out, d_in, r, batch = 128, nq.NQ_MAX_DIM, 64, 17
    ones = lambda rows: oracle.pack_signs(np.ones((rows, r), dtype=np.int8))
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(synth.LinearShape("m", d_out, d_in, r), ones(d_out), ones(d_in),
                                                          np.ones(d_out, dtype=np.float16), np.ones(d_in, dtype=np.float16)))
    nq.nq_binlr_reserve(L.h, batch)
    x = np.empty((batch, d_in))
    for t, low in enumerate(np.resize([128.0, 127.0, -129.0], batch)):
        row = np.full(d_in, low)
        row[0] = 2.0 ** 22 - 2.0 ** 16                    # pins the step of the first quantisation at 1
        s = row.sum()
        row[1] -= s % max(1.0, 2.0 ** (np.frexp(abs(s))[1] - 22))      # and makes t a multiple of the second's
        x[t] = row if t % 2 else -row
    y = new_output(batch, d_out)
    nq.nq_binlr_forward_exact(L.h, to_device(x.astype(np.float32), "f32"), y, batch)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(np.float64), L.oracle(x.astype(np.float32)))
    L.close()
