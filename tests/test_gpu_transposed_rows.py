"""The fixed point of the transposed products at the edges of a thread's four rows, of a wave's and a workgroup's (1024 threads of four) and of the padding: the input
gradient against binary64, tokens of zeros, of one large element (a fifth slice) and not finite among ordinary ones."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, to_device

pytestmark = pytest.mark.gpu


def signs(words, r):
    return nq.nq_unpack_signs(words, r).astype(np.float64)


@pytest.mark.parametrize("d_out", [1, 3, 4, 5, 127, 255, 257, 1021, 4095, 4096, 4097, 8201])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows(d_out, dtype):
    import torch
    d_in, r, batch = 130, 70, 19
    L = Layer(d_out, d_in, r, "f32", seed=14000 + d_out, y_dtype=dtype)
    g = synth.gen_x(batch, d_out, 14001, dtype)
    host = to_device(g, dtype).float()
    host[2] = 0.0
    host[3] *= 2.0 ** -6
    host[3, d_out // 2] = 2.0 ** 18                          # stands out from the others of its token
    host[17, d_out - 1] = float("nan")
    dev = host.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w = torch.empty((batch, d_in), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, dev.contiguous(), w, batch)
    got = w.cpu().numpy().astype(np.float64)
    U, V = signs(L.data.U_words, r), signs(L.data.V_words, r)
    v = dev.double().cpu().numpy() * L.data.s_out.view(np.float16).astype(np.float64)
    assert np.isnan(got[17]).all()
    keep = [b for b in range(batch) if b != 17]
    ref = (v[keep] @ U).astype(np.float32).astype(np.float64) @ V.T
    # one rounding of the intermediate and one of the result to fp32, and fixed point of 31 bits (39 where an element stands out) of sums of r signs
    bound = 3.0 * 2.0 ** -24 * np.abs(v[keep] @ U).sum(axis=1, keepdims=True) + 1e-30
    assert (np.abs(got[keep] - ref) <= bound).all()
    assert (got[2] == 0).all()
    L.close()
