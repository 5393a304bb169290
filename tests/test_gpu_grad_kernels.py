"""The kernels behind the gradients at the edges of their splits: scale_grad's waves and columns in every pair of types; the
exact product and the transposed product where a workgroup takes all, half or a quarter of a tile (the fewer row blocks
and token groups, the fewer)."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000])
@pytest.mark.parametrize("batch", [1, 3, 4, 5, 63, 64, 65, 130])
@pytest.mark.parametrize("ta,tb", [("f32", "f32"), ("f16", "bf16"), ("bf16", "f16"), ("f32", "bf16"), ("f16", "f32")])
def test_scale_grad(n, batch, ta, tb):
    import torch
    a, b = synth.gen_x(batch, n, 7000 + n + batch, ta), synth.gen_x(batch, n, 7500 + n + batch, tb)
    out = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_scale_grad(to_device(a, ta), nq.DTYPE_BY_NAME[ta], to_device(b, tb), nq.DTYPE_BY_NAME[tb], batch, n, out)
    torch.cuda.synchronize()
    prod = synth.x_as_f64(a, ta) * synth.x_as_f64(b, tb)
    # binary64 sums of exact products, one rounding to fp32 (half an ulp, and a last bit for the order of the sums)
    assert np.all(np.abs(out.cpu().numpy() - prod.sum(0)) <= 2.0 ** -24 * np.abs(prod.sum(0)) + 2.0 ** -50 * np.abs(prod).sum(0))


def test_scale_grad_of_very_many_columns():
    """2^28 columns at 61 tokens: 16 waves per 64 columns would be 2^32 threads, more than a launch holds."""
    import torch
    n, batch = 1 << 28, 61
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 34 GB")
    a = torch.zeros((batch, n), dtype=torch.bfloat16, device="cuda")
    at = torch.tensor([0, 63, 64, 12345, 1 << 27, n - 65, n - 1], device="cuda")
    v = (torch.arange(batch * at.numel(), device="cuda") % 13 - 6).reshape(batch, -1)
    a[:, at] = v.bfloat16()
    out = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_scale_grad(a, nq.NQ_BF16, a, nq.NQ_BF16, batch, n, out)
    want = (v * v).sum(0).float()
    assert torch.equal(out[at], want)
    out[at] = 0.0
    assert not bool(out.any())
    del a, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d_out,d_in,r,batch", [
    (600, 70, 40, 40),              # few row blocks: a quarter of a tile's rows each
    (1100, 130, 1000, 128),         # 72 and 64 pairs of row block and token group: half, a quarter
    (2200, 2100, 300, 130),         # more than 128: whole tiles, a last group of two tokens
])
def test_exact_and_transposed_products_in_every_split(d_out, d_in, r, batch):
    import torch
    L = Layer(d_out, d_in, r, "bf16", seed=7700 + r, y_dtype="f32")
    x_np, g_np = synth.gen_x(batch, d_in, 7701, "bf16"), synth.gen_x(batch, d_out, 7702, "f32")
    x = to_device(x_np, "bf16")
    narrow, wide = new_output(batch, d_out), new_output(batch, d_out)
    nq.nq_binlr_forward_exact(L.h, x, narrow, batch)        # nothing reserved: passes of eight through the decode kernels
    nq.nq_binlr_reserve(L.h, batch)
    nq.nq_binlr_forward_exact(L.h, x, wide, batch)
    w = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, to_device(g_np, "f32"), w, batch)
    torch.cuda.synchronize()
    assert torch.equal(narrow, wide) and not torch.isnan(wide).any()
    d = L.data
    U, V = (nq.nq_unpack_signs(m, r).astype(np.float64) for m in (d.U_words, d.V_words))
    ref = ((g_np.astype(np.float64) * d.s_out.astype(np.float64)) @ U) @ V.T
    err = np.linalg.norm(w.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 2 * 2.0 ** -24          # two roundings to fp32; the fixed point's is below a tenth of that
    L.close()
