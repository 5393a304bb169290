"""The products with the transposed sign matrices (nq_binlr_forward_transposed_unscaled, nq_binlr_backward_input) at the
edges of their kernels: 64-column steps, 128-row blocks, eight waves per reduction, groups of 16 tokens, passes."""
import numpy as np
import pytest

import oracle
from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, to_device

pytestmark = pytest.mark.gpu

# u = U^T(..) and w = V u are each rounded once to fp32 (relative 2-norm error 2^-24 / sqrt(3) each for values spread over
# their binade, at most 2^-24); the fixed point behind them is below a tenth of that.
NORM_TOL = 2 * 2.0**-24


def _reference(L, g64):
    d = L.data
    U = nq.nq_unpack_signs(d.U_words, L.r).astype(np.float64)
    V = nq.nq_unpack_signs(d.V_words, L.r).astype(np.float64)
    return ((g64 * d.s_out.astype(np.float64)) @ U) @ V.T


def _norm_err(a, ref):
    return np.linalg.norm(a.astype(np.float64) - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("d_out,d_in,r,batch,dt", [
    (1, 1, 1, 1, "f32"), (64, 64, 64, 16, "bf16"), (127, 63, 65, 17, "f16"), (129, 65, 128, 15, "f32"),
    (1024, 130, 129, 33, "bf16"),            # eight row blocks: one per wave
    (1025, 66, 257, 2, "f16"),               # nine: the second tile of one wave only
    (2051, 321, 1100, 31, "f32"),            # seventeen; rows of an odd length (scalar loads)
    (260, 200, 70, 530, "bf16"),             # more than one pass of 512 tokens
    (9000, 300, 64, 3, "f32"),               # a vector longer than the quantiser keeps in registers
])
def test_transposed_products_at_the_edges(d_out, d_in, r, batch, dt):
    import torch
    L = Layer(d_out, d_in, r, "f32", seed=5100 + r, y_dtype=dt)
    g_np = synth.gen_x(batch, d_out, 5200 + batch, dt)
    g = to_device(g_np, dt)
    w = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    dx = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, g, w, batch)
    nq.nq_binlr_backward_input(L.h, g, dx, batch)
    torch.cuda.synchronize()
    ref = _reference(L, synth.x_as_f64(g_np, dt))
    for t in range(batch):                   # token by token: each has its own fixed-point step
        assert _norm_err(w[t].cpu().numpy(), ref[t]) <= NORM_TOL, t
        assert _norm_err(dx[t].cpu().numpy(), ref[t] * L.data.s_in.astype(np.float64)) <= NORM_TOL, t
    L.close()


def test_one_large_element_among_many_costs_no_precision():
    """The fixed point's step follows a token's maximum: one element 2^20 times the others must not cost the sum of the
    65536 others its precision (a step of 2^-30 of the maximum misses the bound)."""
    import torch
    d_out, d_in, r, batch = 65536, 64, 64, 3
    L = Layer(d_out, d_in, r, "f32", seed=5400)
    g_np = synth.gen_x(batch, d_out, 5401, "f32")
    at = [17, 40000, 65535]
    for t in range(batch):
        g_np[t, at[t]] = np.float32(2.0**20)
    w = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, to_device(g_np, "f32"), w, batch)
    torch.cuda.synchronize()
    ref = _reference(L, g_np.astype(np.float64))
    for t in range(batch):
        assert _norm_err(w[t].cpu().numpy(), ref[t]) <= NORM_TOL, t
    L.close()


@pytest.mark.parametrize("d_out,d_in,r,batch", [(2100, 300, 70, 5), (300, 130, 64, 19), (1500, 200, 4200, 40)])
def test_wide_tokens_are_exact_beside_others(d_out, d_in, r, batch):
    """Two elements of 2^36 that cancel in every column leave sums of small integers, which only a fifth byte slice holds: bit for
    bit, in tokens with and without such a pair side by side, on half and on whole tiles (the last: 66 steps x 3 groups)."""
    import torch
    U_words, V_words = synth.gen_sign_words(d_out, r, 5501), synth.gen_sign_words(d_in, r, 5502)
    rows = [(3, 131), (0, d_out - 1), (d_out // 2, 17)]
    for a, b in rows:
        U_words[b] = U_words[a]
    ones = lambda n: np.ones(n, dtype=np.float16)
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(synth.LinearShape("t", d_out, d_in, r), U_words, V_words, ones(d_out), ones(d_in)))
    g_np = np.random.default_rng(5503).integers(-100, 101, (batch, d_out)).astype(np.float32)
    for t in range(0, batch, 3):
        a, b = rows[t // 3 % 3]
        g_np[t, a], g_np[t, b] = 2.0**36, -2.0**36
    w = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, to_device(g_np, "f32"), w, batch)
    torch.cuda.synchronize()
    assert np.array_equal(w.cpu().numpy(), _reference(L, g_np.astype(np.float64)).astype(np.float32))
    L.close()


@pytest.mark.parametrize("d_out,r", [(1024, 64), (1025, 64), (2049, 70), (4097, 200), (9000, 24), (5000, 1000)])     # 1, 2, 4, 8, 8, 4 parts of one token
@pytest.mark.parametrize("mid", [False, True])
def test_reductions_dealt_out_to_several_workgroups(d_out, r, mid):
    """Few tokens of a tall, narrow first product: its rows are dealt out, and the sums added up by the second product's
    quantisation.  The bits are those of a batch that fills the chip without; the values those of the definition."""
    import torch
    d_in, batch = 150, 530
    L = Layer(d_out, d_in, r, "f32", seed=5600 + r)
    scale = np.ones(r)
    if mid:
        s_mid = (np.random.default_rng(5601).standard_normal(r) * 0.5 + 1.0).astype(np.float16)
        nq.nq_binlr_set_mid_scale(L.h, s_mid)
        scale = s_mid.astype(np.float64)
    g_np = synth.gen_x(batch, d_out, 5602, "f32")
    g_np[2, 1] = np.float32(2.0**24)                      # a wide token
    g = to_device(g_np, "f32")
    w = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    few = [torch.full((n, d_in), float("nan"), dtype=torch.float32, device="cuda") for n in (1, 4, 5, 8, 17)]
    nq.nq_binlr_backward_input(L.h, g, w, batch)
    for f in few:
        nq.nq_binlr_backward_input(L.h, g[: f.shape[0]], f, f.shape[0])
    torch.cuda.synchronize()
    d = L.data
    U, V = (nq.nq_unpack_signs(m, r).astype(np.float64) for m in (d.U_words, d.V_words))
    ref = (((((g_np[:17].astype(np.float64) * d.s_out.astype(np.float64)) @ U) * scale) @ V.T)) * d.s_in.astype(np.float64)
    for f in few:
        n = f.shape[0]
        assert torch.equal(f, w[:n])
        for t in range(n):
            assert _norm_err(f[t].cpu().numpy(), ref[t]) <= NORM_TOL, t
    L.close()


@pytest.mark.parametrize("d_in", [64, 8200])              # half tiles, whole tiles in the second product
def test_accumulators_at_their_extreme_values(d_in):
    """Every sign +1 and 65535 pairs of bytes at -128: the largest joined sums of two slices (below 2^31 over four waves)."""
    import torch
    d_out, r, batch = 65536, 64, 17
    ones = lambda rows: oracle.pack_signs(np.ones((rows, r), dtype=np.int8))
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(synth.LinearShape("m", d_out, d_in, r), ones(d_out), ones(d_in),
                                                          np.ones(d_out, dtype=np.float16), np.ones(d_in, dtype=np.float16)))
    g = np.full((batch, d_out), -(128.0 * 256 + 128))
    g[:, 0] = 2.0**30                                     # (few large elements: five slices)
    g[1::3] = -2.0**30 * 1.96875                          # (none: four; the two upper slices near their ends)
    g[2::3] *= -1.0
    w = torch.full((batch, d_in), float("nan"), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, to_device(g.astype(np.float32), "f32"), w, batch)
    torch.cuda.synchronize()
    u = g.sum(1).astype(np.float32).astype(np.float64)
    assert np.array_equal(w.cpu().numpy(), np.repeat((r * u).astype(np.float32)[:, None], d_in, axis=1))
    L.close()


def test_a_non_finite_gradient_poisons_its_own_token_only():
    import torch
    d_out, d_in, r, batch = 300, 200, 100, 19
    L = Layer(d_out, d_in, r, "f32", seed=5300)
    g_np = synth.gen_x(batch, d_out, 5301, "f32")
    g_np[3, 7], g_np[16, 299], g_np[18] = np.inf, np.nan, 0.0
    w = torch.zeros((batch, d_in), dtype=torch.float32, device="cuda")
    nq.nq_binlr_forward_transposed_unscaled(L.h, to_device(g_np, "f32"), w, batch)
    torch.cuda.synchronize()
    got = w.cpu().numpy()
    assert np.isnan(got[[3, 16]]).all() and not got[18].any()
    clean = [t for t in range(batch) if t not in (3, 16, 18)]
    ref = _reference(L, np.nan_to_num(g_np, nan=0.0, posinf=0.0).astype(np.float64))
    assert _norm_err(got[clean], ref[clean]) <= NORM_TOL
    L.close()
