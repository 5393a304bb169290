"""The dense path on pair sums and differences (sparse matrix instruction): activations of small integers with unit scales make
every step of it exact, so the result must equal the integer product bit for bit -- a wrong pair, position, plane, lane or padding
shows -- at the edges of pairs (8 columns), steps (64), row blocks (128), tiles of 32 and 64 tokens and their groups of
four waves, and in every tiling; then odd row lengths in every type against the oracle, and values at the ends of fp32's range."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, check_rounded, exact_forward, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu

# x'' and T are rounded to fp16 (2^-11 relative each, as pair sums and differences; random signs): a few 1e-4 of the largest output
PREFILL_TOL = 7e-4


@pytest.fixture(autouse=True)
def dense_path(nqopt):
    """Small layers take the exact path where it is the faster one; what is tested here is the dense one."""
    nqopt.set("dense_only", 1)


def unit_layer(d_out, d_in, r, x_dtype, y_dtype, seed):
    ones = lambda n: np.ones(n, dtype=np.float16)
    return Layer(d_out, d_in, r, x_dtype, y_dtype=y_dtype, data=synth.LayerData(
        synth.LinearShape("t", d_out, d_in, r), synth.gen_sign_words(d_out, r, seed + 1), synth.gen_sign_words(d_in, r, seed + 2),
        ones(d_out), ones(d_in)))


def signs(words, r):
    bits = np.unpackbits(np.ascontiguousarray(words).view(np.uint8), axis=1, bitorder="little")[:, :r]
    return bits.astype(np.int64) * 2 - 1


@pytest.mark.parametrize("d_out,d_in,r,batch", [
    (1, 1, 1, 9), (5, 7, 3, 12), (130, 9, 17, 33), (127, 15, 64, 64), (128, 16, 65, 65), (129, 63, 127, 63), (64, 65, 129, 31),
    (513, 257, 200, 100), (640, 1000, 385, 130), (1027, 511, 700, 70), (300, 2047, 520, 257)])
@pytest.mark.parametrize("tg,splits,ks", [(None, None, None), (2, 1, 1), (4, 1, 1), (4, 3, 1), (4, 1, 2), (4, 2, 2)])
def test_small_integers_are_exact(nqopt, d_out, d_in, r, batch, tg, splits, ks):
    for name, v in (("pf_tg", tg), ("pf_splits", splits), ("pf_ks", ks)):
        if v:
            nqopt.set(name + "1", v)
            nqopt.set(name + "2", v)
    L = unit_layer(d_out, d_in, r, "f32", "f32", 8100 + r)
    x = np.random.default_rng(8200 + batch).integers(-1, 2, (batch, d_in))
    t = x @ signs(L.data.V_words, r)
    assert 2 * np.abs(t).max() <= 2048                # pair sums of T are whole numbers that fp16 holds
    y = L.forward(x.astype(np.float32))
    assert np.array_equal(y, (t @ signs(L.data.U_words, r).T).astype(np.float32))
    L.close()


@pytest.mark.parametrize("d_out,d_in,r,batch", [(131, 33, 40, 21), (1001, 1503, 257, 70), (258, 4097, 300, 150)])
@pytest.mark.parametrize("x_dtype,y_dtype", [("f32", "f16"), ("f16", "bf16"), ("bf16", "f32")])
def test_odd_row_lengths(d_out, d_in, r, batch, x_dtype, y_dtype):
    L = Layer(d_out, d_in, r, x_dtype, seed=8300 + r, y_dtype=y_dtype)
    x = synth.gen_x(batch, d_in, 8400 + batch, x_dtype)
    y, ref = L.forward(x), L.oracle(x)
    assert np.isfinite(y).all() and not np.array_equal(y, exact_forward(L, x))
    if y_dtype == "f32":
        assert rel_err(y, ref) <= PREFILL_TOL
    else:
        check_rounded(y, ref, y_dtype, PREFILL_TOL)
    L.close()


@pytest.mark.parametrize("d_out,d_in,r,batch", [
    (1, 1, 1, 9), (5, 7, 3, 12), (130, 9, 17, 33), (127, 15, 64, 64), (128, 16, 65, 65), (129, 63, 127, 63), (64, 65, 129, 31),
    (513, 257, 200, 100), (640, 1000, 385, 130), (1027, 511, 700, 70), (300, 2047, 520, 257)])
@pytest.mark.parametrize("tg,splits,ks", [(None, None, None), (2, 1, 1), (4, 1, 1), (4, 3, 1), (4, 1, 2), (4, 2, 2)])
def test_small_integers_are_exact_in_pairs(nqopt, d_out, d_in, r, batch, tg, splits, ks):
    """The same with s_in = 3: such layers take pairs (fp32 activations times 3 are not in general exact in fp16)."""
    for name, v in (("pf_tg", tg), ("pf_splits", splits), ("pf_ks", ks)):
        if v:
            nqopt.set(name + "1", v)
            nqopt.set(name + "2", v)
    U, V = synth.gen_sign_words(d_out, r, 8801 + r), synth.gen_sign_words(d_in, r, 8802 + r)
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(synth.LinearShape("t", d_out, d_in, r), U, V,
                                                          np.ones(d_out, dtype=np.float16), np.full(d_in, 3.0, dtype=np.float16)))
    x = np.random.default_rng(8900 + batch).integers(-1, 2, (batch, d_in))
    t = 3 * x @ signs(V, r)
    assert 2 * np.abs(t).max() <= 2048
    y = L.forward(x.astype(np.float32))
    assert np.array_equal(y, (t @ signs(U, r).T).astype(np.float32))
    L.close()


@pytest.mark.parametrize("d_out,d_in,r,batch", [(5, 7, 3, 12), (130, 65, 129, 33), (260, 300, 200, 70), (129, 255, 65, 100)])
@pytest.mark.parametrize("tg,splits,ks", [(None, None, None), (2, 1, 1), (4, 1, 1), (4, 3, 1), (4, 1, 2), (4, 2, 2)])
@pytest.mark.parametrize("x_dtype", ["f32", "f16", "bf16"])
def test_exact_scaled_activations_are_not_rounded(nqopt, d_out, d_in, r, batch, tg, splits, ks, x_dtype):
    """Where s_in leaves s_in (.) x exact in fp16 (powers of two; up to 3 significant bits beside bf16) the first product has no
    rounding: T is the exact product rounded once to fp16, and y, whose sums fit fp32 here, follows bit for bit.  Sums of two
    such columns need more than 11 bits."""
    for name, v in (("pf_tg", tg), ("pf_splits", splits), ("pf_ks", ks)):
        if v:
            nqopt.set(name + "1", v)
            nqopt.set(name + "2", v)
    rng = np.random.default_rng(8600 + r + batch)
    s_in = rng.choice([1.0, 1.25, 1.5, 1.75] if x_dtype == "bf16" else [0.25, 0.5, 1.0], d_in).astype(np.float16)
    top = 255 if x_dtype == "bf16" else 2047
    x = rng.integers(-top, top + 1, (batch, d_in)).astype(np.float64)
    x[:, 0] = top                                     # (the token's power of two is then the same for every token)
    U, V = synth.gen_sign_words(d_out, r, 8701), synth.gen_sign_words(d_in, r, 8702)
    L = Layer(d_out, d_in, r, x_dtype, data=synth.LayerData(synth.LinearShape("t", d_out, d_in, r), U, V,
                                                            np.ones(d_out, dtype=np.float16), s_in))
    t = (x * s_in.astype(np.float64)) @ signs(V, r)
    T = t.astype(np.float16).astype(np.float64)
    assert np.abs(t).max() < 65504 and 4 * np.abs(T).sum(1).max() < 2**24
    xs = (x.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16) if x_dtype == "bf16" else x.astype({"f32": np.float32, "f16": np.float16}[x_dtype])
    assert np.array_equal(synth.x_as_f64(xs, x_dtype), x)
    assert np.array_equal(L.forward(xs), (T @ signs(U, r).T).astype(np.float32))
    L.close()


def test_values_at_the_ends_of_the_range():
    """Tokens at the ends of the path's range keep their precision (the per-token power of two is clamped: 2^113 is the first
    maximum that meets the clamp); infinities poison their own token only."""
    d_out, d_in, r = 200, 300, 90
    L = unit_layer(d_out, d_in, r, "f32", "f32", 8500)
    L.close()
    s_out = np.full(d_out, 2.0 ** -14, dtype=np.float16)
    d = L.data
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(d.shape, d.U_words, d.V_words, s_out, d.s_in))
    x = synth.gen_x(40, d_in, 8501, "f32")
    x[3] *= np.float32(2.0 ** 113 / np.abs(x[3]).max())
    x[4] *= np.float32(1e-30)
    x[7, 5] = np.inf
    y, ref = L.forward(x), L.oracle(np.where(np.isfinite(x), x, 0).astype(np.float32))
    for b in range(40):
        if b == 7:
            assert not np.isfinite(y[b]).any()
        else:
            assert np.abs(y[b] - ref[b]).max() <= PREFILL_TOL * np.abs(ref[b]).max(), b
    L.close()


@pytest.mark.parametrize("unit", [True, False])
def test_largest_tokens_that_fp16_operands_hold(unit):
    """x'' fits fp16 up to max|x'| = 65504 * 2^100, and so do the sums of two columns, which have to be scaled down by one more."""
    d_out, d_in, r = 200, 300, 90
    s_in = np.ones(d_in, dtype=np.float16) if unit else synth.gen_scales(d_in, 8601)
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(
        synth.LinearShape("t", d_out, d_in, r), synth.gen_sign_words(d_out, r, 8602), synth.gen_sign_words(d_in, r, 8603),
        np.full(d_out, 2.0 ** -14, dtype=np.float16), s_in))
    x = synth.gen_x(24, d_in, 8604, "f32")
    for b in range(24):                                   # max|x'| = 2^112.125 .. 2^115.0, 2^115.875, 2^115.99
        top = 2.0 ** (112 + (b + 1) / 8) if b < 22 else 2.0 ** (115.875 if b == 22 else 115.99)
        xp = x[b].astype(np.float64) * s_in.astype(np.float64)
        x[b] = (x[b].astype(np.float64) * top / np.abs(xp).max()).astype(np.float32)
        x[b, :8] = np.sign(x[b, :8]) * np.abs(x[b].astype(np.float64) * s_in).max() / s_in[:8].astype(np.float64) * 0.999      # pairs of large columns
    y, ref = L.forward(x), L.oracle(x)
    assert np.isfinite(y).all() and not np.array_equal(y, exact_forward(L, x))
    for b in range(24):
        assert np.abs(y[b] - ref[b]).max() <= PREFILL_TOL * np.abs(ref[b]).max(), b
    L.close()


def test_scales_on_the_device_choose_the_same_form():
    """Layers created from device memory take columns or pairs as those created from host memory do: same bits."""
    import torch
    d_out, d_in, r, batch = 130, 1500, 90, 20
    x = to_device(synth.gen_x(batch, d_in, 9001, "bf16"), "bf16")
    U, V = synth.gen_sign_words(d_out, r, 9002), synth.gen_sign_words(d_in, r, 9003)
    general = synth.gen_scales(d_in, 9004)
    for exact in (0, 93, 94, d_in):                       # powers of two among 1500 scales: 94 are one in sixteen
        s_in = np.where(general.view(np.uint16) & 0xFF, general, np.float16(0.7)).astype(np.float16)
        s_in[:exact] = np.float16(0.5)
        L = Layer(d_out, d_in, r, "bf16", data=synth.LayerData(synth.LinearShape("t", d_out, d_in, r), U, V,
                                                               synth.gen_scales(d_out, 9005), s_in))
        dev = [torch.from_numpy(np.ascontiguousarray(a).view(np.int32 if a.dtype == np.uint32 else np.int16).copy()).cuda()
               for a in (U, V, L.data.s_out, s_in)]
        h = nq.nq_binlr_create_from_device(d_out, d_in, r, *dev, nq.NQ_BF16, nq.NQ_F32)
        a, b = new_output(batch, d_out), new_output(batch, d_out)
        nq.nq_binlr_forward(L.h, x, a, batch)
        nq.nq_binlr_forward(h, x, b, batch)
        torch.cuda.synchronize()
        assert torch.equal(a, b), exact
        nq.nq_binlr_destroy(h)
        L.close()


@pytest.mark.parametrize("d_in", [32769, 65536])
@pytest.mark.parametrize("scale", [1.0, 3.0])             # columns, pairs
def test_rows_longer_than_the_prescale_holds(d_in, scale):
    """Rows of more than 32768 elements are read twice by the pre-scale: integers, bit for bit."""
    d_out, r, batch = 70, 40, 21
    U, V = synth.gen_sign_words(d_out, r, 9101), synth.gen_sign_words(d_in, r, 9102)
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(synth.LinearShape("t", d_out, d_in, r), U, V,
                                                          np.ones(d_out, dtype=np.float16), np.full(d_in, scale, dtype=np.float16)))
    rng = np.random.default_rng(9103 + d_in)
    x = rng.integers(-1, 2, (batch, d_in)) * (rng.random((batch, d_in)) < 0.03)
    x[:, -1] = 1                                          # the last, partial chunk
    t = int(scale) * x @ signs(V, r)
    assert 2 * np.abs(t).max() <= 2048
    assert np.array_equal(L.forward(x.astype(np.float32)), (t @ signs(U, r).T).astype(np.float32))
    L.close()


def test_large_mean_and_uniform_sign_columns_in_pairs():
    """Activations that share a large offset, with columns of V that are all +1 (every pair a sum) or all -1; constant and negative
    tokens; half of the inputs zero."""
    d_out, d_in, r, batch = 640, 8192, 384, 80
    V = synth.gen_sign_words(d_in, r, 9202)
    V[:, 0] = (V[:, 0] | np.uint32(0x0000FFFF)) & np.uint32(0x0000FFFF)       # columns 0..15 all +1, 16..31 all -1
    L = Layer(d_out, d_in, r, "f32", data=synth.LayerData(synth.LinearShape("m", d_out, d_in, r), synth.gen_sign_words(d_out, r, 9201), V,
                                                          synth.gen_scales(d_out, 9203), np.full(d_in, 3.0, dtype=np.float16)))
    x = (np.abs(np.random.default_rng(9204).standard_normal((batch, d_in))) + 3.0).astype(np.float32)
    x[1] = 2.5
    x[2] = -x[2]
    x[3, ::2] = 0.0
    y, ref = L.forward(x), L.oracle(x)
    assert not np.array_equal(y, exact_forward(L, x))
    for b in range(batch):
        assert np.abs(y[b] - ref[b]).max() <= PREFILL_TOL * np.abs(ref[b]).max(), b
    L.close()
