"""The one-launch kernel of small layers at the edges of its rule and of its parts: one to four row blocks of t, one to five tokens and one more than the kernel has columns for, ranks around whole row blocks and
quads, short shares of the reduction, one to eight bit planes in the second stage, and NaN and zeros passing through t.  Output and t against the launches
that quantise separately, bit for bit (the same roundings in the same places: nothing to tolerate), and y against the oracle."""
import numpy as np
import pytest

from paper_2602_06694_amd import synth
from gpu_util import Layer, rel_err
from test_gpu_lone_layers import both

pytestmark = pytest.mark.gpu
TOL = 1e-5          # of the largest output: two fixed-point steps of at least 21 bits and three roundings to fp32, as for all streaming paths


@pytest.mark.parametrize("shape,x_dtype", [
    ((130, 4096, 128), "f32"), ((520, 4097, 100), "bf16"), ((300, 2048, 129), "f16"), ((300, 2049, 256), "bf16"),      # 64 tiles and past them, one row block and two
    ((700, 1024, 384), "f16"), ((700, 768, 512), "f32"), ((700, 770, 513), "bf16"),                                    # 48 tiles of three and four, five row blocks
    ((4100, 250, 255), "f32"), ((8300, 64, 33), "f16"), ((16500, 3, 1), "bf16"), ((32700, 130, 257), "f16"),           # 1, 2, 4 and 8 planes of stage 2
    ((64, 256, 128), "f32"), ((4100, 257, 128), "bf16"), ((8300, 1, 127), "f16"), ((32700, 255, 3), "bf16"),           # five tokens: four tiles, past them, 2 to 8 planes
])
def test_one_launch_equals_two_stages(nqopt, shape, x_dtype):
    L = Layer(*shape, x_dtype, seed=12500 + shape[1])
    for scaled in (False, True):
        if scaled:
            from paper_2602_06694_amd import binding as nq
            nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(shape[2], 12501))
        for batch in (1, 2, 3, 4, 5, 6):
            x = synth.gen_x(batch, shape[1], 12510 + batch, x_dtype)
            (y, t), (y4, t4) = both(L, nqopt, x)
            assert np.array_equal(t, t4) and np.array_equal(y, y4), (shape, batch, scaled)
            if not scaled:
                assert rel_err(y, L.oracle(x)) <= TOL, (shape, batch)
    L.close()


def test_one_token_of_nan_or_zeros_leaves_the_others(nqopt):
    L = Layer(1000, 300, 120, "f32", seed=12600)
    for value in (0.0, np.nan, np.inf):
        x = synth.gen_x(3, 300, 12601, "f32")
        x[1] = value
        (y, t), (y4, t4) = both(L, nqopt, x)
        assert np.array_equal(y, y4, equal_nan=True) and np.array_equal(t, t4, equal_nan=True)
        assert np.isfinite(y[[0, 2]]).all() and (np.isfinite(y[1]).all() if value == 0.0 else np.isnan(y[1]).all())
    L.close()
