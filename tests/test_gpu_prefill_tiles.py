"""The dense path where a last tile of 64 tokens holds 32 or fewer, and 32-token tiles with their reduction in parts: every token against the oracle, and a
reservation that covers every such number of tokens."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, rel_err, to_device

pytestmark = pytest.mark.gpu
TOL = 7e-4          # of the largest output: fp16 operands of both products, 2^-11 each, as for all of the dense path


@pytest.mark.parametrize("batch", [9, 31, 32, 33, 63, 64, 65, 96, 97, 160])
@pytest.mark.parametrize("tg,splits", [(0, 0), (2, 1), (2, 2), (2, 5), (4, 3)])
def test_tokens_around_half_tiles(nqopt, batch, tg, splits):
    L = Layer(700, 900, 330, "f16", seed=13000)
    nqopt.set("dense_only", 1)
    if tg:
        for k in ("1", "2"):
            nqopt.set("pf_tg" + k, tg)
            nqopt.set("pf_splits" + k, splits)
    nq.nq_binlr_set_mid_scale(L.h, synth.gen_scales(330, 13001))
    x = synth.gen_x(batch, 900, 13002 + batch, "f16")
    y = new_output(batch + 1, 700)                           # a row past the last token stays as it is
    nq.nq_binlr_forward(L.h, to_device(x, "f16"), y, batch)
    got = y.cpu().numpy()
    assert np.isnan(got[batch]).all() and np.isfinite(got[:batch]).all()
    plain = L.forward(x)                                     # the same call once more, whatever the workspace held
    assert np.array_equal(plain, got[:batch])
    nqopt.unset("dense_only")
    exact = new_output(batch, 700)
    nq.nq_binlr_reserve(L.h, batch)
    nq.nq_binlr_forward_exact(L.h, to_device(x, "f16"), exact, batch)
    assert rel_err(got[:batch], exact.cpu().numpy()) <= TOL
    L.close()


@pytest.mark.parametrize("shape,batch,tiles", [((2796, 166, 78), 196, (8, 8)), ((2796, 166, 78), 193, (8, 8)), ((2796, 166, 78), 224, (8, 8)), ((2796, 166, 78), 192, (6, 6)),
                                               ((2722, 431, 207), 461, (16, 16)), ((17245, 497, 94), 458, (16, 15))])
def test_short_launches_take_whole_eights_of_tiles(nqopt, capfd, shape, batch, tiles):
    """Seven, 15, .. tiles of 32 tokens that leave every workgroup its CU are launched as eight, 16, ..: the last holds no token, and nothing of it is stored."""
    L = Layer(*shape, "bf16", seed=13400 + batch)
    nqopt.set("dense_only", 1)
    nq.nq_binlr_reserve(L.h, batch)
    nqopt.set("pf_verbose", 1)
    capfd.readouterr()
    x = synth.gen_x(batch, shape[1], 13401, "bf16")
    y = new_output(batch + 1, shape[0])
    nq.nq_binlr_forward(L.h, to_device(x, "bf16"), y, batch)
    got = y.cpu().numpy()
    line = [l for l in capfd.readouterr().err.splitlines() if "prefill tiling B=%d:" % batch in l][-1]
    assert np.isnan(got[batch]).all() and rel_err(got[:batch], L.oracle(x)) <= TOL
    assert tuple(int(w[6:]) for w in line.replace(",", "").split() if w.startswith("tiles=")) == tiles, line
    L.close()


def test_a_reservation_covers_every_number_of_tiles(nqopt):
    nqopt.set("dense_only", 1)
    L = Layer(640, 2300, 300, "bf16", seed=13100)
    nq.nq_binlr_reserve(L.h, 700)
    _, size = nq.nq_binlr_reserved(L.h)
    for batch in (9, 20, 33, 64, 65, 90, 97, 130, 222, 289, 333, 410, 513, 577, 640, 641, 700):
        x = to_device(synth.gen_x(batch, 2300, 13200 + batch, "bf16"), "bf16")
        nq.nq_binlr_forward(L.h, x, new_output(batch, 640), batch)
        assert nq.nq_binlr_reserved(L.h)[1] == size, batch
    L.close()


@pytest.mark.parametrize("shape,batch", [((548, 3214, 192), 207), ((2011, 9600, 997), 149), ((1408, 10245, 1152), 183), ((1330, 5535, 448), 223)])
def test_calls_on_the_exact_path_stay_there(nqopt, shape, batch):
    """Calls just inside the line between the two paths, where 32-token tiles in parts bring the dense path's time below the estimate that the line was fitted to."""
    L = Layer(*shape, "f16", seed=13300 + shape[0])
    nq.nq_binlr_reserve(L.h, batch)
    x = to_device(synth.gen_x(batch, shape[1], 13301, "f16"), "f16")
    y, exact = new_output(batch, shape[0]), new_output(batch, shape[0])
    nq.nq_binlr_forward(L.h, x, y, batch)
    nq.nq_binlr_forward_exact(L.h, x, exact, batch)
    assert np.array_equal(y.cpu().numpy(), exact.cpu().numpy())
    L.close()
