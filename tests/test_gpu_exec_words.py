"""The executor's hand-over by words in two copies that launches take in turn: non-finite values, launches that gave up, inputs that end inside
a lane's group of four, row blocks dealt out by one, two, four and eight bit planes and not at all."""
import numpy as np
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer
from test_gpu_exec import SMALL, Chain

pytestmark = pytest.mark.gpu


def same(c, ref):
    import torch
    for i, (a, b) in enumerate(zip(c.ys, ref)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.nan_to_num(a), torch.nan_to_num(b)), i


def launch(c, e):
    for y in c.ys:
        y.fill_(float("nan"))
    nq.nq_exec_forward(e)
    nq.nq_exec_status(e)


def test_values_that_are_not_finite_are_handed_over():
    """A NaN whose bits are all ones in x, infinities and ordinary inputs in turn: every launch ends and says what single calls say."""
    import torch
    c = Chain(SMALL, 2, seed=13000, first_x="f32")
    e = c.executor()
    for rep, bits in enumerate([None, 0xFFFFFFFF, None, 0x7F800000, 0xFF800000, 0x7FC00000, None]):
        c.set_input(13010 + rep)
        if bits is not None:
            c.x0.view(torch.int32)[0, 5] = int(np.uint32(bits).view(np.int32))
        ref = c.run_as_single_calls()
        launch(c, e)
        same(c, ref)
    nq.nq_exec_destroy(e)
    c.close()


def test_launches_after_some_that_gave_up(nqopt):
    """Launches with a limit of zero leave words of both copies unwritten; whichever copy comes next, no old value is taken for a new one."""
    c = Chain(SMALL, 2, seed=13100)
    e = c.executor()
    for rep, given_up in enumerate([0, 1, 0, 2, 0, 0, 3, 0]):
        for _ in range(given_up):
            nqopt.set("exec_spin_limit_us", 0)
            nq.nq_exec_forward(e)
            with pytest.raises(nq.NQError) as err:
                nq.nq_exec_status(e)
            assert err.value.status == nq.NQ_E_TIMEOUT
            nqopt.unset("exec_spin_limit_us")
        c.set_input(13110 + rep)
        ref = c.run_as_single_calls()
        launch(c, e)
        same(c, ref)
    nq.nq_exec_destroy(e)
    c.close()


# row blocks of a level's stages: 16 (8 planes apart), 17 to 32 (four workgroups each), 33 to 64 (two), 65 to 256 (whole), above (none of its own); lengths
# of every remainder by four, and past 2048 and 16384, where the input is waited for and scaled differently
@pytest.mark.parametrize("shapes", [
    [(2049, 513, 130)] * 3 + [(2050, 2049, 2047), (4097, 2050, 99), (4097, 2050, 99), (513, 4097, 1026)],
    [(5123, 70, 300)] * 3 + [(9001, 5123, 259), (16901, 9001, 2051), (16901, 9001, 2051), (70, 16901, 18)],
    [(32702, 259, 140)] * 3 + [(130, 32702, 64), (300, 130, 64), (300, 130, 64), (259, 300, 64)],
])
def test_row_blocks_dealt_out(shapes):
    c = Chain(shapes, 2, seed=13200)
    e = c.executor()
    for rep in range(3):
        c.set_input(13210 + rep)
        ref = c.run_as_single_calls()
        launch(c, e)
        same(c, ref)
    nq.nq_exec_destroy(e)
    c.close()


@pytest.mark.parametrize("scale", [np.inf, -np.inf, np.nan])
def test_a_scale_that_is_not_finite_stays_in_its_own_layer(scale):
    """Layers whose inputs end inside a step, read from outside and handed over, run by the workgroups that ran a layer with a scale that
    is not finite further up its own, longer input: a lane past the end of an input has no scale, whatever the task before left in it."""
    import torch
    # level 0 has the scale; every later level one layer that reads x and one that reads the level before
    shapes = [(1024, 512, 1024, -1)]
    for k in range(1, 9):
        shapes += [(257 + k, 250 + 5 * k, 1024, -1), (300, 257 + k - 1 if k > 1 else 250, 1024, 2 * k - 3 if k > 1 else -1)]
    layers, xs, ys, level = [], [], [], []
    for i, (d_out, d_in, r, src) in enumerate(shapes):
        lin = synth.LinearShape("t", d_out, d_in, r)
        s_in = synth.gen_scales(d_in, 13300 + i)
        if i == 0:
            s_in[500] = np.float16(scale)
        data = synth.LayerData(lin, synth.gen_sign_words(d_out, r, 13320 + i), synth.gen_sign_words(d_in, r, 13340 + i), synth.gen_scales(d_out, 13360 + i), s_in)
        layers.append(Layer(d_out, d_in, r, "f32", data=data))
        xs.append(torch.from_numpy(synth.gen_x(1, d_in, 13380 + i, "f32")).cuda() if src < 0 else ys[src])
        ys.append(torch.full((1, d_out), float("nan"), device="cuda"))
        level.append((i + 1) // 2)
    for L, x, y in zip(layers, xs, ys):
        nq.nq_binlr_forward(L.h, x, y, 1)
    torch.cuda.synchronize()
    ref = [y.clone() for y in ys]
    assert torch.isnan(ref[0]).all() and not any(torch.isnan(y).any() for y in ref[1:])
    e = nq.nq_exec_create([L.h for L in layers], xs, ys, level)
    for _ in range(3):
        for y in ys:
            y.fill_(7.0)
        nq.nq_exec_forward(e)
        nq.nq_exec_status(e)
        wrong = [shapes[i] for i, (a, b) in enumerate(zip(ys, ref)) if i and not torch.equal(a, b)]
        assert not wrong and torch.isnan(ys[0]).all(), wrong
    nq.nq_exec_destroy(e)
    for L in layers:
        L.close()


@pytest.mark.parametrize("shapes", [SMALL, [(5123, 70, 300)] * 3 + [(9001, 5123, 259), (16901, 9001, 2051), (16901, 9001, 2051), (70, 16901, 18)]])
def test_the_planner_lists_what_the_executor_runs(shapes):
    c = Chain(shapes, 2, seed=13400)
    e = c.executor()
    n_wg, n_tasks, _ = nq.nq_exec_info(e)
    lists = nq.nq_exec_plan_lists([L.d_out for L in c.layers], [L.d_in for L in c.layers], [L.r for L in c.layers], c.level, n_wg)
    assert len(lists) == n_tasks and (lists[:, 8] > 0).any()
    nq.nq_exec_destroy(e)
    c.close()
