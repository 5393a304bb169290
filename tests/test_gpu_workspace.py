"""The workspace of calls with more than eight tokens: what reservations and forwards of growing sizes hold, that a workspace that is
large enough stays where it is, and that graphs captured before it grew stay valid."""
import pytest

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth
from gpu_util import Layer, new_output, to_device

pytestmark = pytest.mark.gpu

SLACK = 4 << 20         # granularity of device allocations


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_a_workspace_that_is_large_enough_is_left_alone():
    d_out, d_in, r = 2048, 4096, 1024
    L = Layer(d_out, d_in, r, "bf16", seed=9100)
    x, y = to_device(synth.gen_x(2048, d_in, 9101, "bf16"), "bf16"), new_output(2048, d_out)
    nq.nq_binlr_forward(L.h, x, y, 2048)                  # nothing reserved: grows on its own
    bytes0, free0 = nq.nq_binlr_reserved(L.h)[1], free_bytes()
    for batch in (9, 64, 512, 512):
        nq.nq_binlr_reserve(L.h, batch)
        assert nq.nq_binlr_reserved(L.h) == (batch, bytes0)
        assert free_bytes() == free0, batch
    L.close()


@pytest.mark.parametrize("steps", [(("reserve", 512), ("reserve", 2048)), (("reserve", 64), ("forward", 1500), ("reserve", 700)),
                                   (("forward", 100), ("reserve", 300), ("forward", 2048))])
def test_nothing_is_held_beside_the_reported_bytes(steps):
    import torch
    d_out, d_in, r = 28672, 8192, 3520
    L = Layer(d_out, d_in, r, "bf16", seed=9200)
    x, y = to_device(synth.gen_x(2048, d_in, 9201, "bf16"), "bf16"), new_output(2048, d_out)
    z0, z1 = new_output(20, d_out), new_output(20, d_out)
    nq.nq_binlr_forward_exact(L.h, x, z0, 20)             # passes of eight, in the layer's small workspace
    assert not torch.equal(z0, z1)                        # (the comparison allocates too, once; so do kernels that need scratch)
    W = Layer(d_out, d_in, r, "bf16", data=L.data)
    for batch in (100, 1500, 2048):
        nq.nq_binlr_forward(W.h, x, y, batch)
    nq.nq_binlr_forward_exact(W.h, x, y, 2048)
    torch.cuda.synchronize()
    W.close()
    free0 = free_bytes()
    for what, batch in steps:
        if what == "reserve":
            nq.nq_binlr_reserve(L.h, batch)
        else:
            nq.nq_binlr_forward(L.h, x, y, batch)
        bytes_ = nq.nq_binlr_reserved(L.h)[1]
        assert free0 - free_bytes() <= bytes_ + SLACK, (what, batch)
        nq.nq_binlr_forward_exact(L.h, x, z1, 20)
        torch.cuda.synchronize()
        assert torch.equal(z0, z1)
        z1.fill_(float("nan"))
    nq.nq_binlr_destroy(L.h)
    L.h = None
    assert free_bytes() >= free0 - SLACK


def test_reservations_without_the_dense_path():
    L = Layer(4096, 4096, 1024, "bf16", seed=9300, flags=nq.NQ_FLAG_NO_PREFILL)
    free0 = free_bytes()
    assert nq.nq_binlr_reserved(L.h) == (8, 0)
    nq.nq_binlr_reserve(L.h, 2048)                        # passes of up to about 8 MiB
    batch, bytes_ = nq.nq_binlr_reserved(L.h)
    assert batch == 8 and 0 < bytes_ <= 9 << 20 and free0 - free_bytes() <= bytes_ + SLACK
    L.close()


@pytest.mark.parametrize("path", ["dense", "exact", "forward"])
def test_graphs_captured_before_the_workspace_grew(nqopt, path):
    import torch
    if path == "dense":
        nqopt.set("dense_only", 1)
    d_out, d_in, r, batch = 600, 1000, 300, 40
    L = Layer(d_out, d_in, r, "bf16", seed=9400)
    call = nq.nq_binlr_forward_exact if path == "exact" else nq.nq_binlr_forward
    x, y, eager = to_device(synth.gen_x(batch, d_in, 9401, "bf16"), "bf16"), new_output(batch, d_out), new_output(batch, d_out)
    big_x, big_y = to_device(synth.gen_x(2048, d_in, 9402, "bf16"), "bf16"), new_output(2048, d_out)
    nq.nq_binlr_reserve(L.h, batch)
    call(L.h, x, y, batch)                                # warm up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(L.h, x, y, batch)
    nq.nq_binlr_forward(L.h, big_x, big_y, 2048)          # the workspace grows
    others = [torch.full((1 << 20,), 3.0, device="cuda") for _ in range(8)]
    for rep in range(4):
        x.copy_(to_device(synth.gen_x(batch, d_in, 9410 + rep, "bf16"), "bf16"))
        call(L.h, x, eager, batch)
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, eager), rep
    assert all(bool((o == 3.0).all()) for o in others)    # nobody else's memory was written
    if path == "dense":
        nq.nq_binlr_forward_exact(L.h, x, eager, batch)
        torch.cuda.synchronize()
        assert not torch.equal(y, eager)
    del graph
    L.close()


def test_the_transposed_products_workspace_follows_the_largest_batch():
    """A first call with one token must not leave a layer in passes of 64: after a call with 512 it holds what a first call with
    512 leaves."""
    import torch
    d = 4096
    w = torch.empty((512, d), dtype=torch.float32, device="cuda")
    g = torch.randn((512, d), device="cuda")
    warm = Layer(d, d, 1024, "f32", seed=9500)
    for batch in (1, 512):
        nq.nq_binlr_backward_input(warm.h, g, w, batch)
    held = []
    for batches in ((512,), (1, 512), (512, 1, 64)):
        L = Layer(d, d, 1024, "f32", data=warm.data)
        free0 = free_bytes()
        for batch in batches:
            nq.nq_binlr_backward_input(L.h, g, w, batch)
        held.append(free0 - free_bytes())
        L.close()
    assert held[0] == held[1] == held[2] and held[0] <= (11 << 20) + SLACK
    warm.close()


def test_transposed_graphs_captured_before_the_workspace_grew():
    """Captured with more tokens than the workspace has room for (several passes), replayed after it has grown."""
    import torch
    d_out, d_in, r, batch = 600, 500, 300, 150
    L = Layer(d_out, d_in, r, "f32", seed=9600)
    g = torch.randn((batch, d_out), device="cuda")
    w, eager = (torch.empty((batch, d_in), dtype=torch.float32, device="cuda") for _ in range(2))
    nq.nq_binlr_backward_input(L.h, g, w, 1)              # a workspace of 64 tokens
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nq.nq_binlr_backward_input(L.h, g, w, batch)
    for rep in range(4):
        g.copy_(torch.randn((batch, d_out), device="cuda"))
        nq.nq_binlr_backward_input(L.h, g, eager, batch)  # (the first one grows it)
        w.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(w, eager), rep
    del graph
    L.close()


FEWER = [((1038, 129, 93), 373, 178), ((1202, 245, 109), 257, 234), ((2623, 351, 86), 249, 156),      # the dense path's call, then fewer tokens on the exact one
         ((1313, 8385, 886), 361, 327), ((13969, 8296, 3202), 164, 138)]                               # both dense, the smaller one with more parts of its reduction


@pytest.mark.parametrize("shape,tokens,fewer", FEWER)
def test_a_forward_leaves_room_for_every_smaller_one(shape, tokens, fewer):
    L = Layer(*shape, "bf16", seed=9700)
    x, y = to_device(synth.gen_x(tokens, shape[1], 9701, "bf16"), "bf16"), new_output(tokens, shape[0])
    nq.nq_binlr_forward(L.h, x, y, tokens)                # nothing reserved
    held = nq.nq_binlr_reserved(L.h)[1]
    for batch in (fewer, 9, 16, 33, tokens // 2, tokens - 1):
        nq.nq_binlr_forward(L.h, x, y, batch)
        assert nq.nq_binlr_reserved(L.h)[1] == held, batch
    L.close()


@pytest.mark.parametrize("shape,tokens,fewer", FEWER)
def test_a_smaller_forward_can_be_captured_without_a_reservation(shape, tokens, fewer):
    import torch
    L = Layer(*shape, "bf16", seed=9700)
    x, y, eager = to_device(synth.gen_x(tokens, shape[1], 9702, "bf16"), "bf16"), new_output(tokens, shape[0]), new_output(tokens, shape[0])
    nq.nq_binlr_forward(L.h, x, y, tokens)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        nq.nq_binlr_forward(L.h, x, y, fewer)
    for rep in range(3):
        x.copy_(to_device(synth.gen_x(tokens, shape[1], 9710 + rep, "bf16"), "bf16"))
        nq.nq_binlr_forward(L.h, x, eager, fewer)
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y[:fewer], eager[:fewer]), rep
    del graph
    L.close()
