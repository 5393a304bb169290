"""Workloads whose speed this repository watches: the calls a program that serves or trains a model made of binary
low-rank factorised linear layers  y = s_out (.) (U (V^T (s_in (.) x)))  makes through paper_2602_06694_amd.binding.

Six kinds of work, each with listed sizes and with a range that draw() samples:

  forward   one nq_binlr_forward call on one layer: batch 1..8 is a decode step, 9 and more a prefill or a training forward
  plan      many independent layers at one small batch through nq_plan_forward (the stored model streamed once)
  block     the seven projections of a decoder block as the four plans a decoder runs one after the other
  chain     the layers of a model in dependency order in one nq_exec_forward (one token through the model)
  grads     the backward of one layer with frozen signs: the gradients of both scale vectors and of the input
  lb_admm   iterations of the LB-ADMM factorisation of one weight matrix in binary64

All inputs are synthetic: signs i.i.d. uniform, scales fp16(|N(0,1)| + 0.1), activations N(0,1), optionally with 1 % of the
channels 20 times larger (outlier channels, as measured in Llama-type models).  Layer shapes are those of the Llama-2-7B and
Llama-2-70B blocks at about 0.55 bit per weight (synth.py), a 1024-wide layer, and odd sizes.
"""
import math

import torch

from paper_2602_06694_amd import binding as nq
from paper_2602_06694_amd import synth

_NQ = {"f32": nq.NQ_F32, "f16": nq.NQ_F16, "bf16": nq.NQ_BF16}
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # the smallest call: one 1024 x 1024 layer, one token, fp32 activations; launches and latency count
        {"name": "forward_1024_b1", "kind": "forward", "d_out": 1024, "d_in": 1024, "r": 256, "batch": 1, "x": "f32", "y": "f32",
         "mid": False, "outliers": False},
        # a lone layer of odd sizes at a small batch (a few sequences decoded together, or a draft being verified)
        {"name": "forward_ragged_b6", "kind": "forward", "d_out": 5003, "d_in": 3001, "r": 777, "batch": 6, "x": "f16", "y": "f16",
         "mid": False, "outliers": False},
        # 16 blocks of a 70B-shaped model streamed once, one token per layer: the weight-bandwidth case
        {"name": "plan_70b_b1", "kind": "plan", "block": "70b", "layers": 112, "batch": 1, "x": "bf16", "y": "f32"},
        # 512 attention-sized layers, eight tokens each: batched decode
        {"name": "plan_4096_b8", "kind": "plan", "block": "4096", "layers": 512, "batch": 8, "x": "bf16", "y": "f32"},
        # one 70B-shaped decoder block, four sequences: q, k, v | o | gate, up | down
        {"name": "block_70b_b4", "kind": "block", "block": "70b", "batch": 4, "x": "bf16", "y": "bf16"},
        # one token through all 32 blocks of a 7B-shaped model, every layer reading the one before it
        {"name": "chain_7b", "kind": "chain", "block": "7b", "blocks": 32},
        # a short prompt, or a few dozen sequences decoded together
        {"name": "prefill_4096_b24", "kind": "forward", "d_out": 4096, "d_in": 4096, "r": 1024, "batch": 24, "x": "bf16", "y": "bf16",
         "mid": False, "outliers": False},
        # a prompt of an odd length on an odd layer
        {"name": "prefill_ragged_b333", "kind": "forward", "d_out": 11005, "d_in": 4095, "r": 1663, "batch": 333, "x": "f16", "y": "f16",
         "mid": True, "outliers": False},
        # prompts of 512 and 2048 tokens on the MLP layers of a 70B-shaped model, with outlier channels
        {"name": "prefill_gate_b512", "kind": "forward", "d_out": 28672, "d_in": 8192, "r": 3520, "batch": 512, "x": "bf16", "y": "f32",
         "mid": False, "outliers": True},
        {"name": "prefill_down_b2048", "kind": "forward", "d_out": 8192, "d_in": 28672, "r": 3520, "batch": 2048, "x": "bf16", "y": "bf16",
         "mid": False, "outliers": True},
        # tuning the scale vectors of one layer with the signs frozen: the backward of 64 tokens
        {"name": "grads_4096_b64", "kind": "grads", "d_out": 4096, "d_in": 4096, "r": 1024, "batch": 64, "x": "bf16", "y": "f32"},
        # four iterations of the factorisation of an attention-sized matrix at 0.5 bit per weight
        {"name": "lb_admm_4096", "kind": "lb_admm", "n": 4096, "m": 4096, "r": 1024, "iters": 4, "power": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo=256, hi=28672):
    """A layer side: half of the time a multiple of 128 as model shapes are, else any number."""
    n = _log(rng, lo, hi)
    return max(128, n // 128 * 128) if rng.random() < 0.5 else n


def _rank(rng, d_out, d_in):
    """The rank of a layer stored at 0.3 to 1 bit per weight."""
    bits = rng.uniform(0.3, 1.0)
    r = int(bits * d_out * d_in / (d_out + d_in)) - 16
    r = max(24, min(r, 4096))
    return max(64, r // 32 * 32) if rng.random() < 0.5 else r


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "prefill", "prefill", "plan", "plan", "block", "chain", "grads", "grads", "lb_admm"])
    if kind in ("forward", "prefill"):
        small = kind == "forward"
        batch = rng.randint(1, 8) if small else _log(rng, 9, 2048)
        d_out, d_in = _side(rng), _side(rng)
        return {"kind": "forward", "d_out": d_out, "d_in": d_in, "r": _rank(rng, d_out, d_in), "batch": batch,
                "x": rng.choice(["bf16", "f16", "f32"]), "y": rng.choice(["f32", "bf16", "f16"]), "mid": rng.random() < 0.2,
                "outliers": rng.random() < 0.4}
    if kind == "plan":
        block = rng.choice(["7b", "70b", "4096"])
        most = {"7b": 224, "70b": 112, "4096": 512}[block]
        return {"kind": "plan", "block": block, "layers": _log(rng, 2, most), "batch": rng.randint(1, 8),
                "x": rng.choice(["bf16", "f16", "f32"]), "y": rng.choice(["f32", "bf16"])}
    if kind == "block":
        return {"kind": "block", "block": rng.choice(["7b", "70b"]), "batch": rng.randint(1, 8), "x": rng.choice(["bf16", "f16", "f32"]),
                "y": rng.choice(["f32", "bf16", "f16"])}
    if kind == "chain":
        block = rng.choice(["7b", "70b"])
        return {"kind": "chain", "block": block, "blocks": rng.randint(1, 32 if block == "7b" else 8)}
    if kind == "grads":
        d_out, d_in = _side(rng, 256, 11008), _side(rng, 256, 11008)
        r = _rank(rng, d_out, d_in)
        most = int(max(4, min(512, 64 * 4096 * 8192 * 8 / (r * (d_out + d_in)))))
        return {"kind": "grads", "d_out": d_out, "d_in": d_in, "r": r, "batch": _log(rng, 1, most), "x": rng.choice(["bf16", "f16", "f32"]),
                "y": rng.choice(["f32", "bf16"])}
    n, m = _side(rng, 256, 4096), _side(rng, 256, 4096)
    return {"kind": "lb_admm", "n": n, "m": m, "r": max(32, min(1024, _rank(rng, n, m))), "iters": rng.randint(1, 4), "power": rng.randint(4, 10)}


# ---- shapes ---------------------------------------------------------------------------------------------------------------

def _block_shapes(block):
    if block == "4096":
        return [synth.LinearShape("q", 4096, 4096, 1024)]
    return synth.llama2_7b_block() if block == "7b" else synth.llama2_70b_block()


def _shapes(case):
    kind = case["kind"]
    if kind in ("forward", "grads"):
        return [synth.LinearShape("lin", case["d_out"], case["d_in"], case["r"])]
    block = _block_shapes(case["block"])
    count = {"plan": lambda: case["layers"], "block": lambda: len(block), "chain": lambda: len(block) * case["blocks"]}[kind]()
    return [block[i % len(block)] for i in range(count)]


def _chain_shift(shapes, src):
    """Powers of two taken out of every layer's scales, so that activations stay near one along the chain (in a model the
    normalisation layers do that); (bits off s_in, bits off s_out) per layer."""
    carry, out = [], []
    for i, s in enumerate(shapes):
        at = carry[src[i]] if src[i] >= 0 else 0.0
        gain = math.log2(1.17 * math.sqrt(s.r * s.d_in))
        k = max(0, min(int(round(at + gain)), 18))
        out.append((k // 2, k - k // 2))
        carry.append(at + gain - k)
    return out


# ---- inputs ---------------------------------------------------------------------------------------------------------------

def _words(g, rows, r):
    w = torch.randint(-2**31, 2**31, (rows, (r + 31) // 32), dtype=torch.int32, device="cuda", generator=g)
    if r % 32:
        w[:, -1] &= (1 << (r % 32)) - 1
    return w


def _scales(g, n, shift=0):
    s = (torch.randn(n, device="cuda", generator=g).abs() + 0.1).half()
    return s * 2.0 ** -shift if shift else s


def _acts(g, batch, n, dtype, outliers=False):
    x = torch.randn(batch, n, device="cuda", generator=g)
    if outliers:
        x[:, torch.randperm(n, device="cuda", generator=g)[: n // 100]] *= 20.0
    return x.to(_TORCH[dtype])


def _inputs(case, seed):
    """The tensors of a case, from the seed alone: prepare() hands them to the library, exact() computes with them."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind = case["kind"]
    if kind == "lb_admm":
        n, m, r = case["n"], case["m"], case["r"]
        f64 = dict(dtype=torch.float64, device="cuda", generator=g)
        k = max(1, min(n, m) // 8)
        decay = 1.0 / torch.sqrt(1.0 + torch.arange(k, dtype=torch.float64, device="cuda"))
        low = (torch.randn(n, k, **f64) * decay) @ torch.randn(k, m, **f64)
        w = 0.02 * (0.7 * low / torch.sqrt((decay**2).sum()) + 0.7 * torch.randn(n, m, **f64))
        s = math.sqrt(0.02 / math.sqrt(r))
        return {"W": w, "U0": s * torch.randn(n, r, **f64), "V0": s * torch.randn(m, r, **f64)}
    shapes = _shapes(case)
    shift = [(0, 0)] * len(shapes)
    if kind == "chain":
        shift = _chain_shift(shapes, synth.chain_spec(case["blocks"])[1])
    layers = [{"U": _words(g, s.d_out, s.r), "V": _words(g, s.d_in, s.r), "s_out": _scales(g, s.d_out, ko), "s_in": _scales(g, s.d_in, ki)}
              for s, (ki, ko) in zip(shapes, shift)]
    if case.get("mid"):
        layers[0]["s_mid"] = _scales(g, case["r"])
    if kind == "chain":
        xs = [_acts(g, 1, shapes[0].d_in, "bf16")]
    elif kind == "block":                  # q, k, v read one input, gate and up another
        a, b, c, d = (_acts(g, case["batch"], shapes[i].d_in, case["x"]) for i in (0, 3, 4, 6))
        xs = [a, a, a, b, c, c, d]
    else:
        xs = [_acts(g, case["batch"], s.d_in, case["x"], case.get("outliers", False)) for s in shapes]
    out = {"layers": layers, "xs": xs}
    if kind == "grads":
        out["g"] = _acts(g, case["batch"], case["d_out"], case["y"])
    return out


class _State:
    """Library objects and buffers of one prepared case; the objects are released with it."""

    def __init__(self, case):
        self.case, self.handles, self.plans, self.exec = case, [], [], None

    def layer(self, shape, data, x_dtype, y_dtype):
        h = nq.nq_binlr_create_from_device(shape.d_out, shape.d_in, shape.r, data["U"], data["V"], data["s_out"], data["s_in"], x_dtype,
                                           y_dtype)
        self.handles.append(h)
        if "s_mid" in data:
            nq.nq_binlr_set_mid_scale(h, data["s_mid"].cpu().numpy())
        return h

    def __del__(self):
        try:
            torch.cuda.synchronize()
            if self.exec is not None:
                nq.nq_exec_destroy(self.exec)
            for p in self.plans:
                nq.nq_plan_destroy(p)
            for h in self.handles:
                nq.nq_binlr_destroy(h)
        except Exception:                  # interpreter shutdown
            pass


def _empty(batch, n, dtype):
    return torch.empty(batch, n, dtype=_TORCH[dtype], device="cuda")


def _outputs(shapes, block, batch, dtype):
    """Output buffers: the layers at one position of the block share a tensor [layers, batch, d_out], each writes its part.
    Returns those tensors and the list of the layers' parts."""
    p = len(_block_shapes(block)) if block else 1
    out = [torch.empty(len(shapes[i::p]), batch, shapes[i].d_out, dtype=_TORCH[dtype], device="cuda") for i in range(min(p, len(shapes)))]
    return out, [out[i % p][i // p] for i in range(len(shapes))]


def prepare(case, seed):
    st = _State(case)
    d = _inputs(case, seed)
    kind = case["kind"]
    if kind == "lb_admm":
        n, m, r = case["n"], case["m"], case["r"]
        st.inputs = d
        st.ws_bytes = nq.nq_lb_admm_workspace_bytes(n, m, r)
        st.ws = torch.empty(st.ws_bytes, dtype=torch.uint8, device="cuda")
        st.out = [torch.empty(rows, r, dtype=torch.float64, device="cuda") for rows in (n, m, n, m, n, m)]
        st.rho = _rho(case)
        return st
    shapes = _shapes(case)
    st.xs = d["xs"]
    if kind == "chain":
        level, src = synth.chain_spec(case["blocks"])
        for s, data, j in zip(shapes, d["layers"], src):
            st.layer(s, data, nq.NQ_BF16 if j < 0 else nq.NQ_F32, nq.NQ_F32)
        st.out, st.ys = _outputs(shapes, case["block"], 1, "f32")
        st.exec = nq.nq_exec_create(st.handles, [st.ys[j] if j >= 0 else st.xs[0] for j in src], st.ys, level)
        return st
    for s, data in zip(shapes, d["layers"]):
        st.layer(s, data, _NQ[case["x"]], _NQ[case["y"]])
    st.out, st.ys = _outputs(shapes, case.get("block"), case["batch"], case["y"])
    if kind == "plan":
        st.plans = [nq.nq_plan_create(st.handles, st.xs, st.ys, case["batch"])]
    elif kind == "block":
        for ids in ((0, 1, 2), (3,), (4, 5), (6,)):
            st.plans.append(nq.nq_plan_create([st.handles[i] for i in ids], [st.xs[i] for i in ids], [st.ys[i] for i in ids], case["batch"]))
    else:
        nq.nq_binlr_reserve(st.handles[0], case["batch"])
    if kind == "grads":
        b = case["batch"]
        st.g, st.z = d["g"], _empty(b, case["d_out"], case["y"])
        st.w, st.dx = _empty(b, case["d_in"], "f32"), _empty(b, case["d_in"], "f32")
        st.ds_out, st.ds_in = _empty(1, case["d_out"], "f32")[0], _empty(1, case["d_in"], "f32")[0]
    return st


def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "forward":
        nq.nq_binlr_forward(st.handles[0], st.xs[0], st.ys[0], case["batch"])
        return st.ys[0]
    if kind in ("plan", "block"):
        for p in st.plans:
            nq.nq_plan_forward(p)
        return st.out
    if kind == "chain":
        nq.nq_exec_forward(st.exec)
        return st.out
    if kind == "grads":
        h, b = st.handles[0], case["batch"]
        nq.nq_binlr_forward_unscaled(h, st.xs[0], st.z, b)
        nq.nq_scale_grad(st.g, _NQ[case["y"]], st.z, _NQ[case["y"]], b, case["d_out"], st.ds_out)
        nq.nq_binlr_forward_transposed_unscaled(h, st.g, st.w, b)
        nq.nq_scale_grad(st.xs[0], _NQ[case["x"]], st.w, nq.NQ_F32, b, case["d_in"], st.ds_in)
        nq.nq_binlr_backward_input(h, st.g, st.dx, b)
        return {"z": st.z, "ds_out": st.ds_out, "w": st.w, "ds_in": st.ds_in, "dx": st.dx}
    d = st.inputs
    nq.nq_lb_admm(d["W"], case["n"], case["m"], case["r"], d["U0"], d["V0"], case["iters"], st.rho[0], st.rho[1], 1e-3, case["power"],
                  *st.out, st.ws, st.ws_bytes)
    return dict(zip(("U", "V", "Z_U", "Z_V", "Lambda_U", "Lambda_V"), st.out))


def _rho(case):
    """The first iterations of a 400-step line from 0.4 to 8 times the scale of the Gram matrix' diagonal."""
    diag = max(case["n"], case["m"]) * 0.02 / math.sqrt(case["r"])
    return 0.4 * diag, (0.4 + 7.6 * (case["iters"] - 1) / 399) * diag


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------

def _weight_bytes(s):
    return s.r * (s.d_out + s.d_in) / 8 + 2 * (s.d_out + s.d_in)


def work(case):
    kind = case["kind"]
    if kind == "lb_admm":
        n, m, r = case["n"], case["m"], case["r"]
        flops = 4.0 * n * m * r + 3.0 * r * r * (n + m) + 2.0 * r**3 / 3    # products, Gram matrices and solves, Cholesky
        return {"bytes": 8.0 * (n * m + 4 * r * (n + m)), "flops": flops * case["iters"]}
    shapes = _shapes(case)
    b = case.get("batch", 1)
    bytes_ = sum(_weight_bytes(s) for s in shapes)
    flops = sum(2.0 * b * s.r * (s.d_out + s.d_in) for s in shapes)
    if kind == "chain":
        return {"bytes": bytes_ + 2 * shapes[0].d_in + sum(4 * s.d_out for s in shapes), "flops": flops}
    n_x = sum(s.d_in for s in shapes)
    if kind == "block":
        n_x = sum(shapes[i].d_in for i in (0, 3, 4, 6))
    bytes_ += b * (_SIZE[case["x"]] * n_x + _SIZE[case["y"]] * sum(s.d_out for s in shapes))
    if case.get("mid"):
        bytes_ += 2 * case["r"]
    if kind == "grads":                    # in: weights, x, g; out: z, w, dx and the two gradients
        s = shapes[0]
        bytes_ += b * (_SIZE[case["y"]] * s.d_out + 8 * s.d_in) + 4 * (s.d_out + s.d_in)
        flops *= 2
    return {"bytes": float(bytes_), "flops": float(flops)}


def tolerance(case):
    """About four times the error against exact() that was measured over the ranges of draw(): 32-bit outputs of the calls
    whose activations are 24-bit fixed point 0.6 to 4e-6, of the fp16-operand path (batch 9 and more) 3e-4; outputs rounded to
    fp16 2.1 to 3.6e-4, to bf16 1.7e-3; LB-ADMM in binary64 1e-14, a rounding of which travels through the iterations."""
    kind = case["kind"]
    if kind == "lb_admm":
        return {"rel": 1e-12, "max": 1e-10}
    if kind == "chain":                    # every layer reads the rounding of those before it
        return {"rel": 4e-5, "max": 4e-4}
    y = case["y"]
    dense = kind == "forward" and case["batch"] > 8
    if y == "f32":
        return {"rel": 1.2e-3, "max": 1.2e-2} if dense else {"rel": 1.5e-5, "max": 1.5e-4}
    if y == "f16":
        return {"rel": 1.5e-3, "max": 1.2e-2} if dense else {"rel": 8e-4, "max": 4e-3}
    return {"rel": 7e-3, "max": 3e-2}


# ---- the same results in binary64, by plain torch -------------------------------------------------------------------------

def _signs(words, r):
    """+-1 as binary64 [rows, r] from packed words (bit k % 32 of word k / 32, 1 -> +1)."""
    bits = (words.unsqueeze(-1) >> torch.arange(32, dtype=torch.int32, device=words.device)) & 1
    return bits.reshape(words.shape[0], -1)[:, :r].double() * 2.0 - 1.0


def _factored(layer, r, x, in_scale, first, second, mid, out_scale):
    """out_scale (.) (A (mid (.) (B^T (in_scale (.) x)))) for A = second, B = first, in binary64."""
    v = x.double() * layer[in_scale].double() if in_scale else x.double()
    t = v @ _signs(layer[first], r)
    if mid and "s_mid" in layer:
        t = t * layer["s_mid"].double()
    z = t @ _signs(layer[second], r).T
    return z * layer[out_scale].double() if out_scale else z


def _svid(p, rounds):
    a_abs = p.abs()
    sign = torch.where(p >= 0, 1.0, -1.0)
    a = torch.ones(p.shape[0], dtype=torch.float64, device=p.device) / math.sqrt(p.shape[0])
    b = None
    if rounds == 0:
        return sign * a_abs.mean()
    for _ in range(rounds):
        b = a_abs.T @ a
        b = b / b.norm()
        a = a_abs @ b
        sigma = a.norm()
        a = a / sigma
    return sign * (sigma * torch.outer(a, b))


def _lb_admm(case, seed):
    d = _inputs(case, seed)
    w, u, v = d["W"], d["U0"], d["V0"]
    r, iters, rounds = case["r"], case["iters"], case["power"]
    rho0, rho1 = _rho(case)
    z_u, z_v = _svid(u, rounds), _svid(v, rounds)
    l_u, l_v = torch.zeros_like(u), torch.zeros_like(v)
    eye = torch.eye(r, dtype=torch.float64, device="cuda")

    def update(w, v, z, l, rho):
        h = v.T @ v + (rho + 1e-3) * eye
        f = torch.cholesky_solve((w @ v + rho * (z - l)).T.contiguous(), torch.linalg.cholesky(h)).T.contiguous()
        z = _svid(f + l, rounds)
        return f, z, l + f - z

    for k in range(iters):
        rho = rho0 if iters == 1 else rho0 + (rho1 - rho0) * k / (iters - 1)
        u, z_u, l_u = update(w, v, z_u, l_u, rho)
        v, z_v, l_v = update(w.T, u, z_v, l_v, rho)
    return {"U": u, "V": v, "Z_U": z_u, "Z_V": z_v, "Lambda_U": l_u, "Lambda_V": l_v}


def exact(case, seed):
    kind = case["kind"]
    if kind == "lb_admm":
        return _lb_admm(case, seed)
    shapes, d = _shapes(case), _inputs(case, seed)
    layers, xs = d["layers"], d["xs"]
    fwd = lambda i, x, scaled=True: _factored(layers[i], shapes[i].r, x, "s_in", "V", "U", True, "s_out" if scaled else None)
    if kind == "forward":
        return fwd(0, xs[0])
    if kind in ("plan", "block", "chain"):
        src = synth.chain_spec(case["blocks"])[1] if kind == "chain" else None
        ys = []
        for i in range(len(shapes)):
            ys.append(fwd(i, xs[i] if src is None else xs[0] if src[i] < 0 else ys[src[i]]))
        p = len(_block_shapes(case["block"]))
        return [torch.stack(ys[i::p]) for i in range(min(p, len(ys)))]
    z = fwd(0, xs[0], False)
    w = _factored(layers[0], case["r"], d["g"], "s_out", "U", "V", True, None)
    return {"z": z, "ds_out": (d["g"].double() * z).sum(0), "w": w,
            "ds_in": (xs[0].double() * w).sum(0), "dx": w * layers[0]["s_in"].double()}
