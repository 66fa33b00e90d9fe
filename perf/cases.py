"""Timed cases of the framework: what its users have it do, over the range they do it in.

A case is a dict of plain values:
  op       "forward" (one layer), "stack" (several residual layers), "backward" (the hard-routed
           gradients from a forward's records) or "train" (a forward with records, then its backward)
  tokens, hidden, depth, trees      the layer's shape (depth counts edges: 2^(depth+1) - 1 nodes)
  x, w, y  "bf16" or "f32": activations in, weights, activations out (gradients dy and dx as y)
  residual, norm                    y = x + FFF(u), with u = x or its LayerNorm
  layers                            layers of a stack (1 otherwise)
  skew                              tokens gathered around a few centres (uneven routing)

Inputs are seeded Gaussians, x ~ N(0, 1) and W ~ N(0, 1/hidden), drawn on the GPU.  A logit that
rounding alone can push to the other side of zero sends its token down another path, where every
correct implementation gives another row; such tokens (a few in ten thousand) are drawn again.
"""
from __future__ import annotations

import math

import torch

import paper_2311_10770_amd as fff

DT = {"f32": torch.float32, "bf16": torch.bfloat16}
EPS = 1e-12  # the LayerNorm's, BERT's value


def _case(op, tokens, hidden, depth, trees, x, w, y, residual=False, norm=False, layers=1, skew=False):
    return {"op": op, "tokens": tokens, "hidden": hidden, "depth": depth, "trees": trees, "x": x, "w": w, "y": y,
            "residual": residual, "norm": norm, "layers": layers, "skew": skew}


def listed():
    cases = {
        # one token through the UltraFastBERT-1x11 layer: a serving step, where latency is everything
        "token_1x11_bf16": _case("forward", 1, 768, 11, 1, "bf16", "bf16", "bf16"),
        # one sequence of 128 tokens through a pre-norm block, y = x + FFF(LN(x))
        "sequence_block_bf16": _case("forward", 128, 768, 11, 1, "bf16", "bf16", "bf16", residual=True, norm=True),
        # a decode batch at LLM width: depth 15 at hidden 4096, where the rows come from HBM
        "decode_4096x15_bf16": _case("forward", 64, 4096, 15, 1, "bf16", "bf16", "bf16"),
        # the paper's speed test: 128 sequences of 128 tokens, hidden 768, single precision
        "speedtest_1x11_f32": _case("forward", 16384, 768, 11, 1, "f32", "f32", "f32"),
        # the throughput workload: a large bf16 batch through the 1x11 layer
        "throughput_1x11_bf16": _case("forward", 65536, 768, 11, 1, "bf16", "bf16", "bf16"),
        # a block of BERT-large's width with fp32 activations and bf16 weights, a ragged batch
        "block_1024_mixed": _case("forward", 30011, 1024, 10, 1, "f32", "bf16", "f32", residual=True, norm=True),
        # a wide shallow member of the KxD family, where a token uses a quarter of the nodes
        "shallow_256x3_bf16": _case("forward", 16384, 768, 3, 256, "bf16", "bf16", "bf16"),
        # a width without its own kernels (512), a ragged batch
        "width_512_bf16": _case("forward", 9001, 512, 10, 1, "bf16", "bf16", "bf16"),
        # the feedforward half of a whole model: twelve UltraFastBERT-4x9 blocks in single precision
        "model_12x4x9_f32": _case("stack", 16384, 768, 9, 4, "f32", "f32", "f32", residual=True, norm=True, layers=12),
        # the gradients of the 1x11 layer at the throughput batch
        "backward_1x11_bf16": _case("backward", 65536, 768, 11, 1, "bf16", "bf16", "bf16"),
        # a training step of a 4x9 layer at the speed test's batch: forward with records, then backward
        "train_4x9_f32": _case("train", 16384, 768, 9, 4, "f32", "f32", "f32"),
        # a training step of a small layer of an odd width
        "train_odd_300_f32": _case("train", 2003, 300, 6, 3, "f32", "f32", "f32"),
    }
    return [dict(name=n, **c) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# layer forms (trees, depth) of the walk, and the family's wide shallow ones
DEEP = [(1, d) for d in range(5, 14)] * 2 + [(2, 8), (2, 10), (2, 11), (4, 7), (4, 8), (4, 9), (8, 6), (8, 8)]
SHALLOW = [(3072, 0), (1536, 1), (512, 2), (256, 3), (128, 4), (64, 5), (32, 4), (32, 6), (16, 5), (16, 7)]
TYPES = [("bf16", "bf16", "bf16")] * 3 + [("f32", "f32", "f32")] * 2 + [("f32", "bf16", "f32"), ("bf16", "bf16", "f32")]


def _fit(c, flops):
    """Fewer tokens where the case would do more than `flops`."""
    per = work(dict(c, tokens=1))["flops"]
    c["tokens"] = max(1, min(c["tokens"], int(flops // per)))
    return c


def draw(rng):
    """A case of the ranges the listed ones stand for."""
    op = rng.choice(["serve", "layer", "layer", "layer", "shallow", "width", "stack", "backward", "train"])
    x, w, y = rng.choice(TYPES)
    if op == "serve":  # token, sequence, decode: 1 to 256 tokens
        hidden = rng.choice([768, 768, 1024, 4096])
        trees, depth = rng.choice([(1, d) for d in range(5, 16)] + [(2, 9), (4, 9), (4, 8)])
        block = rng.random() < 0.3
        return _case("forward", _log_int(rng, 1, 256), hidden, depth, trees, x, w, y, block, block)
    if op == "layer":  # speed test, throughput, blocks: up to 65536 tokens
        trees, depth = rng.choice(DEEP)
        block = rng.random()
        c = _case("forward", _log_int(rng, 257, 65536), rng.choice([768, 768, 1024]), depth, trees, x, w, y,
                  block < 0.4, block < 0.25, skew=rng.random() < 0.25)
        return _fit(c, 8e9)
    if op == "shallow":
        trees, depth = rng.choice(SHALLOW)
        x, w, y = rng.choice([("bf16", "bf16", "bf16"), ("bf16", "bf16", "bf16"), ("f32", "f32", "f32")])
        c = _case("forward", _log_int(rng, 64, 16384), 768, depth, trees, x, w, y)
        return _fit(c, 50e9 if w == "bf16" else 12e9)
    if op == "width":  # any hidden size
        hidden = rng.choice([128 * rng.randint(1, 16), 128 * rng.randint(1, 16), 8 * rng.randint(4, 200),
                             4 * rng.randint(8, 400), rng.randint(33, 1500)])
        c = _case("forward", _log_int(rng, 1, 16384), hidden, rng.randint(2, 11), rng.randint(1, 3), x, w, y,
                  rng.random() < 0.3)
        return _fit(c, 2e9)
    if op == "stack":
        trees, depth = rng.choice([(1, 11), (1, 9), (2, 10), (4, 8), (4, 9)])
        c = _case("stack", _log_int(rng, 128, 16384), 768, depth, trees, "f32", rng.choice(["f32", "bf16"]), "f32",
                  True, rng.random() < 0.7, rng.randint(2, 12))
        return _fit(c, 20e9)
    # gradients and training steps
    if rng.random() < 0.3:
        hidden, forms = 4 * rng.randint(16, 256), [(1, 5), (1, 8), (2, 6), (3, 4)]
        top = 8192
    else:
        hidden, forms = rng.choice([768, 768, 1024]), [(1, d) for d in range(6, 14)] + [(2, 9), (4, 8), (4, 9)]
        top = 65536
    trees, depth = rng.choice(forms)
    c = _case(op, _log_int(rng, 256, top), hidden, depth, trees, x, w, y, skew=rng.random() < 0.25)
    return _fit(c, 8e9)


# ------------------------------------------------------------------ inputs


def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + tag) & 0x7FFFFFFF)
    return g


def _weights(case, seed, tag):
    n = (2 << case["depth"]) - 1
    shape = (case["trees"], n, case["hidden"])
    g = _gen(seed, tag)
    return tuple(torch.randn(shape, generator=g, device="cuda").div_(math.sqrt(case["hidden"])).to(DT[case["w"]])
                 for _ in range(2))


def _norm_params(case, seed, tag):
    g = _gen(seed, tag)
    gamma = 1.0 + 0.1 * torch.randn(case["hidden"], generator=g, device="cuda")
    return gamma, 0.1 * torch.randn(case["hidden"], generator=g, device="cuda")


def _tokens(case, n, g, centres):
    x = torch.randn((n, case["hidden"]), generator=g, device="cuda")
    if centres is not None:
        which = torch.randint(0, centres.shape[0], (n,), generator=g, device="cuda")
        x = centres[which] + 0.7 * x
    return x.to(DT[case["x"]])


def _layer_norm(u, layer):
    return torch.nn.functional.layer_norm(u, (u.shape[1],), layer[2].to(u.dtype), layer[3].to(u.dtype), EPS)


def _walk(u, w_in, depth, t):
    """Nodes and logits [B, depth+1] of tree t, in u's precision."""
    n = torch.zeros(u.shape[0], dtype=torch.int64, device=u.device)
    nodes, logits = [], []
    for _ in range(depth + 1):
        logit = (u * w_in[t][n].to(u.dtype)).sum(1)
        nodes.append(n)
        logits.append(logit)
        n = 2 * n + 1 + (logit > 0).long()
    return torch.stack(nodes, 1), torch.stack(logits, 1)


def _layer_out(u, layer, case):
    """FFF(u) in u's precision; also the smallest branching |logit| of each token over u's rms."""
    y = torch.zeros_like(u)
    closest = torch.full((u.shape[0],), math.inf, dtype=u.dtype, device=u.device)
    for t in range(case["trees"]):
        nodes, logits = _walk(u, layer[0], case["depth"], t)
        act = torch.nn.functional.gelu(logits)
        for l in range(case["depth"] + 1):
            y += act[:, l:l + 1] * layer[1][t][nodes[:, l]].to(u.dtype)
        if case["depth"]:
            closest = torch.minimum(closest, logits[:, :-1].abs().amin(1))
    return y, closest / u.square().mean(1).sqrt()


def _near_ties(x, layers, case):
    """Which tokens have a branch that rounding could turn."""
    margin = 1e-4 if len(layers) > 1 else 2e-5
    out = []
    for xc in x.split(16384):
        u, bad = xc.float(), torch.zeros(xc.shape[0], dtype=torch.bool, device=x.device)
        for layer in layers:
            f, closest = _layer_out(_layer_norm(u, layer) if case["norm"] else u, layer, case)
            bad |= closest < margin
            u = u + f
        out.append(bad)
    return torch.cat(out)


def prepare(case, seed):
    B, H, D, T = case["tokens"], case["hidden"], case["depth"], case["trees"]
    layers = []
    for i in range(case["layers"]):
        layer = _weights(case, seed, 10 + 2 * i)
        layers.append(layer + _norm_params(case, seed, 11 + 2 * i) if case["norm"] else layer)
    g = _gen(seed, 1)
    centres = torch.randn((64, H), generator=g, device="cuda") if case["skew"] else None
    x = _tokens(case, B, g, centres)
    if D:
        check = torch.arange(B, device="cuda")
        for _ in range(8):
            check = check[_near_ties(x[check], layers, case)]
            if check.numel() == 0:
                break
            x[check] = _tokens(case, check.numel(), g, centres)
    state = {"case": case, "x": x, "layers": layers}
    if case["op"] in ("backward", "train"):
        state["dy"] = torch.randn((B, H), generator=g, device="cuda").to(DT[case["y"]])
    if case["op"] == "backward":
        rec = [torch.stack(parts, 1) for parts in zip(*(_records(x, layers[0][0], D, t) for t in range(T)))]
        state["leaves"], state["logits"] = rec[0].to(torch.int32).contiguous(), rec[1].contiguous()
    return state


def _records(x, w_in, depth, t):
    """Leaves [B] and logits [B, depth+1] of tree t as a forward records them, in single precision."""
    parts = [_walk(xc.float(), w_in, depth, t) for xc in x.split(16384)]
    return torch.cat([p[0][:, -1] for p in parts]), torch.cat([p[1] for p in parts])


def run(state):
    case, x = state["case"], state["x"]
    B, H, D, T = case["tokens"], case["hidden"], case["depth"], case["trees"]
    out = "residual" if case["residual"] else "store"
    if case["op"] == "stack":
        return fff.forward_stack(x, state["layers"], D, T, norm="layernorm" if case["norm"] else None, norm_eps=EPS)
    layer = state["layers"][0]
    kw = dict(norm="layernorm", norm_eps=EPS, norm_gamma=layer[2], norm_beta=layer[3]) if case["norm"] else {}
    if case["op"] == "forward":
        return fff.forward(x, layer[0], layer[1], D, T, y_dtype=DT[case["y"]], out=out, **kw)
    if case["op"] == "backward":
        return fff.backward(x, layer[0], layer[1], D, T, state["dy"], state["leaves"], state["logits"])
    nodes = torch.empty((B, T, D + 1), dtype=torch.int32, device=x.device)
    logits = torch.empty((B, T, D + 1), dtype=torch.float32, device=x.device)
    y = fff.forward(x, layer[0], layer[1], D, T, y_dtype=DT[case["y"]], nodes_out=nodes, logits_out=logits)
    leaves = nodes[:, :, D].contiguous()
    return (y,) + fff.backward(x, layer[0], layer[1], D, T, state["dy"], leaves, logits)


# ------------------------------------------------------------------ work and accuracy


def work(case):
    """x, dy and the records in, y and the gradients out, and each weight row that uniform routing
    reaches, once; two flops per multiply-add of the visited nodes."""
    B, H, D, T = case["tokens"], case["hidden"], case["depth"], case["trees"]
    size = {"f32": 4, "bf16": 2}
    sx, sw, sy = size[case["x"]], size[case["w"]], size[case["y"]]
    rows = T * sum(2.0 ** l * -math.expm1(B * math.log1p(-2.0 ** -l)) if l else 1.0 for l in range(D + 1))
    visits = float(B) * T * (D + 1)
    fwd_bytes = B * H * (sx + sy) + case["layers"] * 2 * H * sw * rows
    fwd_flops = case["layers"] * 4.0 * H * visits
    dw = 2.0 * T * ((2 << D) - 1) * H * 4
    bwd_bytes = B * H * (sx + 2 * sy) + 2 * H * sw * rows + dw + 4 * visits + 4 * B * T
    bwd_flops = 8.0 * H * visits
    if case["op"] == "backward":
        return {"bytes": bwd_bytes, "flops": bwd_flops}
    if case["op"] == "train":
        return {"bytes": fwd_bytes + bwd_bytes, "flops": fwd_flops + bwd_flops}
    return {"bytes": fwd_bytes, "flops": fwd_flops}


def tolerance(case):
    # about four times the error against double precision: bf16 outputs 1.7e-3, the store's rounding;
    # fp32 outputs 1e-7 to 2e-7, more where a few tokens with cancelling terms are all there is
    if case["y"] == "bf16":
        return {"rel": 7e-3}
    return {"rel": 1e-6 if case["tokens"] >= 256 else 4e-6}


def _dgelu(z):
    return 0.5 * torch.erfc(-z * math.sqrt(0.5)) + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)


def _exact_backward(case, x, layer, dy, leaves, logits):
    D, T, H = case["depth"], case["trees"], case["hidden"]
    dx = torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    dws = [torch.zeros(layer[0].shape, dtype=torch.float64, device=x.device) for _ in range(2)]
    for b0 in range(0, x.shape[0], 16384):
        b = slice(b0, b0 + 16384)
        xc, gc = x[b].double(), dy[b].double()
        for t in range(T):
            for l in range(D + 1):
                node = ((leaves[b, t].long() + 1) >> (D - l)) - 1
                z = logits[b, t, l].double()
                dl = (gc * layer[1][t][node].double()).sum(1) * _dgelu(z)
                dx[b] += dl[:, None] * layer[0][t][node].double()
                dws[0][t].index_add_(0, node, dl[:, None] * xc)
                dws[1][t].index_add_(0, node, torch.nn.functional.gelu(z)[:, None] * gc)
    return (dx,) + tuple(dws)


def exact(case, seed):
    """What run returns, in double precision."""
    state = prepare(case, seed)
    D, T = case["depth"], case["trees"]
    layer = state["layers"][0]
    if case["op"] == "backward":
        return _exact_backward(case, state["x"], layer, state["dy"], state["leaves"], state["logits"])
    ys = []
    for xc in state["x"].split(16384):
        u = xc.double()
        for lay in state["layers"]:
            f, _ = _layer_out(_layer_norm(u, lay) if case["norm"] else u, lay, case)
            u = u + f if case["residual"] else f
        ys.append(u)
    y = torch.cat(ys)
    if case["op"] != "train":
        return y
    rec = [[], []]
    for t in range(T):
        parts = [_walk(xc.double(), layer[0], D, t) for xc in state["x"].split(16384)]
        rec[0].append(torch.cat([p[0][:, -1] for p in parts]))
        rec[1].append(torch.cat([p[1] for p in parts]))
    leaves, logits = torch.stack(rec[0], 1), torch.stack(rec[1], 1)
    return (y,) + _exact_backward(case, state["x"], layer, state["dy"], leaves, logits)
