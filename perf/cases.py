"""Workloads for timing the framework: one training step of a detached-block
network, one of the detached small transformer, and the embedding-bag input
stage, each through its public entry point.

A case is a plain dict.  ``listed()`` gives the fixed ones, ``draw(rng)`` one
more of the same ranges, ``prepare(case, seed)`` what a training program holds
before the call (inputs, trainer with mid-training Adam state), ``run(state)``
one pass, ``work(case)`` the bytes and operations a pass cannot do without,
``tolerance(case)`` how far two correct implementations may be apart, and
``exact(case, seed)`` the same outputs in float64 from plain torch.
"""
import math

import numpy as np
import torch

from paper_2608_18469_amd import erase, erase_tf, synth

CTR_DENSE, CTR_DIM = 13, 64  # of a CTR input row: dense features, then 64-wide pooled bags
STEP = 1000                  # steps taken before the timed one (Adam's bias corrections)
# Adam as the workloads declare it, at a late-training rate: the timed passes
# repeat one batch, and its gradients should stay those of a training run
ADAM = {"lr": 1e-4, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest step: two fp32 blocks on 64 rows (launch latency and host cost)
        dict(name="tiny_f32", kind="mlp", dtype="f32", batch=64, in_dim=16, blocks=2, widths="32,32",
             schedule="overlap"),
        # the benchmark's CTR step: six subarchitectures on a shared 1677-wide input
        dict(name="ctr_mlp", kind="mlp", dtype="bf16", batch=4096, in_dim=1677, blocks=6, widths="512,256,128",
             schedule="overlap"),
        # the same model at a large batch, steps overlapping one another
        dict(name="ctr_mlp_32k", kind="mlp", dtype="bf16", batch=32768, in_dim=1677, blocks=6, widths="512,256,128",
             schedule="pipeline"),
        # a ragged batch and odd widths: x is copied into the padded buffer, every tile has a remainder
        dict(name="mlp_ragged", kind="mlp", dtype="bf16", batch=1000, in_dim=1003, blocks=3, widths="401,203,99",
             schedule="serial"),
        # the DCNv2 workload at its full size
        dict(name="ctr_dcn", kind="dcn", dtype="bf16", batch=16384, in_dim=1677, blocks=6, cross=2,
             widths="1024,1024,512", schedule="overlap"),
        # a smaller DCN with a ragged batch and odd widths, on one stream
        dict(name="dcn_ragged", kind="dcn", dtype="bf16", batch=3001, in_dim=1003, blocks=2, cross=2,
             widths="600,300,200", schedule="serial"),
        # twelve narrow blocks chained through the stop-gradient (many small launches)
        dict(name="deep_chain", kind="chain", dtype="bf16", batch=1024, in_dim=256, blocks=12, widths="256,256",
             schedule="overlap"),
        # the conventional step of the same network (gradients cross every cut)
        dict(name="chain_undetached", kind="chain", dtype="bf16", batch=1024, in_dim=256, blocks=12, widths="256,256",
             schedule="undetached"),
        # two layers of the full small-transformer shape
        dict(name="tf_c5_2layers", kind="tf", vocab=32768, heads=8, layers=2, seq=1024, batch=16, schedule="overlap"),
        # a small ragged transformer: nothing is a multiple of a tile
        dict(name="tf_ragged", kind="tf", vocab=8000, heads=3, layers=2, seq=300, batch=6, schedule="serial"),
        # the CTR input stage: 26 bags of 1..20 Zipf ids per row, and its backward
        dict(name="bags_forward", kind="bags", dtype="bf16", batch=4096, tables=26, rows=100000, dim=64),
        dict(name="bags_backward", kind="bags_bwd", dtype="bf16", batch=4096, tables=26, rows=100000, dim=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mlp", "mlp", "dcn", "dcn", "chain", "tf", "tf", "bags", "bags_bwd"])
    if kind == "mlp":
        f32 = rng.random() < 0.2
        batch = _log_int(rng, 64, 2048 if f32 else 32768)
        if rng.random() < 0.5:
            batch = max(128, batch // 128 * 128)
        w1 = rng.randint(64, 1024)
        w2 = rng.randint(33, w1)
        w3 = rng.randint(17, w2)
        return dict(kind="mlp", dtype="f32" if f32 else "bf16", batch=batch, in_dim=rng.randint(100, 2000),
                    blocks=rng.randint(1, 6), widths="%d,%d,%d" % (w1, w2, w3),
                    schedule=rng.choice(["overlap", "serial", "pipeline"]))
    if kind == "dcn":
        batch = _log_int(rng, 256, 16384)
        if rng.random() < 0.5:
            batch = batch // 128 * 128
        w1 = rng.randint(128, 1024)
        return dict(kind="dcn", dtype="bf16", batch=batch, in_dim=rng.randint(128, 1677), blocks=rng.randint(1, 4),
                    cross=rng.randint(1, 3), widths="%d,%d,%d" % (w1, rng.randint(128, 1024), rng.randint(64, 512)),
                    schedule=rng.choice(["overlap", "serial", "pipeline"]))
    if kind == "chain":
        w = rng.randint(32, 512)
        return dict(kind="chain", dtype="bf16", batch=_log_int(rng, 64, 4096), in_dim=w, blocks=rng.randint(2, 12),
                    widths="%d,%d" % (rng.randint(32, 512), w),
                    schedule=rng.choice(["overlap", "pipeline", "serial", "undetached"]))
    if kind == "tf":
        seq = _log_int(rng, 16, 1024)
        return dict(kind="tf", vocab=64 * _log_int(rng, 8, 512), heads=rng.randint(1, 8), layers=rng.randint(1, 2),
                    seq=seq, batch=rng.randint(1, 16), schedule=rng.choice(["overlap", "serial"]))
    return dict(kind=kind, dtype=rng.choice(["bf16", "f32"]), batch=_log_int(rng, 64, 4096),
                tables=rng.randint(1, 26), rows=_log_int(rng, 1000, 100000), dim=rng.choice([16, 32, 64]))


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _net(case):
    """The model description of a detached-block case."""
    widths = [int(w) for w in case["widths"].split(",")]
    blocks = []
    for b in range(case["blocks"]):
        layers, cur = [], case["in_dim"]
        for _ in range(case.get("cross", 0)):
            layers.append(("cross", cur, cur))
        for w in widths:
            layers.append(("linear_relu", cur, w))
            cur = w
        blocks.append({"input": "prev" if case["kind"] == "chain" and b > 0 else "x", "layers": layers, "lam": 1.0})
    return synth.custom(case["dtype"], case["batch"], case["in_dim"], blocks, adam=ADAM)


def _mid_training(n, g, scale):
    """Adam moments of a run under way: first moments of both signs, second moments of that size squared."""
    m = torch.randn(n, generator=g, device="cuda") * scale
    v = (torch.rand(n, generator=g, device="cuda") + 0.5) * scale * scale
    return m, v


def _net_inputs(case, seed):
    """(x [M][in_dim] in the activation type, labels, per block flat (param, m, v))."""
    g = _gen(seed)
    M, K = case["batch"], case["in_dim"]
    bf = case["dtype"] == "bf16"
    if case["kind"] == "chain" or K <= CTR_DENSE + CTR_DIM:
        x = torch.randn((M, K), generator=g, device="cuda")
        y = (torch.rand(M, generator=g, device="cuda") < (0.03 if case["kind"] == "chain" else 0.5)).float()
    else:
        # CTR rows: log1p of log-normal dense features, then sums of 1..20 table rows of N(0, 0.01^2)
        dense = torch.log1p(torch.exp(torch.randn((M, CTR_DENSE), generator=g, device="cuda")))
        T = -(-(K - CTR_DENSE) // CTR_DIM)
        bag = torch.randint(1, 21, (M, T, 1), generator=g, device="cuda").float().sqrt() * 0.01
        pooled = (torch.randn((M, T, CTR_DIM), generator=g, device="cuda") * bag).reshape(M, T * CTR_DIM)
        x = torch.cat([dense, pooled[:, :K - CTR_DENSE]], dim=1)
        y = (torch.rand(M, generator=g, device="cuda") < 0.03).float()
    x = x.to(torch.bfloat16 if bf else torch.float32)
    state = []
    for blk in _net(case)["blocks"]:
        parts = []
        for (_k, fin, fout) in blk["layers"]:
            b = 1.0 / math.sqrt(fin)
            parts.append((torch.rand(fout * fin + fout, generator=g, device="cuda") * 2 - 1) * b)
        last = blk["layers"][-1][2]
        parts.append((torch.rand(last + 1, generator=g, device="cuda") * 2 - 1) / math.sqrt(last))
        p = torch.cat(parts)
        state.append((p, *_mid_training(p.numel(), g, 1e-4)))
    return x, y, state


def _tf_cfg(case):
    return {"vocab": case["vocab"], "d": 64 * case["heads"], "heads": case["heads"], "layers": case["layers"],
            "seq": case["seq"], "batch": case["batch"], "lam": 1.0, "adam": dict(ADAM), "dtype": "bf16"}


def _tf_shapes(case, block):
    V, d = case["vocab"], 64 * case["heads"]
    head = [("emb", V, d)] if block == 0 else []
    return head + [("wqkv", 3 * d, d), ("wo", d, d), ("w1", 4 * d, d), ("w2", d, 4 * d), ("wh", V, d)]


def _tf_inputs(case, seed):
    """(tokens int32 [B][T + 1], per block flat (param, m, v))."""
    g = _gen(seed)
    tokens = torch.randint(0, case["vocab"], (case["batch"], case["seq"] + 1), generator=g, device="cuda",
                           dtype=torch.int32)
    state = []
    for b in range(case["layers"]):
        parts = []
        for (name, r, c) in _tf_shapes(case, b):
            if name == "emb":
                parts.append(torch.randn(r * c, generator=g, device="cuda"))
            else:
                parts.append((torch.rand(r * c, generator=g, device="cuda") * 2 - 1) / math.sqrt(c))
        p = torch.cat(parts)
        state.append((p, *_mid_training(p.numel(), g, 1e-5)))
    return tokens, state


def _zipf(rows):
    return np.arange(1, rows + 1, dtype=np.float64) ** -1.1


def _bag_inputs(case, seed):
    """(dense, offsets, indices, tables or the gradient at x): bags of 1..20 bounded-Zipf(1.1) ids."""
    g = _gen(seed)
    M, T, rows, dim = case["batch"], case["tables"], case["rows"], case["dim"]
    lens = torch.randint(1, 21, (T, M), generator=g, device="cuda")
    ends = torch.cumsum(lens.reshape(-1), 0)
    starts = torch.cat([ends.new_zeros(1), ends])  # of every bag, table after table
    offsets = torch.stack([starts[t * M:(t + 1) * M + 1] for t in range(T)]).contiguous()
    cdf = torch.from_numpy(np.cumsum(_zipf(rows) / _zipf(rows).sum())).cuda()
    u = torch.rand(int(ends[-1]), generator=g, device="cuda", dtype=torch.float64)
    indices = torch.searchsorted(cdf, u).clamp_(max=rows - 1).to(torch.int32)
    dense = torch.exp(torch.randn((M, CTR_DENSE), generator=g, device="cuda"))
    if case["kind"] == "bags":
        data = torch.randn((T, rows, dim), generator=g, device="cuda") * 0.01
    else:
        ld = -(-(CTR_DENSE + T * dim) // 128) * 128
        data = torch.zeros((M, ld), device="cuda")
        data[:, :CTR_DENSE + T * dim] = torch.randn((M, CTR_DENSE + T * dim), generator=g, device="cuda") / M
        data = data.to(torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)
    return dense, offsets, indices, data


# ---------------------------------------------------------------------------
# what a program holds before the call
# ---------------------------------------------------------------------------
def _load(tr, state):
    """A checkpoint into a trainer's buffers: parameters, moments and step."""
    for b, (p, m, v) in enumerate(state):
        tr.param[b].copy_(p)
        tr.m[b].copy_(m)
        tr.v[b].copy_(v)
    torch.cuda.synchronize()
    tr.refresh_weights()
    tr.set_step(STEP)
    tr.sync()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "tf":
        tokens, state = _tf_inputs(case, seed)
        cfg = _tf_cfg(case)
        blank = [{n: np.zeros((r, c), np.float32) for (n, r, c) in _tf_shapes(case, b)} for b in range(case["layers"])]
        tr = erase_tf.TfTrainer(cfg, blank)
        _load(tr, state)
        return {"kind": kind, "tr": tr, "tokens": tokens, "schedule": case["schedule"]}
    if kind in ("mlp", "dcn", "chain"):
        x, y, state = _net_inputs(case, seed)
        cfg = _net(case)
        blank = [{"layers": [(np.zeros((o, i), np.float32), np.zeros(o, np.float32)) for (_k, i, o) in blk["layers"]],
                  "head": (np.zeros(blk["layers"][-1][2], np.float32), np.zeros(1, np.float32))}
                 for blk in cfg["blocks"]]
        # rows of x are read where they are when the batch is a multiple of 128
        tr = erase.Trainer(cfg, blank, x_in_place=case["batch"] % 128 == 0, bwd_streams=2)
        xp = torch.zeros((case["batch"], tr.ncfg.x_ld), dtype=x.dtype, device="cuda")
        xp[:, :case["in_dim"]] = x
        _load(tr, state)
        return {"kind": kind, "tr": tr, "x": xp, "y": y, "schedule": case["schedule"]}
    dense, offsets, indices, data = _bag_inputs(case, seed)
    s = {"kind": kind, "dense": dense, "offsets": offsets, "indices": indices, "data": data, "case": dict(case)}
    if kind == "bags":
        ld = -(-(CTR_DENSE + case["tables"] * case["dim"]) // 128) * 128
        s["x"] = torch.empty((case["batch"], ld), device="cuda",
                             dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)
    else:
        s["grad"] = torch.empty((case["tables"], case["rows"], case["dim"]), device="cuda")
    return s


def run(state):
    kind = state["kind"]
    if kind == "bags":
        erase.embed_bags(state["dense"], state["offsets"], state["indices"], state["data"], state["x"])
        return state["x"]
    if kind == "bags_bwd":
        c = state["case"]
        grad, _ = erase.embed_bags_backward(state["offsets"], state["indices"], state["data"], CTR_DENSE, c["rows"],
                                            c["dim"], table_grad=state["grad"])
        return grad
    tr = state["tr"]
    if kind == "tf":
        losses = tr.step(state["tokens"], state["schedule"])
    else:
        losses = tr.step(state["x"], state["y"], state["schedule"])
    return {"losses": losses, "param": tr.param, "m": tr.m, "v": tr.v, "grad": tr.grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "tf":
        V, d, L, T, B = case["vocab"], 64 * case["heads"], case["layers"], case["seq"], case["batch"]
        N = B * T
        body, head, att = 2 * N * d * 12 * d, 2 * N * d * V, 2 * B * d * T * (T + 1)
        # forward, weight gradients, input gradients (none into a detached block input)
        flops = 3 * L * (body + head) - (L - 1) * 2 * N * d * 3 * d + att * L * (1 + 2.5)
        params = L * (12 * d * d + V * d) + V * d
        return {"bytes": 28.0 * params + 4.0 * B * (T + 1), "flops": float(flops)}
    if kind in ("mlp", "dcn", "chain"):
        M, flops, params = case["batch"], 0.0, 0
        cross_cut = case["schedule"].startswith("undetached")
        for b, blk in enumerate(_net(case)["blocks"]):
            for i, (_k, fin, fout) in enumerate(blk["layers"]):
                dgrad = i > 0 or (cross_cut and b > 0)
                flops += 2.0 * M * fin * fout * (3 if dgrad else 2)
                params += fin * fout + fout
            params += blk["layers"][-1][2] + 1
        esz = 2 if case["dtype"] == "bf16" else 4
        # parameters and moments read and written, gradients written, the batch read
        return {"bytes": 28.0 * params + float(esz) * M * case["in_dim"] + 4.0 * M, "flops": flops}
    M, T, rows, dim = case["batch"], case["tables"], case["rows"], case["dim"]
    nnz = M * 10.5
    esz = 2 if case["dtype"] == "bf16" else 4
    used = float(np.sum(-np.expm1(nnz * np.log1p(-_zipf(rows) / _zipf(rows).sum()))))  # rows of a table that occur
    ids = T * (8.0 * (M + 1) + 4.0 * nnz)
    width = -(-(CTR_DENSE + T * dim) // 128) * 128
    if kind == "bags":
        return {"bytes": ids + 4.0 * M * CTR_DENSE + T * used * dim * 4.0 + float(esz) * M * width,
                "flops": T * nnz * dim}
    return {"bytes": ids + float(esz) * M * T * dim + 4.0 * T * rows * dim, "flops": T * nnz * dim}


def tolerance(case):
    kind = case["kind"]
    if kind == "bags":  # one rounding of the sum to x's type
        return {"rel": 5e-3} if case["dtype"] == "bf16" else {"rel": 1e-6}
    if kind == "bags_bwd":  # fp32 sums of up to tens of thousands of terms
        return {"rel": 1e-6}
    if kind == "tf":  # bf16 activations and gradients, attention probabilities as bf16 operands
        return {"rel": 2e-2}
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}


# ---------------------------------------------------------------------------
# the same outputs in float64
# ---------------------------------------------------------------------------
def _adam64(p, m, v, g):
    t = STEP + 1
    b1, b2 = (float(np.float32(ADAM[k])) for k in ("beta1", "beta2"))
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    p = p - ADAM["lr"] / (1 - b1 ** t) * m / (v.sqrt() / math.sqrt(1 - b2 ** t) + ADAM["eps"])
    return p, m, v


def _finish(losses, flats, state):
    """Gradients by autograd, then Adam: the layout of run()'s answer."""
    grads = torch.autograd.grad(sum(losses), flats)
    new = [_adam64(p.double(), m.double(), v.double(), g) for (p, m, v), g in zip(state, grads)]
    return {"losses": torch.stack([l.detach() for l in losses]), "param": [n[0] for n in new],
            "m": [n[1] for n in new], "v": [n[2] for n in new], "grad": list(grads)}


def _exact_net(case, seed):
    x, y, state = _net_inputs(case, seed)
    x, y = x.double(), y.double()
    detach = not case["schedule"].startswith("undetached")
    flats = [p.double().requires_grad_() for (p, _m, _v) in state]
    losses, prev = [], None
    for blk, flat in zip(_net(case)["blocks"], flats):
        a0 = x if blk["input"] == "x" else (prev.detach() if detach else prev)
        h, o = a0, 0
        for (kind, fin, fout) in blk["layers"]:
            W = flat[o:o + fout * fin].view(fout, fin)
            b = flat[o + fout * fin:o + fout * fin + fout]
            o += fout * fin + fout
            u = h @ W.t() + b
            h = torch.relu(u) if kind == "linear_relu" else a0 * u + h
        s = h @ flat[o:-1] + flat[-1]
        losses.append(torch.nn.functional.binary_cross_entropy_with_logits(s, y))
        prev = h
    return _finish(losses, flats, state)


def _rms(x):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + 1e-6)


def _exact_tf(case, seed):
    tokens, state = _tf_inputs(case, seed)
    B, T, H, d = case["batch"], case["seq"], case["heads"], 64 * case["heads"]
    inp, target = tokens[:, :-1].long(), tokens[:, 1:].long().reshape(-1)
    flats = [p.double().requires_grad_() for (p, _m, _v) in state]
    hide = torch.ones((T, T), dtype=torch.bool, device="cuda").triu(1)
    losses, z = [], None
    for b, flat in enumerate(flats):
        w, o = {}, 0
        for (name, r, c) in _tf_shapes(case, b):
            w[name] = flat[o:o + r * c].view(r, c)
            o += r * c
        a0 = w["emb"][inp.reshape(-1)] if b == 0 else z.detach()
        qkv = (_rms(a0) @ w["wqkv"].t()).view(B, T, 3, H, 64).permute(2, 0, 3, 1, 4)
        s = (qkv[0] @ qkv[1].transpose(-1, -2).contiguous()) * 0.125
        att = torch.softmax(s.masked_fill(hide, -math.inf), -1) @ qkv[2]
        a1 = a0 + att.permute(0, 2, 1, 3).reshape(B * T, d) @ w["wo"].t()
        z = a1 + torch.nn.functional.gelu(_rms(a1) @ w["w1"].t(), approximate="tanh") @ w["w2"].t()
        losses.append(torch.nn.functional.cross_entropy(_rms(z) @ w["wh"].t(), target))
        del s, att, qkv
    return _finish(losses, flats, state)


def _exact_bags(case, seed):
    dense, offsets, indices, data = _bag_inputs(case, seed)
    M, T, rows, dim = case["batch"], case["tables"], case["rows"], case["dim"]
    n_used = CTR_DENSE + T * dim
    out = torch.zeros((M, -(-n_used // 128) * 128), dtype=torch.float64, device="cuda")
    if case["kind"] == "bags":
        out[:, :CTR_DENSE] = torch.log1p(dense.double())
    else:
        out = torch.zeros((T, rows, dim), dtype=torch.float64, device="cuda")
    for t in range(T):
        o = offsets[t]
        ids = indices[int(o[0]):int(o[-1])].long()
        bag = torch.repeat_interleave(torch.arange(M, device="cuda"), o[1:] - o[:-1])
        c = CTR_DENSE + t * dim
        if case["kind"] == "bags":
            out[:, c:c + dim].index_add_(0, bag, data[t].double()[ids])
        else:
            out[t].index_add_(0, ids, data[:, c:c + dim].double()[bag])
    return out


def exact(case, seed):
    if case["kind"] == "tf":
        return _exact_tf(case, seed)
    if case["kind"] in ("mlp", "dcn", "chain"):
        return _exact_net(case, seed)
    return _exact_bags(case, seed)
