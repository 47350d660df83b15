"""The work that a training program has this library do, as cases that can be timed and compared.

One pass is one optimizer step of one parameter range: the squared gradient norm and the AdamW
update, taken in one of the ways the library offers.  `path` names the way:

  resident   gs_grad_sqnorm, then gs_accum_adamw over the whole range
  groups     the same for one GPT layer tensor by tensor: weight decay is left out for biases and
             LayerNorm, so every tensor of the layer is a call of its own
  split      the step in two parts, [0,s) and [s,n), with s at a fraction of the layer (delay ratio)
  graph      gs_grad_sqnorm_noalloc and gs_accum_adamw over an unaligned range, captured once in a
             HIP graph and replayed
  staged     gs_grad_accum_sqnorm leaves the fp32 sum behind, gs_adamw_from_acc steps from it
  asyougo    one gs_accum_add per micro-batch (the last one with the norm), then gs_adamw_from_acc
  spec       gs_accum_adamw_spec: step and norm in one pass over the gradients, out of place
  shard      one rank's share [n*r/R, n*(r+1)/R) of a layer whose fp32 gradient sum came back from a
             reduction: gs_acc_sqnorm, then gs_adamw_from_acc
  host       states in pinned host memory, stepped in place over the link: gs_grad_sqnorm, then
             gs_stream_layer_step on an in-place context

`ws` is the device workspace the program brings: "min" = gs_sqnorm_workspace_bytes(), the size every
call accepts, or "full" = gs_sqnorm_workspace_bytes_for(n).
"""
from __future__ import annotations

import math

import torch

from paper_2512_17570_amd import gs
from paper_2512_17570_amd import inputs as I

DEV = "cuda:0"
LR, BETA1, BETA2, EPS, DECAY = 1e-4, 0.9, 0.999, 1e-8, 0.01
NO_DECAY = {"ln1.w", "ln1.b", "qkv.b", "out.b", "ln2.w", "ln2.b", "fc1.b", "fc2.b"}


def _case(name, path, n, k, **more):
    c = {"path": path, "n": n, "k": k, "sigma": 1e-3, "outliers": 0.0, "step": 100, "ws": "min", "begin": 0, "frac": 0.4}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    L = I.layer_numel
    return [
        # the parameters of a layer that take no weight decay, as one small range: launches and host calls
        _case("vectors_h1024_k4", "resident", 13 * 1024, 4, step=10),
        # the small layer of the repository's configurations
        _case("layer_h1024_k4", "resident", L(1024), 4, step=10),
        # the same layer as a program with a decay-free group steps it: 12 calls after one norm
        _case("groups_h1024_k4", "groups", L(1024), 4, step=10),
        # a captured step: small unaligned range, odd k, no workspace from the caller
        _case("graph_ragged_k3", "graph", 3_300_007, 3, begin=13, step=10),
        # middle layer in which clipping fires hard
        _case("layer_h4096_k8_clip", "resident", L(4096), 8, outliers=1e-3),
        # one GPT-65B-shaped layer, the headline workload
        _case("layer_h8192_k16", "resident", L(8192), 16, sigma=5e-4),
        # one GPT-175B-shaped layer, stepped 40 % now and 60 % deferred, at an unaligned split point
        _case("split_h12288_k8", "split", L(12288), 8, sigma=5e-4),
        # one GPT-30B-shaped layer through the fp32 sum, with the workspace made for it
        _case("staged_h7168_k16", "staged", L(7168), 16, sigma=5e-4, ws="full"),
        # the layer's fp32 buffer, added into by every micro-batch's backward
        _case("asyougo_h4096_k8", "asyougo", L(4096), 8),
        # speculative single pass with the workspace every norm call takes
        _case("spec_h4096_k8", "spec", L(4096), 8),
        # one of eight ranks' share of a GPT-65B-shaped layer after the gradients' reduce-scatter
        _case("shard_h8192_rank3of8", "shard", L(8192), 1, ranks=8, rank=3),
        # states in host memory: the link is the bound
        _case("host_h1024_k8", "host", L(1024), 8),
    ]


_MOST_BYTES = 26_000_000_000       # a drawn case's traffic; the largest listed one has 76e9


def draw(rng):
    def span(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))

    path = rng.choice(["resident", "resident", "resident", "groups", "split", "graph", "staged", "asyougo", "spec", "shard", "host"])
    # micro-batches of a layer: mostly the powers of two that are configured, else any number
    k = rng.choice([1, 2, 4, 8, 16, 32]) if rng.random() < 0.5 else rng.randint(1, 32)
    step = rng.choice([1, 10, 100, 5000])
    sigma = rng.choice([5e-4, 1e-3])
    outliers = rng.choice([0.0, 0.0, 1e-3])
    ws = rng.choice(["min", "full"])
    more = {"sigma": sigma, "outliers": outliers, "step": step, "ws": ws}
    if path == "groups":
        return _case(None, path, I.layer_numel(rng.randint(128, 1024)), min(k, 16), **more)
    if path == "host":
        return _case(None, path, span(100_000, 13_000_000), min(k, 16), **more)
    if path == "graph":
        return _case(None, path, span(10_000, 30_000_000), k, begin=rng.randint(0, 5000), **more)
    if path == "shard":
        ranks = rng.choice([2, 4, 8])
        return _case(None, path, span(100_000, 800_000_000), 1, ranks=ranks, rank=rng.randrange(ranks), **more)
    n = min(span(8_000, 800_000_000), _MOST_BYTES // (2 * k + 26))
    if path == "split":
        more["frac"] = rng.uniform(0.1, 0.9)
    return _case(None, path, n, k, **more)


def _range(case):
    n = case["n"]
    if case["path"] == "shard":
        return n * case["rank"] // case["ranks"], n * (case["rank"] + 1) // case["ranks"]
    return min(case["begin"], n), n


def _hp(case, decay=DECAY):
    return gs.HParams(LR, BETA1, BETA2, EPS, decay, 0.0 if case["path"] == "spec" else 1.0, case["step"])


_host_ctx = None


def _host_context():
    """The in-place context a program keeps for its whole run (16 of the chip's CUs fill the link)."""
    global _host_ctx
    if _host_ctx is None:
        _host_ctx = gs.gs_stream_ctx_create_inplace(16)
    return _host_ctx


def _layer_of(n):
    """The tensors of the GPT layer with n parameters as (name, begin, end) of its flat range."""
    h = int(round(math.sqrt(n / 12)))
    while I.layer_numel(h) > n:
        h -= 1
    out, at = [], 0
    for name, size in I.layer_segments(h):
        out.append((name, at, at + size))
        at += size
    assert at == n
    return out


def prepare(case, seed):
    path, n, k = case["path"], case["n"], case["k"]
    b, e = _range(case)
    p, m, v = I.make_states(n, seed, DEV)
    s = {"path": path, "n": n, "b": b, "e": e, "p": p, "m": m, "v": v, "hp": _hp(case),
         "w": torch.zeros(n, dtype=torch.bfloat16, device=DEV),
         "sq": torch.zeros(1, dtype=torch.float64, device=DEV)}
    nbytes = gs.gs_sqnorm_workspace_bytes() if case["ws"] == "min" else gs.gs_sqnorm_workspace_bytes_for(e - b)
    s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    if path == "shard":
        s["acc"] = I.normal_f32(n, case["sigma"] * 4.0, seed, 50, DEV)
        return s
    s["g"] = I.make_grads(n, k, case["sigma"], seed, DEV, case["outliers"])
    if path in ("staged", "asyougo"):
        s["acc"] = torch.zeros(n, dtype=torch.float32, device=DEV)
    elif path == "spec":
        s["out"] = [torch.zeros_like(p) for _ in range(3)]
    elif path == "split":
        s["s"] = int(case["frac"] * n)
    elif path == "groups":
        s["groups"] = [(x, y, _hp(case, 0.0 if name in NO_DECAY else DECAY)) for name, x, y in _layer_of(n)]
    elif path == "host":
        s["ctx"] = _host_context()
        for q in ("p", "m", "v"):
            h = torch.empty(n, dtype=torch.float32, pin_memory=True)
            h.copy_(s[q])
            s[q] = h
    elif path == "graph":
        gs.gs_grad_sqnorm_noalloc(s["g"], b, e, s["sq"])      # outside capture: looks up the library's array
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            gs.gs_grad_sqnorm_noalloc(s["g"], b, e, s["sq"])
            gs.gs_accum_adamw(p, m, v, s["w"], s["g"], b, e, s["hp"], s["sq"])
    return s


def run(s):
    path, p, m, v, w, sq, b, e, hp = (s[x] for x in ("path", "p", "m", "v", "w", "sq", "b", "e", "hp"))
    if path == "graph":
        s["graph"].replay()
    elif path == "resident":
        gs.gs_grad_sqnorm(s["g"], b, e, sq, s["ws"])
        gs.gs_accum_adamw(p, m, v, w, s["g"], b, e, hp, sq)
    elif path == "groups":
        gs.gs_grad_sqnorm(s["g"], b, e, sq, s["ws"])
        for x, y, ghp in s["groups"]:
            gs.gs_accum_adamw(p, m, v, w, s["g"], x, y, ghp, sq)
    elif path == "split":
        gs.gs_grad_sqnorm(s["g"], b, e, sq, s["ws"])
        gs.gs_accum_adamw(p, m, v, w, s["g"], b, s["s"], hp, sq)
        gs.gs_accum_adamw(p, m, v, w, s["g"], s["s"], e, hp, sq)
    elif path == "staged":
        gs.gs_grad_accum_sqnorm(s["g"], b, e, s["acc"], sq, s["ws"])
        gs.gs_adamw_from_acc(p, m, v, w, s["acc"], b, e, hp, sq)
        return {"p": p, "m": m, "v": v, "w": w, "sq": sq, "acc": s["acc"]}
    elif path == "asyougo":
        last = len(s["g"]) - 1
        for j, g in enumerate(s["g"]):
            if j < last:
                gs.gs_accum_add(s["acc"], g, j == 0, b, e)
            else:
                gs.gs_accum_add(s["acc"], g, j == 0, b, e, sq, s["ws"])
        gs.gs_adamw_from_acc(p, m, v, w, s["acc"], b, e, hp, sq)
        return {"p": p, "m": m, "v": v, "w": w, "sq": sq, "acc": s["acc"]}
    elif path == "spec":
        po, mo, vo = s["out"]
        gs.gs_accum_adamw_spec(p, m, v, po, mo, vo, w, s["g"], b, e, hp, sq, s["ws"])
        return {"p": po, "m": mo, "v": vo, "w": w, "sq": sq}
    elif path == "shard":
        gs.gs_acc_sqnorm(s["acc"], b, e, sq, s["ws"])
        gs.gs_adamw_from_acc(p, m, v, w, s["acc"], b, e, hp, sq)
        return {"p": p[b:e], "m": m[b:e], "v": v[b:e], "w": w[b:e], "sq": sq}
    elif path == "host":
        gs.gs_grad_sqnorm(s["g"], b, e, sq, s["ws"])
        gs.gs_stream_layer_step(s["ctx"], p, m, v, w, s["g"], s["n"], hp, sq)
        gs.gs_stream_ctx_sync(s["ctx"])                        # the states are read on the host next
    return {"p": p, "m": m, "v": v, "w": w, "sq": sq}


def work(case):
    """Gradients (bf16, or one fp32 sum) and p, m, v in; p, m, v and the bf16 weight out."""
    b, e = _range(case)
    n, k, path = e - b, case["k"], case["path"]
    grad = 4 if path == "shard" else 2 * k
    acc = 4 if path in ("staged", "asyougo") else 0            # the sum is an output here
    return {"bytes": n * (grad + 12 + 14 + acc), "flops": n * ((0 if path == "shard" else k) + 18)}


def tolerance(case):
    # p, m, v are chains of about ten fp32 roundings: 4e-8 of the 2-norm against 64 bits as measured, so 1e-7
    # between two correct implementations.  w rounds p to bf16: where a last-bit difference of p lies next to a
    # tie (one element in about 2**16) it moves by one bf16 ulp, 2**-8 to 2**-7 of its value, which is 1.5e-5 of
    # the 2-norm and up to 8e-3 of one element.
    return {"rel": 4e-5, "max": 8e-3}


def exact(case, seed):
    """The documented update in 64 bits, chunk by chunk, on the inputs of prepare()."""
    path, n = case["path"], case["n"]
    b, e = _range(case)
    s = prepare(dict(case, path="shard" if path == "shard" else "resident"), seed)
    out = {q: s[q].to(torch.float64) for q in ("p", "m", "v")}
    f32 = lambda x: float(torch.tensor(x, dtype=torch.float32))  # noqa: E731  the hyper-parameters are given in 32 bits
    lr, b1, b2, eps, maxn, t = f32(LR), f32(BETA1), f32(BETA2), f32(EPS), _hp(case).max_grad_norm, case["step"]
    step = 1 << 26
    acc = torch.zeros(n if path in ("staged", "asyougo") else 0, dtype=torch.float64, device=DEV)
    total = torch.zeros(1, dtype=torch.float64, device=DEV)

    def summed(x, y):
        if path == "shard":
            return s["acc"][x:y].to(torch.float64)
        a = torch.zeros(y - x, dtype=torch.float64, device=DEV)
        for g in s["g"]:
            a += g[x:y]
        return a

    for x in range(b, e, step):
        a = summed(x, min(e, x + step))
        total += a.square().sum()
        if acc.numel():
            acc[x:min(e, x + step)] = a
    c = min(1.0, maxn / (math.sqrt(float(total)) + 1e-6)) if maxn > 0 else 1.0
    w = torch.zeros(n, dtype=torch.float64, device=DEV)
    parts = [(x, y, 0.0 if name in NO_DECAY else DECAY) for name, x, y in _layer_of(n)] if path == "groups" else [(b, e, DECAY)]
    for lo, hi, decay in parts:
        for x in range(lo, hi, step):
            y = min(hi, x + step)
            g = summed(x, y) * c
            out["m"][x:y] = b1 * out["m"][x:y] + (1.0 - b1) * g
            out["v"][x:y] = b2 * out["v"][x:y] + (1.0 - b2) * g * g
            d = (out["v"][x:y] / (1.0 - b2 ** t)).sqrt() + eps
            out["p"][x:y] = out["p"][x:y] * (1.0 - lr * f32(decay)) - lr / (1.0 - b1 ** t) * out["m"][x:y] / d
            w[x:y] = out["p"][x:y]
    if path == "shard":
        return {**{q: out[q][b:e] for q in out}, "w": w[b:e], "sq": total}
    if acc.numel():
        return {**out, "w": w, "sq": total, "acc": acc}
    return {**out, "w": w, "sq": total}
