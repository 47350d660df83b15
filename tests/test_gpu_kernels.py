"""Every kernel of the library on the GPU, by the calls of kernel_calls.py, on a range that is ragged at both ends.

The expected values do not come from the call under test: sums are added by torch in fp32, in order (each add is one
rounding, so they are exact equals), norms are torch's fp64 sums of their squares, and a step has to leave the bits
that the same range gives in pieces of up to 300 000 elements, a size whose kernels the parity tests hold against
the oracle element by element."""
from __future__ import annotations

import pytest
import torch

from gpu_util import DEV, gs
from kernel_calls import BEGIN, CALLS
from paper_2512_17570_amd import inputs as I

pytestmark = pytest.mark.gpu

HP = gs.HParams(step=10, max_grad_norm=0.1)
PIECE = 300_000


def in_pieces(p, m, v, w, grads, acc, b, e, hp, sq):
    for x in range(b, e, PIECE):
        y = min(e, x + PIECE)
        if acc is None:
            gs.gs_accum_adamw(p, m, v, w, grads, x, y, hp, sq)
        else:
            gs.gs_adamw_from_acc(p, m, v, w, acc, x, y, hp, sq)


def fp32_sum(grads, b, e):
    a = torch.zeros(e - b, dtype=torch.float32, device=DEV)
    for g in grads:
        a += g[b:e].float()
    return a


def square_sum(a):
    return sum(float(part.double().square().sum()) for part in a.split(1 << 26))


@pytest.mark.parametrize("entry,k,length,ws,cus,first,accumulate", CALLS)
def test_kernel(entry, k, length, ws, cus, first, accumulate):
    print(f"[kernel] {entry} k={k} length={length} ws={ws} cus={cus} first={first} accumulate={accumulate}", flush=True)
    b, e = BEGIN, BEGIN + length
    n = e + 2
    grads = [I.normal_f32(n, 1e-3, 7, j, DEV).to(torch.bfloat16) for j in range(k)] if entry != "acc_norm" else []
    sq = torch.full((1,), 4.0 if accumulate or entry in ("step", "oop", "from_acc") else float("nan"), dtype=torch.float64, device=DEV)
    nbytes = gs.gs_sqnorm_workspace_bytes() if ws == "min" else gs.gs_sqnorm_workspace_bytes_for(length)
    work = torch.full((nbytes,), 0xff, dtype=torch.uint8, device=DEV)          # NaNs: nothing may be taken from it unwritten
    raw = gs.gs_cu_stream_create(cus) if cus < 256 else None
    torch.cuda.synchronize()
    try:
        S = 0.0
        if entry in ("step", "oop", "from_acc", "spec"):
            states = I.make_states(n, 3, DEV)
            acc = fp32_sum(grads, 0, n) if entry == "from_acc" else None
            want = [x.clone() for x in states] + [torch.zeros(n, dtype=torch.bfloat16, device=DEV)]
            in_pieces(*want, grads, acc, b, e, HP, None if entry == "spec" else sq)
            got = [x.clone() for x in states] + [torch.zeros(n, dtype=torch.bfloat16, device=DEV)]
            torch.cuda.synchronize()
            if entry == "step":
                gs.gs_accum_adamw(*got, grads, b, e, HP, sq, stream=raw)
            elif entry == "oop":
                gs.gs_accum_adamw_oop(*states, *got, grads, b, e, HP, sq, stream=raw)
            elif entry == "from_acc":
                gs.gs_adamw_from_acc(*got, acc, b, e, HP, sq, stream=raw)
            else:
                gs.gs_accum_adamw_spec(*states, *got, grads, b, e, HP, sq, work, stream=raw)
            torch.cuda.synchronize()
            for name, x, y in zip("pmvw", got, want):
                assert torch.equal(x, y), name           # outside the range both hold what was there
            if entry == "spec":
                S = square_sum(fp32_sum(grads, b, e))
        else:
            start = torch.full((n,), 3.0, dtype=torch.float32, device=DEV)
            acc = start.clone()
            if entry == "norm":
                want = fp32_sum(grads, b, e)
            elif entry == "acc_norm":
                acc[b:e] = want = I.normal_f32(length, 1e-3, 5, 0, DEV)
            else:
                want = fp32_sum(grads, b, e) + (3.0 if entry.startswith("add") and not first else 0.0)
            torch.cuda.synchronize()
            if entry == "norm":
                gs.gs_grad_sqnorm(grads, b, e, sq, work, accumulate=bool(accumulate), stream=raw)
            elif entry == "acc_norm":
                gs.gs_acc_sqnorm(acc, b, e, sq, work, accumulate=bool(accumulate), stream=raw)
            elif entry == "staged":
                gs.gs_grad_accum_sqnorm(grads, b, e, acc, sq, work, accumulate=bool(accumulate), stream=raw)
            elif entry == "add":
                gs.gs_accum_add(acc, grads[0], bool(first), b, e, stream=raw)
            else:
                gs.gs_accum_add(acc, grads[0], bool(first), b, e, sq, work, accumulate=bool(accumulate), stream=raw)
            torch.cuda.synchronize()
            if entry != "norm":
                assert torch.equal(acc[b:e], want)
                assert bool((acc[:b] == 3.0).all()) and bool((acc[e:] == 3.0).all())
            if entry != "add":
                S = square_sum(want)
        if S:
            total = float(sq.item()) - (4.0 if accumulate else 0.0)
            # two fp64 trees over exact squares, each within (depth of the tree) x 2^-53 of the sum; with an earlier
            # norm of 4 in the scalar, one rounding of that
            assert abs(total - S) <= 1e-12 * S + (1e-15 if accumulate else 0.0), (total, S)
    finally:
        if raw is not None:
            gs.gs_cu_stream_destroy(raw)
