"""GPU tests at the sizes where the launchers change the shape of a pass: the last range of one shape and
the first of the next, with ragged begins and every remainder of the gradient batches.

Sizes are lengths of [begin,end); the limits are those of csrc/gs_internal.h.
"""
from __future__ import annotations

import pytest
import torch

from gpu_util import DEV, DeviceCase, O, assert_bf16_close, assert_f32_close, gs, np_bf16, np_f32

pytestmark = pytest.mark.gpu

LATENCY, RESIDENT, FEW, SERIAL = 1 << 19, 1 << 21, 7_000_000, 1 << 27
HP = gs.HParams(step=10, max_grad_norm=0.1)


def check(got, want, b, e, tag):
    """p, m, v, w of [b,e) against the oracle; nothing outside the range may have moved."""
    for nm, g, w in zip("pmv", got[:3], want[:3]):
        assert_f32_close(np_f32(g)[b:e], w[b:e], f"{tag}.{nm}")
    assert_bf16_close(np_bf16(got[3])[b:e], want[3][b:e], f"{tag}.w")


def untouched(got, before, b, e):
    for g, o in zip(got, before):
        assert torch.equal(g[:b], o[:b]) and torch.equal(g[e:], o[e:])


# (length, k): both sides of every line; k covers whole batches and every kind of remainder
EDGES = [(1, 1), (2, 9), (255, 3), (257, 17), (LATENCY, 8), (LATENCY, 9), (LATENCY + 1, 7), (LATENCY + 1, 19),
         (RESIDENT // 4 * 3, 7), (RESIDENT // 4 * 3 + 1, 7), (RESIDENT // 4 * 3 + 1, 8), (RESIDENT, 5), (RESIDENT, 32),
         (RESIDENT + 1, 6), (FEW, 2), (FEW + 1, 1), (FEW + 1, 11)]


@pytest.mark.parametrize("length,k", EDGES)
@pytest.mark.parametrize("begin", [0, 1, 6])
def test_step_and_staged_step_at_shape_edges(length, k, begin):
    n = begin + length + 3
    case = DeviceCase(n, k, seed=length % 97 + k)
    e = begin + length
    S = case.gpu_sqnorm(begin, e)
    c = O.clip_coef(O.grad_sqnorm(case.h_g, begin, e), HP.max_grad_norm)
    want = case.oracle_step(HP, c, begin, e)
    before = case.clone_states()
    got = case.clone_states()
    gs.gs_accum_adamw(*got, case.grads, begin, e, HP, case.sq)
    check(got, want, begin, e, f"step S={S}")
    untouched(got, before, begin, e)
    acc = torch.zeros(n, dtype=torch.float32, device=DEV)
    for j, g in enumerate(case.grads):
        gs.gs_accum_add(acc, g, j == 0, begin, e)
    staged = case.clone_states()
    gs.gs_adamw_from_acc(*staged, acc, begin, e, HP, case.sq)
    for a, b in zip(got, staged):
        assert torch.equal(a, b)                 # same sum, same update: same bits


@pytest.mark.parametrize("k", [1, 2, 3, 9, 32])
@pytest.mark.parametrize("staged", [False, True])
def test_every_cut_of_short_ranges(k, staged):
    """Begins and ends at every offset within a group, with and without whole groups between them: the
    elements that a range end cuts off a group are stepped on their own."""
    n = 160
    case = DeviceCase(n, k, seed=k)
    case.sq.fill_(4.0)
    c = O.clip_coef(4.0, HP.max_grad_norm)
    full = case.oracle_step(HP, c)
    acc = torch.zeros(n, dtype=torch.float32, device=DEV)
    for j, g in enumerate(case.grads):
        gs.gs_accum_add(acc, g, j == 0, 0, n)
    for b in list(range(0, 9)) + [126, 127, 128, 129]:
        for e in [b + 1, b + 2, b + 3, b + 5, b + 8, 130, 133, n - 1, n]:
            if e <= b or e > n:
                continue
            got = case.clone_states()
            if staged:
                gs.gs_adamw_from_acc(*got, acc, b, e, HP, case.sq)
            else:
                gs.gs_accum_adamw(*got, case.grads, b, e, HP, case.sq)
            check(got, full, b, e, f"[{b},{e})")
            untouched(got, (case.p, case.m, case.v, case.w), b, e)


# (with the smallest workspace, which holds a partial per 256 elements up to 67 M: test_gpu_kernels.py has
# longer ranges with both workspaces)
@pytest.mark.parametrize("length,k", EDGES + [(RESIDENT, 2), (FEW, 16), (FEW + 1, 12)])
def test_speculative_step_at_shape_edges(length, k):
    begin, n = 5, length + 9
    case = DeviceCase(n, k, seed=length % 89 + k)
    e = begin + length
    want = case.oracle_step(HP, 1.0, begin, e)
    out = [torch.full((n,), 7.0, device=DEV) for _ in range(3)] + [torch.zeros_like(case.w)]
    before = [x.clone() for x in out]
    case.sq.fill_(float("nan"))                  # overwritten, not added to
    gs.gs_accum_adamw_spec(case.p, case.m, case.v, *out, case.grads, begin, e, HP, case.sq, case.ws)
    check(out, want, begin, e, "spec")
    untouched(out, before, begin, e)
    S = O.grad_sqnorm(case.h_g, begin, e)
    # every square is exact in fp64; the oracle adds the `length` non-negative terms one after another, which
    # is within length * 2^-53 of the exact sum (the kernel's tree is far closer)
    assert abs(float(case.sq.item()) - S) <= max(length * 2.0 ** -53, 1e-13) * S


@pytest.mark.parametrize("k", [8, 9, 10, 11, 13, 14, 15])
@pytest.mark.parametrize("length", [FEW + 1, 80_000_001])
def test_speculative_step_leftover_streams(length, k):
    """Batches of four streams and 0 to 3 left over, in the shapes of long ranges: the step's own bits (c = 1)
    and the norm's value."""
    b, e = 1, 1 + length
    case = DeviceCase(e + 2, k, seed=k, keep_host=False)
    ws = torch.empty(gs.gs_sqnorm_workspace_bytes_for(length), dtype=torch.uint8, device=DEV)
    want = case.clone_states()
    gs.gs_accum_adamw(*want, case.grads, b, e, HP, None)
    S = case.gpu_sqnorm(b, e)
    out = [x.clone() for x in (case.p, case.m, case.v)] + [torch.zeros_like(case.w)]
    gs.gs_accum_adamw_spec(case.p, case.m, case.v, *out, case.grads, b, e, HP, case.sq, ws)
    for a, w in zip(out, want):
        assert torch.equal(a, w)
    assert abs(float(case.sq.item()) - S) <= 1e-12 * S           # two fp64 trees over exact squares


# the norm's lines: one workgroup | many, and the sizes where the workgroups change; each with a range that
# ends inside a group and one that does not
NORM_SIZES = [1, 3, 4096, 4097, 16384, 16385, (1 << 20), (1 << 20) + 1, (1 << 21) + 2, (1 << 22) + 1, (1 << 23) + 3]


@pytest.mark.parametrize("length", NORM_SIZES)
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 16, 23])
@pytest.mark.parametrize("begin", [0, 7])
def test_norms_at_shape_edges(length, k, begin):
    e = begin + length
    case = DeviceCase(e + 5, k, seed=length % 83 + k)
    tol = max(length * 2.0 ** -53, 1e-13)        # the oracle's serial fp64 sum, as above
    S = O.grad_sqnorm(case.h_g, begin, e)
    case.sq.fill_(float("nan"))
    got = case.gpu_sqnorm(begin, e)
    assert abs(got - S) <= tol * S
    assert abs(case.gpu_sqnorm(begin, e, accumulate=True) - 2 * got) <= 1e-15 * got
    acc = torch.full((case.n,), 3.0, device=DEV)
    gs.gs_grad_accum_sqnorm(case.grads, begin, e, acc, case.sq, case.ws)
    assert abs(float(case.sq.item()) - S) <= tol * S
    assert bool((acc[:begin] == 3.0).all()) and bool((acc[e:] == 3.0).all())
    case.sq.fill_(float("nan"))
    gs.gs_acc_sqnorm(acc, begin, e, case.sq, case.ws)
    assert abs(float(case.sq.item()) - S) <= tol * S
    case.sq.fill_(1.0)
    gs.gs_acc_sqnorm(acc, begin, begin, case.sq, case.ws)
    gs.gs_grad_sqnorm(case.grads, begin, begin, case.sq, case.ws, accumulate=True)
    assert float(case.sq.item()) == 0.0           # an empty range writes 0, or adds nothing


# the adding and the staged kernels' lines (2^19, 2^22, 2^23, 2^25) with the smallest workspace, as above
@pytest.mark.parametrize("length,k", [(1, 3), (LATENCY, 8), (LATENCY + 1, 5), ((1 << 22) + 2, 9), ((1 << 22) + 3, 2),
                                      ((1 << 23) + 1, 4), ((1 << 25) + 5, 8)])
def test_staged_and_adding_kernels_at_shape_edges(length, k):
    begin, e = 3, 3 + length
    case = DeviceCase(e + 2, k, seed=length % 79 + k, keep_host=False)
    want = torch.zeros(e - begin, dtype=torch.float32, device=DEV)
    for g in case.grads:
        want += g[begin:e].float()                # fp32, in order: the exact same sum
    S = float((want.double() ** 2).sum())
    for staged in (True, False):
        acc = torch.full((case.n,), 5.0, device=DEV)
        case.sq.fill_(float("nan"))
        if staged:
            gs.gs_grad_accum_sqnorm(case.grads, begin, e, acc, case.sq, case.ws)
        else:
            for j, g in enumerate(case.grads):
                last = j == k - 1
                gs.gs_accum_add(acc, g, j == 0, begin, e, case.sq if last else None, case.ws if last else None)
        assert torch.equal(acc[begin:e], want)
        assert bool((acc[:begin] == 5.0).all()) and bool((acc[e:] == 5.0).all())
        assert abs(float(case.sq.item()) - S) <= 1e-12 * S       # two fp64 trees over exact squares


@pytest.mark.parametrize("k", [1, 3, 6])
def test_norms_of_long_runs(k):
    """From 2^29 gradient elements (2^27 of the fp32 buffer) on a workgroup reads longer runs."""
    n = (1 << 29) + 1
    g = [torch.ones(n, dtype=torch.bfloat16, device=DEV)] * k          # one buffer k times: read only
    sq = torch.zeros(1, dtype=torch.float64, device=DEV)
    ws = torch.empty(gs.gs_sqnorm_workspace_bytes(), dtype=torch.uint8, device=DEV)
    gs.gs_grad_sqnorm(g, 1, n, sq, ws)
    assert float(sq.item()) == float(k * k * (n - 1))                   # whole numbers: exact in fp64
    acc = torch.full(((1 << 27) + 7,), 2.0, device=DEV)
    gs.gs_acc_sqnorm(acc, 3, acc.numel(), sq, ws)
    assert float(sq.item()) == 4.0 * (acc.numel() - 3)


@pytest.mark.parametrize("k", [2, 7, 8])
def test_largest_shape_equals_its_pieces(k):
    """From 2^27 elements on (the shallow shape up to 7 streams): bit for bit what the other shapes give
    over the range cut into pieces of every size class."""
    n = SERIAL + 3
    case = DeviceCase(n, k, seed=k, keep_host=False)
    case.gpu_sqnorm()
    whole, parts = case.clone_states(), case.clone_states()
    gs.gs_accum_adamw(*whole, case.grads, 0, n, HP, case.sq)
    cuts = [0, 77, LATENCY + 77, LATENCY + RESIDENT + 77, LATENCY + RESIDENT + FEW + 78, n // 2 + 1, n]
    for x, y in zip(cuts, cuts[1:]):
        gs.gs_accum_adamw(*parts, case.grads, x, y, HP, case.sq)
    for a, b in zip(whole, parts):
        assert torch.equal(a, b)


@pytest.mark.parametrize("k", [1, 8, 9])
def test_cu_budget_shapes_give_the_same_bits(k):
    """A stream on some of the CUs takes shapes of its own above 2^21 elements (and 2^25 for the staged
    norm): same bits as on all of them; the look-up works under capture."""
    n = (1 << 25) + 3
    case = DeviceCase(n, k, seed=k, keep_host=False)
    case.gpu_sqnorm()
    ws = torch.empty(gs.gs_sqnorm_workspace_bytes_for(n), dtype=torch.uint8, device=DEV)
    raw = gs.gs_cu_stream_create(64)
    try:
        results = []
        for stream in (None, raw):
            got = case.clone_states()
            acc = torch.zeros(n, dtype=torch.float32, device=DEV)
            out = [torch.zeros(n, device=DEV) for _ in range(3)] + [torch.zeros_like(case.w)]
            sq = torch.zeros(3, dtype=torch.float64, device=DEV)
            torch.cuda.synchronize()
            gs.gs_accum_adamw(*got, case.grads, 1, n, HP, case.sq, stream=stream)
            gs.gs_grad_accum_sqnorm(case.grads, 1, n, acc, sq[0:1], ws, stream=stream)
            gs.gs_adamw_from_acc(*got, acc, 1, n, HP, case.sq, stream=stream)
            gs.gs_accum_add(acc, case.grads[0], False, 1, n, sq[1:2], ws, stream=stream)
            gs.gs_accum_adamw_spec(case.p, case.m, case.v, *out, case.grads, 1, n, HP, sq[2:3], ws, stream=stream)
            torch.cuda.synchronize()
            results.append((*got, acc, *out, sq))
        for a, b in zip(results[0][:-1], results[1][:-1]):
            assert torch.equal(a, b)
        assert torch.allclose(results[0][-1], results[1][-1], rtol=1e-13, atol=0.0)     # fp64 trees of other shapes
    finally:
        gs.gs_cu_stream_destroy(raw)
    # the look-up of a stream's CUs under capture, on an ordinary stream
    got = case.clone_states()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gs.gs_accum_adamw(*got, case.grads, 1, n, HP, case.sq)
    want = case.clone_states()
    for _ in range(3):
        graph.replay()
        gs.gs_accum_adamw(*want, case.grads, 1, n, HP, case.sq)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)
