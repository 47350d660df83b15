"""GPU tests of the shapes that bound how many workgroups a CU holds, at the lengths and stream counts where they
begin and end: the same bits as the range taken in pieces short enough for the shapes of small ranges, which
test_gpu_shapes.py holds against the oracle."""
from __future__ import annotations

import pytest
import torch

from gpu_util import DEV, DeviceCase, gs

pytestmark = pytest.mark.gpu

HP = gs.HParams(step=10, max_grad_norm=0.1)
PIECE = 1 << 19


def in_pieces(call, b, e):
    for x in range(b, e, PIECE):
        call(x, min(e, x + PIECE))


# the step's lines: 2^21 elements; five and eight streams; 2^25 elements from eight streams on
@pytest.mark.parametrize("length,k", [((1 << 21) + 1, 4), ((1 << 21) + 1, 5), ((1 << 25), 8), ((1 << 25) + 1, 8), ((1 << 25) + 1, 7),
                                      ((1 << 25) + 3, 13), ((1 << 25) + 2, 1)])
@pytest.mark.parametrize("begin", [0, 3])
def test_step_has_the_bits_of_short_ranges(length, k, begin):
    case = DeviceCase(begin + length + 2, k, seed=k, keep_host=False)
    b, e = begin, begin + length
    case.sq.fill_(4.0)
    got, want = case.clone_states(), case.clone_states()
    gs.gs_accum_adamw(*got, case.grads, b, e, HP, case.sq)
    in_pieces(lambda x, y: gs.gs_accum_adamw(*want, case.grads, x, y, HP, case.sq), b, e)
    for g, w in zip(got, want):
        assert torch.equal(g, w)
    acc = torch.zeros(begin + length + 2, dtype=torch.float32, device=DEV)
    for j, g in enumerate(case.grads):
        gs.gs_accum_add(acc, g, j == 0, b, e)
    staged = case.clone_states()
    gs.gs_adamw_from_acc(*staged, acc, b, e, HP, case.sq)
    for g, w in zip(staged, want):
        assert torch.equal(g, w)


# 7 M elements, below five streams and from five on; 2^24 and 2^26 elements with streams left over; whole batches of eight
@pytest.mark.parametrize("length,k", [(7_000_000, 4), (7_000_001, 4), (7_000_000, 5), (7_000_001, 5), ((1 << 24), 9), ((1 << 24) + 1, 9),
                                      ((1 << 26) + 1, 10), ((1 << 24) + 1, 21), ((1 << 25), 16), ((1 << 25) + 1, 16), (8_000_000, 24), (8_000_000, 32)])
def test_step_lines_by_streams(length, k):
    test_step_has_the_bits_of_short_ranges(length, k, 1)


# (length, k, workspace): written through or not up to 7 M elements; a partial per 256 or 512 elements; runs
@pytest.mark.parametrize("length,k,ws", [(1 << 21, 7, "min"), ((1 << 21) + 1, 7, "min"), (7_000_000, 2, "min"), (7_000_001, 2, "min"),
                                         (7_000_001, 9, "min"), (66_000_000, 5, "min"), (68_000_000, 4, "min"), (68_000_000, 5, "min"),
                                         (135_000_000, 3, "min"), (135_000_000, 6, "full"), (1 << 28, 2, "min"), ((1 << 28) + 1, 3, "min")])
def test_speculative_pass_has_the_bits_of_the_step(length, k, ws):
    b, e = 3, 3 + length
    case = DeviceCase(e + 1, k, seed=k, keep_host=False)
    space = torch.empty(gs.gs_sqnorm_workspace_bytes() if ws == "min" else gs.gs_sqnorm_workspace_bytes_for(length), dtype=torch.uint8, device=DEV)
    want = case.clone_states()
    gs.gs_accum_adamw(*want, case.grads, b, e, HP, None)
    S = case.gpu_sqnorm(b, e)
    out = [x.clone() for x in (case.p, case.m, case.v)] + [case.w.clone()]
    gs.gs_accum_adamw_spec(case.p, case.m, case.v, *out, case.grads, b, e, HP, case.sq, space)
    for g, w in zip(out, want):
        assert torch.equal(g, w)
    # two orders of adding `length` non-negative fp64 terms in trees no deeper than 2^13 sequential additions a partial
    assert abs(float(case.sq.item()) - S) <= 2 * (1 << 13) * 2.0 ** -53 * S


# the runs of the norm of one stream (2^23, 2^26, 2^28 elements) and of three, against fp64 sums
@pytest.mark.parametrize("length,k", [((1 << 23) - 1, 1), (1 << 23, 1), (1 << 26, 1), ((1 << 28) + 1, 1), ((1 << 22) + 1, 3), ((1 << 25) + 7, 3)])
def test_norm_runs(length, k):
    b, e = 3, 3 + length
    case = DeviceCase(e + 2, k, seed=k, keep_host=False)
    S = case.gpu_sqnorm(b, e)
    want = 0.0
    for x in range(b, e, 1 << 24):
        a = torch.zeros(min(e, x + (1 << 24)) - x, dtype=torch.float32, device=DEV)
        for g in case.grads:
            a += g[x:x + a.numel()].float()
        want += float(a.double().square().sum())
    # as above: both sides' partials are trees of at most 2^13 sequential additions
    assert abs(S - want) <= 2 * (1 << 13) * 2.0 ** -53 * want


@pytest.mark.parametrize("length", [(1 << 22) + 1, (64 << 20) + 3, (64 << 20) + 1021])
def test_later_micro_batches_written_through_and_cached(length):
    """Both sides of the last 256 MB of the buffer, whose stores stay in the cache."""
    b, e = 5, 5 + length
    case = DeviceCase(e + 3, 2, seed=3, keep_host=False)
    acc = torch.full((e + 3,), 9.0, dtype=torch.float32, device=DEV)
    gs.gs_accum_add(acc, case.grads[0], True, b, e)
    gs.gs_accum_add(acc, case.grads[1], False, b, e)
    assert torch.equal(acc[b:e], case.grads[0][b:e].float() + case.grads[1][b:e].float())
    assert bool((acc[:b] == 9.0).all()) and bool((acc[e:] == 9.0).all())


@pytest.mark.parametrize("cus", [0, 16, 32, 60, 64, 128, 192])
@pytest.mark.parametrize("n,k", [(130, 2), (100_003, 9), (700_001, 8), ((1 << 23) + 3, 3)])
def test_step_on_host_memory_by_cus(n, k, cus):
    """Each number of workgroups that a CU is given over the link, and none: the resident step's bits."""
    case = DeviceCase(n, k, seed=k, keep_host=False)
    case.sq.fill_(4.0)
    host = []
    for x in (case.p, case.m, case.v):
        h = torch.empty(n, dtype=torch.float32, pin_memory=True)
        h.copy_(x)
        host.append(h)
    want = case.clone_states()
    gs.gs_accum_adamw(*want, case.grads, 0, n, HP, case.sq)
    ctx = gs.gs_stream_ctx_create_inplace(cus)
    w = torch.zeros_like(case.w)
    gs.gs_stream_layer_step(ctx, *host, w, case.grads, n, HP, case.sq)
    gs.gs_stream_ctx_sync(ctx)
    gs.gs_stream_ctx_destroy(ctx)
    for h, x in zip(host + [w.cpu()], want):
        assert torch.equal(h, x.cpu())
