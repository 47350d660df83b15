"""The ways in which a kernel is given its arguments: addresses, or distances from p where everything lies near it."""
from __future__ import annotations

import pytest
import torch

from gpu_util import DEV, gs
from paper_2512_17570_amd import inputs as I

pytestmark = pytest.mark.gpu

B = 5                                        # begin of every range
LENGTHS = [1, 2, 3, 127, 130, 1001, 200_000, 267_000, 267_001, 312_001, 430_000, 430_001, 1 << 19, (1 << 19) + 1, 960_001, 1_200_000, 1_200_001, 3 << 19, (1 << 21) + 1, 5_000_000, 5_000_001]


def the_same(k, length, hp, sq, place=None):
    """A step in place against the same step out of place, which is always given addresses: the same bits."""
    n = B + length + 2
    new = place or (lambda name, like: like.clone())
    states = I.make_states(n, 11, DEV)
    grads = [new(f"g{j}", I.normal_f32(n, 1e-3, 9, j, DEV).to(torch.bfloat16)) for j in range(k)]
    want = [torch.zeros_like(x) for x in states] + [torch.zeros(n, dtype=torch.bfloat16, device=DEV)]
    gs.gs_accum_adamw_oop(*states, *want, grads, B, B + length, hp, sq)
    got = [new(name, x) for name, x in zip("pmv", states)] + [new("w", torch.zeros(n, dtype=torch.bfloat16, device=DEV))]
    gs.gs_accum_adamw(*got, grads, B, B + length, hp, sq)
    torch.cuda.synchronize()
    for name, x, y, was in zip("pmvw", got, want, [*states, torch.zeros(n, dtype=torch.bfloat16, device=DEV)]):
        assert torch.equal(x[B:B + length], y[B:B + length]), name
        assert torch.equal(x[:B], was[:B]) and torch.equal(x[B + length:], was[B + length:]), name


@pytest.mark.parametrize("k", range(1, 10))
@pytest.mark.parametrize("clip", ["clipped", "no norm", "max_grad_norm 0"])
def test_step_by_distances(k, clip):
    hp = gs.HParams(step=10, max_grad_norm=0.0 if clip == "max_grad_norm 0" else 0.1)
    sq = None if clip == "no norm" else torch.full((1,), 4.0, dtype=torch.float64, device=DEV)
    for length in LENGTHS:
        print(f"[near] k={k} {clip} length={length}", flush=True)
        the_same(k, length, hp, sq)


@pytest.mark.parametrize("far", ["nothing", "p", "m", "v", "w", "g0", "g7", "sq"])
@pytest.mark.parametrize("odd", [0, 16])
def test_step_with_one_array_far_away(far, odd):
    """Distances of up to 32 GB fit, longer ones only in units of 256 bytes; any array may lie farther than that, before or behind p."""
    gib = 1 << 30
    free = torch.cuda.mem_get_info()[0]
    if free < 60 * gib:
        pytest.skip("needs 44 GB")
    big = torch.empty(44 * gib, dtype=torch.uint8, device=DEV)
    at = {"near": 0}

    def place(name, like):
        nbytes = (like.numel() * like.element_size() + 255) // 256 * 256
        start = (42 * gib if name == far else at["near"]) + (odd if name in ("g3", far) else 0)
        if name != far:
            at["near"] += nbytes + 256
        t = big[start:start + like.numel() * like.element_size()].view(like.dtype)
        return t.copy_(like)

    sq = place("sq", torch.full((1,), 4.0, dtype=torch.float64, device=DEV))
    for length in (1, 1001, 300_001, 600_001):
        at["near"] = 256
        print(f"[far] {far} length={length}", flush=True)
        the_same(8, length, gs.HParams(step=10, max_grad_norm=0.1), sq, place)


@pytest.mark.parametrize("k", [1, 4, 5, 6, 7, 8, 9, 17])
def test_norm_with_each_table_of_streams(k):
    for length in (1, 3, 4095, 4096, 4097, 65536 // k, 65536 // k + 1, 16384, 16385, 100_001, (1 << 21) + 5):
        n = B + length + 2
        grads = [I.normal_f32(n, 1e-3, 9, j, DEV).to(torch.bfloat16) for j in range(k)]
        a = torch.zeros(length, dtype=torch.float32, device=DEV)
        for g in grads:
            a += g[B:B + length].float()
        want = float(a.double().square().sum())
        sq = torch.full((1,), 4.0, dtype=torch.float64, device=DEV)
        ws = torch.full((gs.gs_sqnorm_workspace_bytes(),), 0xff, dtype=torch.uint8, device=DEV)
        for accumulate in (False, True):
            gs.gs_grad_sqnorm(grads, B, B + length, sq, ws, accumulate=accumulate)
            got = float(sq.item())
            # two fp64 trees over exact squares (deeper than 2^-40 of the sum needs more than 2^12 additions in a chain)
            assert abs(got - want * (2 if accumulate else 1)) <= 1e-12 * want, (k, length, accumulate)


@pytest.mark.parametrize("k", [5, 6, 7, 8, 9, 10, 13, 15])
@pytest.mark.parametrize("begin", [0, 5, 1021, 1024, 3000, 4093])
def test_captured_norm_of_a_few_tiles_has_the_same_bits(k, begin):
    """Captured, such a range is read by one workgroup less often than called one after the other."""
    top = 65536 // k
    lengths = sorted({4097, 40960 // k, 40960 // k + 1, top, top + 1, 8200 - begin, 8192, (4097 + top) // 2, 4096 * 3 - begin} & set(range(4097, top + 2)))
    n = begin + top + 3
    grads = [I.normal_f32(n, 1e-3, 9, j, DEV).to(torch.bfloat16) for j in range(k)]
    sq, eager = (torch.zeros(len(lengths), dtype=torch.float64, device=DEV) for _ in range(2))
    gs.gs_grad_sqnorm_noalloc(grads, begin, n, sq)
    ws = torch.full((gs.gs_sqnorm_workspace_bytes(),), 0xff, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for i, length in enumerate(lengths):
            gs.gs_grad_sqnorm_noalloc(grads, begin, begin + length, sq[i:])
    for times in (1, 3, 5):
        for g in grads:
            g.mul_(times)
        for i, length in enumerate(lengths):
            gs.gs_grad_sqnorm(grads, begin, begin + length, eager[i:], ws)
        torch.cuda.synchronize()
        sq.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(sq, eager), (lengths, (sq - eager).tolist())
