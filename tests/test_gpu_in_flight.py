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
