"""The ways in which a kernel is given its arguments."""
from __future__ import annotations

import pytest
import torch

from gpu_util import DEV, gs
from paper_2512_17570_amd import inputs as I

pytestmark = pytest.mark.gpu

B = 5                                        # begin of every range


@pytest.mark.parametrize("k", [1, 4, 5, 7, 8, 9, 17])
def test_norm_with_each_table_of_streams(k):
    for length in (1, 3, 4095, 4096, 16384, 16385, 100_001, (1 << 21) + 5):
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
