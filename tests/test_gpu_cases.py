"""The workloads of perf/cases.py against their 64-bit results with a bound for each output.

The one tolerance that a case states there is set by the bf16 weight, which a last bit of p next to a tie moves by
2^-8 of its value; it lets a step without weight decay (1e-6 of p) pass.  Here p, m, v, the fp32 sum and the norm
have bounds of their own, element by element, and the planted mistakes have to exceed them."""
from __future__ import annotations

import pytest
import torch

from perf import cases as C

pytestmark = pytest.mark.gpu

# every path at its listed size, or at a ragged million elements where that is a large layer
CASES = [c if c["n"] <= 13_000_000 else dict(c, n=8_000_003 if c["path"] == "shard" else 1_000_003) for c in C.listed()]
SEED = 5


def excess(got, want, p0, m0):
    """The largest error of each output in units of its bound; p0, m0: the states before the step."""
    out = {}
    for name, w in want.items():
        g = got[name].to(torch.float64).to(w.device)
        if name == "sq":             # fp32 sums of k terms, squared and summed in fp64: rounding errors of 2^-24 average out
            bound = 1e-8 * w
        elif name == "w":            # one bf16 rounding of p, and p's own last bits next to a tie: at most an ulp, 2^-7
            bound = 2.0 ** -7 * w.abs() + 1e-9
        elif name in ("m", "v", "acc"):
            # k adds (the sum), then two products and an add, each within 2^-24: with cancellation that is relative to
            # the operands, of which the gradients' part is at most 32 * 0.1 (outliers) * 0.1
            bound = 4e-7 * w.abs() + {"m": 2e-8, "v": 1e-10, "acc": 2e-6}[name]
        else:
            # p = p0 * decay - s: the product and the difference round within 2^-24 of p or s; s = step_size * m / d comes of
            # about ten roundings (16 * 2^-24 = 1e-6 of s), and where m cancels, three of them are relative to m's operands
            m, step = want["m"], p0 * (1.0 - C.LR * C.DECAY) - w
            cancelled = (0.9 * m0).abs() + (m - 0.9 * m0).abs()
            bound = 4e-7 * w.abs() + step.abs() * (1e-6 + 2e-7 * cancelled / m.abs().clamp_min(1e-30)) + 1e-12
        out[name] = float(((g - w).abs() / bound).max())
    return out


@pytest.mark.parametrize("case", CASES, ids=[c["name"] for c in CASES])
def test_case_within_each_outputs_bound(case, monkeypatch):
    before = C.prepare(dict(case, path="shard" if case["path"] == "shard" else "resident"), SEED)
    p0, m0 = before["p"].double(), before["m"].double()
    if case["path"] == "shard":
        p0, m0 = (x[before["b"]:before["e"]] for x in (p0, m0))
    got = C.run(C.prepare(case, SEED))
    torch.cuda.synchronize()
    worst = excess(got, C.exact(case, SEED), p0, m0)
    print(case["name"], {k: round(v, 3) for k, v in worst.items()}, flush=True)
    assert max(worst.values()) <= 1.0, worst
    # expected values with a planted mistake are told apart
    with monkeypatch.context() as mp:
        mp.setattr(C, "DECAY", 0.0)
        assert excess(got, C.exact(case, SEED), p0, m0)["p"] > 1.0
    if case["path"] == "groups":
        with monkeypatch.context() as mp:
            mp.setattr(C, "NO_DECAY", set())
            assert excess(got, C.exact(case, SEED), p0, m0)["p"] > 1.0
    with monkeypatch.context() as mp:
        mp.setattr(C, "BETA2", C.BETA2 - 1e-5)
        assert max(excess(got, C.exact(case, SEED), p0, m0)[x] for x in "pv") > 1.0
