"""GPU tests of the binding's native marshalling (_gs_call): for every form of argument that it takes, the same
results as the general reading in gs.py; every other form is left to that reading, which accepts or refuses it
as it does on its own."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_util import DEV, DeviceCase, gs

pytestmark = pytest.mark.gpu

HP = gs.HParams(step=10, max_grad_norm=0.1)
N, K = 5003, 3


class General:
    """_gs_call that takes no call, so that the general reading takes them all."""

    def __getattr__(self, name):
        return lambda *args: None


class Counting:
    def __init__(self, call):
        self.call, self.taken = call, 0

    def __getattr__(self, name):
        def f(*args):
            st = getattr(self.call, name)(*args)
            self.taken += st is not None
            return st
        return f


def both(monkeypatch, use):
    """use(case): its result or exception, natively and in the general way; and the calls taken natively."""
    out = []
    for call in (Counting(gs._call), General()):
        case = DeviceCase(N, K, seed=5)
        case.sq.fill_(2.0)
        case.acc = case.grads[0].float()
        with monkeypatch.context() as mp:
            mp.setattr(gs, "_call", call)
            try:
                r = use(case)
            except Exception as err:  # noqa: BLE001  its type and text are what is compared
                r = (type(err), str(err))
        torch.cuda.synchronize()
        out.append((r, [x.clone() for x in (case.p, case.m, case.v, case.w, case.sq, case.acc)], getattr(call, "taken", 0)))
    (r, state, taken), (want, want_state, _) = out
    assert r == want
    for a, b in zip(state, want_state):
        assert torch.equal(a, b)
    return r, taken


def step(c, p=None, grads=None, begin=1, end=N - 1, hp=HP, sq=0, **kw):
    return gs.gs_accum_adamw(c.p if p is None else p, c.m, c.v, c.w, c.grads if grads is None else grads, begin, end, hp,
                             c.sq if sq == 0 else sq, **kw)


def spec(c, **kw):
    out = [torch.zeros_like(c.p) for _ in range(3)]
    st = gs.gs_accum_adamw_spec(c.p, c.m, c.v, *out, c.w, c.grads, 2, N, HP, c.sq, c.ws, **kw)
    c.p, c.m, c.v = out
    return st


def oop(c):
    out = [torch.zeros_like(c.p) for _ in range(3)]
    st = gs.gs_accum_adamw_oop(c.p, c.m, c.v, *out, c.w, c.grads, 2, N, HP, c.sq)
    c.p, c.m, c.v = out
    return st


TAKEN = [
    lambda c: step(c),
    lambda c: step(c, grads=tuple(c.grads)),
    lambda c: step(c, p=torch.nn.Parameter(c.p)),
    lambda c: step(c, sq=None),
    lambda c: step(c, k=K),
    lambda c: step(c, stream=torch.cuda.current_stream()),
    lambda c: step(c, stream=torch.cuda.current_stream().cuda_stream),
    lambda c: step(c, begin=7, end=7),
    lambda c: step(c, begin=9, end=3, check=False),
    lambda c: step(c, begin=-1, check=False),
    lambda c: step(c, begin=-1),
    lambda c: step(c, hp=gs.HParams(step=0)),
    lambda c: step(c, hp=gs.HParams(lr=float("nan")), check=False),
    lambda c: step(c, hp=gs.HParams(lr=1e300), check=False),
    lambda c: step(c, grads=[g[3:] for g in c.grads], end=N - 4, check=False),        # misaligned addresses
    lambda c: step(c, p=c.p[4:], end=N - 5),
    lambda c: gs.gs_grad_sqnorm(c.grads, 0, N, c.sq, c.ws),
    lambda c: gs.gs_grad_sqnorm(c.grads, 0, N, c.sq, c.ws, accumulate=True),
    lambda c: gs.gs_grad_sqnorm(c.grads, 0, N, c.sq, c.ws, workspace_bytes=100, check=False),
    lambda c: gs.gs_grad_sqnorm(c.grads, 0, N, c.sq, None, check=False),
    lambda c: gs.gs_grad_sqnorm_noalloc(c.grads, 3, N, c.sq),
    lambda c: gs.gs_grad_accum_sqnorm(c.grads, 3, N, c.acc, c.sq, c.ws),
    lambda c: gs.gs_accum_add(c.acc, c.grads[1], False, 1, N),
    lambda c: gs.gs_accum_add(c.acc, c.grads[1], True, 1, N, c.sq, c.ws),
    lambda c: gs.gs_acc_sqnorm(c.acc, 1, N, c.sq, c.ws, accumulate=True),
    lambda c: gs.gs_adamw_from_acc(c.p, c.m, c.v, c.w, c.acc, 1, N, HP, c.sq),
    lambda c: spec(c), lambda c: spec(c, accumulate=True), lambda c: oop(c),
]


@pytest.mark.parametrize("i", range(len(TAKEN)))
def test_taken_natively_with_the_same_result(monkeypatch, i):
    _, taken = both(monkeypatch, TAKEN[i])
    assert taken == 1


class OwnStruct(gs.HParams):
    def c_struct(self):
        return gs.HParams(step=3).c_struct()


class Sub(torch.Tensor):
    pass


def in_mode(c):
    with torch.overrides.BaseTorchFunctionMode():
        return step(c)


LEFT = [
    lambda c: step(c, hp=OwnStruct(step=10)),
    lambda c: step(c, hp=HP.c_struct()),
    lambda c: step(c, hp=None, check=False),
    lambda c: step(c, hp=gs.HParams(lr=1)),
    lambda c: step(c, hp=gs.HParams(step=2.5)),
    lambda c: step(c, hp=gs.HParams(step=1 << 40), check=False),
    lambda c: step(c, begin=True),
    lambda c: step(c, begin=np.int64(1)),
    lambda c: step(c, end=1 << 70),
    lambda c: step(c, end=N + 1),
    lambda c: step(c, p=c.p[:100]),
    lambda c: step(c, p=c.p.double()),
    lambda c: step(c, p=torch.empty(2 * N, device=DEV)[::2]),
    lambda c: step(c, p=c.p.as_subclass(Sub)),
    lambda c: step(c, p=c.p.data_ptr()),
    lambda c: step(c, p="p"),
    lambda c: step(c, grads=[]),
    lambda c: step(c, grads=[c.grads[0]] * 33, check=False),
    lambda c: step(c, grads=[g.data_ptr() for g in c.grads]),
    lambda c: step(c, grads=torch.stack(c.grads)),
    lambda c: step(c, grads=[c.grads[0], c.grads[1].float()]),
    lambda c: step(c, k=2),
    lambda c: step(c, sq=c.sq.data_ptr()),
    lambda c: step(c, stream="s"),
    lambda c: gs.gs_grad_sqnorm(c.grads, 0, N, c.sq, c.ws.data_ptr(), workspace_bytes=c.ws.numel()),
    lambda c: gs.gs_grad_sqnorm(c.grads, 0, N, c.sq, c.ws, accumulate=1),
    lambda c: gs.gs_accum_add(c.acc, c.grads[1], 0, 1, N),
    in_mode,
]


@pytest.mark.parametrize("i", range(len(LEFT)))
def test_left_to_the_general_reading(monkeypatch, i):
    _, taken = both(monkeypatch, LEFT[i])
    assert taken == 0


def test_native_part_is_loaded():
    assert gs._call.__file__.endswith("_gs_call.so")


def test_current_stream_is_the_callers(monkeypatch):
    """A side stream that is current at the call gets the launch: it is ordered behind what that stream holds."""
    side = torch.cuda.Stream()
    case = DeviceCase(N, K, seed=2)
    want = case.clone_states()
    case.sq.fill_(4.0)
    gs.gs_accum_adamw(*want, case.grads, 0, N, HP, case.sq)
    got = case.clone_states()
    g0 = case.grads[0].clone()
    case.grads[0].zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(2_000_000)
        case.grads[0].copy_(g0)
        gs.gs_accum_adamw(*got, case.grads, 0, N, HP, case.sq)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)
