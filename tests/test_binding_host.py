"""When the native marshalling (_gs_call) asks torch whether this process may use the GPU at all: a child that was forked after its
parent used the GPU may not, and its calls are left to the general reading, which raises torch's own error.  On the CPU: tensors
that say they are on a GPU, over host memory, and an entry point that only counts its calls."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MODULE = os.path.join(ROOT, "paper_2512_17570_amd", "_gs_call.so")

SCRIPT = """
import ctypes, importlib.util, os, sys
import torch

bad, fork_first, fork_after = (x == "1" for x in sys.argv[2:])
asked, called = [], []

def in_bad_fork():
    asked.append(1)
    return bad

def on_gpu(n, dtype, size):
    host = ctypes.create_string_buffer(n * size)
    dev = torch.device("cuda", 0)
    storage = torch._C._construct_storage_from_data_pointer(ctypes.addressof(host), dev, n * size)
    meta = dict(size=(n,), stride=(1,), dtype=dtype, device=dev, storage_offset=0, nbytes=n * size, data_ptr=ctypes.addressof(host))
    return torch._C._construct_CUDA_Tensor_From_Storage_And_Metadata(meta, storage), host

@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p,
                  ctypes.c_size_t, ctypes.c_void_p)
def entry(*args):
    called.append(args)
    return 0

class HParams:
    pass

def in_child():
    pid = os.fork()
    if pid:
        os._exit(os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]))

if fork_first:
    in_child()
spec = importlib.util.spec_from_file_location("_gs_call", sys.argv[1])
call = importlib.util.module_from_spec(spec)
spec.loader.exec_module(call)
call.setup(*[ctypes.cast(entry, ctypes.c_void_p).value] * 9, HParams, in_bad_fork)
if fork_after:
    in_child()
acc, keep = on_gpu(64, torch.float32, 4)
sq, keep_sq = on_gpu(1, torch.float64, 8)
for stream in (None, None, 0x5000):
    asked.clear(), called.clear()
    st = call.acc_sqnorm(acc, 0, 64, sq, sq, None, False, stream)
    print(len(asked), len(called), st, flush=True)
os._exit(0)
"""


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("fork", ["never", "before the set-up", "after the set-up"])
def test_torch_is_asked_where_the_gpu_may_not_be_usable(bad, fork):
    args = [str(int(x)) for x in (bad, fork == "before the set-up", fork == "after the set-up")]
    r = subprocess.run([sys.executable, "-c", SCRIPT, MODULE, *args], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    *current, given = [tuple(x.split()) for x in r.stdout.strip().split("\n")]
    for asked, called, status in current:
        # the parent of a child that imports the binding itself is known by torch only: what torch says at the set-up is the sign
        assert int(asked) == (bad or fork == "after the set-up"), r.stdout
        if bad:
            assert (called, status) == ("0", "None")
    assert given == ("0", "1", "0")                # a stream that is given is the caller's own
