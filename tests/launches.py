"""Builds the library's launchers for the host only, against a HIP runtime that records launches instead of
making them (hipmock/launch_recorder.cpp), and reads back what each call would have launched."""
from __future__ import annotations

import ctypes
import os
import re
import subprocess
from dataclasses import dataclass

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_17570_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = [os.path.join(CSRC, f) for f in ("gs_kernels.hip", "gs_api.hip", "gs_noalloc.hip")]

MIN_WS = 2_098_176                      # gs_sqnorm_workspace_bytes(): 262144 partials and 128 slices
FULL = -1                               # gs_sqnorm_workspace_bytes_for(range)
# far-apart addresses: never dereferenced, and no two arrays may overlap over the longest range used here
P, M, V, PO, MO, VO, W, ACC, SQ, WS = ((i + 1) << 50 for i in range(10))
GRADS = [(64 + j) << 42 for j in range(32)]
STREAM = 0x5000


class _Launch(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_char * 128), ("grid", ctypes.c_uint64), ("block", ctypes.c_uint64),
                ("stream", ctypes.c_uint64), ("lds", ctypes.c_uint64), ("begin", ctypes.c_int64), ("end", ctypes.c_int64), ("extra", ctypes.c_int64),
                ("keep_from", ctypes.c_int64), ("partials", ctypes.c_uint64), ("out", ctypes.c_uint64),
                ("status", ctypes.c_int32)]


class HP(ctypes.Structure):
    _fields_ = [(x, ctypes.c_float) for x in ("lr", "beta1", "beta2", "eps", "wd", "max_norm")] + [("step", ctypes.c_int32)]


@dataclass
class Launch:
    kernel: str            # without its template arguments
    targs: tuple           # those, as numbers (false/true as 0/1)
    grid: int
    block: int
    lds: int               # bytes of LDS asked for beyond what the kernel itself declares
    begin: int
    end: int
    extra: int
    keep_from: int
    partials: int
    out: int
    status: int

    @property
    def name(self):
        return f"{self.kernel}<{','.join(map(str, self.targs))}>"


def parse_name(name: str):
    m = re.fullmatch(r"(\w+)(?:<(.*)>)?", name)
    args = [{"false": 0, "true": 1}.get(x.strip(), x.strip()) for x in (m[2] or "").split(",") if x.strip()]
    return m[1], tuple(int(x) for x in args)


def build(out_dir: str):
    """The recorder library, loaded."""
    objs = []
    for src in SOURCES + [os.path.join(ROOT, "tests", "hipmock", "launch_recorder.cpp")]:
        o = os.path.join(out_dir, os.path.basename(src) + ".o")
        subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-fuse-cuid=none", "-std=c++17", "-O1",
                        "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", o],
                       check=True, capture_output=True, text=True)
        objs.append(o)
    so = os.path.join(out_dir, "liblaunches.so")
    # -z defs: nothing may come from the real runtime; -Bsymbolic: not even if it is loaded in this process;
    # -z muldefs: each object carries an empty mark of its own under the same name
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-Wl,-z,muldefs", *objs, "-o", so], check=True, capture_output=True, text=True)
    lib = ctypes.CDLL(so)
    lib.gs_sqnorm_workspace_bytes_for.restype = ctypes.c_size_t
    lib.gs_sqnorm_workspace_bytes_for.argtypes = [ctypes.c_int64]
    lib.rec_mask_query.restype = ctypes.c_uint64
    return lib


class Recorder:
    def __init__(self, lib):
        self.lib = lib
        self.hp = HP(1e-4, 0.9, 0.999, 1e-8, 0.01, 1.0, 10)

    def kernels(self):
        buf = ctypes.create_string_buffer(1 << 16)
        self.lib.rec_kernels(buf, len(buf))
        return sorted(buf.value.decode().split("\n")[:-1])

    def call(self, entry: str, k: int, begin: int, end: int, ws: int = MIN_WS, accumulate: int = 0, first: int = 0,
             cus: int = 256, stream: int = STREAM):
        """(status, launches, stream handles whose CUs were asked for, bytes of workspace handed over)"""
        i64, vp, hp = ctypes.c_int64, ctypes.c_void_p, ctypes.byref(self.hp)
        lib = self.lib
        lib.rec_reset(cus)
        tab = (vp * k)(*GRADS[:k]) if k else None
        b, e, s = i64(begin), i64(end), vp(stream)
        wsb = lib.gs_sqnorm_workspace_bytes_for(end - begin) if ws == FULL else ws
        norm = (vp(SQ), accumulate, vp(WS), ctypes.c_size_t(wsb), s)
        st = {
            "step": lambda: lib.gs_accum_adamw(vp(P), vp(M), vp(V), vp(W), tab, k, b, e, hp, vp(SQ), s),
            "oop": lambda: lib.gs_accum_adamw_oop(vp(P), vp(M), vp(V), vp(PO), vp(MO), vp(VO), vp(W), tab, k, b, e, hp, vp(SQ), s),
            "from_acc": lambda: lib.gs_adamw_from_acc(vp(P), vp(M), vp(V), vp(W), vp(ACC), b, e, hp, vp(SQ), s),
            "host_step": lambda: lib.rec_step_on_host_memory(k, b, e, s),
            "spec": lambda: lib.gs_accum_adamw_spec(vp(P), vp(M), vp(V), vp(PO), vp(MO), vp(VO), vp(W), tab, k, b, e, hp, *norm),
            "norm": lambda: lib.gs_grad_sqnorm(tab, k, b, e, *norm),
            "noalloc": lambda: lib.gs_grad_sqnorm_noalloc(tab, k, b, e, vp(SQ), accumulate, s),
            "staged": lambda: lib.gs_grad_accum_sqnorm(tab, k, b, e, vp(ACC), *norm),
            "acc_norm": lambda: lib.gs_acc_sqnorm(vp(ACC), b, e, *norm),
            "add": lambda: lib.gs_accum_add(vp(ACC), vp(GRADS[0]), first, b, e, None, 0, None, ctypes.c_size_t(0), s),
            "add_norm": lambda: lib.gs_accum_add(vp(ACC), vp(GRADS[0]), first, b, e, *norm),
        }[entry]()
        out = []
        for i in range(lib.rec_count()):
            r = _Launch()
            lib.rec_get(i, ctypes.byref(r))
            kernel, targs = parse_name(r.kernel.decode())
            out.append(Launch(kernel, targs, r.grid, r.block, r.lds, r.begin, r.end, r.extra, r.keep_from, r.partials, r.out, r.status))
        asked = [lib.rec_mask_query(i) for i in range(lib.rec_mask_queries())]
        return st, out, asked, wsb


WORK = ("k_accum_adamw", "k_accum_adamw_spec", "k_grad_sqnorm", "k_grad_accum_sqnorm", "k_accum_add", "k_acc_sqnorm")


def shape(l: Launch):
    """(lanes, elements per lane, tiles a workgroup takes at a time) of a kernel, from its template arguments."""
    t = l.targs
    return {"k_accum_adamw": lambda: (t[0], t[1], 1), "k_accum_adamw_spec": lambda: (t[0], t[1], 1),
            "k_grad_sqnorm": lambda: (t[2], 4, t[1]), "k_grad_accum_sqnorm": lambda: (t[0], t[1], 1),
            "k_accum_add": lambda: (t[2], t[3], 1), "k_acc_sqnorm": lambda: (t[1], 4, t[0])}[l.kernel]()


def check(entry, launches, begin, end, wsb):
    """Every launch is one the runtime accepts; the work launches together take exactly [begin,end); every
    workgroup's partial lies in the workspace, and the folds read exactly what was written."""
    assert launches
    work = [l for l in launches if l.kernel in WORK]
    at = begin
    for l in work:
        assert l.status == 0, f"{l.name} grid {l.grid} x {l.block} refused"
        block, el, group = shape(l)
        assert l.block == block and l.begin == at and (l.end > l.begin or begin == end)
        at = l.end
        tile = block * el
        first = l.begin // tile
        tiles = (l.end - 1) // tile - first + 1 if l.end > l.begin else 1
        if l.kernel == "k_accum_adamw":
            whole = -(-l.begin // el) < l.end // el
            assert l.extra == int(l.begin % el != 0 or l.end % el != 0)
            assert l.grid - l.extra == (tiles if whole else 0) and l.grid >= 1
        else:
            span = l.extra
            assert span >= 1 and span % group == 0 and (l.grid - 1) * span < tiles <= l.grid * span
    assert at == end
    folds = [l for l in launches if l.kernel not in WORK]
    base, cap = (1 << 60, MIN_WS // 8) if entry == "noalloc" else (WS, wsb // 8)
    norm = entry in ("spec", "norm", "noalloc", "staged", "acc_norm", "add_norm")
    if not norm:
        assert not folds
        return
    assert len(work) == 1
    l = work[0]
    if l.kernel in ("k_grad_sqnorm", "k_acc_sqnorm") and l.targs[3 if l.kernel == "k_grad_sqnorm" else 2]:   # in a single workgroup
        assert l.grid == 1 and l.out == SQ and not folds
        return
    assert l.partials == base and l.grid <= cap - 128
    if l.grid > 8192:
        sl, fin = folds
        assert (sl.kernel, sl.partials, sl.extra, sl.grid) == ("k_sqnorm_fold_slices", base, l.grid, 128)
        assert sl.out == base + 8 * (cap - 128) and (fin.partials, fin.extra) == (sl.out, 128)
    else:
        fin, = folds
        assert (fin.partials, fin.extra) == (base, l.grid)
    assert fin.kernel == "k_sqnorm_finalize" and fin.out == SQ and all(f.status == 0 for f in folds)
