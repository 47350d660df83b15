"""Builds the library's launchers for the host only, against a HIP runtime that records launches instead of
making them (hipmock/launch_recorder.cpp), and reads back what each call would have launched."""
from __future__ import annotations

import copy
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
STREAM = 0x5000


class Arrays:
    """Where a call's arrays lie: addresses that are never dereferenced, `apart` bytes between each and the next, p among the others."""
    NAMES = ("p", "m", "v", "po", "mo", "vo", "w", "acc", "sq", "ws")

    def __init__(self, apart: int):
        for i, name in enumerate(self.NAMES):
            setattr(self, name, (1 << 50) + (i - 3) * apart)
        self.g = [(1 << 50) + (len(self.NAMES) + j) * apart for j in range(32)]

    def moved(self, name: str, by: int):
        """The same with one array elsewhere ("g3": the fourth stream)."""
        other = copy.deepcopy(self)
        if name[0] == "g":
            other.g[int(name[1:])] += by
        else:
            setattr(other, name, getattr(other, name) + by)
        return other


# Arrays of the longest range used here do not overlap in the first; in the others they lie as an allocator deals them out to a
# training program, at multiples of 256 bytes (up to 2^28 elements) or of 16 (up to 2^24).
FAR = Arrays(1 << 44)
NEAR = Arrays(6 << 28)
NEAR16 = Arrays((1 << 26) + 16)


class _Launch(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_char * 512), ("grid", ctypes.c_uint64), ("block", ctypes.c_uint64),
                ("stream", ctypes.c_uint64), ("lds", ctypes.c_uint64), ("begin", ctypes.c_int64), ("end", ctypes.c_int64), ("extra", ctypes.c_int64),
                ("keep_from", ctypes.c_int64), ("keep_block", ctypes.c_int64), ("partials", ctypes.c_uint64), ("out", ctypes.c_uint64),
                ("states", ctypes.c_uint64 * 6), ("w", ctypes.c_uint64), ("acc", ctypes.c_uint64), ("sqnorm", ctypes.c_uint64),
                ("streams", ctypes.c_uint64 * 32), ("consts", ctypes.c_float * 9), ("k", ctypes.c_int32), ("accumulate", ctypes.c_int32), ("status", ctypes.c_int32)]


class HP(ctypes.Structure):
    _fields_ = [(x, ctypes.c_float) for x in ("lr", "beta1", "beta2", "eps", "wd", "max_norm")] + [("step", ctypes.c_int32)]


@dataclass
class Launch:
    kernel: str            # without its template arguments
    targs: tuple           # those, as numbers (false/true as 0/1)
    params: str            # its parameter list: kernels of one name are told apart by it
    grid: int
    block: int
    lds: int               # bytes of LDS asked for beyond what the kernel itself declares
    begin: int
    end: int
    extra: int
    keep_from: int         # the first element that is left in the cache: the range's end if none is
    partials: int
    out: int
    accumulate: int
    consts: tuple          # a step's constants and largest norm
    status: int

    @property
    def name(self):
        return f"{self.kernel}<{','.join(map(str, self.targs))}>"

    @property
    def near(self):
        """A step whose arrays are given by their distances from p."""
        return "NearRest" in self.params


def parse_name(name: str):
    """(name, template arguments, parameter list)"""
    m = re.fullmatch(r"(\w+)(?:<([^()]*)>)?\((.*)\)", name)
    args = [{"false": 0, "true": 1}.get(x.strip(), x.strip()) for x in (m[2] or "").split(",") if x.strip()]
    return m[1], tuple(int(x) for x in args), m[3]


def _launch(r: _Launch):
    kernel, targs, params = parse_name(r.kernel.decode())
    l = Launch(kernel, targs, params, r.grid, r.block, r.lds, r.begin, r.end, r.extra, r.keep_from, r.partials, r.out, r.accumulate, tuple(r.consts), r.status)
    if r.keep_block >= 0:
        block, el, _ = shape(l)
        # kernels that are made without the choice leave nothing in the cache, whatever they are told
        keeps = targs[3] if kernel == "k_grad_accum_sqnorm" else not targs[3] and (targs[2] > 256 or 1 <= targs[0] <= 4)
        first = l.begin // (block * el) * block * el + r.keep_block * l.extra * block * el
        l.keep_from = max(l.begin, first) if keeps and r.keep_block < l.grid else l.end
    return l


def check_arrays(entry, r: _Launch, l: Launch, at: Arrays, k: int, sqnorm: int, accumulate: int):
    """A launch is given the arrays, the number of streams and the norm of the call."""
    grads = list(r.streams[:r.k])
    step = l.kernel in ("k_accum_adamw", "k_accum_adamw_spec")
    if step and entry != "host_step":
        out = (at.p, at.m, at.v) if entry in ("step", "from_acc") else (at.po, at.mo, at.vo)
        assert list(r.states) == [at.p, at.m, at.v, *out] and r.w == at.w, (entry, l.name)
        assert r.sqnorm == sqnorm, (entry, l.name)
    if step and entry == "from_acc" or l.kernel in ("k_grad_accum_sqnorm", "k_accum_add", "k_acc_sqnorm"):
        assert r.acc == at.acc
    if l.kernel == "k_accum_add":
        assert grads == at.g[:1]
    elif l.kernel in WORK and entry not in ("from_acc", "acc_norm", "host_step"):
        assert r.k == k and grads == at.g[:k], (entry, l.name)
        assert l.kernel != "k_grad_sqnorm" or l.targs[0] in (0, k)
    if l.out == at.sq:
        assert l.accumulate == accumulate


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
             cus: int = 256, stream: int = STREAM, at: Arrays = FAR, capturing: bool = False, sqnorm: bool = True, max_norm: float = 1.0):
        """(status, launches, stream handles whose CUs were asked for, bytes of workspace handed over)"""
        self.hp.max_norm = max_norm
        i64, vp, hp = ctypes.c_int64, ctypes.c_void_p, ctypes.byref(self.hp)
        lib = self.lib
        lib.rec_reset(cus, int(capturing))
        tab = (vp * k)(*at.g[:k]) if k else None
        b, e, s = i64(begin), i64(end), vp(stream)
        wsb = lib.gs_sqnorm_workspace_bytes_for(end - begin) if ws == FULL else ws
        sq = vp(at.sq) if sqnorm else None
        norm = (vp(at.sq), accumulate, vp(at.ws), ctypes.c_size_t(wsb), s)
        st = {
            "step": lambda: lib.gs_accum_adamw(vp(at.p), vp(at.m), vp(at.v), vp(at.w), tab, k, b, e, hp, sq, s),
            "oop": lambda: lib.gs_accum_adamw_oop(vp(at.p), vp(at.m), vp(at.v), vp(at.po), vp(at.mo), vp(at.vo), vp(at.w), tab, k, b, e, hp, sq, s),
            "from_acc": lambda: lib.gs_adamw_from_acc(vp(at.p), vp(at.m), vp(at.v), vp(at.w), vp(at.acc), b, e, hp, sq, s),
            "host_step": lambda: lib.rec_step_on_host_memory(k, b, e, s),
            "spec": lambda: lib.gs_accum_adamw_spec(vp(at.p), vp(at.m), vp(at.v), vp(at.po), vp(at.mo), vp(at.vo), vp(at.w), tab, k, b, e, hp, *norm),
            "norm": lambda: lib.gs_grad_sqnorm(tab, k, b, e, *norm),
            "noalloc": lambda: lib.gs_grad_sqnorm_noalloc(tab, k, b, e, vp(at.sq), accumulate, s),
            "staged": lambda: lib.gs_grad_accum_sqnorm(tab, k, b, e, vp(at.acc), *norm),
            "acc_norm": lambda: lib.gs_acc_sqnorm(vp(at.acc), b, e, *norm),
            "add": lambda: lib.gs_accum_add(vp(at.acc), vp(at.g[0]), first, b, e, None, 0, None, ctypes.c_size_t(0), s),
            "add_norm": lambda: lib.gs_accum_add(vp(at.acc), vp(at.g[0]), first, b, e, *norm),
        }[entry]()
        out = []
        for i in range(lib.rec_count()):
            r = _Launch()
            lib.rec_get(i, ctypes.byref(r))
            l = _launch(r)
            check_arrays(entry, r, l, at, k, at.sq if sqnorm and max_norm > 0 and entry != "spec" else 0, accumulate)
            out.append(l)
        asked = [lib.rec_mask_query(i) for i in range(lib.rec_mask_queries())]
        return st, out, asked, wsb


WORK = ("k_accum_adamw", "k_accum_adamw_spec", "k_grad_sqnorm", "k_grad_accum_sqnorm", "k_accum_add", "k_acc_sqnorm")


def shape(l: Launch):
    """(lanes, elements per lane, tiles a workgroup takes at a time) of a kernel, from its template arguments."""
    t = l.targs
    return {"k_accum_adamw": lambda: (t[0], t[1], 1), "k_accum_adamw_spec": lambda: (t[0], t[1], 1),
            "k_grad_sqnorm": lambda: (t[2], 4, t[1]), "k_grad_accum_sqnorm": lambda: (t[0], t[1], 1),
            "k_accum_add": lambda: (t[2], t[3], 1), "k_acc_sqnorm": lambda: (t[1], 4, t[0])}[l.kernel]()


def check(entry, launches, begin, end, wsb, arrays=FAR):
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
    base, cap = (1 << 60, MIN_WS // 8) if entry == "noalloc" else (arrays.ws, wsb // 8)
    norm = entry in ("spec", "norm", "noalloc", "staged", "acc_norm", "add_norm")
    if not norm:
        assert not folds
        return
    assert len(work) == 1
    l = work[0]
    if l.kernel in ("k_grad_sqnorm", "k_acc_sqnorm") and l.targs[3 if l.kernel == "k_grad_sqnorm" else 2]:   # in a single workgroup
        assert l.grid == 1 and l.out == arrays.sq and not folds
        return
    assert l.partials == base and l.grid <= cap - 128
    if l.grid > 8192:
        sl, fin = folds
        assert (sl.kernel, sl.partials, sl.extra, sl.grid) == ("k_sqnorm_fold_slices", base, l.grid, 128)
        assert sl.out == base + 8 * (cap - 128) and (fin.partials, fin.extra) == (sl.out, 128)
    else:
        fin, = folds
        assert (fin.partials, fin.extra) == (base, l.grid)
    assert fin.kernel == "k_sqnorm_finalize" and fin.out == arrays.sq and all(f.status == 0 for f in folds)
