"""What the compiler makes of places in the kernels whose speed depends on it: the gfx950 assembly of the
library's own source, read on the CPU."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2512_17570_amd import build as B


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name with template arguments and parameter list: assembly lines}"""
    out = str(tmp_path_factory.mktemp("asm") / "gs_kernels.s")
    flags = [f for f in B.FLAGS if f != "-shared"]
    subprocess.run([B.HIPCC, *flags, "--offload-device-only", "-S", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
                    os.path.join(B.CSRC, "gs_kernels.hip"), "-o", out], check=True, capture_output=True, text=True)
    text = open(out).read()
    marks = [(m.start(), m[1]) for m in re.finditer(r"^(_ZN2gs\w+):", text, re.M)]
    names = subprocess.run(["c++filt"], input="\n".join(n for _, n in marks), capture_output=True, text=True, check=True).stdout.split("\n")
    ends = [a for a, _ in marks[1:]] + [len(text)]
    found = {re.sub(r"^(void )?gs::", "", name): text[a:e].split(".section")[0].split("\n") for (a, _), e, name in zip(marks, ends, names)}
    assert len(found) == len(marks) == len(re.findall(r"^\s*\.amdhsa_kernel ", text, re.M))
    return found


def test_no_kernel_uses_scratch_memory(kernels, tmp_path):
    """Arrays that are not resolved into registers go to memory and cost many times the kernel (a cut group's
    batch did once: the norm of 1 element 2.5 -> 11 us)."""
    assert len(kernels) > 40
    for name, lines in kernels.items():
        assert not any(re.search(r"\b(scratch|buffer)_(load|store)", l) for l in lines), name


def test_late_arguments_are_read_where_they_are_needed(kernels):
    """Read late, a wave's arguments are not all behind the wait at its entry: there is none of the states' loads'
    addresses, the gradients' or the hyper-parameters' before the range's ends, and the last are read after the gradients."""
    late = [lines for name, lines in kernels.items() if re.fullmatch(r"k_accum_adamw<(\d+, \d+, false, .*, )true>\(.*\)", name)]
    assert len(late) == 2
    for lines in late:
        code = [l.strip() for l in lines]
        first = next(i for i, l in enumerate(code) if "lgkmcnt" in l)
        assert sum(l.startswith("s_load") for l in code[:first]) <= 2
        body = code[next(i for i, l in enumerate(code) if l.startswith("global_load")):]
        loads = [i for i, l in enumerate(body) if l.startswith("global_load")]
        assert any(l.startswith("s_load_dwordx8") for l in body[loads[3]:])


def test_leftover_streams_of_the_speculative_pass_are_in_flight_together(kernels):
    found = 0
    for name, lines in kernels.items():
        if not re.match(r"k_accum_adamw_spec<\d+, \d+, 4,", name):
            continue
        for i, line in enumerate(lines):
            m = re.search(r"; (\d) streams? left", line)
            if not m:
                continue
            found += 1
            rest = lines[i:]
            wait = next(j for j, l in enumerate(rest) if "s_waitcnt" in l and "vmcnt" in l)
            loads = sum("global_load" in l for l in rest[:wait])
            assert loads == int(m[1]), (name, line.strip(), loads)
    assert found == 12         # four kernels, each with 1, 2 and 3 streams left
