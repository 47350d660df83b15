"""How the kernels are given their arguments, from the gfx950 assembly of the library's own source, read on the CPU."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2512_17570_amd import build as B


@pytest.fixture(scope="module")
def arguments(tmp_path_factory):
    """[(kernel with template and function arguments, bytes of arguments, registers filled before a wave starts)]"""
    out = str(tmp_path_factory.mktemp("asm") / "gs_kernels.s")
    flags = [f for f in B.FLAGS if f != "-shared"]
    subprocess.run([B.HIPCC, *flags, "--offload-device-only", "-S", "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC,
                    os.path.join(B.CSRC, "gs_kernels.hip"), "-o", out], check=True, capture_output=True, text=True)
    found = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", open(out).read(), re.S)
    names = subprocess.run(["c++filt"], input="\n".join(n for n, _ in found), capture_output=True, text=True, check=True).stdout.split("\n")
    number = lambda key, block: int(re.search(rf"{key} (\d+)", block)[1])  # noqa: E731
    return [(name, number("kernarg_size", block), number("kernarg_preload_length", block)) for name, (_, block) in zip(names, found)]


def test_arguments_of_short_ranges_are_in_registers_and_few(arguments):
    """Up to 112 bytes of arguments the host's launch is shorter (by 0.05 us, on a shared core by 0.6), and what fits 14 registers is not
    fetched by the waves."""
    steps = [a for a in arguments if "k_accum_adamw<" in a[0] and "NearRest" in a[0]]
    norms = [a for a in arguments if "k_grad_sqnorm<" in a[0]]
    few = [a for a in norms if "GradTable" not in a[0]]
    eight = [a for a in norms if "GradTableOf<8>" in a[0]]
    assert steps and few and eight
    for name, size, registers in steps + few:
        assert size <= 112 and registers == 14, name
    for name, size, registers in eight:
        assert size <= 112 and registers >= 6, name
    for name, size, registers in arguments:
        if "k_acc_sqnorm<" in name or "k_sqnorm_" in name:
            assert registers * 4 >= size - 3, name           # all of them
