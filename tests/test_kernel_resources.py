"""Register use of the attention kernels as built (the metadata of the library's
own code objects, no GPU): none spills vector registers or uses scratch memory,
and those that are meant to run three waves per SIMD (168 vector registers at
most) do.
"""
import os
import re
import shutil
import subprocess

import pytest
import yaml

from paper_2606_08476_amd import flashcp as F

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name<template arguments> -> the code object's metadata of the kernel."""
    if not os.path.exists(F._LIB_PATH):
        from paper_2606_08476_amd import build
        build.build()
    if shutil.which(READELF) is None:
        pytest.skip("needs llvm-readelf")
    blob, out = open(F._LIB_PATH, "rb").read(), {}
    # code objects: the ELF images behind each bundle header
    ends = [m.start() for m in re.finditer(rb"__CLANG_OFFLOAD_BUNDLE__", blob)] + [len(blob)]
    for a, b in zip(ends, ends[1:]):
        path = tmp_path_factory.mktemp("co") / "k.elf"
        path.write_bytes(blob[blob.index(b"\x7fELF", a):b])
        text = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                              check=True).stdout
        for k in yaml.safe_load(text[text.index("---"):text.index("\n...")])["amdhsa.kernels"]:
            t = re.match(r"_ZN3fck\d+(\w+?)I(.*?)EEv", k[".name"])
            if t:
                args = re.findall(r"L[ib](\d+)", t.group(2))
                out[f"{t.group(1)}<{', '.join(args)}>"] = k
    return out


def test_no_attention_kernel_spills(kernels):
    assert len(kernels) > 60 and "attn_bwd_grid_kernel<128, 4, 4>" in kernels
    bad = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"])
           for n, k in kernels.items()
           if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not bad, bad


# <head dim, heads per iteration or tile>
THREE_WAVES = [f"{k}<64, {h}>" for k in ("attn_bwd_kernel", "attn_bwd_atomic_kernel") for h in (1, 2, 4)]


@pytest.mark.parametrize("name", THREE_WAVES + ["attn_bwd_dq_kernel<64, 4>"])
def test_three_waves_per_simd(kernels, name):
    assert kernels[name][".vgpr_count"] <= 168 and kernels[name][".agpr_count"] == 0
