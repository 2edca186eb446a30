"""Register budgets of the built kernels, from the code objects in libdpb.so:
a kernel whose launch is sized for a number of waves per SIMD must fit that many,
and none but one may put registers in scratch memory.  (A SIMD has 512
vector registers a lane, handed out in blocks of eight: 128 for four waves,
168 for three.)  Read on the CPU; needs no GPU.
"""
import os
import re
import struct
import subprocess

import pytest

from paper_2607_20652_amd import binding

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def code_objects(path):
    data = open(path, "rb").read()
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := data.find(magic, at)) >= 0:
        n = struct.unpack_from("<Q", data, at + len(magic))[0]
        pos = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + idlen].decode()
            pos += 24 + idlen
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at += len(magic)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(READELF):
        pytest.skip(f"no {READELF}")
    binding.load()
    out, tmp = {}, tmp_path_factory.mktemp("co")
    for i, co in enumerate(code_objects(binding.lib_path)):
        p = tmp / f"{i}.co"
        p.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"\n\s+- \.(?:agpr_count|args)", notes)[1:]:
            field = lambda f: int(re.search(rf"\.{f}:\s+(\d+)", block).group(1))
            name = re.search(r"\.symbol:\s+'?([\w.]+?)\.kd", block)
            if name:
                out[name.group(1)] = {f: field(f) for f in ("vgpr_count", "vgpr_spill_count", "private_segment_fixed_size")}
    assert len(out) > 100
    return out


BUDGETS = [
    # (kernel, vector registers)
    (r"col_decode_kernelILi(4|8|16)E", 128),
    (r"col_decode_kernelILi0E", 64),
    (r"col_bwd_kernelILi(4|8|16)E", 128),
    (r"col_bwd_kernelILi0ELi\dELb1E", 96),                  # bf16 gradients: five waves
    (r"14decode2_kernelILb1E", 168),                         # bf16 output: three waves
    (r"18decode_bwd2_kernelILb1E", 168),                    # bf16 gradients: three waves
    (r"encode3_kernelILb1ELi(8|16)ELi4ELb0E", 128),
]


@pytest.mark.parametrize("pattern,most", BUDGETS)
def test_register_budget(kernels, pattern, most):
    found = {k: v["vgpr_count"] for k, v in kernels.items() if re.search(pattern, k)}
    assert found, f"no kernel matches {pattern}"
    over = {k: v for k, v in found.items() if v > most}
    assert not over, over


# fp32 output, sixteen columns, over 24 index bits: a few registers, where one wave fewer is slower
MAY_SPILL = r"col_decode_kernelILi16ELi8ELb0E"


def test_no_kernel_spills_to_scratch(kernels):
    spilled = {k: v for k, v in kernels.items() if v["vgpr_spill_count"] or v["private_segment_fixed_size"]}
    few = [k for k in spilled if re.search(MAY_SPILL, k) and spilled[k]["vgpr_spill_count"] <= 8]
    for k in few:
        del spilled[k]
    assert not spilled, spilled
