"""Registers and LDS of kernels whose speed hangs on them, read from the code
objects' metadata in the built library: what a change of the source around a
kernel costs there shows in no result."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1912_05371_amd", "libwacm.so")


@pytest.fixture(scope="module")
def kernels():
    """demangled name (no argument list) -> metadata of the kernel"""
    data = open(LIB, "rb").read()
    found = {}
    # AMDGPU metadata notes: namesz 7, descsz, type 32, "AMDGPU\0" padded to 8
    for m in re.finditer(rb"\x07\x00\x00\x00(....)\x20\x00\x00\x00AMDGPU\x00\x00", data, re.S):
        size = struct.unpack("<I", m.group(1))[0]
        for k in msgpack.unpackb(data[m.end():m.end() + size]).get("amdhsa.kernels", []):
            found[k[".name"]] = k
    names = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True,
                           check=True).stdout.splitlines()
    return {n.split("(")[0].replace("void ", ""): k for n, k in zip(names, found.values())}


def pick(kernels, pattern):
    got = {n: k for n, k in kernels.items() if re.fullmatch(pattern, n)}
    assert got, pattern
    return got


def test_penalized_rhs_of_small_blocks_does_not_spill(kernels):
    # 48 registers spilled before the mask's factor tables, 71 with them: the rhs
    # of 904 blocks of 16^3 FP64 with a sphere took 180 and 184 us
    for n, k in pick(kernels, r"wacm::stage_kernel<double, 16, 16, 0, true, \w+, \d>").items():
        assert k[".vgpr_spill_count"] == 0, n


def test_force_gradient_of_a_sphere_holds_no_factor_tables(kernels):
    for n, k in pick(kernels, r"wacm::force_adj_kernel<\w+, \d+, false>").items():
        assert k[".group_segment_fixed_size"] == 3 * 256 * 8, n  # its reduction


def test_diagnostics_without_a_mask_hold_nothing_for_one(kernels):
    # with a mask's registers (129) and LDS three of four waves fit a SIMD
    for n, k in pick(kernels, r"wacm::diag_kernel<\w+, \d+, 0>").items():
        assert k[".vgpr_count"] <= 64 and k[".group_segment_fixed_size"] <= 20480, n


def test_rhs_of_large_2d_blocks_leaves_room_for_two_workgroups(kernels):
    for n, k in pick(kernels, r"wacm::d2::stage2d_kernel<\w+, 32, 0>").items():
        assert k[".vgpr_count"] <= 64 and k[".vgpr_spill_count"] == 0, n
