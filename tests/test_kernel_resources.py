"""Registers, scratch and LDS of kernels whose residency the host code and the
notes beside the kernels count on, from the metadata of the built library's
gfx950 code objects."""
import re
import struct

import msgpack
import pytest

from paper_2101_05886_amd import build as B

CU_LDS = 160 * 1024


def code_objects(lib):
    """the amdhsa ELF images in the library's offload bundles"""
    at = lib.find(b"\x7fELF\x02\x01\x01\x40")
    while at >= 0:
        yield lib[at:]
        at = lib.find(b"\x7fELF\x02\x01\x01\x40", at + 8)


def metadata(elf):
    """the AMDGPU metadata note (type 32) of one code object"""
    phoff, phnum = struct.unpack_from("<Q", elf, 32)[0], struct.unpack_from("<H", elf, 56)[0]
    for i in range(phnum):
        ptype, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + 56 * i)
        end = off + size
        while ptype == 4 and off < end:
            nlen, dlen, kind = struct.unpack_from("<III", elf, off)
            data = off + 12 + (nlen + 3) // 4 * 4
            if kind == 32:
                return msgpack.unpackb(elf[data:data + dlen])
            off = data + (dlen + 3) // 4 * 4
    raise ValueError("no metadata note")


@pytest.fixture(scope="module")
def kernels():
    """{name: [(template arguments, metadata)]}"""
    with open(B.LIB, "rb") as f:
        lib = f.read()
    out = {}
    for elf in code_objects(lib):
        for k in metadata(elf)["amdhsa.kernels"]:
            m = re.match(r"_ZN3fpk(\d+)(\w+)", k[".name"])
            name = m.group(2)[:int(m.group(1))]
            args = tuple(int(v) for v in re.findall(r"L[ib](\d+)E", k[".name"]))
            out.setdefault(name, []).append((args, k))
    return out


def test_two_workgroups_of_the_sweeps_fit_a_cu(kernels):
    # four waves each, one per SIMD: 256 registers a wave and half of the LDS;
    # the batched FP64 WENO7 sweeps in 3D run alone, to hold all registers
    for name in ("kb_sweep_wg", "k_sweep_wg", "kb_sweep_x", "k_sweep_x", "k_row_2d"):
        for args, k in kernels[name]:
            assert 2 * k[".group_segment_fixed_size"] <= CU_LDS, (name, args)
            if name == "kb_sweep_wg" and args[0] == 3 and args[2] == 2 and args[4] == 0:
                assert k[".private_segment_fixed_size"] == 0, args
            else:
                assert k[".vgpr_count"] <= 256, (name, args)


def test_metrics_2d_registers(kernels):
    # a lane per node: latency is hidden by other waves, four per SIMD or more
    for args, k in kernels["k_metrics2"]:
        assert k[".vgpr_count"] <= 128 and k[".private_segment_fixed_size"] == 0, args
