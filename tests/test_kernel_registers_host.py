"""Registers of the marches that are measured with a given number of wavefronts per SIMD, from the metadata
of the library built here: 512 vector registers a SIMD lane, so four wavefronts with at most 128 each, six
with at most 80, and none of them in scratch memory."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2204_14241_amd import build

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of the library's bundles."""
    for at in (m.start() for m in re.finditer(MAGIC, data)):
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n]
            p += 24 + n
            if build.ARCH.encode() in name:
                yield data[at + off:at + off + size]


def kernels(elf):
    """amdhsa.kernels of a code object's metadata note."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entry, num = struct.unpack_from("<HH", elf, 58)
    for i in range(num):
        kind, = struct.unpack_from("<I", elf, shoff + i * entry + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * entry + 24)
        if kind != 7:
            continue
        p, end = off, off + size
        while p < end:
            namesz, descsz, _ = struct.unpack_from("<III", elf, p)
            name = elf[p + 12:p + 12 + namesz]
            desc = p + 12 + (namesz + 3) // 4 * 4
            if name.startswith(b"AMDGPU"):
                yield from msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]
            p = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def found():
    if not os.path.exists(build.LIB):
        build.build_library()
    with open(build.LIB, "rb") as f:
        data = f.read()
    ks = [k for elf in code_objects(data) for k in kernels(elf)]
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in ks), capture_output=True,
                           text=True).stdout.splitlines()
    return {n.split("(")[0]: k for n, k in zip(names, ks)}


@pytest.mark.parametrize("kernel", [
    "k_cg_b_march<hmc::MGeoOne, false>", "k_cg_b2_march<hmc::MGeoOne, false>",
    "k_ru_resid_march<float, hmc::MGeoOne, false>", "k_ru_resid_march<double, hmc::MGeoOne, false>",
    "k_ru_apply_march<hmc::MGeoOne, false>", "k_mdm_march<512>", "k_mdm2_march<512>"])
def test_four_wavefronts_a_simd(found, kernel):
    k = found["void hmc::" + kernel]
    assert k[".vgpr_count"] <= 128
    assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0


@pytest.mark.parametrize("geo", ["GeoOne", "GeoBatch"])
@pytest.mark.parametrize("full", ["true", "false"])
def test_six_wavefronts_a_simd(found, geo, full):
    k = found[f"void hmc::k_pc_t<float, hmc::{geo}, {full}>"]
    assert k[".vgpr_count"] <= 80
    assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0
