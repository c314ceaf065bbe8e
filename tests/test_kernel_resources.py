"""Registers of the built kernels whose speed rests on them, from the metadata of
the library's own gfx950 code objects.  CPU only."""
import os
import re
import struct
import subprocess

import pytest

import paper_2510_17335_amd as ddm

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJCOPY = "/opt/rocm/llvm/bin/llvm-objcopy"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: {metadata key: value}} of every kernel of the library."""
    if not (os.path.exists(ddm.LIB_PATH) and os.path.exists(READELF) and os.path.exists(OBJCOPY)):
        pytest.skip("needs the built library and ROCm's binutils")
    tmp = tmp_path_factory.mktemp("co")
    fat = str(tmp / "fatbin")
    subprocess.run([OBJCOPY, "--dump-section", f".hip_fatbin={fat}", ddm.LIB_PATH, str(tmp / "copy.so")], check=True)
    data = open(fat, "rb").read()
    out = {}
    for start in [m.start() for m in re.finditer(re.escape(MAGIC), data)]:
        at = start + len(MAGIC)
        count, at = struct.unpack_from("<Q", data, at)[0], at + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, at)
            triple, at = data[at + 24:at + 24 + n].decode(), at + 24 + n
            if "gfx950" not in triple or size == 0:
                continue
            obj = tmp / f"{start}.co"
            obj.write_bytes(data[start + off:start + off + size])
            text = subprocess.run([READELF, "--notes", str(obj)], check=True, capture_output=True, text=True).stdout
            for block in re.split(r"\n  - ", text)[1:]:
                meta = dict(re.findall(r"^    \.(\w+): +(\S+)$", "\n" + "    " + block, re.M))
                if "name" in meta:
                    out[meta["name"]] = meta
    return out


# the separate G2P: 8 waves per SIMD, without which its gathers wait one by one
@pytest.mark.parametrize("name", ["_ZN3ddm5k_g2pIfLi3ELb0EEE"])
def test_fits_64_registers_without_scratch(kernels, name):
    found = [m for k, m in kernels.items() if k.startswith(name)]
    assert len(found) == 1, sorted(kernels)[:5]
    assert int(found[0]["vgpr_count"]) <= 64
    assert int(found[0]["vgpr_spill_count"]) == 0
    assert int(found[0]["private_segment_fixed_size"]) == 0


# P2G joined with the G2P before it, FP32, 256 and 512 threads: 128 registers, four
# waves per SIMD, and nothing of a particle in scratch
@pytest.mark.parametrize("block", [256, 512])
def test_joined_p2g_without_scratch(kernels, block):
    found = [m for k, m in kernels.items() if k.startswith(f"_ZN3ddm5k_p2gIfLi3ELb0ELi{block}ELb1EEE")]
    assert len(found) == 1
    assert int(found[0]["vgpr_count"]) <= 128
    assert int(found[0]["vgpr_spill_count"]) == 0
    assert int(found[0]["private_segment_fixed_size"]) == 0
