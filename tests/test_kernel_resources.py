"""What the compiler made of the kernels, from the notes of the code objects in the built library: the registers leave room for the
workgroups that the selector reckons with, and nothing spills but where that is known."""
import os
import re
import shutil
import struct
import subprocess
import tempfile

import pytest

import paper_2511_16041_amd as atb
from paper_2511_16041_amd import build

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
pytestmark = pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The device code objects in a library, one per translation unit: magic, number of entries, then offset, size and name of each."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24: p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in name and size:
                yield data[at + off: at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def kernels(path):
    """{mangled name: its notes}"""
    out = {}
    for obj in code_objects(path):
        with tempfile.NamedTemporaryFile(suffix=".elf") as f:
            f.write(obj)
            f.flush()
            text = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n  - (?=\.)", text):
            m = re.search(r"\.symbol: +'?(\S+?)\.kd", part)
            if m:
                out[m[1]] = {k: int(v) for k, v in re.findall(r"\.(\w+): +(\d+)\s", part)}
    return out


@pytest.fixture(scope="module")
def all_kernels():
    return kernels(build.ensure_built())


@pytest.fixture(scope="module")
def tile_kernels(all_kernels):
    """{tiles: [(even N, notes)]} of the tile pipeline"""
    out = {}
    for name, k in all_kernels.items():
        m = re.search(r"atb_gemm_kernel.*?ShapeILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E.*?EEELb(\d)", name)
        if m:
            out.setdefault(tuple(int(x) for x in m.groups()[:4]), []).append((m[5] == "1", k))
    assert sorted(out) == sorted(atb.instances())
    return out


def waves_per_simd(k):
    """512 registers per lane and SIMD, handed out in eights; vgpr_count has the accumulation registers in it."""
    return min(8, 512 // (-(-k["vgpr_count"] // 8) * 8))


def test_registers_leave_room_for_the_workgroups_that_share_a_cu(tile_kernels):
    for i, tiles in enumerate(atb.instances()):
        want = atb.instance_geometry(i)[2]
        for _, k in tile_kernels[tiles]:
            got = waves_per_simd(k) * 256 // k["max_flat_workgroup_size"]
            assert got >= want, (tiles, k)


def test_nothing_spills_but_in_the_epilogue_of_the_four_wave_tiles(all_kernels, tile_kernels):
    """The 256-row tiles on four waves use all 512 registers; what they spill (10 at most) they do outside the K loop."""
    four_waves = [(32, 256, 64, 256), (32, 256, 128, 256)]
    spilled = {tiles: max(k["vgpr_spill_count"] for _, k in ks) for tiles, ks in tile_kernels.items()}
    assert all(n <= 10 for n in (spilled.pop(t) for t in four_waves)) and not any(spilled.values()), spilled
    others = {name: k for name, k in all_kernels.items() if "atb_gemm_kernel" not in name}
    assert others and not any(k["vgpr_spill_count"] for k in others.values())
