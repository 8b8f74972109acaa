"""The streaming kernel's forms for 64 rows that take B through LDS (two panels in flight, row-major bf16 B of even N), against the oracle:
tiles cut by M and by N, one column of tiles and many, reductions that end in a whole panel, in one of 8 rows, and with waves that have a
panel fewer than others."""
import os
import re
import subprocess
import tempfile

import pytest

import test_gpu_skinny as skinny
from paper_2511_16041_amd import build
from test_kernel_resources import READELF, code_objects

# (M, N, K); above 64 rows 64 x 128 tiles, at 49 to 64 rows 64 x 64
SHAPES = [(16300, 66, 1536), (4161, 194, 1544), (8130, 250, 1600), (129, 5634, 2040), (49, 8194, 1032), (64, 8264, 1096), (50, 16384, 1160)]


@pytest.mark.gpu
@pytest.mark.parametrize("exact", [True, False])
@pytest.mark.parametrize("c_format", skinny.BOTH)
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_through_lds(shape, c_format, exact, monkeypatch, capfd):
    print(f"rows {shape} C={c_format} exact={exact}", flush=True)
    monkeypatch.setenv("ATB_LOG", "1")
    capfd.readouterr()
    g = skinny.plan(shape, "bf16", c_format)
    assert skinny.variants(capfd.readouterr().err) == {("bf16", 64, 128 if shape[0] > 64 else 64, 256, 2)}
    skinny._check(g, exact, seed=27)


@pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-objdump")
def test_only_the_requests_use_m0():
    """The kernels with two panels in LDS set M0 for their requests and leave it so: nothing that the compiler made in them may use it."""
    objdump = os.path.join(os.path.dirname(READELF), "llvm-objdump")
    seen = 0
    for obj in code_objects(build.ensure_built()):
        with tempfile.NamedTemporaryFile(suffix=".elf") as f:
            f.write(obj)
            f.flush()
            text = subprocess.run([objdump, "-d", "--mcpu=gfx950", f.name], capture_output=True, text=True, check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*skinny_kernelILi0ELi4ELi[48]ELi4ELi2E\S*)>:\n((?:.+\n)*)", text, re.M):
            uses = re.findall(r"^\s*(\S+ .*\bm0\b.*?)\s*//", body, re.M)
            assert len(uses) > 20 and all(re.match(r"s_add_u32 m0, s\d+, (0x[0-9a-f]+|\d+)$", u) for u in uses), (name, uses)
            seen += 1
    assert seen == 2
