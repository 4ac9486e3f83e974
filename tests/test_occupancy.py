"""CPU: every sweep kernel leaves room on a CU for the blocks that its tile shape counts on there
(shapes.hpp: two of the second float shape, whose launches are priced by that), by the registers and
the LDS recorded in the library built here: 512 registers a SIMD lane, given out in eights, 160 KB of
LDS.  The kernels with the sextic term need more registers and have one block in every shape."""
import re
import shutil
import subprocess
from pathlib import Path

import pytest

from paper_2604_25876_amd import build

LLVM = Path("/opt/rocm/llvm/bin")


def test_blocks_per_cu(tmp_path):
    if not build.LIB.exists():
        pytest.skip("the library is not built here")
    lib = tmp_path / "lib.so"
    shutil.copy(build.LIB, lib)
    subprocess.check_call([str(LLVM / "llvm-objdump"), "--offloading", str(lib)], stdout=subprocess.DEVNULL)
    shapes = (build.PKG / "csrc" / "shapes.hpp").read_text()
    per_cu = {}
    for name, prec in (("SKYR_SHAPES_F64", "d"), ("SKYR_SHAPES_F32", "f")):
        entries = re.search(name + r"\(X\) \\\n(.*)", shapes).group(1)
        for e in re.findall(r"X\(([^)]*)\)", entries):
            v = [float(x) for x in e.split(",")]
            per_cu[(prec, *map(int, v[:4]))] = int(v[4])
    assert sorted(per_cu.values()) == [1, 1, 1, 1, 1, 2]
    seen = 0
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        notes = subprocess.check_output([str(LLVM / "llvm-readelf"), "--notes", str(obj)], text=True)
        for k in re.split(r"(?m)^  - \.agpr_count", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", k).group(1)
            m = re.match(r"_ZN4skyr\d+(batch_)?sweep_kernelI([df])NS_3GeoILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)EEE(.*)", name)
            if not m:
                continue
            args = [int(x) for x in re.findall(r"Li(\d+)E", m.group(7))]
            ext = args[0] if m.group(1) else args[1]
            shape = (m.group(2), *(int(x) for x in m.groups()[2:6]))
            blocks = 1 if ext == 2 else per_cu[shape]
            waves = (shape[1] + shape[2]) * blocks
            regs = -(-int(re.search(r"\.vgpr_count:\s+(\d+)", k).group(1)) // 8) * 8
            lds = int(re.search(r"\.group_segment_fixed_size:\s+(\d+)", k).group(1))
            assert regs * -(-waves // 4) <= 512, (name, regs)
            assert lds * blocks <= 160 * 1024, (name, lds)
            seen += 1
    assert seen == 2 * 3 * 3 * (3 + 1 + 2)  # precision, shape, variant: step policies, gradient, batch policies
