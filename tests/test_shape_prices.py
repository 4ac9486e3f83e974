"""CPU: every tile shape carries its own prices, also in lists that a build defines for itself (more
shapes than the default ones, and in another order)."""
import subprocess
from pathlib import Path

CSRC = Path(__file__).resolve().parent.parent / "paper_2604_25876_amd" / "csrc"

DRIVER = """
#include "shapes.hpp"
#include <cstdio>
int main()
{
    for (const skyr::Shape& s : skyr::kShapesF64) std::printf("%d %g %g %g\\n", s.cols, s.cost, s.step, s.step_full);
    for (const skyr::Shape& s : skyr::kShapesF32) std::printf("%d %g %g %g\\n", s.cols, s.cost, s.step, s.step_full);
}
"""


def _prices(tmp_path, *defines):
    (tmp_path / "p.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-I", str(CSRC), *defines, "-o", str(tmp_path / "p"), str(tmp_path / "p.cpp")])
    out = subprocess.check_output([str(tmp_path / "p")], text=True)
    return [tuple(float(v) for v in line.split()) for line in out.splitlines()]


def test_prices_belong_to_their_shapes(tmp_path):
    from paper_2604_25876_amd import skyr
    default = _prices(tmp_path)
    assert len(default) == len(skyr.tile_variants(skyr.F64)) + len(skyr.tile_variants(skyr.F32_BULK))
    assert all(c > 0 and a > 0 and f > 0 for _, c, a, f in default)
    own = ("-DSKYR_SHAPES_F64(X)=X(6, 2, 2, 32, 1, 4.0, 4.1, 4.2) X(4, 4, 1, 16, 1, 1.0, 1.1, 1.2) "
           "X(4, 4, 1, 32, 1, 2.0, 2.1, 2.2) X(8, 8, 1, 16, 1, 3.0, 3.1, 3.2)")
    assert _prices(tmp_path, own)[:4] == [(32, 4.0, 4.1, 4.2), (16, 1.0, 1.1, 1.2), (32, 2.0, 2.1, 2.2),
                                          (16, 3.0, 3.1, 3.2)]
