"""Host-side rules of the launches, checked without a GPU."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1010_4782_amd", "csrc")


def test_solver_scalars_keep_their_type():
    """Scal holds doubles and ints, which type-based alias analysis takes to be apart: a slot that is written as an
    array of one of them and then through its members may keep the old state or iteration count."""
    cast = re.compile(r"reinterpret_cast<(?:const )?(?:double|float|int|long|unsigned|int\d+_t|uint\d+_t)\s*\*>\("
                      r"\s*(?:&\s*)?(?:pre|sc|next|scal|B\.scal|bh\.d_scal|R\.h_scal)\b")
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".cpp", ".h")):
            hits = [m.group(0) for m in cast.finditer(open(os.path.join(CSRC, name)).read())]
            assert not hits, (name, hits)


def test_wide_launches_are_one_workgroup_per_cu(tmp_path):
    """Every workgroup of a wide CG launch walks the same number of tiles, the fewest that leave at most 256
    workgroups; more right-hand sides than that are not taken."""
    import shutil
    import subprocess

    import pytest

    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler on this host")
    src = tmp_path / "wide.cpp"
    src.write_text("""
#include <cstdio>
#include "wide_grid.h"
int main() {
  int tiles[16], slots[16], n;
  while (std::scanf("%d", &n) == 1) {
    for (int i = 0; i < n; ++i) std::scanf("%d %d", tiles + i, slots + i);
    std::printf("%d\\n", stag::wide_tiles(tiles, slots, n));
  }
}
""")
    exe = tmp_path / "wide"
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    cases = [[(t, s)] for t in (1, 2, 65, 80, 157, 324, 1029, 2048) for s in (1, 2, 3, 5, 8, 12, 13, 19, 28, 256, 257)]
    cases += [[(1, 2), (80, 2), (1, 3)], [(157, 13), (5, 1)], [(32, 4), (324, 12), (1024, 8)], [(70, 200), (1, 60)]]
    text = "".join(f"{len(c)} " + " ".join(f"{t} {s}" for t, s in c) + "\n" for c in cases)
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split()
    for c, per in zip(cases, map(int, out)):
        grid = lambda k: sum(-(-t // k) * s for t, s in c)  # noqa: E731
        if sum(s for _, s in c) > 256:
            assert per == 0, c
        else:
            assert grid(per) <= 256 and (per == 1 or grid(per - 1) > 256), (c, per, grid(per))
