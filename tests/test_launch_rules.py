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
