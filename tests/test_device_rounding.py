"""A cell gets the same bits from every kernel that updates it only if no
rounding in the update is left to the compiler: the update compiled with its
own contraction of products and sums allowed and forbidden has to be the same
code.  Compiles for gfx950; no GPU."""
import os
import re
import subprocess

import pytest

from paper_2102_01305_amd import build

SOURCE = r"""
#include "update_dev.h"
using namespace ibmk;
template <bool IBM, bool FORCE, bool ZH>
__global__ void cell(Geo g, Phys p, const CollideArgs* a, const float* S, float* D) {
  const int x = threadIdx.x, y = blockIdx.x, z = blockIdx.y;
  float f[kQ];
  pull19<StF32, true>(S, g, x, y, z, f);
  update_cell<StF32, IBM, FORCE, ZH, false>(g, p, *a, x, y, z, f);
  store_cell<StF32>(D, g, p, x, y, z, f);
}
#define K(i, f, z) template __global__ void cell<i, f, z>(Geo, Phys, const CollideArgs*, const float*, float*)
K(false, false, false); K(false, true, false); K(true, false, false); K(true, true, false);
K(false, false, true); K(false, true, true); K(true, false, true); K(true, true, true);
"""


def test_no_rounding_of_the_cell_update_is_left_to_the_compiler(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src = tmp_path / "cell.hip"
    src.write_text(SOURCE)
    code = []
    for extra in ([], ["-ffp-contract=off"]):
        out = tmp_path / f"cell{len(extra)}.s"
        flags = [f for f in build.FLAGS if f not in ("-fPIC", "-shared", "-Wall")]
        subprocess.run([build.HIPCC, *flags, *extra, "-cuid=cell", "-I", build.CSRC, "--cuda-device-only", "-S", str(src),
                        "-o", str(out)], check=True, capture_output=True)
        code.append([line for line in (re.sub(r"\s*;.*", "", t).strip() for t in out.read_text().splitlines()) if line])
    assert len(code[0]) > 5000                         # (the kernels are in it)
    assert code[0] == code[1]
