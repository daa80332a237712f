"""The inner stopping test's norms on FP32 rows that do not fill whole waves are
sums of FP64 products: in the code that the compiler makes of the residual sweeps,
each cell pair of a plane has its two FP64 products per norm, which the sweeps on
rows of whole waves do without.  Compiles kernels to gfx950 assembly; runs nothing."""
import os
import re
import subprocess

import pytest

from paper_1601_05448_amd import build as B

SOURCE = """
#include "poisson_resid.hpp"
namespace pois {
template __global__ void k_resid_dhtx_z<float, %(n)d, 0, 0, 0>(GridArgs, const Slot*, Tables, int, int);
template __global__ void k_resid_dhtx_s<float, %(n)d, 2, 0, 0>(GridArgs, const Slot*, Tables, int);
}  // namespace pois
"""


def _fp64_products(n, tmp_path):
    """FP64 products in the marching and in the small-tile kernel."""
    src, out = os.path.join(str(tmp_path), f"n{n}.hip"), os.path.join(str(tmp_path), f"n{n}.s")
    with open(src, "w") as f:
        f.write(SOURCE % {"n": n})
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    r = subprocess.run([B.HIPCC, *flags, "-I", B.CSRC, "--cuda-device-only", "-S", src, "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        asm = f.read()
    counts = []
    for kernel in ("k_resid_dhtx_z", "k_resid_dhtx_s"):
        body = re.search(r"^_Z\w*%s\w*:.*?^\.Lfunc_end" % kernel, asm, re.S | re.M)
        assert body, kernel
        counts.append(len(re.findall(r"\bv_(?:fma|fmac|mul)_f64", body.group(0))))
    return counts


@pytest.mark.parametrize("n", [16, 24, 32, 48, 96])
def test_short_rows_square_in_fp64(n, tmp_path):
    # beside the decision's: two rows x two norms per plane, 8 planes of a flush, 2
    # of a small tile
    march, small = _fp64_products(n, tmp_path)
    march64, small64 = _fp64_products(64, tmp_path)
    assert march - march64 >= 4 * 8 and small - small64 >= 4 * 2
