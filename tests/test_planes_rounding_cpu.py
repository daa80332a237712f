"""The fused y, z and y sweeps of small grids stand for two y sweeps and a z sweep
and promise their bits: in the code that the compiler makes of them the fused kernel
has as many fused FP64 multiply-adds as those three kernels (contraction across
statements differs from kernel to kernel; products and sums on their own round alike
wherever they stand).  Compiles to gfx950 assembly; runs nothing."""
import os
import re
import subprocess

import pytest

from paper_1601_05448_amd import build as B


@pytest.fixture(scope="module")
def operations(tmp_path_factory):
    """{kernel<its template arguments>: fused multiply-adds}"""
    out = str(tmp_path_factory.mktemp("planes") / "f64.s")
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    r = subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(B.CSRC, "poisson_planes_f64.hip"),
                        "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        asm = f.read()
    ops = {}
    for m in re.finditer(r"^_ZN4pois\d+(k_dht_\w+?)IdLi(\d+)ELi(\d+)EE\w*:.*?^\.Lfunc_end", asm, re.S | re.M):
        ops[m.group(1), int(m.group(2)), int(m.group(3))] = len(re.findall(r"\bv_fmac?_f64", m.group(0)))
    return ops


def test_the_fused_kernel_contracts_as_the_sweeps(operations):
    one = {}  # per length: the same for wide and narrow line groups
    for (kernel, n, _), ops in operations.items():
        if kernel != "k_dht_planes":
            assert one.setdefault((kernel, n), ops) == ops, (kernel, n)
    fused = [(ny, nz) for kernel, ny, nz in operations if kernel == "k_dht_planes"]
    lengths = (16, 24, 32, 48, 64)
    assert sorted(fused) == [(ny, nz) for ny in lengths for nz in lengths if ny * nz <= 48 * 48]
    for ny, nz in fused:
        y, z = one["k_dht_cols", ny], one["k_dht_z_solve", nz]
        assert operations["k_dht_planes", ny, nz] == 2 * y + z, (ny, nz)
