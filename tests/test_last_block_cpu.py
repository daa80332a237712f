"""The hand-over to a launch's last block, in the code that the compiler makes of
it: the last block may write the solve's state as soon as every block's thread 0
has arrived, so a block must not arrive before all its waves have read that state
and all its stores are out.  Compiles kernels to gfx950 assembly; runs nothing."""
import os
import re
import subprocess

import pytest

from paper_1601_05448_amd import build as B

PROBE = """
#include "poisson_device.hpp"
namespace pois {
__global__ void __launch_bounds__(256) k_probe(const Slot* __restrict__ slots, double* out) {
    const Slot& s = slots[blockIdx.y];
    if (s.st->stage != 2) return;
    const double scale = s.st->inv_s;
    out[blockIdx.x * 256 + threadIdx.x] = scale;
    if (last_block(s) && threadIdx.x == 0) s.st->stage = 0;
}
}  // namespace pois
"""


def _assembly(src, tmp_path):
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    out = os.path.join(str(tmp_path), "out.s")
    r = subprocess.run([B.HIPCC, *flags, "-I", B.CSRC, "--cuda-device-only", "-S", str(src), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def _instructions(asm, kernel):
    """The kernel's instructions in program order."""
    body = re.search(r"^_Z\w*%s\w*:.*?s_endpgm" % kernel, asm, re.S | re.M)
    assert body, kernel
    return [line.split(";")[0].strip() for line in body.group(0).splitlines()
            if re.match(r"\s+[a-z]\w+", line)]


@pytest.mark.parametrize("kernel", ["k_probe", "k_setup", "k_outer_update"])
def test_a_block_arrives_after_all_its_waves(kernel, tmp_path):
    src = os.path.join(B.CSRC, "poisson_kernels.hip")
    if kernel == "k_probe":
        src = tmp_path / "probe.hip"
        src.write_text(PROBE)
    ins = _instructions(_assembly(src, tmp_path), kernel)
    arrive = next(i for i, x in enumerate(ins) if re.match(r"(flat|global)_atomic_add", x))
    barrier = [i for i in range(arrive) if ins[i] == "s_barrier"]
    assert barrier, "thread 0 arrives with no barrier after the waves' reads of the state"
    # up to that barrier: every vector access of global memory is waited for
    access = [i for i in range(barrier[-1]) if re.match(r"(flat|global|buffer)_(load|store)", ins[i])]
    waits = [i for i in range(barrier[-1]) if ins[i].startswith("s_waitcnt") and "vmcnt(0)" in ins[i]]
    assert access and waits and waits[-1] > access[-1], ins[access[-1]:barrier[-1] + 1]
    # and none between it and the arrival but what the arrival itself needs (loads)
    assert not [x for x in ins[barrier[-1]:arrive] if re.match(r"(flat|global|buffer)_store", x)]
