"""Every device helper that the kernels' headers define has a caller (the build does
not warn of unused functions: a header's kernels are not all taken by each file)."""
import glob
import os
import re

from paper_1601_05448_amd import build as B


def test_device_helpers_are_called_and_constants_defined_once():
    text = {f: open(f).read() for f in glob.glob(os.path.join(B.CSRC, "*.h*"))}
    code = re.sub(r"//[^\n]*", "", "\n".join(text.values()))
    helpers = set(re.findall(r"__device__ __forceinline__ (?:constexpr )?[\w:<>*& ]+?\b(\w+)\(", code))
    assert "hartley" in helpers and "last_block" in helpers
    unused = sorted(n for n in helpers if len(re.findall(r"\b%s\b" % n, code)) < 2)
    assert not unused, unused
    constants = re.findall(r"^constexpr \w+ (k\w+) =", code, re.M)
    twice = sorted({c for c in constants if constants.count(c) > 1})
    assert not twice, twice
