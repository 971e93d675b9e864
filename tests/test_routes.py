"""The rule that picks the kernel of a plain attention call, compiled for the host, against the Python statement of it that the GPU
tests use to say which kernel they reach (helpers.route)."""
import os
import subprocess

import pytest

from helpers import route

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "intfa_internal.h"
#include <cstdio>
int main() {
    int heads, Nq, Nk, d, half;
    while (scanf("%d %d %d %d %d", &heads, &Nq, &Nk, &d, &half) == 5)
        puts(!half && ifa_packed_queries(heads, Nq, Nk, d) ? "packed" : ifa_few_queries(heads, Nq, Nk, d, half) ? "few" : "fused");
    return 0;
}
"""


def test_helpers_route_is_the_librarys_rule(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "route.hip", tmp_path / "route"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2409_16997_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    cases = [(heads, Nq, Nk, d, half) for d in (64, 128) for half in (0, 1) for Nq in (1, 31, 32, 33, 64, 65, 127, 128, 1000)
             for heads in (1, 4, 8, 64, 65, 128, 129, 171, 256, 257, 300, 512, 513, 1000, 5 << 20, (5 << 20) + 1)
             for Nk in (1, 64, 65, 127, 128, 129, 256, 257, 384, 385, 1024, 1025, 1280, 1281, 2047, 2048, 16384)]
    text = "".join("%d %d %d %d %d\n" % c for c in cases)
    out = subprocess.run([str(exe)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    assert out == [route(*c) for c in cases]
