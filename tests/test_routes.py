"""The rule that picks the kernel of a plain attention call, compiled for the host, against the Python statement of it that the GPU
tests use to say which kernel they reach (helpers.route)."""
import os
import subprocess

import pytest

from helpers import route, unsplit

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "intfa_internal.h"
#include <cstdio>
int main() {
    const char *const name[] = {"fused", "pair", "packed", "few"};
    int heads, Nq, Nk, d, causal, half;
    while (scanf("%d %d %d %d %d %d", &heads, &Nq, &Nk, &d, &causal, &half) == 6)
        puts(half ? name[ifa_few_queries(heads, Nq, Nk, d, true) ? IFA_KERNEL_FEW : IFA_KERNEL_FUSED] : name[ifa_fwd_kernel(heads, Nq, Nk, d, causal)]);
    return 0;
}
"""


def library_says(tmp_path, program, cases):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "route.hip", tmp_path / "route"
    src.write_text(program)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2409_16997_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    text = "".join(" ".join(str(int(x)) for x in c) + "\n" for c in cases)
    return subprocess.run([str(exe)], input=text, stdout=subprocess.PIPE, text=True, check=True).stdout.split()


def test_helpers_route_is_the_librarys_rule(tmp_path):
    cases = [(heads, Nq, Nk, d, causal, half) for d in (64, 128) for causal, half in ((0, 0), (1, 0), (0, 1)) for Nq in (1, 31, 32, 33, 64, 65, 127, 128, 1000, 4100, 8192)
             for heads in (1, 2, 4, 8, 9, 64, 65, 128, 129, 171, 256, 257, 300, 512, 513, 1000, 1024, 1025, 5 << 20, (5 << 20) + 1)
             for Nk in (1, 64, 65, 127, 128, 129, 256, 257, 383, 384, 385, 511, 512, 768, 769, 1024, 1025, 1152, 1153, 1280, 1281, 2047, 2048, 7168, 7169, 16384, 28672, 28673)]
    assert library_says(tmp_path, PROGRAM, cases) == [route(*c) for c in cases]


SPLIT_PROGRAM = r"""
#include "intfa_internal.h"
#include <cstdio>
int main() {
    int heads, Nq, Nk, d;
    while (scanf("%d %d %d %d", &heads, &Nq, &Nk, &d) == 4) puts(ifa_unsplit_queries(heads, Nq, Nk, d) ? "1" : "0");
    return 0;
}
"""


def test_helpers_unsplit_is_the_librarys_rule(tmp_path):
    cases = [(heads, Nq, Nk, d) for d in (64, 128) for Nq in range(1, 33) for heads in (1, 2, 8, 15, 16, 17, 31, 32, 33, 64, 71, 72, 95, 96, 112, 129, 160, 6_000_000)
             for Nk in (1, 2, 2047, 2048, 2049, 2304, 2305, 3000, 4096, 4097, 8192, 16384, 32768, 1 << 20, 1 << 24)]
    assert library_says(tmp_path, SPLIT_PROGRAM, cases) == ["01"[unsplit(*c)] for c in cases]


# Calls of the key-split entry points beside which the other side measured at least 11 % slower, on the same K and V and on K and V in rotation
@pytest.mark.parametrize("heads,Nq,Nk,d,few", [
    (56, 4, 2500, 128, True), (56, 1, 2500, 128, True), (32, 32, 2100, 128, True), (48, 32, 8192, 128, True), (144, 4, 8192, 64, True), (48, 32, 2100, 64, True),
    (88, 32, 6000, 64, True), (64, 16, 8192, 128, True), (32, 1, 16384, 128, False), (32, 16, 8192, 128, False), (48, 9, 16384, 128, False), (40, 16, 8192, 64, False),
    (64, 5, 16384, 64, False), (24, 32, 16384, 128, False), (48, 1, 8192, 64, False)])
def test_key_split_calls_on_the_faster_side(heads, Nq, Nk, d, few):
    assert unsplit(heads, Nq, Nk, d) == few
