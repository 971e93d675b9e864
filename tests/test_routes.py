"""The rules that pick the kernel of a call, compiled for the host, against a Python statement of them.  (The GPU tests ask the library: helpers.route, helpers.unsplit.)"""
import os
import subprocess

import pytest

from helpers import route, unsplit, wavefronts

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def stated_route(heads, Nq, Nk, d, causal=None, half=False, vblock=False):
    """The rule of helpers.route, stated again."""
    groups = heads * -(-Nq // 32)
    if not half:
        assert causal is not None
        if Nq > 32 and groups > 256:
            wgs, uneven = heads * -(-Nq // 64), causal and 2 * Nq >= Nk
            if wgs <= 256:
                pair = Nk >= (512 if d == 128 else 384) and not (uneven and Nk >= 2048 and (heads == 1 or wgs <= 192))
            else:
                keys = heads * Nk
                if not causal or (4 if not vblock else 3 if d == 64 else 3.5) * Nq < Nk:
                    pair = False
                elif wgs <= 512:
                    a, b, c = {(64, 0): (3, 2.5, 200), (64, 1): (3, 7, 200), (128, 0): (4, 3, 100), (128, 1): (4.5, 5, 400)}[d, int(vblock)]
                    pair = (Nk + c) * Nq >= wgs * (a * Nq + b * max(Nk - 1.125 * Nq, 0))
                elif vblock:
                    pair = (wgs <= ((680 if d == 128 else 640) if heads <= 8 else 576 if heads <= 10 else 0) and 4 * Nk <= (6 if d == 128 else 5) * Nq and
                            keys <= (48 if d == 128 else 40) << 10)
                else:
                    pair = uneven and Nk >= 2048 and keys <= 56 << 10 and (heads <= 8 and wgs <= 768 or wgs <= 576 and Nk >= (4000 if d == 128 else 3000) and
                                                                           (heads <= 10 or 4 * Nk <= 5 * Nq))
            if pair:
                return "pair"
        if Nk <= 128 if groups <= 256 else d == 64 and (Nk <= (768 if groups <= 1024 else 1152) if Nq <= 32 else
                                                        Nq <= 64 and groups <= 512 and 128 <= Nk < 384):
            return "packed"
    short_keys = {(True, 128): 256, (True, 64): 64, (False, 128): 384, (False, 64): 0}[half, d]
    if groups <= 5 << 20 and (groups <= 256 or (Nk > short_keys if Nq <= 32 else groups <= 512 and Nk >= 2048)):
        return "few"
    return "fused"


def stated_unsplit(heads, Nq, Nk, d):
    """The rule of helpers.unsplit, stated again."""
    if heads <= (64 if d == 128 else 128) and (Nq == 1 or Nq <= 8 and Nk > 384):      # the decode kernel's
        return Nk <= 3000 + 75 * heads or heads >= 108 if Nq == 1 else Nk <= 2000 + (86 + 4 * Nq) * heads or heads >= 120 - 3 * Nq
    if Nq <= 8:
        E, S, H = (2048, 1536, 134 - 5 * Nq) if d == 128 else (1024, 1536, 146 - 7 * Nq)
    else:
        E, S, H = 1024, 2304, (104 if d == 128 else 122) - Nq
    return Nk <= 2048 or heads * (Nk + E) >= H * (Nk - S)


PROGRAM = r"""
#include "intfa_internal.h"
#include <cstdio>
int main() {
    const char *const name[] = {"fused", "pair", "packed", "few"};
    int heads, Nq, Nk, d, causal, half, vblock;
    while (scanf("%d %d %d %d %d %d %d", &heads, &Nq, &Nk, &d, &causal, &half, &vblock) == 7)
        puts(half ? name[ifa_few_queries(heads, Nq, Nk, d, true) ? IFA_KERNEL_FEW : IFA_KERNEL_FUSED] : name[ifa_fwd_kernel(heads, Nq, Nk, d, causal, vblock)]);
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
    cases = [(heads, Nq, Nk, d, causal, half, vblock) for d in (64, 128) for causal, half, vblock in ((0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 0, 1)) for Nq in (1, 31, 32, 33, 64, 65, 127, 128, 1000, 4100, 8192)
             for heads in (1, 2, 4, 8, 9, 64, 65, 128, 129, 171, 256, 257, 300, 512, 513, 1000, 1024, 1025, 5 << 20, (5 << 20) + 1)
             for Nk in (1, 64, 65, 127, 128, 129, 256, 257, 383, 384, 385, 511, 512, 768, 769, 1024, 1025, 1152, 1153, 1280, 1281, 2047, 2048, 7168, 7169, 16384, 28672, 28673)]
    assert library_says(tmp_path, PROGRAM, cases) == [stated_route(*c) for c in cases] == [route(*c) for c in cases]


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
    assert library_says(tmp_path, SPLIT_PROGRAM, cases) == ["01"[stated_unsplit(*c)] for c in cases] == ["01"[unsplit(*c)] for c in cases]


# Causal calls with more workgroups of 64 queries than CUs: the side on which a call ran at least 8 % faster
@pytest.mark.parametrize("heads,Nq,Nk,d,vblock,kernel", [
    (12, 1444, 1444, 128, False, "pair"), (3, 5898, 14531, 128, False, "pair"), (10, 3380, 3380, 64, False, "pair"), (23, 995, 1791, 128, False, "fused"), (43, 526, 2081, 64, False, "fused"),
    (39, 565, 922, 64, False, "fused"), (12, 1444, 1444, 128, True, "pair"), (12, 3047, 4490, 64, True, "fused"), (43, 526, 2081, 64, True, "fused"), (21, 1419, 5215, 64, True, "fused"),
    (26, 846, 1479, 128, True, "fused"), (5, 9696, 9696, 64, True, "fused"), (13, 2813, 3520, 64, True, "fused")])
def test_calls_with_a_second_wave_on_the_faster_side(heads, Nq, Nk, d, vblock, kernel):
    assert route(heads, Nq, Nk, d, True, vblock=vblock) == kernel


# Calls of the key-split entry points beside which the other side measured at least 11 % slower, on the same K and V and on K and V in rotation
@pytest.mark.parametrize("heads,Nq,Nk,d,few", [
    (56, 4, 2500, 128, True), (56, 1, 2500, 128, True), (32, 32, 2100, 128, True), (48, 32, 8192, 128, True), (144, 4, 8192, 64, True), (48, 32, 2100, 64, True),
    (88, 32, 6000, 64, True), (64, 16, 8192, 128, True), (32, 1, 16384, 128, False), (32, 16, 8192, 128, False), (48, 9, 16384, 128, False), (40, 16, 8192, 64, False),
    (64, 5, 16384, 64, False), (24, 32, 16384, 128, False), (48, 1, 8192, 64, False)])
def test_key_split_calls_on_the_faster_side(heads, Nq, Nk, d, few):
    assert unsplit(heads, Nq, Nk, d) == few


# Wavefronts per SIMD where a call ran at least 4 % faster with two, or with more
@pytest.mark.parametrize("heads,Nq,Nk,d,causal,half,more", [
    (45, 5740, 5740, 64, True, False, False), (50, 6174, 6174, 64, True, False, False), (88, 3016, 3016, 64, True, False, False), (100, 1732, 1732, 64, True, False, False),
    (83, 2116, 2116, 64, True, False, True), (128, 4096, 4096, 64, True, False, True), (300, 250, 250, 64, False, False, True), (50, 4446, 4446, 64, True, True, False),
    (40, 4948, 4948, 64, True, True, False), (82, 2008, 2008, 64, True, True, True), (490, 180, 685, 128, True, True, False), (32, 5120, 5120, 128, False, True, True),
    (267, 768, 768, 128, True, True, True), (192, 668, 668, 128, True, True, False)])
def test_wavefronts_on_the_faster_side(heads, Nq, Nk, d, causal, half, more):
    assert (wavefronts(heads, Nq, Nk, d, causal, half) > 2) == more
