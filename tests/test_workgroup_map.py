"""The mapping of workgroups of the fused kernels (two of which share a CU) and the two-group kernel (one to a CU) to (head, query block), compiled for the host: every pair exactly once, the whole
heads of a call on one XCD each, and the order that the mask asks for."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "intfa_device.h"
#include <cstdio>
#include <vector>
static int check(int heads, int T_r, int group, bool causal, bool paired) {
    const int W = heads * T_r;
    std::vector<int> seen(W, 0), last(8, -1);
    for (int L = 0; L < W; ++L) {
        int h = -1, q = -1;
        ifa_dev::map_workgroup(L, heads, T_r, group, causal, h, q, paired);
        if (h < 0 || h >= heads || q < 0 || q >= T_r || seen[h * T_r + q]++) return 1;
        const bool dealt = !causal && (heads & 7) && T_r >= 16;
        if (!dealt && h < heads / 8 * 8 && (h & 7) != (L & 7)) return 2;
        // one group: the ranks of an XCD never fall, except in the backward half of a call that starts all at once, where they never rise
        if (causal && heads / 8 <= group) {
            const bool back = paired && W <= 512 && (L >> 3) > 32;
            if ((!paired || (L >> 3) != 32) && (back ? q > last[L & 7] : q < last[L & 7])) return 3;
        }
        last[L & 7] = q;
    }
    return 0;
}
int main() {
    const int ranks[] = {1, 2, 3, 5, 7, 8, 15, 16, 17, 33, 64, 129};
    for (int heads = 1; heads <= 130; ++heads)
        for (int T_r : ranks)
            for (int group : {1, 2, 4, 8})
                for (int causal = 0; causal < 2; ++causal)
                    for (int paired = 0; paired < 2; ++paired)
                        if (int rc = check(heads, T_r, group, causal, paired)) { printf("heads %d blocks %d group %d causal %d paired %d: %d\n", heads, T_r, group, causal, paired, rc); return 1; }
    return 0;
}
"""


def test_every_query_block_once_in_the_stated_order(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "map.hip", tmp_path / "map"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2409_16997_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert res.returncode == 0, res.stdout
