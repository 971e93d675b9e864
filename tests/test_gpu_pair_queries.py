"""The two-group kernel (two groups of 32 queries of a head per workgroup): the rows of the other kernels, bit for bit, and the
calls its rule takes."""
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")

import oracle
from test_gpu_few_query_dispatch import problem

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (heads, Nq, Nk): an odd number of key blocks and a ragged one, a last workgroup without its second group (Nq = 33, 65, 96: all but or half
# empty), more than one query per key block of the mask, and (the last two, under the mask only) more workgroups than CUs
SHAPES = [(129, 64, 512), (130, 33, 513), (90, 65, 640), (65, 96, 1023), (37, 200, 1025), (24, 384, 700), (16, 1000, 1000), (8, 2048, 2048), (9, 1999, 2049)]


def taken(heads, Nq, Nk, d, causal):
    if Nq <= 32 or heads * -(-Nq // 32) <= 256:
        return False
    wgs, uneven = heads * -(-Nq // 64), causal and 2 * Nq >= Nk
    if wgs <= 256:
        return Nk >= (512 if d == 128 else 384) and not (uneven and Nk >= 2048 and (heads == 1 or wgs <= 192))
    return uneven and Nk >= 2048 and (wgs <= 512 or heads <= 8 and wgs <= 768 and heads * Nk <= 56 << 10)


def test_rule_is_the_librarys(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "pair.hip", tmp_path / "pair"
    src.write_text('#include "intfa_internal.h"\n#include <cstdio>\nint main() { int h, q, k, d, c; '
                   'while (scanf("%d %d %d %d %d", &h, &q, &k, &d, &c) == 5) puts(ifa_pair_queries(h, q, k, d, c) ? "1" : "0"); }\n')
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2409_16997_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    cases = [(h, q, k, d, c) for h in (1, 2, 8, 9, 64, 65, 128, 129, 256, 257, 5 << 20) for q in (1, 32, 33, 64, 65, 2000, 4100, 6000, 8192, 16384, 24000, 32768, 48000)
             for k in (64, 383, 384, 511, 512, 2047, 2048, 4000, 4001, 7168, 7169, 16384, 28672, 28673, 32768, 57344, 57345) for d in (64, 128) for c in (0, 1)]
    out = subprocess.run([str(exe)], input="".join("%d %d %d %d %d\n" % c for c in cases), stdout=subprocess.PIPE, text=True, check=True).stdout.split()
    assert out == ["01"[taken(*c)] for c in cases]


@pytest.mark.gpu
@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("heads,Nq,Nk,d,causal", [s + (d, c) for s in SHAPES for d in (64, 128) for c in (False, True) if taken(*s, d, c)])
def test_rows_of_the_two_group_kernel(heads, Nq, Nk, d, causal, vblock):
    import paper_2409_16997_amd as ifa
    q8, k8, v8, sq, sk = problem(heads, Nk, d, heads + Nk)
    q8, sq = q8[:, :, Nk - Nq:].contiguous(), sq[:, :, Nk - Nq:].contiguous()
    Bc = ifa.block_cols(d, causal)
    g = torch.Generator(device="cuda").manual_seed(Nk)
    sv = 0.005 + 0.02 * torch.rand((1, heads) + ((-(-Nk // Bc),) if vblock else ()), generator=g, device="cuda")
    call = lambda *t: ifa.int_flash_attn_fwd(*t, causal=causal, out_dtype=torch.float32)
    full = call(q8, k8, v8, sq, sk, sv)
    few = 4 if Nq < 1999 else 2                                  # heads whose calls have at most 256 groups of 32 queries
    assert not taken(few, Nq, Nk, d, causal)
    for h in range(0, heads - few + 1, max(1, heads // 3)):
        assert torch.equal(call(*[t[:, h:h + few].contiguous() for t in (q8, k8, v8, sq, sk, sv)]), full[:, h:h + few])
    n = lambda t: t[0, :1].cpu().numpy()
    if Nq <= 384:
        res = oracle.compare_up_to_ties(full[0, 0].cpu().numpy(), n(q8), n(k8), n(v8), n(sq), n(sk), n(sv), causal, Bc)
        assert float(res["err"].max()) <= 1e-3 * float(res["scale"])
