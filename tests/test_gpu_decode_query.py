"""The decode kernel (one query per head) and its form for two to eight: the rows of the few-query kernel, bit for bit, and the oracle's."""
import pytest

torch = pytest.importorskip("torch")

import oracle
from helpers import route
from test_gpu_few_query_dispatch import problem
from test_routes import library_says


def taken(heads, Nq, Nk, d):
    return (Nq == 1 or Nq <= 8 and Nk > 384) and heads <= (64 if d == 128 else 128) and route(heads, Nq, Nk, d, True) == "few"


def test_rule_is_the_librarys(tmp_path):
    program = ('#include "intfa_internal.h"\n#include <cstdio>\nint main() { int h, q, k, d; while (scanf("%d %d %d %d", &h, &q, &k, &d) == 4) '
               'puts(ifa_fwd_kernel(h, q, k, d, true) == IFA_KERNEL_FEW && ifa_decode_query(h, q, k, d) ? "1" : "0"); }\n')
    cases = [(h, q, k, d) for h in (1, 8, 63, 64, 65, 127, 128, 129, 300) for q in (1, 2, 8, 9, 32) for k in (1, 128, 129, 384, 385, 5000) for d in (64, 128)]
    assert library_says(tmp_path, program, cases) == ["01"[taken(*c)] for c in cases]


def check(heads, Nq, Nk, d, vblock, masks):
    import paper_2409_16997_amd as ifa
    more = 65 if d == 128 else 129                               # heads of a call that runs the few-query kernel
    assert taken(heads, Nq, Nk, d) and not taken(more, Nq, Nk, d) and route(more, Nq, Nk, d, True) == "few"
    q8, k8, v8, sq, sk = problem(heads, Nk, d, heads + Nk)
    q8, sq = q8[:, :, Nk - Nq:].contiguous(), sq[:, :, Nk - Nq:].contiguous()
    Bc = ifa.block_cols(d, True)
    g = torch.Generator(device="cuda").manual_seed(Nk)
    sv = 0.005 + 0.02 * torch.rand((1, heads) + ((-(-Nk // Bc),) if vblock else ()), generator=g, device="cuda")
    ops = (q8, k8, v8, sq, sk, sv)
    wide = [torch.cat([t] * -(-more // heads), 1)[:, :more].contiguous() for t in ops]
    for causal in masks:
        ref = ifa.int_flash_attn_fwd(*wide, causal=causal, out_dtype=torch.float32)[:, :heads]
        got = ifa.int_flash_attn_fwd(*ops, causal=causal, out_dtype=torch.float32)
        assert torch.equal(got, ref), causal
        for dtype in (torch.float16, torch.bfloat16):            # the fp32 rows rounded once, nothing around them written
            n = heads * Nq
            buf = torch.full((8 + n + 8, d), 77.0, dtype=dtype, device="cuda")
            ifa.int_flash_attn_fwd(*ops, causal=causal, out=buf[8:8 + n].view(1, heads, Nq, d))
            assert torch.equal(buf[8:8 + n].view(1, heads, Nq, d), got.to(dtype))
            assert bool((buf[:8] == 77.0).all()) and bool((buf[8 + n:] == 77.0).all())
        n = lambda t: t[0, heads - 1:].cpu().numpy()
        res = oracle.compare_up_to_ties(got[0, heads - 1].cpu().numpy(), n(q8), n(k8), n(v8), n(sq), n(sk), n(sv), causal, Bc)
        assert float(res["err"].max()) <= 1e-3 * float(res["scale"])


# Lengths at the edges of a key quad, a key tile, a block and a window of 2048 keys, the last window with one block, with all, with a block of one key;
# head counts that fill no round of eight XCDs, and the most it takes
@pytest.mark.gpu
@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,Nk", [(1, 129), (3, 131), (8, 160), (5, 161), (64, 255), (64, 256), (7, 257), (9, 1025), (4, 2047), (8, 2048), (3, 2049), (5, 2176), (2, 2177), (33, 4095), (8, 4097),
                                      (1, 20001)])
def test_rows_of_the_decode_kernel(heads, Nk, d, vblock):
    check(heads, 1, Nk, d, vblock, (True, False))


# ... and, under the mask, queries whose last keys lie in one block, in two (Nk - Nq < a multiple of 128 < Nk) and in two windows
@pytest.mark.gpu
@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Nq", [2, 3, 7, 8])
@pytest.mark.parametrize("heads,Nk", [(1, 385), (3, 515), (64, 512), (9, 1027), (4, 2047), (8, 2048), (3, 2050), (5, 2180), (33, 4095), (8, 4101)])
def test_rows_of_its_form_for_a_few_queries(heads, Nk, Nq, d, vblock):
    check(heads, Nq, Nk, d, vblock, (True, False))
