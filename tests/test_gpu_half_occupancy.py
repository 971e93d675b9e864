"""The half-INT8 kernel with three (d = 64: four) wavefronts per SIMD, for calls with many workgroups, against the same heads in a call that has
two, bit for bit, and against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from helpers import route, wavefronts
from test_gpu_few_query_dispatch import problem

pytestmark = pytest.mark.gpu


# (heads, heads of the call with two, Nq, Nk, causal, d): just beyond a line of the rule and at it or below; whole, ragged and single key blocks
@pytest.mark.parametrize("heads,few,Nq,Nk,causal,d", [
    (129, 128, 449, 449, False, 64), (513, 512, 65, 640, False, 64), (257, 256, 511, 512, True, 64), (520, 500, 128, 128, True, 64), (600, 512, 100, 127, True, 64),
    (129, 128, 449, 449, False, 128), (257, 256, 450, 385, False, 128), (513, 512, 66, 641, False, 128), (313, 312, 500, 500, True, 128), (208, 173, 1664, 1664, True, 128), (560, 250, 600, 600, True, 128), (209, 208, 768, 768, True, 128), (520, 500, 128, 128, True, 128),
    (172, 170, 257, 300, True, 128), (129, 128, 400, 1000, True, 128), (32, 31, 4400, 4400, True, 128), (66, 65, 3800, 3800, True, 64)])
def test_rows_do_not_depend_on_the_wavefronts_per_simd(heads, few, Nq, Nk, causal, d):
    import paper_2409_16997_amd as ifa
    assert route(heads, Nq, Nk, d, half=True) == route(few, Nq, Nk, d, half=True) == "fused"
    assert (wavefronts(heads, Nq, Nk, d, causal, half=True), wavefronts(few, Nq, Nk, d, causal, half=True)) == (4 if d == 64 else 3, 2)
    q8, k8, v8, sq, sk = problem(heads, max(Nq, Nk), d, heads + Nk)
    q8, sq = q8[:, :, :Nq].contiguous(), sq[:, :, :Nq].contiguous()
    k8, sk = (t[:, :, :Nk].contiguous() for t in (k8, sk))
    v = v8[:, :, :Nk].to(torch.float16) / 64
    ops = (q8, k8, v, sq, sk)
    for dtype in (torch.float32, torch.float16, torch.bfloat16):
        full = ifa.int_flash_attn_fwd_half(*ops, causal=causal, out_dtype=dtype)
        assert torch.equal(ifa.int_flash_attn_fwd_half(*[t[:, :few].contiguous() for t in ops], causal=causal, out_dtype=dtype), full[:, :few])
        assert torch.equal(ifa.int_flash_attn_fwd_half(*[t[:, heads - few:].contiguous() for t in ops], causal=causal, out_dtype=dtype), full[:, heads - few:])
    full = ifa.int_flash_attn_fwd_half(*ops, causal=causal, out_dtype=torch.float32)
    h = heads - 1
    n = lambda t: t[0, h:h + 1].cpu().numpy()
    rows = np.arange(Nq) if Nq < 2000 else np.arange(0, Nq, 37)
    ref = oracle.int_flash_attn_fwd_half(n(q8), n(k8), n(v), n(sq), n(sk), causal, ifa.block_cols_half(d, causal), row_idx=rows)["O"]
    assert np.abs(full[0, h].cpu().numpy()[rows] - ref).max() <= 1e-3 * np.abs(ref).max()


# s_Q and s_K are any positive fp32.  A power of two moved from one to the other leaves every product, and so every row, as it is: for all rows, and for one row of a
# call that alone leaves the range in which the kernels of many workgroups carry the scores.  (s_K is 2^-8.5 at least: at 2^-117 of it still a normal number.)
@pytest.mark.parametrize("power", [80, 97, 110, 117])
@pytest.mark.parametrize("d,heads,N,causal", [(128, 260, 400, False), (64, 300, 385, True), (128, 520, 128, True)])
def test_rows_with_scales_far_from_one(d, heads, N, causal, power):
    import paper_2409_16997_amd as ifa
    q8, k8, v8, sq, sk = problem(heads, N, d, power)
    v = v8.to(torch.float16) / 64
    call = lambda a, b: ifa.int_flash_attn_fwd_half(q8, k8, v, a, b, causal=causal, out_dtype=torch.float32)
    ref = call(sq, sk)
    assert torch.equal(call(sq * 2.0 ** power, sk * 2.0 ** -power), ref)
    one = torch.where(torch.arange(N, device="cuda") == 77, sq, sq * 2.0 ** -power)     # the other rows see scores of about zero
    assert torch.equal(call(one * 2.0 ** power, sk * 2.0 ** -power)[:, :, 77], ref[:, :, 77])
