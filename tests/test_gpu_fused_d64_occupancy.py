"""The fused kernel at d = 64 with three wavefronts per SIMD (those of ifa_fused_wavefronts()) against the same
heads in a call that has two, bit for bit, and against the oracle."""
import pytest

torch = pytest.importorskip("torch")

import oracle
from helpers import route, wavefronts
from test_gpu_few_query_dispatch import problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("heads,few,Nq,Nk,causal", [
    (129, 128, 385, 385, False), (129, 128, 512, 511, False), (513, 512, 66, 641, False),         # 516 and 513 workgroups against 512
    (217, 216, 500, 500, True), (173, 172, 513, 513, True),                                        # 868 and 865 against 864 and 860, uneven
    (188, 187, 1500, 1500, True), (79, 78, 2001, 2001, True),                                      # 2256 against 2244, 1264 against 1248
    (520, 500, 128, 128, True), (172, 170, 257, 300, True), (260, 250, 130, 900, True),            # one, three and two query blocks a head
    (257, 256, 400, 401, False), (112, 111, 2500, 2500, True)])                                    # beyond two rounds of 512; beyond one and a half groups of heads
def test_rows_do_not_depend_on_the_wavefronts_per_simd(heads, few, Nq, Nk, causal, vblock):
    import paper_2409_16997_amd as ifa
    d = 64
    assert route(heads, Nq, Nk, d, causal) == route(few, Nq, Nk, d, causal) == "fused"
    assert (wavefronts(heads, Nq, Nk, d, causal), wavefronts(few, Nq, Nk, d, causal)) == (3, 2)
    q8, k8, v8, sq, sk = problem(heads, max(Nq, Nk), d, heads + Nk)
    q8, sq = q8[:, :, :Nq].contiguous(), sq[:, :, :Nq].contiguous()
    k8, v8, sk = (t[:, :, :Nk].contiguous() for t in (k8, v8, sk))
    Bc = ifa.block_cols(d, causal)
    g = torch.Generator(device="cuda").manual_seed(Nk)
    sv = 0.005 + 0.02 * torch.rand((1, heads) + ((-(-Nk // Bc),) if vblock else ()), generator=g, device="cuda")
    ops = (q8, k8, v8, sq, sk, sv)
    for dtype in (torch.float32, torch.float16, torch.bfloat16):
        full = ifa.int_flash_attn_fwd(*ops, causal=causal, out_dtype=dtype)
        assert torch.equal(ifa.int_flash_attn_fwd(*[t[:, :few].contiguous() for t in ops], causal=causal, out_dtype=dtype), full[:, :few])
        assert torch.equal(ifa.int_flash_attn_fwd(*[t[:, heads - few:].contiguous() for t in ops], causal=causal, out_dtype=dtype), full[:, heads - few:])
    full = ifa.int_flash_attn_fwd(*ops, causal=causal, out_dtype=torch.float32)
    h = heads - 1
    n = lambda t: t[0, h:h + 1].cpu().numpy()
    res = oracle.compare_up_to_ties(full[0, h].cpu().numpy(), n(q8), n(k8), n(v8), n(sq), n(sk), n(sv), causal, Bc)
    assert float(res["err"].max()) <= 1e-3 * float(res["scale"])
