"""The two-group kernel (two groups of 32 queries of a head per workgroup): the rows of the other kernels, bit for bit, and the
calls its rule takes."""
import pytest

torch = pytest.importorskip("torch")

import oracle
from helpers import route
from test_gpu_few_query_dispatch import problem

# (heads, Nq, Nk): an odd number of key blocks and a ragged one, a last workgroup without its second group (Nq = 33, 65, 96: all but or half
# empty), more than one query per key block of the mask, and (the last two, under the mask only) more workgroups than CUs
SHAPES = [(129, 64, 512), (130, 33, 513), (90, 65, 640), (65, 96, 1023), (37, 200, 1025), (24, 384, 700), (16, 1000, 1000), (8, 2048, 2048), (9, 1999, 2049)]


def taken(heads, Nq, Nk, d, causal):
    return route(heads, Nq, Nk, d, causal) == "pair"


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
