"""Key-split calls of 9 to 32 queries around the run length from which the second pass keeps three blocks of K and V in its ring (d = 64, nine
blocks), with ragged last blocks and short last runs, against the rows of the plain call."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_few_query_dispatch import problem

pytestmark = pytest.mark.gpu


def run_length(heads, Nk):
    blocks = -(-Nk // 128)
    return min(blocks, max(4, -(-blocks // max(1, 1024 // heads))))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,Nq", [(64, 9), (64, 32), (128, 16)])
@pytest.mark.parametrize("heads,Nk,run", [(64, 16384, 8), (64, 16385, 9), (62, 17000, 9), (32, 33000, 9), (40, 40000, 13), (1, 600, 4)])
def test_runs_of_either_ring(heads, Nk, run, d, Nq, causal):
    import paper_2409_16997_amd as ifa
    assert run_length(heads, Nk) == run
    q8, k8, v8, sq, sk = problem(heads, Nk, d, heads + Nk)
    q8, sq = q8[:, :, Nk - Nq:].contiguous(), sq[:, :, Nk - Nq:].contiguous()
    sv = 0.005 + 0.02 * torch.rand((1, heads), device="cuda", generator=torch.Generator(device="cuda").manual_seed(Nk))
    ref = ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, sv, causal=causal, out_dtype=torch.float32)
    out = ifa.int_flash_attn_fwd_splitk(q8, k8, v8, sq, sk, sv, causal=causal, out_dtype=torch.float32)
    # P and the integer sums are the same; the fp32 additions of O and l have another order (a few ulp of the largest value)
    assert float((out - ref).abs().max()) <= 4e-6 * float(ref.abs().max())
