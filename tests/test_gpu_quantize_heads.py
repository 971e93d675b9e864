"""Tensor-level quantization of V where its ways of walking a head meet: a head held in registers by one workgroup, read a
second time by it, or cut into parts and regions over two launches.  Bit for bit against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu

# 6144 chunks of 8 elements stay in registers (4-byte ones: 3072), 4096 more per step of the loop behind (2048).  Whole heads up to 64 KB
# + 4 KB per head or from 96 heads on, except long ones that leave CUs without one (V alone, not in quantize_qkv); heads of up to
# 16 KB of more than 512 heads go to smaller workgroups (V alone).
SHAPES = [
    (1, 1, 64), (1, 272, 64), (1, 273, 64), (1, 544, 64), (1, 545, 64),   # one workgroup or parts: 68 KB at 4 and at 2 bytes
    (3, 577, 128), (2, 1151, 64),                        # parts: remainders in the last part and region
    (1, 16384, 128), (5, 4099, 128),                     # 64 and more parts wanted
    (96, 767, 64), (96, 768, 64), (97, 769, 64),         # whole heads at the end of the registers (6144 chunks)
    (96, 1279, 64), (96, 1280, 64), (96, 1281, 64),      # ... and at one full step of the loop (10240 chunks)
    (96, 1025, 128), (100, 1793, 64),
    (96, 4096, 128), (96, 4097, 128), (260, 1024, 128), (260, 1025, 128),   # 1 MB and 256 KB per head at 2 bytes: whole up to here, then in parts
    (513, 1, 64), (513, 63, 64), (513, 64, 64), (513, 65, 64), (520, 128, 64), (520, 129, 64), (512, 7, 64),   # 16 KB per head at 4 and at 2 bytes
    (96, 2741, 128), (33, 4099, 128),                    # more rows of Q and K than one sweep of the launch (whole 262144, parts 131072)
]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("heads,N,d", SHAPES)
def test_headwise_codes_and_scales(heads, N, d, dtype):
    import paper_2409_16997_amd as ifa
    g = torch.Generator(device="cuda").manual_seed(heads * 7919 + N)
    V = torch.randn((1, heads, N, d), generator=g, device="cuda").to(dtype)
    at = torch.randint(0, N * d, (heads,), generator=g, device="cuda")
    V.view(heads, -1)[torch.arange(heads, device="cuda"), at] = 9.0     # the maximum of each head, once, anywhere in it
    V[0, 0, N - 1, d - 1] = -11.0                                       # ... and at the very end of the first
    V[0, heads // 2] *= 0.0 if heads > 1 else 1.0
    pick = sorted({0, heads // 2, heads - 1})
    rq, rs = oracle.quantize_headwise(V[0, pick].float().cpu().numpy())
    q, s = ifa.quantize_headwise(V)
    assert np.array_equal(q[0, pick].cpu().numpy(), rq) and np.array_equal(s[0, pick].cpu().numpy(), rs)
    Q, K = (torch.randn((1, heads, N, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    out = tuple(torch.full((1, heads, N, d), 77, dtype=torch.int8, device="cuda") for _ in range(3)) + tuple(
        torch.full(sh, 3.0e38, device="cuda") for sh in ((1, heads, N), (1, heads, N), (1, heads)))
    ifa.quantize_qkv(Q, K, V, out=out)
    assert torch.equal(out[2], q) and torch.equal(out[5], s)
    for x, c, sc in ((Q, out[0], out[3]), (K, out[1], out[4])):
        rq, rs = ifa.quantize_tokenwise(x)
        assert torch.equal(c, rq) and torch.equal(sc, rs)


# In shares: 32 KB a head (two shares) up to 256 or 384 KB (twelve), 64 heads; shares that do not divide the head, ends of the registers (96 KB a share
# with 64 heads of 256 KB + and 48 of 384), head counts that fill no round of eight, and the sizes on the other side of each line.
SHARES = [
    (1, 127, 128), (1, 128, 128), (1, 255, 64), (1, 256, 64), (3, 129, 128), (8, 131, 128), (9, 1023, 128), (1, 1024, 128), (1, 1025, 128),
    (7, 1537, 64), (8, 1536, 128), (8, 1537, 128), (16, 769, 64), (31, 333, 128), (48, 768, 128), (48, 1536, 128), (49, 1023, 64), (63, 512, 128), (64, 511, 128),
    (64, 1024, 128), (65, 512, 128), (64, 1025, 64)]


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("heads,N,d", SHARES)
def test_heads_in_shares(heads, N, d, dtype):
    test_headwise_codes_and_scales(heads, N, d, dtype)
