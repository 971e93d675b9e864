"""The two-group kernel (two groups of 32 queries of a head per workgroup): the rows of the other kernels, bit for bit, and the
calls its rule takes."""
import pytest

torch = pytest.importorskip("torch")

import oracle
from helpers import route
from test_gpu_few_query_dispatch import problem
from test_routes import library_says

# (heads, Nq, Nk): an odd number of key blocks and a ragged one, a last workgroup without its second group (Nq = 33, 65, 96: all but or half
# empty), more than one query per key block of the mask, exactly as many workgroups as CUs (8 x 2048) and, under the mask only, more (9 x 1999)
SHAPES = [(129, 64, 512), (130, 33, 513), (90, 65, 640), (90, 96, 1023), (37, 200, 1025), (24, 384, 700), (16, 1000, 1000), (8, 2048, 2048), (9, 1999, 2049)]


def taken(heads, Nq, Nk, d, causal):
    return route(heads, Nq, Nk, d, causal) == "pair"


def test_rule_is_the_librarys(tmp_path):
    program = ('#include "intfa_internal.h"\n#include <cstdio>\nint main() { int h, q, k, d, c; '
               'while (scanf("%d %d %d %d %d", &h, &q, &k, &d, &c) == 5) puts(ifa_pair_queries(h, q, k, d, c) ? "1" : "0"); }\n')
    cases = [(h, q, k, d, c) for h in (1, 2, 8, 9, 64, 65, 128, 129, 256, 257, 5 << 20) for q in (1, 32, 33, 64, 65, 2000, 4100, 6000, 8192, 16384, 24000, 32768, 48000)
             for k in (64, 383, 384, 511, 512, 2047, 2048, 4000, 4001, 7168, 7169, 16384, 28672, 28673, 32768, 57344, 57345) for d in (64, 128) for c in (0, 1)]
    assert library_says(tmp_path, program, cases) == ["01"[taken(*c)] for c in cases]


def test_every_shape_is_the_kernels():
    assert all(taken(*s, d, True) for s in SHAPES for d in (64, 128)) and all(taken(*s, d, False) for s in SHAPES[:-1] for d in (64, 128))


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


def windows(shape, d, causal, vblock):
    """Operands of a call and a function that gives rows a .. b - 1 of it from a call with those queries alone, which is another kernel's."""
    import paper_2409_16997_amd as ifa
    heads, Nq, Nk = shape
    q8, k8, v8, sq, sk = problem(heads, Nk, d, heads + Nk)
    q8, sq = q8[:, :, Nk - Nq:].contiguous(), sq[:, :, Nk - Nq:].contiguous()
    Bc = ifa.block_cols(d, causal)
    sv = 0.005 + 0.02 * torch.rand((1, heads) + ((-(-Nk // Bc),) if vblock else ()), generator=torch.Generator(device="cuda").manual_seed(Nk), device="cuda")

    def rows(a, b):
        n = Nk - Nq + b if causal else Nk                        # keys that the last of them sees
        assert not taken(heads, b - a, n, d, causal)
        return ifa.int_flash_attn_fwd(q8[:, :, a:b].contiguous(), k8[:, :, :n].contiguous(), v8[:, :, :n].contiguous(), sq[:, :, a:b].contiguous(),
                                      sk[:, :, :n].contiguous(), sv[:, :, :-(-n // Bc)].contiguous() if vblock else sv, causal=causal, out_dtype=torch.float32)
    return (q8, k8, v8, sq, sk, sv), rows


# More workgroups than CUs, up to the limits of the rule: 512, and 768 for up to 8 heads (which the mapping shares out over all XCDs)
@pytest.mark.gpu
@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,Nq,Nk", [(1, 17000, 17000), (4, 8192, 8192), (16, 2000, 2048), (8, 4096, 4500), (8, 6100, 6100), (5, 9000, 10001), (2, 24500, 24500)])
def test_rows_of_calls_with_more_workgroups_than_cus(heads, Nq, Nk, d, vblock):
    import paper_2409_16997_amd as ifa
    assert taken(heads, Nq, Nk, d, True) and heads * -(-Nq // 64) > 256
    args, rows = windows((heads, Nq, Nk), d, True, vblock)
    full = ifa.int_flash_attn_fwd(*args, causal=True, out_dtype=torch.float32)
    assert bool(torch.isfinite(full).all())
    step = Nq // 7
    for a in list(range(0, Nq - 64, step)) + [Nq - 64]:
        b = min(a + 64 + a % 5, Nq)
        out, ref = full[:, :, a:b], rows(a, b)
        # per-block V scales: a row may go through the scale of a block that only other rows of its group of 32 see, one change of unit (below 2^-21)
        assert bool(((out - ref).abs() <= 2.0 ** -21 * ref.abs()).all()) if vblock else torch.equal(out, ref), (a, b)


# ... on fewer keys, the sooner the fewer workgroups, with up to four times as many keys as queries, and a little beyond 512 of them
@pytest.mark.gpu
@pytest.mark.parametrize("vblock", [False, True])
@pytest.mark.parametrize("heads,Nq,Nk,d", [(12, 1444, 1444, 128), (10, 1996, 1996, 64), (26, 659, 659, 64), (19, 1000, 1117, 128), (3, 5898, 14531, 128), (8, 2050, 8200, 64),
                                           (10, 3380, 3380, 64), (9, 4010, 4010, 128)])
def test_rows_of_calls_with_a_short_second_wave(heads, Nq, Nk, d, vblock):
    test_rows_of_calls_with_more_workgroups_than_cus(heads, Nq, Nk, d, vblock)


# 2-byte outputs are the fp32 rows rounded once, and nothing around O is written
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("heads,Nq,Nk,d", [(130, 33, 513, 64), (130, 33, 513, 128), (90, 96, 1023, 64), (65, 100, 1023, 128), (37, 200, 1025, 128), (24, 384, 700, 64), (9, 1999, 2049, 128)])
def test_output_types_and_what_lies_around_them(heads, Nq, Nk, d, causal, dtype):
    import paper_2409_16997_amd as ifa
    if not taken(heads, Nq, Nk, d, causal):
        assert (heads, causal) == (9, False)                     # beyond 256 workgroups only under the mask
        return
    args, _ = windows((heads, Nq, Nk), d, causal, False)
    ref = ifa.int_flash_attn_fwd(*args, causal=causal, out_dtype=torch.float32)
    guard, n = 256, heads * Nq
    buf = torch.full((guard + n + guard, d), 77.0, dtype=dtype, device="cuda")
    ifa.int_flash_attn_fwd(*args, causal=causal, out=buf[guard:guard + n].view(1, heads, Nq, d))
    assert torch.equal(buf[guard:guard + n].view(1, heads, Nq, d), ref.to(dtype))
    assert bool((buf[:guard] == 77.0).all()) and bool((buf[guard + n:] == 77.0).all())
