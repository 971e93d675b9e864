"""The plain calls of the binding, which go through its native module, and the same calls on the general path behind it: the same
results and the same refusals.  (An active torch function mode sends every call the general way.)"""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def general(f):
    with torch.device("cuda"):                                   # a torch function mode
        return f()


def tensors(r):
    return r if isinstance(r, tuple) else (r,)


def calls(B, H, Nq, Nk, d, dtype):
    import paper_2409_16997_amd as ifa
    g = torch.Generator(device="cuda").manual_seed(Nk)
    mk = lambda n, t=dtype: torch.randn((B, H, n, d), generator=g, device="cuda").to(t)
    Q, K, V, W = mk(Nq), mk(Nk), mk(Nk), mk(Nk, torch.float16)
    q8, sq = ifa.quantize_tokenwise(Q, scale_mul=d ** -0.5)
    k8, sk = ifa.quantize_tokenwise(K)
    v8, sv = ifa.quantize_headwise(V)
    vb, svb = ifa.quantize_blockwise(V, ifa.block_cols(d, True))
    ws = torch.empty(max(ifa.splitk_workspace_bytes(B, H, Nq, Nk, d), 256), dtype=torch.uint8, device="cuda")
    out = [lambda: ifa.quantize_tokenwise(Q, scale_mul=2), lambda: ifa.quantize_headwise(V), lambda: ifa.quantize_qkv(K, V, K, s_Q_mul=0.5),
           lambda: ifa.quantize_qk(K, V), lambda: ifa.quantize_qk(K, V, hadamard=True)]
    for causal in (True, False):
        for dt in (None, torch.float32, torch.bfloat16):
            out += [lambda c=causal, t=dt: ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, sv, causal=c, out_dtype=t),
                    lambda c=causal, t=dt: ifa.int_flash_attn_fwd(q8, k8, vb, sq, sk, svb, causal=c, out_dtype=t),
                    lambda c=causal, t=dt: ifa.int_flash_attn_fwd_half(q8, k8, W, sq, sk, causal=c, out_dtype=t)]
            if Nq <= 32:
                out += [lambda c=causal, t=dt, w=w: ifa.int_flash_attn_fwd_splitk(q8, k8, v8, sq, sk, sv, causal=c, out_dtype=t, workspace=w) for w in (ws, "static", None)]
    return out


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1, 64), (2, 3, 5, 300, 128), (1, 2, 129, 129, 64), (2, 5, 32, 2100, 128)])
def test_both_paths_agree(shape, dtype):
    from paper_2409_16997_amd import binding
    assert not isinstance(binding._load_native(), binding._NoNative)
    for f in calls(*shape, dtype):
        a, b = tensors(f()), tensors(general(f))
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert x.dtype is y.dtype and x.shape == y.shape and x.stride() == y.stride() and torch.equal(x, y)
    side = torch.cuda.Stream()                                   # ... and on a stream other than the default one
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = [tensors(f()) for f in calls(*shape, dtype)[:6]]
    torch.cuda.current_stream().wait_stream(side)
    for x, f in zip(got, calls(*shape, dtype)[:6]):
        assert all(torch.equal(p, q) for p, q in zip(x, tensors(f())))


class Sub(torch.Tensor):
    pass


def test_refusals_are_those_of_the_general_path():
    import paper_2409_16997_amd as ifa
    X = torch.randn((1, 2, 64, 64), device="cuda").half()
    q8, k8, v8, sq, sk, sv = ifa.quantize_qkv(X, X, X)
    fwd, cut = ifa.int_flash_attn_fwd, torch.zeros((1, 2, 65, 64), dtype=torch.int8, device="cuda")
    bad = [lambda: ifa.quantize_tokenwise(X.cpu()), lambda: ifa.quantize_tokenwise(X.transpose(2, 3)), lambda: ifa.quantize_tokenwise(X.double()),
           lambda: ifa.quantize_tokenwise(X, scale_mul=0.0), lambda: ifa.quantize_tokenwise(X, scale_mul="x"), lambda: ifa.quantize_tokenwise(X[:0]), lambda: ifa.quantize_tokenwise(None),
           lambda: ifa.quantize_headwise(X[0, 0, 0]), lambda: ifa.quantize_qkv(X, X, X[:, :1]), lambda: ifa.quantize_qk(X, X.float()),
           lambda: fwd(q8, k8, v8, sq, sk, sv[:, :1].expand(1, 2)), lambda: fwd(q8, k8, v8, sq[:, :1], sk, sv), lambda: fwd(X, k8, v8, sq, sk, sv),
           lambda: fwd(cut, k8, v8, torch.ones((1, 2, 65), device="cuda"), sk, sv, causal=True), lambda: fwd(q8, k8, v8, sq, sk, sv.view(1, 2, 1).repeat(1, 1, 2)),
           lambda: fwd(q8, k8, v8, sq, sk, sv[:, :1].contiguous()), lambda: fwd(q8, k8, v8, sq, sk, sv[0, 0]), lambda: fwd(q8, k8, v8, sq, sk, sv[0, :1]),
           lambda: fwd(q8, k8, v8, sq, sk, sv, out_dtype=torch.float64), lambda: fwd(q8[0], k8[0], v8[0], sq[0], sk[0], sv[0]),
           lambda: ifa.int_flash_attn_fwd_half(q8, k8, X.float(), sq, sk), lambda: ifa.int_flash_attn_fwd_splitk(q8, k8, v8, sq, sk, sv, workspace="static"),
           lambda: ifa.int_flash_attn_fwd_splitk(q8[:, :, :2].contiguous(), k8, v8, sq[:, :, :2].contiguous(), sk, sv, workspace=torch.empty(8, dtype=torch.uint8, device="cuda"))]
    for i, f in enumerate(bad):
        seen = []
        for path in (lambda: f(), lambda: general(f)):
            with pytest.raises(Exception) as e:
                path()
            seen.append((e.type, str(e.value)))
        assert seen[0] == seen[1], i
    for f in (lambda x: ifa.quantize_tokenwise(x), lambda x: ifa.quantize_headwise(x)):       # accepted before, accepted still
        assert all(torch.equal(a, b) for a, b in zip(f(X.as_subclass(Sub)), f(X)))
    assert torch.equal(fwd(q8, k8, v8, sq, sk, sv[0]), fwd(q8, k8, v8, sq, sk, sv))
    assert torch.equal(fwd(q8, k8, v8, sq, sk, sv, causal=1), fwd(q8, k8, v8, sq, sk, sv, causal=True))


def test_a_tensor_whose_address_cannot_be_had_is_refused():
    # data_ptr() raises for it (C++ exception inside the module): the call ends in the same error on both paths, and the process goes on
    import paper_2409_16997_amd as ifa
    bad = torch.randn((1, 2, 64, 64), device="cuda").half()
    torch._C._set_throw_on_mutable_data_ptr(bad)
    for f in (lambda: ifa.quantize_tokenwise(bad), lambda: ifa.quantize_headwise(bad), lambda: ifa.quantize_qkv(bad, bad, bad), lambda: ifa.quantize_qk(bad, bad)):
        for path in (lambda: f(), lambda: general(f)):
            with pytest.raises(RuntimeError, match="data pointer"):
                path()
    good = torch.randn((1, 2, 64, 64), device="cuda").half()
    assert ifa.quantize_tokenwise(good)[0].shape == good.shape


def test_a_hip_error_is_raised_and_the_call_not_repeated():
    # a stand-in for the C ABI whose every launch fails once behind the module; the library on the general path would succeed
    import ctypes
    from paper_2409_16997_amd import binding
    ifa = binding
    B, H, N, d = 1, 2, 64, 64
    X = torch.randn((B, H, N, d), device="cuda").half()
    q8, k8, v8, sq, sk, sv = ifa.quantize_qkv(X, X, X)
    svb = ifa.quantize_blockwise(X, 128)[1]
    ws = torch.empty(ifa.splitk_workspace_bytes(B, H, 8, N, d), dtype=torch.uint8, device="cuda")
    few = (q8[:, :, :8].contiguous(), k8, v8, sq[:, :, :8].contiguous(), sk, sv)
    calls = [lambda: ifa.quantize_tokenwise(X), lambda: ifa.quantize_headwise(X), lambda: ifa.quantize_qkv(X, X, X), lambda: ifa.quantize_qk(X, X),
             lambda: ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, sv), lambda: ifa.int_flash_attn_fwd(q8, k8, v8, sq, sk, svb),
             lambda: ifa.int_flash_attn_fwd_half(q8, k8, X, sq, sk), lambda: ifa.int_flash_attn_fwd_splitk(*few, workspace=ws),
             lambda: ifa.int_flash_attn_fwd_splitk(*few, workspace="static")]
    fail = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: -5)            # IFA_ERR_HIP
    module = binding._load_native()
    addresses = [binding._address(getattr(binding.lib(), name)) for name in binding._NATIVE_CALLS]
    try:
        module.init(binding._check, *([binding._address(fail)] * (len(addresses) - 1) + addresses[-1:]))
        for i, f in enumerate(calls):
            with pytest.raises(binding.IntfaError, match="IFA_ERR_HIP"):
                f()
    finally:
        module.init(binding._check, *addresses)
    for f in calls:
        f()


def test_calls_run_on_the_current_stream():
    # the inputs are written by the side stream after a wait of some milliseconds; a launch on another stream would find what was there before
    import paper_2409_16997_amd as ifa
    torch.manual_seed(5)
    new = torch.randn((1, 4, 300, 128), device="cuda").half()
    want = ifa.quantize_qkv(new, new, new)
    want_O = ifa.int_flash_attn_fwd(*want, causal=True)
    X, side = torch.zeros_like(new), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(10_000_000)
        X.copy_(new)
        got = ifa.quantize_qkv(X, X, X) + ifa.quantize_tokenwise(X) + ifa.quantize_headwise(X) + ifa.quantize_qk(X, X)
        O = [ifa.int_flash_attn_fwd(*got[:6], causal=True), ifa.int_flash_attn_fwd_half(got[0], got[1], X, got[3], got[4], causal=True),
             ifa.int_flash_attn_fwd_splitk(got[0][:, :, -8:].contiguous(), *got[1:3], got[3][:, :, -8:].contiguous(), *got[4:6], causal=True, workspace="static")]
    torch.cuda.synchronize()
    q8, k8, v8, sq, sk, sv = want
    for a, b in zip(got, (q8, k8, v8, sq, sk, sv, q8, sq, v8, sv, q8, k8, sq, sk)):
        assert torch.equal(a, b)
    assert torch.equal(O[0], want_O) and torch.equal(O[1], ifa.int_flash_attn_fwd_half(q8, k8, new, sq, sk, causal=True))
    assert torch.equal(O[2], want_O[:, :, -8:])


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("shape,block", [((2, 3, 300, 128), 128), ((1, 1, 1, 64), 64), ((5, 129, 64), 128), ((7, 8, 32), 3), ((2, 2, 2, 33, 64), 256), ((4, 100, 8), 100)])
def test_quantize_blockwise_on_both_paths(shape, block, dtype):
    import paper_2409_16997_amd as ifa
    from paper_2409_16997_amd import binding
    X = torch.randn(shape, device="cuda").to(dtype)
    a, b = ifa.quantize_blockwise(X, block), general(lambda: ifa.quantize_blockwise(X, block))
    for x, y in zip(a, b):
        assert x.dtype is y.dtype and x.shape == y.shape and x.stride() == y.stride() and torch.equal(x, y)
    for bad in (0, -1, 1 << 40):                                 # the same refusals
        refusals = []
        for path in (lambda f: f(), general):
            with pytest.raises((binding.IntfaError, ZeroDivisionError, RuntimeError)) as e:
                path(lambda: ifa.quantize_blockwise(X, bad))
            refusals.append((e.type, str(e.value)))
        assert refusals[0] == refusals[1]


# A tensor is contiguous whatever the stride of a dimension of one: the outputs of either path have it, too
@pytest.mark.parametrize("whole,cut", [((1, 4, 33, 64), (slice(None), slice(0, 1))), ((5, 2, 40, 64), (slice(2, 3), slice(0, 1))), ((3, 2, 7, 128), (slice(1, 2), slice(1, 2), slice(4, 5)))])
def test_strides_of_dimensions_of_one(whole, cut):
    import paper_2409_16997_amd as ifa
    X = torch.randn(whole, device="cuda", dtype=torch.float16)[cut]
    assert X.is_contiguous() and X.stride() != torch.empty(X.shape).stride()
    for call in (lambda: ifa.quantize_blockwise(X, 128), lambda: ifa.quantize_tokenwise(X), lambda: ifa.quantize_headwise(X), lambda: ifa.quantize_qkv(X, X, X)):
        for x, y in zip(call(), general(call)):
            assert x.dtype is y.dtype and x.shape == y.shape and x.stride() == y.stride() and torch.equal(x, y)
