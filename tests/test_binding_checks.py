"""What the binding's general path refuses before the C ABI is reached, on host tensors with a stand-in for the library."""
import os
import warnings

import pytest

torch = pytest.importorskip("torch")

from paper_2409_16997_amd import binding


class Library:
    """Every function of it succeeds and is noted."""
    def __init__(self):
        self.called = []

    def __getattr__(self, name):
        def call(*args):
            if not name.startswith("ifa_"):
                self.called.append(name)
            return {"ifa_block_cols": 128, "ifa_splitk_workspace_bytes": 256}.get(name, 0)
        return call


@pytest.fixture
def library(monkeypatch):
    stand_in = Library()
    monkeypatch.setattr(torch.Tensor, "is_cuda", True, raising=False)
    monkeypatch.setattr(binding, "lib", lambda: stand_in)
    monkeypatch.setattr(binding, "_stream", lambda: 0)
    monkeypatch.setattr(binding, "_native", binding._NoNative())
    return stand_in


def operands(B=2, H=3, Nq=5, Nk=7, d=64):
    i8 = lambda n: torch.zeros((B, H, n, d), dtype=torch.int8)
    return i8(Nq), i8(Nk), i8(Nk), torch.ones((B, H, Nq)), torch.ones((B, H, Nk))


# s_V is read at every head: a tensor with fewer scales than heads would be read past its end
@pytest.mark.parametrize("shape,taken", [((2, 3), True), ((6,), True), ((2, 3, 1), True), ((2, 3, 1, 1), True), ((1,), False), ((), False), ((2, 2), False),
                                         ((5,), False), ((2, 3, 2), False), ((1, 1, 1), False)])
def test_v_scales_of_every_head(library, shape, taken):
    call = lambda: binding.int_flash_attn_fwd(*operands(), torch.ones(shape))
    if taken:
        call()
        assert len(library.called) == 1
    else:
        with pytest.raises(binding.IntfaError):
            call()
        assert not library.called


# an `out` with fewer elements than the call writes would be written past its end
def test_outputs_have_room(library):
    q, k, v, sq, sk = operands(Nq=5, Nk=5)
    sv = torch.ones((2, 3))
    X = torch.zeros((2, 3, 5, 64), dtype=torch.float16)
    small, room, flat = torch.empty((2, 3, 4, 64)), torch.empty((2, 3, 5, 64)), torch.empty(2 * 3 * 5 * 64)
    for fn, args in ((binding.int_flash_attn_fwd, (q, k, v, sq, sk, sv)), (binding.int_flash_attn_fwd_half, (q, k, X, sq, sk)),
                     (binding.int_flash_attn_fwd_splitk, (q, k, v, sq, sk, sv))):
        for out in (room, flat):
            assert fn(*args, out=out) is out
        before = len(library.called)
        with pytest.raises(binding.IntfaError):
            fn(*args, out=small)
        assert len(library.called) == before
    codes, rows = torch.empty((2, 3, 5, 64), dtype=torch.int8), torch.empty((2, 3, 5))
    for fn, args, outs in ((binding.quantize_qkv, (X, X, X), [codes, codes, codes, rows, rows, sv]), (binding.quantize_qk, (X, X), [codes, codes, rows, rows])):
        fn(*args, out=tuple(outs))
        before = len(library.called)
        for i, t in enumerate(outs):
            with pytest.raises(binding.IntfaError):
                fn(*args, out=tuple(outs[:i] + [t.flatten()[:-1]] + outs[i + 1:]))
        assert len(library.called) == before


# Without a host module that fits (none, one that does not load, one built for another torch) the general path serves every call.
@pytest.mark.parametrize("fault", ["missing", "broken", "other torch"])
def test_calls_without_the_host_module(monkeypatch, tmp_path, fault):
    monkeypatch.setattr(binding, "_native", None)
    if fault == "other torch":
        if not os.path.exists(binding._NATIVE_PATH):
            pytest.skip("not built")
        monkeypatch.setattr(torch, "__version__", "1.0.0")
    else:
        path = tmp_path / "_intfa_host.so"
        if fault == "broken":
            path.write_bytes(b"not a library")
        monkeypatch.setattr(binding, "_NATIVE_PATH", str(path))
    with pytest.warns(RuntimeWarning, match="cannot be used"):
        with pytest.raises(binding.IntfaError, match="contiguous tensor in GPU memory"):
            binding.quantize_tokenwise(torch.zeros((4, 64)))
    with warnings.catch_warnings():                              # said once
        warnings.simplefilter("error")
        with pytest.raises(binding.IntfaError, match="contiguous tensor in GPU memory"):
            binding.quantize_headwise(torch.zeros((4, 64)))
