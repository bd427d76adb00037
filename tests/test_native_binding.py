"""The native part of the binding: it answers a call only if every argument is what it expects, and then gives what the Python
code gives, errors included."""
import ctypes as C

import pytest
import torch

from paper_2512_24449_amd import binding, synth


def _calls(handle):
    binding.lib()
    calls = binding._native.Calls(1, 2, 4, "cpu")
    calls.set_handle(handle)
    return calls


class _Sub(torch.Tensor):
    pass


def test_leaves_what_it_does_not_expect():
    """With an address that must never be called: every one of these is left to the Python code."""
    never = _calls(0xDEAD0)
    k = torch.zeros(1, 3, 2, 128, dtype=torch.float16)
    q = torch.zeros(1, 4, 128, dtype=torch.float16)
    p = torch.zeros(1, 4, 8)
    bad_k = [None, 1, k.numpy(), k.float(), k[:, :, :1], k.expand(2, 3, 2, 128), k.transpose(1, 2), k[0], k.as_subclass(_Sub), k.to_sparse()]
    for b in bad_k:
        assert never.append(b, b, 0) is NotImplemented
        assert never.append(k, b, 0) is NotImplemented
    assert never.append(k, k.to(torch.bfloat16), 0) is NotImplemented
    assert never.append(k, k, torch.zeros(1)) is NotImplemented and never.append(k, k, 1.0) is NotImplemented
    for b in (None, q.float(), q[:, :2], q[:, :, :64], q.transpose(0, 1), q[..., None], q.as_subclass(_Sub)):
        assert never.k_matvec(b, 0.1, None, 0) is NotImplemented
        assert never.attention(b, 0.1, 0) is NotImplemented
    for scale in (None, "1", 1, torch.tensor(0.1)):
        assert never.k_matvec(q, scale, p, 0) is NotImplemented and never.attention(q, scale, 0) is NotImplemented
    for b in (None, p.double(), p[:, :2], p[:, :, ::2], p[0], p[..., None], p.as_subclass(_Sub)):
        assert never.softmax(b, 0) is NotImplemented and never.v_matvec(b, 0) is NotImplemented
        assert b is None or b.shape == (1, 2, 8) or never.k_matvec(q, 0.1, b, 0) is NotImplemented
    for tokens in (None, 1.0, 1 << 70, torch.tensor(3)):
        assert never.restore(tokens) is NotImplemented
    with torch.overrides.BaseTorchFunctionMode():
        assert never.append(k, k, 0) is NotImplemented and never.softmax(p, 0) is NotImplemented
    closed = _calls(0)
    assert closed.append(k, k, 0) is NotImplemented and closed.attention(q, 0.1, 0) is NotImplemented
    assert closed.restore(0) is NotImplemented and closed.release(0) is NotImplemented


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_same_results_and_errors_as_the_python_code(dtype):
    B, H, Hq, L = 2, 3, 6, 200
    K, V, q = synth.make_kv(B, L, H, Hq, 3, device="cuda:0")
    K, V = K.to(dtype), V.to(dtype)
    side = torch.cuda.Stream()
    got = []
    for native in (True, False):
        cache = binding.PackedKVCache(B, H, Hq, L)
        if not native:
            cache._calls.set_handle(0)
        cache.kv_compress_append(K[:, :150].contiguous(), V[:, :150].contiguous())
        cache.kv_compress_append(K[:, 150:].contiguous(), V[:, 150:].contiguous(), torch.cuda.current_stream())
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            s = cache.kv_k_matvec(q, 0.09)
            p = cache.kv_softmax(s.clone())
            o = cache.kv_v_matvec(p)
            f = cache.kv_decode_attention(q, 0.09, stream=side.cuda_stream)
        side.synchronize()
        mine = torch.empty(B, Hq, L + 5, device="cuda:0")
        assert cache.kv_k_matvec(q, 0.09, mine) is mine and cache.kv_softmax(mine) is mine
        assert torch.equal(mine[..., :L], p) and cache.tokens == L
        errors = []
        for call in (lambda: cache.kv_compress_append(K, V), lambda: cache.kv_compress_append(K[:, :1], V[:, :1]),
                     lambda: cache.kv_compress_append(None, V), lambda: cache.kv_k_matvec(q, 0.1, mine[..., :8].contiguous()),
                     lambda: cache.kv_k_matvec(q.float(), 0.1), lambda: cache.kv_k_matvec(q, "x"), lambda: cache.kv_v_matvec(p[..., :8].contiguous()),
                     lambda: cache.kv_softmax(p[:1]), lambda: cache.kv_cache_restore(-1), lambda: cache.kv_cache_restore("1"),
                     lambda: cache.kv_decode_attention(q, float("nan"))):
            with pytest.raises(Exception) as e:
                call()
            errors.append((type(e.value), getattr(e.value, "code", None), str(e.value).split("\n")[0]))
        cache.kv_cache_restore(100)
        assert cache.tokens == 100
        cache.kv_cache_release()
        assert cache.tokens == 0
        cache.close()
        with pytest.raises(binding.PackKVError):
            cache.kv_cache_restore(0)
        got.append((s, p, o, f, errors))
    assert all(torch.equal(a, b) for a, b in zip(got[0][:4], got[1][:4]))
    assert got[0][4] == got[1][4]
