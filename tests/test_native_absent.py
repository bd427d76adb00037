"""Without its native part the binding works in Python: no compiler for it, no headers, or a file that was built against
another Python or torch (whose name differs) or cannot be loaded."""
import pytest
import torch

from paper_2512_24449_amd import binding, build, synth


def _reload(monkeypatch, native_path):
    binding.lib()
    monkeypatch.setattr(build, "native_path", lambda: native_path)
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    return binding.lib


@pytest.mark.parametrize("compiler", ["/nonexistent/g++", "false"])
def test_no_compiler(monkeypatch, tmp_path, compiler):
    load = _reload(monkeypatch, str(tmp_path / "_native.so"))
    monkeypatch.setenv("CXX", compiler)
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        assert load().kv_strerror(0)
    assert binding._native is None and binding.lib() is binding._lib


def test_file_that_cannot_be_loaded(monkeypatch, tmp_path):
    path = tmp_path / "_native.so"
    path.write_bytes(b"not a library")
    load = _reload(monkeypatch, str(path))
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        assert load().kv_strerror(0)
    assert binding._native is None


def test_the_name_says_what_it_was_built_against(monkeypatch):
    here = build.native_path()
    monkeypatch.setattr(torch, "__version__", "0.0.1")
    assert build.native_path() != here


def test_library_builds_without_the_native_part(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libpackkv.so"))
    monkeypatch.setattr(build, "sources", lambda: [build.CSRC + "/softmax.hip"])
    monkeypatch.setenv("CXX", "/nonexistent/g++")
    with pytest.warns(UserWarning, match="native part was not built"):
        assert build.build() == str(tmp_path / "libpackkv.so")
    assert (tmp_path / "libpackkv.so").exists()


@pytest.mark.gpu
def test_same_results(monkeypatch, tmp_path):
    B, H, Hq, L = 2, 3, 6, 200
    K, V, q = synth.make_kv(B, L, H, Hq, 3, device="cuda:0")
    got = []
    for absent in (False, True):
        if absent:
            load = _reload(monkeypatch, str(tmp_path / "_native.so"))
            monkeypatch.setenv("CXX", "false")
            with pytest.warns(RuntimeWarning):
                load()
        cache = binding.PackedKVCache(B, H, Hq, L)
        cache.kv_compress_append(K, V)
        p = cache.kv_softmax(cache.kv_k_matvec(q, 0.09))
        got.append((p, cache.kv_v_matvec(p), cache.kv_decode_attention(q, 0.09)))
        cache.kv_cache_restore(100)
        assert cache.tokens == 100
        cache.kv_cache_release()
        assert cache.tokens == 0
        cache.close()
        with pytest.raises(binding.PackKVError):
            cache.kv_cache_restore(0)
    assert all(torch.equal(a, b) for a, b in zip(*got))
