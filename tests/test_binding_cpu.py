"""The binding's native half against its general path in Python: the same answers and errors, without a GPU (every call here is
refused before the device is touched, or never made)."""
import os
import shutil
import signal
import subprocess
import sys
import textwrap
import types

import pytest
import torch


@pytest.fixture(scope="module")
def B():
    from paper_2403_17312_amd import binding, build
    if not os.path.exists(binding.LIB_PATH) or not os.path.exists(build.NATIVE_PATH):
        build.build()
    binding.lib()
    return binding


@pytest.fixture(params=["native", "general"])
def path(request, B, monkeypatch):
    if request.param == "general":
        class Nothing:
            def __getattr__(self, name):
                return lambda *args: None
        monkeypatch.setattr(B, "_native", Nothing())
    return request.param


def _calls(B, p, t, stream=0):
    """Every call with tensors t for its pointers; R and ring rows are 4 and 1."""
    return [lambda: B.swa_decode_step(p, t, t, t, t, t, t, t, t, t, None, t, t, None, t, stream),
            lambda: B.swa_decode_step_q8(p, t, t, t, t, t, t, t, t, t, t, None, t, t, None, t, stream),
            lambda: B.swa_decode_step_window(p, t, t, t, t, t, t, 4, 1, t, t, t, t, None, t, t, None, t, stream),
            lambda: B.swa_decode_step_window_q8(p, t, t, t, t, t, t, t, 4, 1, t, t, t, t, None, t, t, None, t, stream),
            lambda: B.swa_decode_step_static(p, t, t, t, t, t, t, t, t, t, None, t, t, None, stream),
            lambda: B.swa_compact_kv(p, t, t, t, t, t, t, t, t, stream),
            lambda: B.swa_prefill_scores(p, t, 4, t, t, t, t, stream),
            lambda: B.swa_prefill_rows(p, t, 4, t, t, t, t, stream),
            lambda: B.swa_prefill_attention(p, t, t, t, t, t, 4, t, t, stream),
            lambda: B.swa_quantize_kv(p, t, t, t, t, t, t, stream)]


def test_the_librarys_refusals_come_through(B, path):
    bad = B.make_params(1, 1, 65, 8, 1, 5000, torch.float16)          # no such head dimension
    t = torch.zeros(64)
    for call in _calls(B, bad, t):
        with pytest.raises(B.SwaError) as e:
            call()
        assert e.value.code == B.SWA_ERR_UNSUPPORTED_D
    good = B.make_params(1, 1, 64, 8, 1, 5000, torch.float16)
    with pytest.raises(B.SwaError) as e:
        B.swa_prefill_scores(good, None, 4, t, t, t, t, 0)
    assert e.value.code == B.SWA_ERR_NULL
    for R in (0, -1, B.SWA_MAX_PREFILL_ROWS + 1, True and 129, 129.0):
        with pytest.raises(B.SwaError) as e:
            B.swa_prefill_scores(good, t, R, t, t, t, t, 0)
        assert e.value.code == B.SWA_ERR_BAD_SHAPE
    with pytest.raises(B.SwaError) as e:
        B.swa_prefill_scores(good, t[1:], 4, t, t, t, t, 0)           # 4 bytes beyond a 16-byte boundary
    assert e.value.code == B.SWA_ERR_ALIGNMENT


def test_what_is_no_contiguous_tensor_is_refused(B, path):
    p = B.make_params(1, 1, 65, 8, 1, 5000, torch.float16)
    for call in _calls(B, p, torch.zeros(8, 8).t()):
        with pytest.raises(ValueError, match="contiguous"):
            call()
    for thing in (5, "x", [1]):
        with pytest.raises(AttributeError):
            _calls(B, p, thing)[0]()
    for other in (b"0" * 40, None, 7, object()):
        with pytest.raises((TypeError, AttributeError)):
            _calls(B, other, torch.zeros(64))[0]()
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda t: _calls(B, p, t)[0]())(torch.zeros(2, 64))


def test_a_stream_object_and_a_parameter_are_taken(B, path):
    class Stream:
        cuda_stream = 0
    p = B.make_params(1, 1, 65, 8, 1, 5000, torch.float16)
    for t in (torch.nn.Parameter(torch.zeros(64)), torch.zeros(64, requires_grad=True)):
        for call in _calls(B, p, t, Stream()):
            with pytest.raises(B.SwaError):
                call()


@pytest.mark.parametrize("module", [None, types.SimpleNamespace(torch_version="1.0"), types.SimpleNamespace()])
def test_without_a_native_half_of_this_torch_the_general_path_serves(B, monkeypatch, module):
    """No native half, or one that was built for another torch."""
    name = "paper_2403_17312_amd._swa_native"
    monkeypatch.setitem(sys.modules, name, module)
    if module is None:
        monkeypatch.delattr(sys.modules["paper_2403_17312_amd"], "_swa_native", raising=False)
    else:
        monkeypatch.setattr(sys.modules["paper_2403_17312_amd"], "_swa_native", module, raising=False)
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_native", None)
    with pytest.warns(UserWarning, match="in Python"):
        B.lib()
    bad = B.make_params(1, 1, 65, 8, 1, 5000, torch.float16)
    for call in _calls(B, bad, torch.zeros(64)):
        with pytest.raises(B.SwaError) as e:
            call()
        assert e.value.code == B.SWA_ERR_UNSUPPORTED_D


def test_a_build_without_a_host_compiler_leaves_no_native_half(tmp_path, monkeypatch):
    from paper_2403_17312_amd import build
    stale = tmp_path / "_swa_native.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(build, "NATIVE_PATH", str(stale))
    monkeypatch.setenv("PATH", str(tmp_path))
    with pytest.warns(UserWarning, match="not built, for want of g"):
        assert build.build_native() is None
    assert not stale.exists()


@pytest.mark.skipif(not shutil.which("g++"), reason="builds a library that throws")
def test_an_exception_out_of_the_library_ends_the_process(B, tmp_path):
    """As by way of ctypes: it is not taken for an argument that the general path has to look at, with the interpreter's lock released
    and the call made again."""
    if isinstance(B._native, B._General):
        pytest.skip("no native half here")
    (tmp_path / "throws.cpp").write_text('extern "C" int swa_compact_kv(...) { throw 1; }\n')
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(tmp_path / "throws.so"), str(tmp_path / "throws.cpp")], check=True)
    code = textwrap.dedent(f"""
        import ctypes, torch
        from paper_2403_17312_amd import binding as B
        B.lib()
        fn = ctypes.CDLL({str(tmp_path / "throws.so")!r}).swa_compact_kv
        B._native.bind({{"swa_compact_kv": ctypes.cast(fn, ctypes.c_void_p).value}}, B.SwaParams)
        t = torch.zeros(64)
        print("came back", B._native.swa_compact_kv(B.make_params(1, 1, 64, 8, 1, 5000, torch.float16), t, t, t, t, t, t, t, t, 0))
    """)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == -signal.SIGABRT and "terminate called" in r.stderr and "came back" not in r.stdout, r
