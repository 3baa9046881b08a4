"""The native calls of the torch layer (csrc/fq_binding.cpp) against the Python they stand in for: the same outputs, and None --
the Python way, with its errors -- wherever a call is out of the ordinary."""
import ctypes

import pytest

from paper_2308_09723_amd import fq


class _Python:
    """Stands in for the native module: every call goes the Python way."""

    def __getattr__(self, name):
        return lambda *args: None


def _native():
    fq._torch()
    return fq._native


def test_host_tensors_and_wrong_arguments_go_the_python_way():
    import torch
    native = _native()
    A, W = torch.zeros((4, 128), dtype=torch.float16), torch.zeros((128, 16), dtype=torch.float16)
    assert native.gemm(A, W, W, 4, 128, None, None) is None
    assert native.gemm(A, W, W) is None and native.gemm() is None and native.gemm(1, 2, 3, 4, 5, 6, 7) is None
    assert native.gemm_grouped(A, [0, 4], W, W, 4, 128, 16, None) is None
    assert native.quantize_act_i8(A) is None and native.quantize_act_i8("A") is None
    assert native.gemm_w4a8(A, A, A, A, A, 128, torch.float16, None, None) is None
    assert native.quantize(W, 4, 128, 0) is None and native.quantize_w4a8(W, 128) is None
    for call in (lambda: fq.gemm(A, W, W, 4, 128), lambda: fq.quantize(W, 4, 128), lambda: fq.quantize_act_i8(A),
                 lambda: fq.quantize_w4a8(W, 128)):
        with pytest.raises(AssertionError):
            call()


@pytest.mark.parametrize("fault", ["no torch", "no compiler", "compile error"])
def test_the_library_builds_without_the_native_calls(monkeypatch, tmp_path, fault):
    """libfq.so is linked where the native calls cannot be compiled, and no earlier build of them stays beside it."""
    import importlib.util

    from paper_2308_09723_amd import build

    commands, find_spec = [], importlib.util.find_spec

    def run(cmd):
        commands.append(cmd)
        if cmd[0] != "g++":
            return 0, ""
        if fault == "no compiler":
            raise FileNotFoundError("g++")
        return 1, "error"

    monkeypatch.setattr(build, "_run", run)
    monkeypatch.setattr(build, "_resource_report", lambda rows, verbose: None)
    for name, value in (("OBJ_DIR", "obj"), ("LIB_PATH", "libfq.so"), ("NATIVE_PATH", "_fqcall.so")):
        monkeypatch.setattr(build, name, str(tmp_path / value))
    if fault == "no torch":
        monkeypatch.setattr(importlib.util, "find_spec", lambda name, *a: None if name == "torch" else find_spec(name, *a))
    (tmp_path / "_fqcall.so").write_bytes(b"an earlier build")
    with pytest.warns(RuntimeWarning, match="not built"):
        assert build.build_lib(verbose=False) == str(tmp_path / "libfq.so")
    assert "-shared" in commands[-1] and commands[-1][-1] == str(tmp_path / "libfq.so")
    assert not (tmp_path / "_fqcall.so").exists()


@pytest.mark.parametrize("there", ["missing", "not a library"])
def test_without_the_native_calls_everything_goes_the_python_way(monkeypatch, tmp_path, there):
    path = tmp_path / "_fqcall.so"
    if there == "not a library":
        path.write_bytes(b"something else")
    import torch
    for name, value in (("NATIVE_PATH", str(path)), ("_lib", None), ("_native", None), ("_torch_mod", None)):
        monkeypatch.setattr(fq, name, value)
    assert fq.load(build_if_missing=False) is not None       # the C interface needs libfq.so alone
    A = torch.zeros((4, 128), dtype=torch.float16)
    with pytest.warns(RuntimeWarning, match="issued from Python"):
        fq._torch()
    assert fq._native.gemm(A, A, A, 4, 128, None, None) is None and fq._native.quantize_act_i8(A) is None
    with pytest.raises(AssertionError):                      # (host tensors: the Python way's own check)
        fq.quantize_act_i8(A)


@pytest.mark.gpu
def test_same_outputs_and_errors_as_the_python_way(monkeypatch):
    import torch
    native = _native()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    K, N = 1024, 1040
    W = (torch.randn((K, N), generator=gen, device="cuda") * 0.02).to(torch.float16)
    A = torch.randn((7, K), generator=gen, device="cuda").to(torch.bfloat16)

    def everything():
        out = []
        for bits, g, fmt in ((4, 128, 0), (8, 0, 1), (3, 64, 0)):
            codes, scales = fq.quantize(W, bits, g, fmt)
            out += [codes, scales, fq.gemm(A, codes, scales, bits, g)]
            C, ws = torch.empty((7, N), dtype=A.dtype, device="cuda"), torch.empty(1 << 20, dtype=torch.float32, device="cuda")
            assert fq.gemm(A, codes, scales, bits, g, out=C, workspace=ws) is C
            small = torch.empty(16, dtype=torch.uint8, device="cuda")     # too small a workspace: one is made
            out += [C, fq.gemm(A, codes, scales, bits, g, workspace=small)]
            two, s2 = torch.cat([codes, codes]), torch.cat([scales, scales])
            for offsets in ([0, 3, 7], (0, 7, 7), [0, torch.tensor(3), 7], bytes([0, 3, 7])):
                out.append(fq.gemm_grouped(A, offsets, two, s2, bits, g, N))
        codes, z, t = fq.quantize_w4a8(W, 64)
        Aq, alpha = fq.quantize_act_i8(A)
        out += [codes, z, t, Aq, alpha, fq.gemm_w4a8(Aq, alpha, codes, z, t, 64, torch.float16),
                fq.gemm_w4a8(Aq, alpha, codes, z, t, 64, torch.bfloat16, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))]
        return out

    def errors():
        codes, scales = fq.quantize(W, 4, 128)
        calls = (lambda: fq.gemm(A[:, ::2], codes, scales, 4, 128), lambda: fq.gemm(A.float(), codes, scales, 4, 128),
                 lambda: fq.gemm(A, codes, scales.float(), 4, 128), lambda: fq.gemm(A, codes, scales, 5, 128),
                 lambda: fq.gemm(A.half(), codes, scales.to(torch.bfloat16), 4, 128), lambda: fq.gemm(A, codes, scales, 4, 96),
                 lambda: fq.quantize(W, 4, 100), lambda: fq.quantize(W.float(), 4, 128), lambda: fq.quantize_w4a8(W[:, :8], 128),
                 lambda: fq.gemm_grouped(A, [0, 9, 7], codes, scales, 4, 128, N), lambda: fq.quantize_act_i8(A.t()))
        got = []
        for call in calls:
            with pytest.raises(Exception) as e:
                call()
            got.append((type(e.value), str(e.value)))
        return got

    mine, mine_errors = everything(), errors()
    monkeypatch.setattr(fq, "_native", _Python())
    python, python_errors = everything(), errors()
    monkeypatch.undo()
    assert mine_errors == python_errors
    for a, b in zip(mine, python):
        assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    # a subclass, a function mode and a transformed tensor are not plain
    class Sub(torch.Tensor):
        pass
    assert native.quantize_act_i8(A.as_subclass(Sub)) is None
    from torch.overrides import TorchFunctionMode

    class Mode(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))
    with Mode():
        assert native.quantize_act_i8(A) is None
    seen = []
    torch.vmap(lambda x: (seen.append(native.quantize_act_i8(x)), x)[1])(A.unsqueeze(0))
    assert seen == [None]
    # the current stream
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        x = torch.randn((64, 4096), device="cuda").to(torch.float16)
        Aq, alpha = fq.quantize_act_i8(x)
    s.synchronize()
    assert torch.equal(Aq, fq.quantize_act_i8(x)[0])


@pytest.mark.gpu
def test_an_error_of_the_runtime_is_raised_and_the_call_not_made_again(monkeypatch):
    """FQ_ERR_HIP can follow launches that were enqueued.  The library's functions are stubs here, which launch nothing."""
    import torch
    native = _native()
    W = (torch.randn((1024, 1040), device="cuda") * 0.02).to(torch.float16)
    A = torch.randn((7, 1024), device="cuda").to(torch.float16)
    codes, scales = fq.quantize(W, 4, 128)
    c8, z, t = fq.quantize_w4a8(W, 128)
    Aq, alpha = fq.quantize_act_i8(A)
    calls, real = [], fq.load()

    class Library:
        def __getattr__(self, name):
            if name not in stubs:
                return getattr(real, name)
            return stubs[name]

    names = [n for n in fq._NATIVE_FUNCTIONS if not n.endswith("_bytes")]
    stubs = {n: ctypes.CFUNCTYPE(ctypes.c_int)(lambda n=n: (calls.append(n), fq.FQ_ERR_HIP)[1]) for n in names}
    monkeypatch.setattr(fq, "load", lambda *args: Library())
    try:
        monkeypatch.setattr(fq, "_native", fq._load_native())
        for name, call in (("fq_gemm_sf", lambda: fq.gemm(A, codes, scales, 4, 128)),
                           ("fq_gemm_grouped_sf", lambda: fq.gemm_grouped(A, [0, 7], codes, scales, 4, 128, 1040)),
                           ("fq_gemm_w4a8", lambda: fq.gemm_w4a8(Aq, alpha, c8, z, t, 128, torch.float16)),
                           ("fq_quantize_act_i8", lambda: fq.quantize_act_i8(A)), ("fq_quantize_sf", lambda: fq.quantize(W, 4, 128)),
                           ("fq_quantize_w4a8", lambda: fq.quantize_w4a8(W, 128))):
            with pytest.raises(fq.FqError) as e:
                call()
            assert (e.value.status, str(e.value)) == (fq.FQ_ERR_HIP, f"{name}: FQ_ERR_HIP")
            assert calls == [name]
            calls.clear()
    finally:
        monkeypatch.undo()
        fq._load_native()                # the library's own functions again
    assert fq._native is native and torch.equal(fq.quantize_act_i8(A)[0], Aq)
