"""The native entry of matmul() and conv2d_nchw() (csrc/torch_binding.cpp): it
takes the plain calls and leaves every other one to the Python path, with the
same results and the same errors."""
import pytest

import paper_2512_16512_amd as x

torch = pytest.importorskip("torch")


def test_everything_but_plain_gpu_tensors_is_left_to_the_python_path():
    a = torch.zeros(4, 4)
    for args in [(a, a, None, False), (a, None, None, False), ([1], a, None, False), (a, a, None, 1), (a, a)]:
        assert x._fast.matmul(*args) is None
    k = torch.zeros(1, 1, 3, 3)
    for args in [(k, k, 1, 1, None, False), (k, k, "1", 1, None, False), (k,)]:
        assert x._fast.conv2d_nchw(*args) is None
    with pytest.raises(ValueError, match="CUDA"):
        x.matmul(a, a)
    with pytest.raises(TypeError, match="same dtype"):
        x.matmul(a, a.bfloat16())


@pytest.mark.parametrize("binding", [None, b"no shared object"])
def test_the_library_imports_without_its_binding(tmp_path, binding):
    """A binding that is missing or does not load is reported and leaves the C
    ABI usable."""
    import os
    import shutil
    import subprocess
    import sys
    pkg = os.path.dirname(x.__file__)
    dst = tmp_path / "paper_2512_16512_amd"
    dst.mkdir()
    for f in ("__init__.py", "libxtc.so"):
        shutil.copy(os.path.join(pkg, f), dst / f)
    if binding is not None:
        (dst / "_binding.so").write_bytes(binding)
    code = ("import paper_2512_16512_amd as x\n"
            "assert x.__file__.startswith(%r)\n"
            "print(x._fast, x.xtc_version(), len(x.xtc_sched_list(0, 0)) > 0)" % str(tmp_path))
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert r.stdout.split() == ["None", "100", "True"]
    assert "native binding does not load" in r.stderr and "build.py" in r.stderr


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_native_and_python_paths_agree(dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    dt = getattr(torch, dtype)
    a = torch.randn(37, 50, device="cuda").to(dt)[:, 1:]     # rows off a 16-byte boundary
    b = torch.randn(49, 30, device="cuda").to(dt)
    sched = x.xtc_default_schedule(x.XTC_OP_MATMUL, x.XTC_F32 if dt == torch.float32 else x.XTC_BF16, 37, 30, 49)
    for relu in (False, True):
        want = x.matmul(a, b, sched=sched, relu=relu)         # an explicit schedule takes the Python path
        got = x._fast.matmul(a, b, None, relu)
        out = torch.full((37, 40), 7.0, device="cuda")[:, :30]
        assert x.matmul(a, b, out=out, relu=relu) is out
        torch.cuda.synchronize()
        assert torch.equal(got, want) and torch.equal(out, want) and got.dtype == torch.float32
    X = torch.randn(2, 8, 9, 7, device="cuda").to(dt)
    W = torch.randn(5, 8, 3, 3, device="cuda").to(dt)
    for stride, pad in ((1, 1), ((2, 1), (0, 2))):
        y = x._fast.conv2d_nchw(X, W, stride, pad, None, True)
        want = x.conv2d_nchw(X, W, list(stride) if isinstance(stride, tuple) else stride, pad, relu=True)
        torch.cuda.synchronize()
        assert torch.equal(y, want)


@pytest.mark.gpu
def test_transforms_modes_and_bad_operands_take_the_python_path():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    from torch.utils._python_dispatch import TorchDispatchMode

    class Mode(TorchDispatchMode):
        def __torch_dispatch__(self, f, types, args=(), kwargs=None):
            return f(*args, **(kwargs or {}))

    class Sub(torch.Tensor):
        pass

    a, b = torch.randn(8, 8, device="cuda"), torch.randn(8, 8, device="cuda")
    seen = []
    with Mode():
        seen.append(x._fast.matmul(a, b, None, False))
    with torch.device("cuda"):
        seen.append(x._fast.matmul(a, b, None, False))
    torch.vmap(lambda t: (seen.append(x._fast.matmul(t, b, None, False)), t)[1])(torch.randn(2, 8, 8, device="cuda"))
    torch.func.jvp(lambda t: (seen.append(x._fast.matmul(t, b, None, False)), t)[1], (a,), (a,))
    seen.append(x._fast.matmul(a.as_subclass(Sub), b, None, False))
    seen.append(x._fast.matmul(a.t(), b, None, False))
    seen.append(x._fast.matmul(a, b[:7], None, False))
    seen.append(x._fast.matmul(a, b.bfloat16(), None, False))
    seen.append(x._fast.matmul(a, b, torch.empty(8, 8), False))
    assert seen == [None] * 9
    with pytest.raises(ValueError, match="inner dimensions"):
        x.matmul(a, b[:7])
    with pytest.raises(x.XtcError):                      # C*R*S past the k-offset table
        x.conv2d_nchw(torch.zeros(1, 1024, 4, 4, device="cuda"), torch.zeros(1, 1024, 3, 3, device="cuda"))
