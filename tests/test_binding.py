"""The binding's native part without a GPU: device tensors are stand-ins in host memory, entry points are the test's own."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2302_06646_amd as lc
from paper_2302_06646_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    """Folder with the compiled helper module."""
    d = tmp_path_factory.mktemp("stub")
    subprocess.run(build.host_command(os.path.join(HERE, "device_tensor_stub.cpp"), str(d / "device_tensor_stub.so")), check=True,
                   capture_output=True, text=True)
    return str(d)


def _python(stub, code):
    """`code` in an interpreter of its own, which may crash."""
    env = dict(os.environ, PYTHONPATH=os.pathsep.join([ROOT, stub]))
    return subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=300)


def test_an_exception_in_the_library_becomes_a_python_error(stub):
    # the library is entered without the GIL: an exception that leaves it must not keep the interpreter without one, nor send
    # the call through the Python way a second time
    r = _python(stub, """
import torch, device_tensor_stub as stub
import paper_2302_06646_amd as lc
from paper_2302_06646_amd import _native
_native.bind({name: stub.throwing() for name in lc.EXPORTS})
class Stream: cuda_stream = 0
k = stub.tensor(2, 256)
assert type(k) is torch.Tensor and k.is_cuda
for again in range(3):
    try:
        print("returned", _native.kreg_fwd(k, None, k, 1, 0.5, Stream()))
    except MemoryError:
        print("MemoryError")
assert _native.kreg_fwd(k, None, k, 1, 1, Stream()) is None      # not the usual call (an integer threshold): not entered
print("alive", sum(range(10)))
""")
    assert r.returncode == 0, r.stderr[-2000:]
    assert r.stdout.split() == ["MemoryError"] * 3 + ["alive", "45"], r.stdout


def test_calls_are_served_without_the_native_part(monkeypatch):
    # a library built by itself, or for another interpreter: the Python way looks at every call
    monkeypatch.setattr(lc, "_bound", None)
    monkeypatch.setitem(sys.modules, "paper_2302_06646_amd._native", None)
    monkeypatch.delattr(lc, "_native", raising=False)
    k = torch.zeros(2, 256)
    with pytest.warns(RuntimeWarning, match="native part"):
        with pytest.raises(lc.LongconvError, match="k must be a contiguous device tensor"):
            lc.longconv_kreg_fwd(k, None, k, 1, 0.5)
    with pytest.raises(lc.LongconvError, match="u must be a contiguous device tensor"):       # (and warns once)
        lc.longconv_fwd(torch.zeros(1, 2, 256), k, torch.zeros(2), torch.zeros(1, 2, 256), torch.zeros(1))


def test_the_library_builds_without_a_host_compiler(monkeypatch, tmp_path, capsys):
    monkeypatch.setenv("CXX", "/nonexistent/c++")
    monkeypatch.setattr(build, "NATIVE", str(tmp_path / "_native.so"))
    assert build.build_binding() is None
    assert "/nonexistent/c++" in capsys.readouterr().out


def test_the_native_part_is_of_this_interpreter():
    import importlib.machinery
    assert build.NATIVE.endswith(importlib.machinery.EXTENSION_SUFFIXES[0])
