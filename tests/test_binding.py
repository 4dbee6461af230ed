"""The binding's native part without a GPU: device tensors are stand-ins in host memory, entry points are the test's own."""
import os
import subprocess
import sys

import pytest

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
