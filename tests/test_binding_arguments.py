"""What the binding makes of its arguments before the library sees them, with calls that the library refuses on the host: no
GPU.  What could end the interpreter runs in one of its own."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2604_21221_amd import pbsa  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def in_child(code):
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    return r.returncode, r.stdout + r.stderr


def test_a_tensor_without_memory_is_an_error():
    """A wrapped tensor of a function transform that says it is on the GPU and has no memory: torch's exception, as from
    its data_ptr(), and not the end of the process."""
    rc, out = in_child("""
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2604_21221_amd import pbsa
with FakeTensorMode(allow_non_fake_inputs=True):
    x = torch.empty(2, 3, 4, device="cuda:0")
def call(x):
    try:
        pbsa.pbsa_pool_blocks(pbsa.make_params(2, 128, 64, 200, 16, 16, 4, 3, 0.088), x, 0x1000, -1, 0x1000, stream=0)
    except RuntimeError as e:
        print("refused:", e)
    return x
torch.vmap(call)(x)
""")
    assert rc == 0 and "refused: Cannot access data pointer" in out, out[-2000:]


A = 0x10000          # an aligned address that nothing looks at
EINVAL, EALIGN, EWS = pbsa.PBSA_EINVAL, pbsa.PBSA_EALIGN, pbsa.PBSA_EWS


def params():
    return pbsa.make_params(2, 128, 64, 200, 16, 16, 4, 3, 0.088)


class Duck:          # whatever answers like a tensor
    is_cuda = True

    def is_contiguous(self):
        return True

    def dim(self):
        return 3

    def data_ptr(self):
        return A


class Index:
    def __index__(self):
        return -1


def check(want, call, *args, **kw):
    """want: the exception of the binding, or the code of the library's refusal."""
    try:
        call(*args, **kw)
    except pbsa.PbsaError as e:
        assert e.code == want
    except Exception as e:
        assert not isinstance(want, int) and isinstance(e, want), repr(e)
    else:
        raise AssertionError("nothing was refused")


def test_the_parameters_are_the_structure_and_nothing_else():
    rc, out = in_child("""
import ctypes, torch
from paper_2604_21221_amd import pbsa
class Sub(pbsa.pbsa_params):
    pass
p = pbsa.make_params(2, 128, 64, 200, 16, 16, 4, 3, 0.088)
g = pbsa.make_grid(3, 8, 8, 1, 8, 8, 2, 128, 64)
for x, want in ((5, TypeError), (None, TypeError), (torch.zeros(3), TypeError), (g, ctypes.ArgumentError),
                ((ctypes.c_char * 200)(), ctypes.ArgumentError), (ctypes.pointer(p), ctypes.ArgumentError),
                (p, pbsa.PbsaError), (Sub.from_buffer_copy(p), pbsa.PbsaError)):
    for call in (lambda: pbsa.pbsa_pool_blocks(x, 0x10000, 0x10000, -1, 0x10000, stream=0),
                 lambda: pbsa.pbsa_select_blocks(x, None, 0, 0, 0, 0, 0, 0, stream=0)):
        try:
            call()
        except want as e:
            assert want is not pbsa.PbsaError or e.code == pbsa.PBSA_EINVAL
        else:
            raise AssertionError((x, "taken"))
        try:
            pbsa.pbsa_unblockify(x, 0x10000, 0, 0x10001, stream=0)
        except (TypeError, ctypes.ArgumentError):
            assert x is not g
        except pbsa.PbsaError as e:
            assert x is g and e.code == pbsa.PBSA_EALIGN
print("all seen")
""")
    assert rc == 0 and "all seen" in out, out[-2000:]


@pytest.mark.parametrize("n,want", [
    (-1, EINVAL), (np.int64(-1), EINVAL), (torch.tensor(-1), EINVAL), (Index(), EINVAL), (ctypes.c_int32(-1), EINVAL),
    (2 ** 40 - 1, EINVAL),                   # the low 32 bits count
    (True, EINVAL),                          # one block, and no address for it
    (-1.0, ctypes.ArgumentError), (None, ctypes.ArgumentError), ("a", ctypes.ArgumentError),
    ((ctypes.c_char * 200)(), ctypes.ArgumentError), (ctypes.c_int64(-1), ctypes.ArgumentError)])
def test_a_count_is_an_integer(n, want):
    check(want, pbsa.pbsa_pool_blocks, params(), A, A, n, None, stream=0)


@pytest.mark.parametrize("x,want", [
    (A, EINVAL), (None, EINVAL), (True, EINVAL), (-16, EINVAL), (2 ** 70, EINVAL), (Duck(), EINVAL),
    (torch.zeros(3), TypeError), (torch.nn.Parameter(torch.zeros(3, 4, 5)), TypeError),
    (np.int64(A), AttributeError), (Index(), AttributeError), (ctypes.c_void_p(A), AttributeError),
    ((ctypes.c_char * 200)(), AttributeError), (1.0, AttributeError)])
def test_an_address_is_a_tensors_or_an_integer(x, want):
    check(want, pbsa.pbsa_pool_blocks, params(), x, A, -1, A, stream=0)


@pytest.mark.parametrize("ws,want", [
    (None, EWS), ((A, 5), EWS), ((None, 5), EWS), ((A, 5, 6), EWS), ((A, torch.tensor(5)), EWS), ((A, np.int64(5)), EWS),
    (torch.zeros(300), EWS), ((torch.zeros(2), 5), TypeError), ((A, 5.0), ctypes.ArgumentError), ([A, 5], AttributeError)])
def test_a_workspace_is_a_tensor_or_address_and_size(ws, want):
    check(want, pbsa.pbsa_memory_update_apply, params(), A, A, A, A, A, A, A, ws, stream=0)


@pytest.mark.parametrize("stream,want", [(0, EINVAL), (False, EINVAL), (np.int64(0), AttributeError),
                                         (ctypes.c_void_p(0), AttributeError), (1.0, AttributeError)])
def test_a_stream_is_an_address_or_has_one(stream, want):
    check(want, pbsa.pbsa_pool_blocks, params(), A, A, -1, A, stream=stream)
    check(EINVAL, pbsa.pbsa_pool_blocks, params(), A, A, -1, A, stream=type("S", (), {"cuda_stream": 0})())


def test_signatures_match_the_header():
    """The kinds of arguments the binding passes, against include/pbsa.h."""
    import re
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(ROOT, "include", "pbsa.h")).read(), flags=re.S)
    for name, kinds in pbsa._SIGNATURES.items():
        args = re.search(rf"\b{name}\(([^)]*)\)", text).group(1).split(",")
        assert len(args) == len(kinds), name
        for arg, kind in zip(args, kinds):
            arg = " ".join(arg.split())
            want = ("p" if "pbsa_params" in arg else "g" if "pbsa_grid" in arg else "P" if "* const*" in arg else
                    "o" if arg.startswith("size_t*") else "L" if arg == "const int64_t* blk_stride_h" and "giPPL" in kinds else
                    "w" if arg in ("void* ws", "void* split_ws", "void* hip_stream") else "t" if "*" in arg else
                    {"int32_t": "i", "int64_t": "l", "size_t": "z"}[arg.split()[0]])
            assert kind == want, (name, arg)
