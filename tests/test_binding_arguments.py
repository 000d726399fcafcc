"""What the binding makes of its arguments before the library sees them, with calls that the library refuses on the host: no
GPU.  What could end the interpreter runs in one of its own."""
import os
import subprocess
import sys

import pytest

pytest.importorskip("torch")

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
