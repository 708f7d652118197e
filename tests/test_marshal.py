"""Errors of the native argument marshalling that are found late.  No GPU needed: the tensors are fake device tensors."""
import os
import subprocess
import sys

import pytest

pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import sys
sys.path.insert(0, %r)
from collections import deque
import torch
from torch._subclasses.fake_tensor import FakeTensor, FakeTensorMode
import paper_2512_05746_amd as hq
f16, f32, i32 = torch.float16, torch.float32, torch.int32
mode = FakeTensorMode()
d = lambda *shape, dtype=torch.uint8: FakeTensor(mode, torch.empty(shape, dtype=dtype, device="meta"), torch.device("cuda"))
for k, error in ((1 << 31, ValueError), (64, RuntimeError)):   # a size beyond 32 bits; a tensor without memory
    for name, call in (
        ("linear", lambda: hq.hq_int_linear(d(1, k // 2), None, d(1, k // 2), None, y_dtype=i32, out=d(1, 1, dtype=i32))),
        ("linear_static", lambda: hq.hq_int_linear_static(d(1, k // 2), None, d(1, k // 2), None, y_dtype=i32,
                                                          out=d(1, 1, dtype=i32))),
        ("linear_single", lambda: hq.hq_int_linear_single(d(1, k // 2), None, d(1, 3, k // 2), None, y_dtype=i32,
                                                          out=d(1, 3, 1, dtype=i32))),
        ("conv2d", lambda: hq.hq_int_conv2d(d(1, 1, 1, k // 2), None, d(1, 1, k // 2), None, ksize=1, y_dtype=i32,
                                            out=d(1, dtype=i32))),
        ("conv2d_width", lambda: hq.hq_int_conv2d_width(d(3, 1, 1, 1, k // 2), None, d(1, 9, k // 2), None, y_dtype=i32,
                                                        out=d(1, dtype=i32))),
        ("quant", lambda: hq.hq_act_hadamard_quant(d(1, k, dtype=f16), out=(d(1, k // 2), d(1, dtype=f32)))),
        ("quant, pair of another type", lambda: hq.hq_act_hadamard_quant(d(1, k, dtype=f16),
                                                                         out=deque([d(1, k // 2), d(1, dtype=f32)]))),
    ):
        print(name, k, flush=True)
        try:
            call()
        except error as e:
            print("raised", type(e).__name__, e, flush=True)
print("done")
"""


def test_late_errors_are_raised():
    """In a process of its own, which an error raised without the interpreter's lock would end."""
    res = subprocess.run([sys.executable, "-c", PROGRAM % ROOT], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True,
                         timeout=300)
    assert res.returncode == 0 and res.stdout.endswith("done\n"), res.stdout
    assert res.stdout.count("raised ValueError") == res.stdout.count("raised RuntimeError") == 7, res.stdout


def test_a_library_of_another_pytorch_is_stale(monkeypatch):
    from paper_2512_05746_amd import build
    if build.is_stale():
        build.build_lib()
    assert not build.is_stale()
    monkeypatch.setattr(build, "built_for", lambda: "built for Python 0.0, PyTorch 0.0")
    assert build.is_stale()
