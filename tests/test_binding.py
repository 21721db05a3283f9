"""The extension behind the grouping calls, as far as it can be seen without a GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

TENSOR_THAT_THROWS = """
import torch
from paper_2510_11062_amd import api

class Odd(torch.Tensor):
    @staticmethod
    def __new__(cls, dtype):
        return torch.Tensor._make_wrapper_subclass(cls, (8,), dtype=dtype, device="cuda:0", dispatch_sizes_strides_policy="strides")

    @classmethod
    def __torch_dispatch__(cls, func, types, args=(), kwargs=None):
        raise ValueError("no strides here")

api.load_library()
ids = Odd(torch.int32)
try:
    api._binding.group_advantage(0, ids, ids, ids, Odd(torch.float32), None, 0.0, 2, 2, 2, 1e-6, 0, 0, True, False, 0, 0, 0)
except ValueError as e:
    print("raised", e)
"""


def test_a_tensor_that_throws_when_it_is_looked_at_raises():
    """In a process of its own: an exception that leaves the C function ends the process."""
    r = subprocess.run([sys.executable, "-c", TENSOR_THAT_THROWS], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "raised no strides here", (r.returncode, r.stdout, r.stderr[-500:])
