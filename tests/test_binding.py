"""The extension behind the grouping calls, as far as it can be seen without a GPU."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2510_11062_amd
from paper_2510_11062_amd import api

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

binding = api.load_binding()
ids = Odd(torch.int32)
try:
    binding.group_advantage(0, ids, ids, ids, Odd(torch.float32), None, 0.0, 2, 2, 2, 1e-6, 0, 0, True, False, 0, 0, 0)
except ValueError as e:
    print("raised", e)
"""


def test_a_tensor_that_throws_when_it_is_looked_at_raises():
    """In a process of its own: an exception that leaves the C function ends the process."""
    r = subprocess.run([sys.executable, "-c", TENSOR_THAT_THROWS], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "raised no strides here", (r.returncode, r.stdout, r.stderr[-500:])


def test_without_the_extension_only_its_own_calls_are_gone(monkeypatch):
    """An extension that does not load (built for another torch, say) takes the two calls with it that go through it."""
    monkeypatch.setitem(sys.modules, "paper_2510_11062_amd._binding", None)
    monkeypatch.delattr(paper_2510_11062_amd, "_binding", raising=False)
    monkeypatch.setattr(api, "_binding", None)
    monkeypatch.setattr(api, "_lib", None)
    assert api.load_library().at_grpo_version() > 0
    b = api._Batch()
    b.V, b.n_heads, b.n_tok, b.n_resp = 10, 1, 8, 4
    assert api.load_library().at_grpo_workspace_bytes(api.CALL_SURROGATE, api.C.byref(b), 0, 0, 0, 0) > 0
    ids, reward = torch.zeros(8, dtype=torch.int32), torch.zeros(8)
    with pytest.raises(api.AtGrpoError, match="_binding.so"):
        api.at_grpo_group_advantage(ids, ids, ids, reward, 2, 2, 2)
    with pytest.raises(api.AtGrpoError, match="_binding.so"):
        api.at_grpo_group_advantage_mixed(ids, ids, ids, reward, reward, 1.0, 2, 2, 2)
