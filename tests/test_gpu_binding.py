"""How the grouping call's outputs are allocated by the extension: errors keep their Python types, other threads run."""
import ctypes
import os
import subprocess
import sys
import sysconfig

import pytest
import torch

from paper_2510_11062_amd import api


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def inputs(R, dev):
    """R responses in groups of four under R / 4 environments."""
    env = (torch.arange(R, device=dev) // 4).to(torch.int32)
    zero = torch.zeros(R, dtype=torch.int32, device=dev)
    return env, zero, zero, torch.rand(R, generator=torch.Generator(device=dev).manual_seed(3), device=dev), R // 4, 1, 1


@pytest.mark.gpu
def test_out_of_memory_keeps_its_type(gpu_device):
    """A program that shrinks its batch when memory runs out catches torch.OutOfMemoryError.  The allocator's limit is set to what the
    process holds, so that it refuses the outputs by itself; afterwards the same call goes through."""
    R = 1 << 24
    args = inputs(R, gpu_device)
    first = api.at_grpo_group_advantage(*args)["adv"].clone()      # the scratch memory is there from here on
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(gpu_device).total_memory
    say(f"[binding] outputs of {R} responses past the limit of memory")
    torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved(gpu_device) / total, gpu_device)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            api.at_grpo_group_advantage(*args)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0, gpu_device)
    assert torch.equal(api.at_grpo_group_advantage(*args)["adv"], first)


HOOK = r"""
#include <Python.h>
#include <hip/hip_runtime_api.h>
static long calls = 0, held = 0;
extern "C" {
void* hook_alloc(ssize_t bytes, int, hipStream_t) {
  void* p = nullptr;
  ++calls;
  held += PyGILState_Check();
  return hipMalloc(&p, static_cast<size_t>(bytes)) == hipSuccess ? p : nullptr;
}
void hook_free(void* p, ssize_t, int, hipStream_t) { (void)hipFree(p); }
long hook_calls(void) { return calls; }
long hook_held(void) { return held; }
}
"""


@pytest.mark.gpu
def test_other_threads_run_while_memory_is_allocated(gpu_device, tmp_path):
    """torch.empty lets go of the interpreter's lock while the allocator works; an allocation that has to reach the driver under it
    stops every other Python thread, and two locks taken in turn can wait for each other.  The pool's allocator notes who holds it."""
    src, lib = tmp_path / "hook.cpp", tmp_path / "hook.so"
    src.write_text(HOOK)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", sysconfig.get_paths()["include"], str(src), "-o", str(lib), "-L", os.path.join(rocm, "lib"), "-lamdhip64"],
                   check=True)
    R = 1 << 20
    args = inputs(R, gpu_device)
    want = api.at_grpo_group_advantage(*args)["adv"].clone()       # the scratch memory is there from here on
    torch.cuda.synchronize()
    say(f"[binding] {R} responses, outputs from a pool of their own")
    hook = ctypes.PyDLL(str(lib))
    allocator = torch.cuda.memory.CUDAPluggableAllocator(str(lib), "hook_alloc", "hook_free")
    pool = torch.cuda.MemPool(allocator.allocator())
    with torch.cuda.use_mem_pool(pool):
        out = api.at_grpo_group_advantage(*args)
    assert torch.equal(out["adv"], want)
    calls, held = hook.hook_calls(), hook.hook_held()
    torch.cuda.synchronize()
    del out, pool
    assert calls > 0 and held == 0, (calls, held)
