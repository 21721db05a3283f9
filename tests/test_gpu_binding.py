"""How the grouping call's outputs are allocated by the extension: errors keep their Python types."""
import sys

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
