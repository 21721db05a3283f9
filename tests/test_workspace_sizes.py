"""Scratch memory that is asked for once, for the largest batch, serves the smaller ones: sizes do not fall where responses, their rows
or heads are added, on both sides of every rule that picks how many workgroups share a batch's responses.  Host only."""
import itertools

import pytest

from paper_2510_11062_amd import api

RESPONSES = [1, 2, 15, 16, 17, 511, 512, 513, 600, 1024, 4095, 4096, 4097, 8192, 8193, 32768, 32769, 100000]
ROWS = [1, 20, 59, 60, 159, 160, 511, 512, 600]
HEADS = [1, 2, 3, 16]


def size(call, n_tok, n_resp, n_heads, dtype=0):
    b = api._Batch()
    b.dtype, b.H, b.V, b.n_heads, b.n_tok, b.n_resp = dtype, 64, 1000, n_heads, n_tok, n_resp
    return api.load_library().at_grpo_workspace_bytes(call, api.C.byref(b), 0, 0, 0, 0)


def test_monitors_need_the_number_of_responses_only():
    for n in RESPONSES:
        sizes = {size(api.CALL_DIAGNOSTICS, n * rows, n, heads) for rows in ROWS for heads in HEADS}
        assert len(sizes) == 1 and sizes.pop() >= 28 * n, n


@pytest.mark.parametrize("call", [api.CALL_DIAGNOSTICS, api.CALL_SURROGATE])
def test_stage_sizes_do_not_fall(call):
    batches = sorted(itertools.product(RESPONSES, ROWS, HEADS))
    got = {(n, rows, heads): size(call, n * rows, n, heads) for n, rows, heads in batches}
    assert min(got.values()) > 0
    for axis, values in enumerate((RESPONSES, ROWS, HEADS)):
        for key in batches:
            at = values.index(key[axis])
            if at:
                less = key[:axis] + (values[at - 1],) + key[axis + 1:]
                assert got[less] <= got[key], (less, key)


@pytest.mark.parametrize("call", [api.CALL_SURROGATE, api.CALL_TOKEN_LOGPROB, api.CALL_TOKEN_ENTROPY, api.CALL_POLICY_LOSS_FWD,
                                  api.CALL_POLICY_LOSS_BWD, api.CALL_POLICY_LOSS_FWD_BWD])
@pytest.mark.parametrize("n_tok", [600, 2 ** 15, 2 ** 18])
@pytest.mark.parametrize("dtype", [0, 1])
def test_sizes_do_not_fall_with_more_responses_of_the_same_rows(call, n_tok, dtype):
    for heads in HEADS:
        got = [size(call, n_tok, n, heads, dtype) for n in RESPONSES if n <= n_tok]
        assert min(got) > 0 and got == sorted(got), (heads, got)
