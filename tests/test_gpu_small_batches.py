"""Preparation of small batches (routing, counts, lists and coefficients in one workgroup) at the edges of its range and
just past them, where the general kernels take over: one-pass step, two calls and the entropy call against the CPU oracle at
the tolerances of tests/test_gpu_parity.py.  The gradients of rows are products of the same operands on both sides of the
edge, so nothing but the lists, counts and coefficients can differ there."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2510_11062_amd import api, synth
from tests import helpers
from tests.gpu_case import DeviceCase, host
from tests.test_gpu_onepass import check_step_against_oracle
from tests.test_gpu_parity import say, tolerances


@pytest.mark.gpu
@pytest.mark.parametrize("E,N,K,lo,hi,padded,heads,agg", [
    (1, 1, 2, 1, 1, False, 1, "token_mean"),                    # two rows
    (256, 2, 2, 8, 32, False, 2, "seq_mean_token_mean"),        # 1024 responses on 16 lanes: the last that fit
    (205, 1, 5, 8, 32, False, 1, "seq_mean_token_mean"),        # 1025: general
    (8, 2, 4, 100, 512, True, 2, "token_mean"),                 # 64 responses of 512 slots: 32768 rows, the last that fit
    (13, 1, 5, 100, 512, True, 1, "token_mean"),                # 33280 rows: general
    (9, 3, 3, 60, 130, False, 3, "seq_mean_token_mean"),        # 32 lanes; lists that cross an 8192-row tile or not
])
def test_small_batch_preparation(gpu_device, E, N, K, lo, hi, padded, heads, agg):
    cfg = replace(synth.CONFIGS["C1"], name=f"small-{E * N * K}-{hi}", H=32, V=66, n_heads=heads, E=E, N=N, T=1, K=K, len_lo=lo,
                  len_hi=hi, padded=padded, reward_kind="bernoulli", forced_equal_groups=0 if E == 1 else 2,
                  old_sigma=0.02)
    say(f"[small] building {cfg.name}")
    c = helpers.build_case(cfg, device=gpu_device)
    ref = helpers.oracle_bwd(c, agg=agg)
    dc = DeviceCase(c, gpu_device)
    tol = tolerances(cfg)
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip, agg=agg)
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip, cfg.eps_clip,
                                      agg=agg)
    torch.cuda.synchronize()
    assert api.error_word(bwd["workspace"]) == 0
    check_step_against_oracle(dict(fwd, **{k: bwd[k] for k in ("d_hidden", "dW")}), ref, c, cfg, tol, "small, two calls")
    ent = host(api.at_grpo_token_entropy(dc.batch())["entropy"])
    assert np.all(ent[ref["w"] == 0] == 0) and np.all(ent[ref["w"] != 0] > 0)

    cfg16 = replace(cfg, H=64, dtype="bf16")
    c = helpers.build_case(cfg16, device=gpu_device)
    ref = helpers.oracle_bwd(c, agg=agg)
    dc = DeviceCase(c, gpu_device)
    out = api.at_grpo_policy_loss_fwd_bwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip, agg=agg)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    check_step_against_oracle(out, ref, c, cfg16, tolerances(cfg16), "small, one pass")
