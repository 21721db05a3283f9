"""Head contractions at the sizes where the launch plan changes: last tiles of every dimension, tiles split along k,
weights read transposed or as they stand.  One-pass step and two-call sequence against the CPU oracle with the bf16
tolerances of tests/test_gpu_parity.py (the logit gradient and d_hidden are rounded to bf16, 2^-9 per element,
against 2e-2)."""
from dataclasses import replace

import pytest
import torch

from paper_2510_11062_amd import api, synth
from tests import helpers
from tests.gpu_case import DeviceCase
from tests.test_gpu_onepass import check_step_against_oracle
from tests.test_gpu_parity import say, tolerances


@pytest.mark.gpu
@pytest.mark.parametrize("H,V,E,K,length", [
    (64, 64, 5, 4, 2),          # one k-step of the logits and of dHidden, one tile everywhere
    (128, 321, 2048, 6, 1),     # 12288 rows: the most that dHidden reads W untransposed for; V no multiple of 64
    (128, 321, 2050, 6, 1),     # 12300 rows: W is transposed
    (320, 8192, 65, 8, 1),      # 520 rows: 6 tiles of 128 k-steps in dHidden, split; ragged tiles along H and rows
    (256, 300, 128, 8, 4),      # 4096 rows: 2 tiles of 64 k-steps in dW, split; ragged last vocabulary tile
    (192, 4100, 9, 5, 17),      # 765 rows: parts of unequal length, 60 columns in the last k-step
])
def test_tiles_and_split_contractions(gpu_device, H, V, E, K, length):
    cfg = replace(synth.CONFIGS["C3"], name=f"tiles-{H}-{V}-{E * K * length}", dtype="bf16", H=H, V=V, n_heads=1, E=E, N=1,
                  T=1, K=K, len_lo=length, len_hi=length, reward_kind="uniform", old_sigma=0.02)
    say(f"[tiles] building {cfg.name}")
    c = helpers.build_case(cfg, device=gpu_device)
    ref = helpers.oracle_bwd(c)
    dc = DeviceCase(c, gpu_device)
    tol = tolerances(cfg)
    out = api.at_grpo_policy_loss_fwd_bwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    check_step_against_oracle(out, ref, c, cfg, tol, "tiles, one pass")
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    check_step_against_oracle(dict(fwd, **{k: bwd[k] for k in ("d_hidden", "dW")}), ref, c, cfg, tol, "tiles, two calls")


@pytest.mark.gpu
@pytest.mark.parametrize("H,V,E,K,length", [
    (32, 3, 3, 2, 1),           # one k-step everywhere, fewer vocabulary rows than a lane pair sums
    (32, 66, 31, 3, 7),         # 651 rows: one column past a tile, rows and k ragged
    (96, 333, 700, 4, 6),       # 16800 rows: dW split into the most parts, dHidden whole
    (64, 5000, 20, 4, 2),       # 160 rows: dHidden split along the vocabulary
    (64, 4200, 128, 8, 2),      # 2048 rows: 128 x 128 tiles in dZ
    (512, 200, 512, 8, 4),      # 16384 rows: 128 x 128 tiles in dHidden
    (1024, 8190, 5, 4, 2),      # 128 x 128 tiles in dW
])
def test_fp32_tiles(gpu_device, H, V, E, K, length):
    """The fp32 contractions at the edges of their tiles and of the rules that choose tile and split, against the oracle
    at the fp32 tolerances (sums of up to 16800 fp32 products against 1e-4)."""
    cfg = replace(synth.CONFIGS["C1"], name=f"f32-tiles-{H}-{V}-{E * K * length}", H=H, V=V, E=E, N=1, T=1, K=K,
                  len_lo=length, len_hi=length, reward_kind="uniform", forced_equal_groups=0, old_sigma=0.02)
    say(f"[tiles] building {cfg.name}")
    c = helpers.build_case(cfg, device=gpu_device)
    ref = helpers.oracle_bwd(c)
    dc = DeviceCase(c, gpu_device)
    out = api.at_grpo_policy_loss_fwd_bwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    check_step_against_oracle(out, ref, c, cfg, tolerances(cfg), "fp32 tiles")
