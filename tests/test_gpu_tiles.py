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


@pytest.mark.gpu
@pytest.mark.parametrize("accumulate", [False, True], ids=["overwrite", "accumulate"])
@pytest.mark.parametrize("over", [0, 1], ids=["one launch", "two launches"])
def test_fp32_gradients_of_three_heads_in_one_launch_or_two(gpu_device, over, accumulate):
    """The last size at which the workgroups of dHidden and dW fit the chip together (three per compute unit), and the first at
    which they do not: 210 rows are 4 tiles of dHidden in 32 parts each, and dW has a tile per 64 vocabulary rows.  The
    profile says which of them were launched.  Against torch in 64 bits: fp32 sums of up to V products, 1e-5."""
    dev, H, heads = gpu_device, 64, 3
    V = 64 * (3 * torch.cuda.get_device_properties(dev).multi_processor_count - 4 * 32) + over
    say(f"[tiles] fp32 V={V} accumulate={accumulate}")
    gen = torch.Generator(device=dev).manual_seed(V)
    n, R = 210, 6
    hidden = torch.randn(n, H, generator=gen, device=dev)
    W = [torch.randn(V, H, generator=gen, device=dev) * 0.05 for _ in range(heads)]
    y = torch.randint(0, V, (n,), generator=gen, device=dev, dtype=torch.int32)
    y[-1] = V - 1
    cu = torch.arange(R + 1, device=dev) * (n // R)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device=dev)
    adv = torch.tensor([1.0, -0.5, 0.8, 0.0, 2.0, -1.0], device=dev)
    batch = api.Batch(hidden, W, y, cu, None, i32([0, 1, 2, 0, 1, 2]), i32([0, 1, 2]))
    old = api.at_grpo_token_logprob(batch)["logp"].clone()
    dW0 = [torch.randn(V, H, generator=gen, device=dev) * 1e-3 for _ in range(heads)]
    dW = [w.clone() for w in dW0]
    api.at_grpo_profile_enable(True)
    out = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, 0.2, 0.2, dW=dW, accumulate_dW=accumulate)
    torch.cuda.synchronize()
    prof = api.at_grpo_profile_read()
    api.at_grpo_profile_enable(False)
    assert prof["head_dh"][0] >= heads and (prof["head_dw"][0] >= heads) == bool(over)
    rows = torch.arange(n, device=dev)
    for m in range(heads):
        mine = (rows // (n // R)) % heads == m
        h, t = hidden[mine].double(), y[mine].long()
        g = -adv[rows[mine] // (n // R)].double() / int(mine.sum())       # ratio 1
        dz = -g[:, None] * torch.softmax(h @ W[m].double().T, 1)
        dz[torch.arange(len(t), device=dev), t] += g
        for got, ref in ((out["d_hidden"][mine], dz @ W[m].double()), (dW[m], dz.T @ h + (dW0[m].double() if accumulate else 0))):
            assert float((got.double() - ref).norm() / ref.norm()) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("one_pass", [True, False], ids=["one_pass", "two_calls"])
@pytest.mark.parametrize("dtype,V,H,n", [(torch.bfloat16, 34_200_003, 64, 300), (torch.bfloat16, 8_600_001, 64, 12_400),
                                         (torch.float32, 8_500_003, 32, 300)],
                         ids=["64 k-rows of 4 GiB", "256 transposed rows of 4 GiB", "fp32"])
def test_vocabulary_of_millions(gpu_device, dtype, V, H, n, one_pass):
    """Rows of dZ so long that a tile of them spans 4 GiB and more.  With p about 1 / V, row y_t of dW is g_t h_t up to
    n / V, and d_hidden of a row is g (W[y] - E_p[W]), which fp32 torch gives for sampled rows."""
    say(f"[tiles] V={V} H={H} n={n} {dtype} one_pass={one_pass}")
    gen = torch.Generator(device=gpu_device).manual_seed(3)
    W = torch.randn(V, H, generator=gen, device=gpu_device, dtype=dtype).mul_(0.02)
    hidden = torch.randn(n, H, generator=gen, device=gpu_device, dtype=dtype)
    y = torch.randint(0, V, (n,), generator=gen, device=gpu_device, dtype=torch.int32)
    y[-1] = V - 1
    cu = torch.arange(0, n + 1, 100, device=gpu_device)
    adv = torch.where(torch.arange(cu.numel() - 1, device=gpu_device) % 2 == 0, 1.0, -0.5).float()
    batch = api.Batch(hidden, [W], y, cu)
    old = api.at_grpo_token_logprob(batch)["logp"]
    if one_pass:
        out = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, 0.2, 0.2)
    else:
        fwd = api.at_grpo_policy_loss_fwd(batch, old, adv, 0.2, 0.2)
        out = api.at_grpo_policy_loss_bwd(batch, old, adv, fwd["logp"], fwd["lse"], 0.2, 0.2)
        out["logp"] = fwd["logp"]
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    g = (-adv / n).repeat_interleave(100)
    rows = torch.unique(torch.cat([torch.arange(0, n, max(1, n // 60), device=gpu_device),
                                   torch.arange(250, n, 256, device=gpu_device), torch.arange(n - 3, n, device=gpu_device)]))
    h, step = hidden[rows].float(), 1 << 20
    lse = torch.full((rows.numel(),), -float("inf"), device=gpu_device)
    for v in range(0, V, step):
        lse = torch.logaddexp(lse, torch.logsumexp(h @ W[v:v + step].float().T, 1))
    target = W[y.long()].float()
    mean = torch.zeros(rows.numel(), H, device=gpu_device)
    for v in range(0, V, step):
        w = W[v:v + step].float()
        mean += torch.exp(h @ w.T - lse[:, None]) @ w
    close = lambda a, r: float((a - r).norm() / r.norm())
    tol = 2e-2 if dtype == torch.bfloat16 else 1e-3
    assert (out["logp"][rows] - ((h * target[rows]).sum(1) - lse)).abs().max() <= 1e-3
    assert close(out["d_hidden"][rows].float(), g[rows, None] * (target[rows] - mean)) <= tol
    one = torch.bincount(y.long() - y.min(), minlength=1)[y.long() - y.min()] == 1      # tokens drawn once
    want = g[:, None] * hidden.float()
    assert close(out["dW"][0][y.long()][one], want[one]) <= tol
    del W, out, batch
    api.release_workspace()
    torch.cuda.empty_cache()
