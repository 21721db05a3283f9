"""Parity of the HIP library (through its C ABI) against the CPU oracle.

Tolerances:
  * integers (group ids, segment offsets, permutations, counts) and clip masks: bit-exact;
  * fp32 path: 1e-4 relative;
  * bf16 path (fp32 accumulation): 1e-2 absolute on log-probs, 2e-2 relative on the loss;
  * gradients (d_hidden, dW): every row within tol of its reference in norm, every element within
    tol * (|ref| + rms of its row), and the Frobenius ratio within tol; tol = 2e-2 (bf16), 1e-4 (fp32)
    (tests.helpers.assert_grad_close).
Clip masks are compared bit-exactly when both sides see the same logp (stage parity); end to end
the tokens whose d = logp - old_logp lies within the logp tolerance of a threshold are excluded
and counted.
"""
import re
import os
import sys
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import at_grpo_oracle as orc
from paper_2510_11062_amd import api, synth
from tests import helpers
from tests.gpu_case import DeviceCase, host

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


# ---------------------------------------------------------------------------- host-only checks
def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "at_grpo.h")).read()
    declared = sorted(set(re.findall(r"\b(at_grpo_[a-z_]+)\s*\(", header)))
    assert set(declared) == set(api.EXPORTS)
    lib = api.load_library()
    for name in declared:
        assert hasattr(lib, name), name
    assert api.at_grpo_version() >= 100
    assert lib.at_grpo_status_string(0) == b"ok"
    assert lib.at_grpo_status_string(3).startswith(b"workspace")


def test_workspace_query_and_argument_errors_on_host():
    lib = api.load_library()
    assert lib.at_grpo_workspace_bytes(api.CALL_GROUP_ADVANTAGE, None, 64, 4, 2, 2) > 0
    assert lib.at_grpo_workspace_bytes(api.CALL_GROUP_ADVANTAGE, None, 0, 4, 2, 2) == 0
    assert lib.at_grpo_workspace_bytes(99, None, 64, 4, 2, 2) == 0
    b = api._Batch()
    b.dtype, b.H, b.V, b.n_heads, b.n_tok, b.n_resp = 1, 2048, 151936, 1, 1 << 19, 1024
    fwd = lib.at_grpo_workspace_bytes(api.CALL_POLICY_LOSS_FWD, b, 0, 0, 0, 0)
    bwd = lib.at_grpo_workspace_bytes(api.CALL_POLICY_LOSS_BWD, b, 0, 0, 0, 0)
    assert 0 < fwd < bwd < (40 << 30)
    # the one-pass step needs the backward's buffers plus its lists and partial sums; fp32 runs the two calls
    step = lib.at_grpo_workspace_bytes(api.CALL_POLICY_LOSS_FWD_BWD, b, 0, 0, 0, 0)
    assert bwd < step < bwd + (1 << 30)
    b.dtype = 0
    f32 = [lib.at_grpo_workspace_bytes(c, b, 0, 0, 0, 0)
           for c in (api.CALL_POLICY_LOSS_FWD, api.CALL_POLICY_LOSS_BWD, api.CALL_POLICY_LOSS_FWD_BWD)]
    assert f32[2] == max(f32[0], f32[1]) > 0
    b.dtype = 1
    # null outputs of the one-pass call are rejected before anything is launched
    assert lib.at_grpo_policy_loss_fwd_bwd(b, None, None, 0.2, 0.2, 0, None, None, None, None, None, None, None,
                                           None, 0, None, 0, None) == 1
    b.H = 2050                       # not a multiple of 64 elements for bf16
    assert lib.at_grpo_workspace_bytes(api.CALL_POLICY_LOSS_FWD, b, 0, 0, 0, 0) == 0
    # null pointers are rejected before anything is launched
    st = lib.at_grpo_group_advantage(4, 1, 1, 1, None, None, None, None, 1e-6, 0, 0,
                                     None, None, None, None, None, None, None, None, 0, None)
    assert st == 1
    st = lib.at_grpo_group_advantage_mixed(4, 1, 1, 1, None, None, None, None, None, 1.0, 1e-6, 0, 0, None,
                                           None, None, None, None, None, None, None, None, None, 0, None)
    assert st == 1
    b.H = 2048
    assert lib.at_grpo_token_logprob(b, None, None, None, 0, None) == 1
    # head update: fixed-size workspace; null arrays, bf16 without fp32 weights and step 0 are rejected
    assert lib.at_grpo_workspace_bytes(api.CALL_HEAD_UPDATE, None, 0, 0, 0, 0) > 0
    opt = api._Adam(1e-6, 0.9, 0.999, 1e-8, 0.01, 1.0, 1, 1)
    assert lib.at_grpo_head_update(1, 64, 64, 1, None, None, None, None, None, opt, None, None, 0, None) == 1
    one = (api.C.c_void_p * 1)(256)
    assert lib.at_grpo_head_update(1, 64, 64, 1, one, None, one, one, one, opt, 256, None, 0, None) == 1
    opt.step = 0
    assert lib.at_grpo_head_update(0, 64, 64, 1, one, None, one, one, one, opt, 256, None, 0, None) == 1
    opt.step = 1
    assert lib.at_grpo_head_update(0, 64, 64, 1, one, None, one, one, one, opt, 256, None, 0, None) == 3
    assert lib.at_grpo_workspace_bytes(api.CALL_DIAGNOSTICS, b, 0, 0, 0, 0) > 7 * 4 * 1024
    assert lib.at_grpo_surrogate_diagnostics(b, None, None, None, 0.2, 0.2, None, None, None, 0, None) == 1


def test_room_for_partial_results():
    """Of a small head no more than its few k-steps can be cut into (here dHidden's one tile of 16 steps into four parts, 1 MiB), of a
    large one 1024 partial tiles."""
    b = api._Batch()
    b.dtype, b.n_heads, b.n_resp = 1, 1, 8
    b.H, b.V, b.n_tok = 64, 1000, 256
    assert api.load_library().at_grpo_workspace_bytes(api.CALL_POLICY_LOSS_BWD, b, 0, 0, 0, 0) < 2 << 20
    b.H, b.V, b.n_tok = 2048, 151936, 2300
    rest = api.load_library().at_grpo_workspace_bytes(api.CALL_POLICY_LOSS_BWD, b, 0, 0, 0, 0) - 2304 * (151936 + 2048) * 2
    assert 0 <= rest - (256 << 20) < 1 << 20


# ---------------------------------------------------------------------------- S1 + S2
def run_group_advantage(dev, st, cfg, **kw):
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(dev)
    out = api.at_grpo_group_advantage(i32(st.env_id), i32(st.agent_id), i32(st.turn_id),
                                      torch.from_numpy(st.reward).to(dev), cfg.E, cfg.N, cfg.T, **kw)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    return out


def check_group_advantage(out, st, cfg, eps_std=1e-6, ddof=0, norm="std"):
    key = orc.group_key(st.env_id, st.agent_id, st.turn_id, cfg.N, cfg.T)
    gid, G, offs, perm = orc.group_segments(key)
    adv, mean, std = orc.group_advantage(st.reward, gid, G, eps_std=eps_std, ddof=ddof, norm=norm)
    assert int(out["n_groups"].item()) == G
    assert np.array_equal(host(out["group_id"]), gid)
    assert np.array_equal(host(out["seg_offsets"])[:G + 1], offs)
    assert np.array_equal(host(out["perm"]), perm)
    got = host(out["adv"]).astype(np.float64)
    assert np.all(got[std[gid] == 0] == 0)                   # all-equal groups: exactly zero
    assert np.allclose(got, adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[:G], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[:G], std, rtol=1e-4, atol=1e-7)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4", "C5"])
def test_group_advantage_matches_oracle_full_size(gpu_device, name):
    cfg = synth.CONFIGS[name]
    say(f"[group_advantage] {name} R={cfg.n_resp}")
    st = synth.make_structure(cfg)
    check_group_advantage(run_group_advantage(gpu_device, st, cfg), st, cfg)


@pytest.mark.gpu
@pytest.mark.parametrize("variant", ["early_termination", "singletons", "large_groups", "ddof1", "norm_none",
                                     "many_keys", "many_keys_early_termination"])
def test_group_advantage_variants(gpu_device, variant):
    base = synth.CONFIGS["C4"]
    kw = {}
    if variant == "early_termination":
        cfg = replace(base, E=40, drop_tail_frac=0.3)
    elif variant == "singletons":
        cfg = replace(base, E=50, K=1)
    elif variant == "large_groups":
        cfg = replace(base, E=3, N=1, T=2, K=700, reward_kind="uniform", forced_equal_groups=1)
    elif variant == "many_keys":
        # more keys and responses than the one-workgroup path takes: the multi-launch pipeline
        cfg = replace(base, E=2100, N=2, T=2, K=8, reward_kind="mixed")
    elif variant == "many_keys_early_termination":
        cfg = replace(base, E=1200, N=2, T=4, K=3, drop_tail_frac=0.3)
    elif variant == "ddof1":
        cfg = replace(base, E=30)
        kw = dict(ddof=1)
    else:
        cfg = replace(base, E=30, reward_kind="uniform")
        kw = dict(norm="none")
    say(f"[group_advantage] variant {variant} R={cfg.n_resp}")
    st = synth.make_structure(cfg)
    check_group_advantage(run_group_advantage(gpu_device, st, cfg, **kw), st, cfg, **kw)


@pytest.mark.gpu
def test_group_advantage_key_box_beyond_one_scan_block(gpu_device):
    """80000 keys, 240000 responses: the three-kernel scan.  Integers are compared in full; the
    advantages on a sample of groups the oracle handles one by one."""
    cfg = replace(synth.CONFIGS["C4"], E=40000, N=2, T=1, K=3, reward_kind="uniform", forced_equal_groups=50)
    st = synth.make_structure(cfg)
    say(f"[group_advantage] large key box R={cfg.n_resp} keys={cfg.E * cfg.N * cfg.T}")
    out = run_group_advantage(gpu_device, st, cfg)
    key = orc.group_key(st.env_id, st.agent_id, st.turn_id, cfg.N, cfg.T)
    gid, G, offs, perm = orc.group_segments(key)
    assert int(out["n_groups"].item()) == G
    assert np.array_equal(host(out["group_id"]), gid)
    assert np.array_equal(host(out["seg_offsets"])[:G + 1], offs)
    assert np.array_equal(host(out["perm"]), perm)
    pick = np.random.default_rng(1).choice(G, size=400, replace=False)
    pick.sort()
    members = np.concatenate([perm[offs[g]:offs[g + 1]] for g in pick])
    sub_gid = np.repeat(np.arange(400), [offs[g + 1] - offs[g] for g in pick])
    adv, mean, std = orc.group_advantage(st.reward[members], sub_gid, 400)
    got = host(out["adv"]).astype(np.float64)[members]
    assert np.all(got[std[sub_gid] == 0] == 0)
    assert np.allclose(got, adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[pick], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[pick], std, rtol=1e-4, atol=1e-7)


@pytest.mark.gpu
def test_group_advantage_mixed_group_sizes_and_determinism(gpu_device):
    rng = np.random.default_rng(5)
    E, N, T = 7, 2, 3
    sizes = rng.choice([1, 2, 5, 16, 17, 40, 64, 65, 130], size=E * N * T)
    e, i, t = np.meshgrid(np.arange(E), np.arange(N), np.arange(T), indexing="ij")
    env = np.repeat(e.ravel(), sizes)
    agent = np.repeat(i.ravel(), sizes)
    turn = np.repeat(t.ravel(), sizes)
    sh = rng.permutation(env.shape[0])
    st = type("S", (), {})()
    st.env_id, st.agent_id, st.turn_id = env[sh], agent[sh], turn[sh]
    st.reward = rng.random(env.shape[0]).astype(np.float32)
    cfg = type("C", (), dict(E=E, N=N, T=T))()
    say(f"[group_advantage] mixed sizes R={env.shape[0]}")
    first = run_group_advantage(gpu_device, st, cfg)
    check_group_advantage(first, st, cfg)
    again = run_group_advantage(gpu_device, st, cfg)
    for k in ("group_id", "seg_offsets", "perm", "adv", "group_mean", "group_std"):
        assert torch.equal(first[k], again[k])


@pytest.mark.gpu
@pytest.mark.parametrize("name,alpha", [("C1", 1.0), ("C2", 1.0), ("C3", 0.3), ("C4", 1.0), ("C5", 0.7)])
def test_group_advantage_mixed_matches_oracle(gpu_device, name, alpha):
    """Eq. (3) mixing + Eq. (1) + the tree-sampling arg max, at the configurations' real R."""
    cfg = synth.CONFIGS[name]
    st = synth.make_structure(cfg)
    r_team, r_loc = synth.make_team_local_rewards(cfg, cfg.n_resp)
    if name == "C3":
        r_loc = (r_loc * np.float32(1.7) + np.float32(0.1)).astype(np.float32)   # inexact products and sums
    say(f"[group_advantage_mixed] {name} R={cfg.n_resp} alpha={alpha}")
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(gpu_device)
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(gpu_device)
    out = api.at_grpo_group_advantage_mixed(i32(st.env_id), i32(st.agent_id), i32(st.turn_id), f32(r_team),
                                            f32(r_loc), alpha, cfg.E, cfg.N, cfg.T)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    mixed = orc.mix_rewards(r_team, r_loc, alpha)
    assert np.array_equal(host(out["reward"]).view(np.uint32), mixed.view(np.uint32))    # bit-exact
    st.reward = mixed
    check_group_advantage(out, st, cfg)
    key = orc.group_key(st.env_id, st.agent_id, st.turn_id, cfg.N, cfg.T)
    gid, G, _, _ = orc.group_segments(key)
    assert np.array_equal(host(out["best"])[:G], orc.select_candidates(mixed, gid, G))


@pytest.mark.gpu
def test_group_advantage_mixed_large_groups_and_no_best(gpu_device):
    cfg = replace(synth.CONFIGS["C4"], E=3, N=1, T=2, K=700)
    st = synth.make_structure(cfg)
    r_team, r_loc = synth.make_team_local_rewards(cfg, cfg.n_resp, levels=4)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(gpu_device)
    f32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(gpu_device)
    say(f"[group_advantage_mixed] large groups R={cfg.n_resp}")
    out = api.at_grpo_group_advantage_mixed(i32(st.env_id), i32(st.agent_id), i32(st.turn_id), f32(r_team),
                                            f32(r_loc), 0.5, cfg.E, cfg.N, cfg.T)
    torch.cuda.synchronize()
    mixed = orc.mix_rewards(r_team, r_loc, 0.5)
    st.reward = mixed
    check_group_advantage(out, st, cfg)
    key = orc.group_key(st.env_id, st.agent_id, st.turn_id, cfg.N, cfg.T)
    gid, G, _, _ = orc.group_segments(key)
    assert np.array_equal(host(out["best"])[:G], orc.select_candidates(mixed, gid, G))
    skipped = api.at_grpo_group_advantage_mixed(i32(st.env_id), i32(st.agent_id), i32(st.turn_id),
                                                f32(r_team), f32(r_loc), 0.5, cfg.E, cfg.N, cfg.T,
                                                want_best=False, want_stats=False)
    torch.cuda.synchronize()
    assert skipped["best"] is None and torch.equal(skipped["adv"], out["adv"])


@pytest.mark.gpu
def test_group_advantage_flags_ids_out_of_range(gpu_device):
    cfg = replace(synth.CONFIGS["C1"])
    st = synth.make_structure(cfg)
    st.env_id = st.env_id.copy()
    st.env_id[3] = cfg.E + 2
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(gpu_device)
    out = api.at_grpo_group_advantage(i32(st.env_id), i32(st.agent_id), i32(st.turn_id),
                                      torch.from_numpy(st.reward).to(gpu_device), cfg.E, cfg.N, cfg.T)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) & 1
    assert int(out["group_id"][3].item()) == -1 and float(out["adv"][3].item()) == 0.0


@pytest.mark.gpu
@pytest.mark.parametrize("group_by", ["trajectory", "parallel", "agent_turn"])
@pytest.mark.parametrize("name", ["C4", "C2"])
def test_group_advantage_under_the_other_keys(gpu_device, name, group_by):
    """Trajectory-level groups (every candidate of a task, Sec. 5.3) and the groups parallel sampling
    leaves (one response each after the first turn, Sec. 4.1) at the configurations' real sizes:
    integers bit-exact, advantages as for the paper's key; C4 takes the multi-launch path, C2 the
    one-workgroup path."""
    cfg = synth.CONFIGS[name]
    st = synth.make_structure(cfg)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(gpu_device)
    say(f"[group_advantage_keyed] {name} {group_by} R={cfg.n_resp}")
    out = api.at_grpo_group_advantage_keyed(group_by, i32(st.env_id), i32(st.agent_id), i32(st.turn_id),
                                            torch.from_numpy(st.reward).to(gpu_device), cfg.E, cfg.N, cfg.T,
                                            sample_id=i32(st.sample_id), n_sample=cfg.K)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    key = orc.group_key_by(st.env_id, st.agent_id, st.turn_id, st.sample_id, cfg.N, cfg.T, cfg.K, group_by)
    gid, G, offs, perm = orc.group_segments(key)
    adv, mean, std = orc.group_advantage(st.reward, gid, G)
    assert int(out["n_groups"]) == G
    assert np.array_equal(host(out["group_id"]), gid)
    assert np.array_equal(host(out["seg_offsets"])[:G + 1], offs)
    assert np.array_equal(host(out["perm"]), perm)
    got = host(out["adv"]).astype(np.float64)
    assert np.all(got[std[gid] == 0] == 0) and np.allclose(got, adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[:G], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[:G], std, rtol=1e-4, atol=1e-7)
    if group_by == "parallel":
        assert np.all(got[st.turn_id > 0] == 0) and np.abs(got[st.turn_id == 0]).max() > 0
    if group_by == "trajectory":
        assert G == cfg.E
    if group_by == "agent_turn":
        plain = api.at_grpo_group_advantage(i32(st.env_id), i32(st.agent_id), i32(st.turn_id),
                                            torch.from_numpy(st.reward).to(gpu_device), cfg.E, cfg.N, cfg.T)
        torch.cuda.synchronize()
        assert torch.equal(plain["adv"], out["adv"]) and torch.equal(plain["perm"], out["perm"])


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["C1", "C4"])
def test_group_advantage_non_finite_rewards_take_no_part(gpu_device, name):
    """A NaN and an infinite reward raise the data flag and drop out: no group id, advantage 0, and the
    rest of their groups is what the oracle gives without them (both launch shapes)."""
    cfg = synth.CONFIGS[name]
    st = synth.make_structure(cfg)
    reward = st.reward.copy()
    bad = np.array([3, cfg.n_resp - 2])
    reward[bad[0]] = np.nan
    reward[bad[1]] = np.inf
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(gpu_device)
    say(f"[group_advantage] {name}: non-finite rewards at {bad.tolist()}")
    out = api.at_grpo_group_advantage(i32(st.env_id), i32(st.agent_id), i32(st.turn_id),
                                      torch.from_numpy(reward).to(gpu_device), cfg.E, cfg.N, cfg.T)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 2
    keep = np.ones(cfg.n_resp, bool)
    keep[bad] = False
    kept = np.nonzero(keep)[0]
    key = orc.group_key(st.env_id[kept], st.agent_id[kept], st.turn_id[kept], cfg.N, cfg.T)
    gid, G, offs, perm = orc.group_segments(key)
    adv, mean, std = orc.group_advantage(reward[kept], gid, G)
    got_gid, got_adv = host(out["group_id"]), host(out["adv"]).astype(np.float64)
    assert np.all(got_gid[bad] == -1) and np.all(got_adv[bad] == 0)
    assert int(out["n_groups"]) == G
    assert np.array_equal(got_gid[kept], gid)
    assert np.array_equal(host(out["seg_offsets"])[:G + 1], offs)
    assert np.array_equal(host(out["perm"])[:kept.size], kept[perm])
    assert np.all(np.isfinite(got_adv)) and np.allclose(got_adv[kept], adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[:G], mean, rtol=1e-4, atol=1e-7)


# ---------------------------------------------------------------------------- S3..S8 on oracle-sized cases
def mini_cfg(name):
    """Oracle-sized twins: same heads, H, layout and reward structure as the named config.  C2 keeps
    the full vocabulary (594 vocabulary tiles with a ragged tail); the others use V = 4736
    (18 tiles and a half) so that the fp64 oracle stays within seconds."""
    base = synth.CONFIGS[name]
    if name == "C1":
        return base
    if name == "C2":
        return replace(base, name="C2-mini", E=1, len_lo=2, len_hi=9)
    if name == "C3":
        return replace(base, name="C3-mini", E=2, len_lo=3, len_hi=10, V=4736)
    if name == "C4":
        return replace(base, name="C4-mini", E=8, len_lo=1, len_hi=2, V=4736)
    if name == "C5":
        return replace(base, name="C5-mini", E=2, len_kind="uniform", len_lo=1, len_hi=6, V=4736)
    raise KeyError(name)


def tolerances(cfg):
    if cfg.dtype == "f32":
        return dict(logp_abs=None, logp_rel=1e-4, loss_rel=1e-4, grad_rel=1e-4)
    return dict(logp_abs=1e-2, logp_rel=None, loss_rel=2e-2, grad_rel=2e-2)


def assert_logp_close(got, ref, tol, what):
    got = np.asarray(got, np.float64)
    if tol["logp_abs"] is not None:
        err = np.abs(got - ref).max()
        assert err <= tol["logp_abs"], f"{what}: max abs err {err}"
    else:
        err = (np.abs(got - ref) / np.maximum(np.abs(ref), 1.0)).max()
        assert err <= tol["logp_rel"], f"{what}: max rel err {err}"
    return err


def compare_clip_masks(got_mask, ref, old_logp, cfg, logp_tol):
    lo32, hi32 = orc.clip_thresholds(cfg.eps_clip, cfg.eps_clip)
    d = ref["logp"].astype(np.float32) - old_logp
    near = (np.abs(d - lo32) <= logp_tol) | (np.abs(d - hi32) <= logp_tol)
    same = got_mask == ref["clip_mask"]
    assert np.all(same | near), "clip mask differs away from the thresholds"
    return int(near.sum())


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4", "C5"])
def test_policy_loss_fwd_bwd_matches_oracle(gpu_device, name):
    cfg = mini_cfg(name)
    tol = tolerances(cfg)
    say(f"[fwd/bwd] building {cfg.name}: H={cfg.H} V={cfg.V} heads={cfg.n_heads}")
    c = helpers.build_case(cfg, device=gpu_device)
    # more drift on one config so that the clipped branches carry real weight
    if name == "C5":
        c.old_logp = (c.old_logp + c.noise).astype(np.float32)
    say(f"[fwd/bwd] oracle on {c.st.n_tok} rows ({c.st.n_valid} response tokens)")
    grad_loss = None if cfg.n_heads == 1 else np.linspace(1.0, 0.5, cfg.n_heads)
    ref = helpers.oracle_bwd(c, grad_loss=grad_loss)
    dc = DeviceCase(c, gpu_device)

    say("[fwd/bwd] at_grpo_token_logprob")
    lp = api.at_grpo_token_logprob(dc.batch())
    torch.cuda.synchronize()
    assert api.error_word(lp["workspace"]) == 0
    assert_logp_close(host(lp["logp"]), ref["logp"], tol, "token_logprob.logp")
    assert_logp_close(host(lp["lse"]), ref["lse"], tol, "token_logprob.lse")

    say("[fwd/bwd] at_grpo_policy_loss_fwd")
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    assert api.error_word(fwd["workspace"]) == 0
    err = assert_logp_close(host(fwd["logp"]), ref["logp"], tol, "fwd.logp")
    assert_logp_close(host(fwd["lse"]), ref["lse"], tol, "fwd.lse")
    assert torch.equal(fwd["logp"], lp["logp"])
    assert np.array_equal(host(fwd["n_valid"]), ref["n_valid"])
    loss = host(fwd["loss"]).astype(np.float64)
    assert np.all(np.abs(loss - ref["loss"]) <= tol["loss_rel"] * np.abs(ref["loss"]) + 1e-5), (loss, ref["loss"])
    n_near = compare_clip_masks(host(fwd["clip_mask"]), ref, c.old_logp, cfg, max(10 * err, 1e-6))
    say(f"[fwd/bwd] loss {loss} vs {ref['loss']}; logp err {err:.2e}; {n_near} tokens next to a threshold")
    off = ref["w"] == 0
    assert np.all(host(fwd["logp"])[off] == 0) and np.all(host(fwd["clip_mask"])[off] == 0)

    say("[fwd/bwd] at_grpo_policy_loss_bwd")
    gl = None if grad_loss is None else torch.from_numpy(grad_loss.astype(np.float32)).to(gpu_device)
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"],
                                      cfg.eps_clip, cfg.eps_clip, grad_loss=gl)
    torch.cuda.synchronize()
    assert api.error_word(bwd["workspace"]) == 0
    dH = host(bwd["d_hidden"]).astype(np.float64)
    # rows without gradient are exactly zero; tokens next to a threshold may flip
    lo32, hi32 = orc.clip_thresholds(cfg.eps_clip, cfg.eps_clip)
    d = ref["logp"].astype(np.float32) - c.old_logp
    near = (np.abs(d - lo32) <= max(10 * err, 1e-6)) | (np.abs(d - hi32) <= max(10 * err, 1e-6))
    zero_rows = (ref["g"] == 0) & ~near
    assert np.all(dH[zero_rows] == 0)
    keep = ~near
    assert not near.any(), "a token sits on a clip threshold: its branch may differ between the two sides"
    r_dh = helpers.assert_grad_close(dH[keep], ref["d_hidden"][keep], tol["grad_rel"], "d_hidden")
    say(f"[fwd/bwd] d_hidden worst row {r_dh[0]:.3e}, worst element {r_dh[1]:.3e}, Frobenius {r_dh[2]:.3e}")
    for k in range(cfg.n_heads):
        dWk = host(bwd["dW"][k]).astype(np.float64)
        r_dw = helpers.assert_grad_close(dWk, ref["dW"][k], tol["grad_rel"], f"dW[{k}]")
        say(f"[fwd/bwd] dW[{k}] worst row {r_dw[0]:.3e}, worst element {r_dw[1]:.3e}, Frobenius {r_dw[2]:.3e}; "
            f"column-sum residual {np.abs(dWk.sum(axis=0)).max():.2e}")

    say("[fwd/bwd] accumulate_dW adds onto an existing gradient")
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(5)
    # what is already there has the size of the gradient itself, so a lost or doubled add shows everywhere
    base = [torch.randn(g.shape, generator=gen, device=gpu_device) * g.abs().mean() for g in bwd["dW"]]
    before = [b.clone() for b in base]
    acc = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"],
                                      cfg.eps_clip, cfg.eps_clip, grad_loss=gl, dW=base, accumulate_dW=True)
    torch.cuda.synchronize()
    for k in range(cfg.n_heads):
        added = host(acc["dW"][k]).astype(np.float64) - host(before[k]).astype(np.float64)
        helpers.assert_grad_close(added, ref["dW"][k], max(tol["grad_rel"], 1e-3), f"accumulated dW[{k}]")
        assert torch.allclose(acc["dW"][k], before[k] + bwd["dW"][k], rtol=0, atol=1e-6 * float(bwd["dW"][k].abs().max()))
    assert torch.equal(acc["d_hidden"], bwd["d_hidden"])


@pytest.mark.gpu
@pytest.mark.parametrize("agg", ["token_mean", "seq_mean_token_mean"])
@pytest.mark.parametrize("name", ["C1", "C3"])
def test_surrogate_stage_is_bit_exact_on_masks(gpu_device, name, agg):
    """Given identical logp on both sides, clip masks and counts are bit-exact and the loss agrees
    to fp32 accuracy (stage parity of the ratio / clip / masked averaging step)."""
    cfg = replace(mini_cfg(name), H=64, V=256, name=name + "-stage")
    if name == "C3":
        cfg = replace(cfg, E=16, len_lo=40, len_hi=300, padded=True)
    c = helpers.build_case(cfg)
    c.old_logp = (c.old_logp + 2 * c.noise).astype(np.float32)
    on = helpers.oracle_fwd(c, agg=agg)
    logp32 = on["logp"].astype(np.float32)
    ref = orc.policy_loss_from_logp(logp32, c.old_logp, c.adv, c.st.mask, on["head_of_tok"], on["resp_of_tok"],
                                    cfg.n_heads, cfg.eps_clip, cfg.eps_clip, agg)
    dc = DeviceCase(c, gpu_device)
    say(f"[surrogate] {cfg.name} agg={agg} rows={c.st.n_tok}")
    out = api.at_grpo_surrogate_from_logp(dc.layout_only(), torch.from_numpy(logp32).to(gpu_device),
                                          dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip, agg)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    assert np.array_equal(host(out["clip_mask"]), ref[1])
    assert np.array_equal(host(out["n_valid"]), ref[2])
    assert (ref[1] & orc.CLIP_ZERO_GRAD).astype(bool).sum() > 0
    loss = host(out["loss"]).astype(np.float64)
    assert np.all(np.abs(loss - ref[0]) <= 1e-4 * np.abs(ref[0]) + 1e-6), (loss, ref[0])
    again = api.at_grpo_surrogate_from_logp(dc.layout_only(), torch.from_numpy(logp32).to(gpu_device),
                                            dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip, agg)
    assert torch.equal(again["loss"], out["loss"])            # fixed-order reduction


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C5"])
def test_token_entropy_matches_oracle(gpu_device, name):
    """Entropy of the next-token distribution from the same pass as the log-probs; the log-probs of
    this variant are bit-identical to those of the plain call."""
    cfg = mini_cfg(name)
    c = helpers.build_case(cfg, device=gpu_device)
    st = c.st
    ref = orc.token_entropy(c.hidden, c.W, st.mask, c.head_of_tok)
    dc = DeviceCase(c, gpu_device)
    say(f"[entropy] {cfg.name} rows={st.n_tok} V={cfg.V}")
    out = api.at_grpo_token_entropy(dc.batch())
    plain = api.at_grpo_token_logprob(dc.batch())
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    assert torch.equal(out["logp"], plain["logp"]) and torch.equal(out["lse"], plain["lse"])
    got = host(out["entropy"]).astype(np.float64)
    tol = tolerances(cfg)
    if tol["logp_abs"] is not None:
        assert np.abs(got - ref).max() <= tol["logp_abs"]
    else:
        assert (np.abs(got - ref) / np.maximum(np.abs(ref), 1.0)).max() <= tol["logp_rel"]
    on = ref != 0
    assert on.any() and np.all(got[~on] == 0)
    assert np.all(got[on] > 0) and np.all(got[on] <= np.log(cfg.V) + 1e-3)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["C1", "C3", "C5"])
def test_surrogate_diagnostics_match_oracle(gpu_device, name):
    """Clip counts are integers: exact given identical log-probs.  KL estimate and mean ratio to fp32
    accuracy.  Two calls give identical bits (fixed-order sums)."""
    cfg = replace(mini_cfg(name), H=64, V=256, name=name + "-diag")
    if name == "C3":
        cfg = replace(cfg, E=16, len_lo=40, len_hi=300, padded=True)
    if name == "C5":
        cfg = replace(cfg, E=8, len_lo=1, len_hi=90)
    c = helpers.build_case(cfg)
    c.old_logp = (c.old_logp + 2 * c.noise).astype(np.float32)
    on = helpers.oracle_fwd(c)
    logp32 = on["logp"].astype(np.float32)
    counts, kl, ratio = orc.surrogate_diagnostics(logp32, c.old_logp, c.adv, c.st.mask, on["head_of_tok"],
                                                  on["resp_of_tok"], cfg.n_heads, cfg.eps_clip, cfg.eps_clip)
    dc = DeviceCase(c, gpu_device)
    say(f"[diagnostics] {cfg.name} rows={c.st.n_tok} heads={cfg.n_heads}")
    out = api.at_grpo_surrogate_diagnostics(dc.layout_only(), torch.from_numpy(logp32).to(gpu_device), dc.old_logp,
                                            dc.adv, cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    assert np.array_equal(host(out["counts"]).astype(np.int64), counts)
    assert counts[:, 1].sum() > 0 and counts[:, 2].sum() > 0 and counts[:, 3].sum() > 0
    stats = host(out["stats"]).astype(np.float64)
    assert np.allclose(stats[:, 0], kl, rtol=1e-4, atol=1e-7)
    assert np.allclose(stats[:, 1], ratio, rtol=1e-5, atol=0)
    again = api.at_grpo_surrogate_diagnostics(dc.layout_only(), torch.from_numpy(logp32).to(gpu_device),
                                              dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    assert torch.equal(again["stats"], out["stats"]) and torch.equal(again["counts"], out["counts"])
    # the counts are the bit counts of the clip mask the surrogate stage writes
    sur = api.at_grpo_surrogate_from_logp(dc.layout_only(), torch.from_numpy(logp32).to(gpu_device), dc.old_logp,
                                          dc.adv, cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    cm = host(sur["clip_mask"])
    assert [(cm & b != 0).sum() for b in (1, 2, 4)] == counts[:, 1:].sum(axis=0).tolist()
    assert host(sur["n_valid"]).tolist() == counts[:, 0].tolist()


@pytest.mark.gpu
def test_seq_mean_aggregation_end_to_end(gpu_device):
    cfg = mini_cfg("C1")
    c = helpers.build_case(cfg)
    ref = helpers.oracle_bwd(c, agg="seq_mean_token_mean")
    dc = DeviceCase(c, gpu_device)
    say("[seq-mean] fwd + bwd on C1")
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip,
                                      agg="seq_mean_token_mean")
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                      cfg.eps_clip, agg="seq_mean_token_mean")
    torch.cuda.synchronize()
    assert abs(float(fwd["loss"][0]) - ref["loss"][0]) <= 1e-4 * abs(ref["loss"][0]) + 1e-6
    helpers.assert_grad_close(host(bwd["d_hidden"]), ref["d_hidden"], 1e-4, "d_hidden")
    helpers.assert_grad_close(host(bwd["dW"][0]), ref["dW"][0], 1e-4, "dW")


@pytest.mark.gpu
def test_data_errors_are_flagged_and_masked(gpu_device):
    cfg = mini_cfg("C1")
    c = helpers.build_case(cfg)
    bad = c.token_id.copy()
    bad[5] = cfg.V + 3
    dc = DeviceCase(c, gpu_device, token_id=bad)
    say("[errors] token id out of range")
    out = api.at_grpo_token_logprob(dc.batch())
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) & 4
    assert float(out["logp"][5]) == 0.0
    good = np.ones(c.st.n_tok, bool)
    good[5] = False
    ref = helpers.oracle_fwd(c)
    assert_logp_close(host(out["logp"])[good], ref["logp"][good], tolerances(cfg), "logp with one bad row")


@pytest.mark.gpu
def test_empty_head_and_all_masked_rows(gpu_device):
    """A head that receives no token gives loss 0 and dW 0; a fully masked batch runs cleanly."""
    cfg = replace(mini_cfg("C1"), n_heads=2)
    c = helpers.build_case(cfg)
    c.st.head_of_agent[:] = 0                           # every agent -> head 0; head 1 stays empty
    c.resp_of_tok, c.head_of_tok = orc.token_heads(c.st.n_tok, c.st.cu_seqlens, c.st.agent_id, c.st.head_of_agent)
    c.token_id, c.old_logp = helpers.oracle_rollout_standin(c.hidden, c.W, c.st.mask, c.head_of_tok, c.u, c.noise)
    ref = helpers.oracle_bwd(c)
    dc = DeviceCase(c, gpu_device)
    say("[edge] empty head")
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    dW = [torch.full((cfg.V, cfg.H), 7.0, device=gpu_device) for _ in range(2)]
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                      cfg.eps_clip, dW=dW)
    torch.cuda.synchronize()
    assert host(fwd["n_valid"]).tolist() == [c.st.n_valid, 0]
    assert float(fwd["loss"][1]) == 0.0
    assert abs(float(fwd["loss"][0]) - ref["loss"][0]) <= 1e-4 * abs(ref["loss"][0]) + 1e-6
    assert float(bwd["dW"][1].abs().max()) == 0.0
    helpers.assert_grad_close(host(bwd["dW"][0]), ref["dW"][0], 1e-4, "dW[0]")
    helpers.assert_grad_close(host(bwd["d_hidden"]), ref["d_hidden"], 1e-4, "d_hidden")
    say("[edge] all rows masked")
    dc.mask = torch.zeros(c.st.n_tok, dtype=torch.uint8, device=gpu_device)
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                      cfg.eps_clip)
    torch.cuda.synchronize()
    assert host(fwd["n_valid"]).tolist() == [0, 0] and float(fwd["loss"].abs().max()) == 0.0
    assert float(fwd["logp"].abs().max()) == 0.0
    assert float(bwd["d_hidden"].abs().max()) == 0.0
    assert all(float(g.abs().max()) == 0.0 for g in bwd["dW"])


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,H,V", [("bf16", 192, 1001), ("f32", 96, 1001), ("bf16", 64, 130), ("bf16", 320, 8192)])
@pytest.mark.parametrize("padded", [False, True])
def test_odd_shapes_and_empty_responses(gpu_device, dtype, H, V, padded):
    """Ragged everything: V not a multiple of the 64-wide k padding (or below one tile), H below one
    tile, responses of length 0 and 1, row counts that are not multiples of 4, three heads."""
    cfg = replace(synth.CONFIGS["C1"], name=f"odd-{dtype}-{H}-{V}", dtype=dtype, H=H, V=V, n_heads=3, E=5, N=3,
                  T=2, K=3, len_lo=0, len_hi=9, padded=padded, reward_kind="uniform", forced_equal_groups=1,
                  seed=synth.BASE_SEED + 77 + H)
    tol = tolerances(cfg)
    c = helpers.build_case(cfg, device=gpu_device)
    assert (c.st.lengths == 0).any() and (c.st.lengths == 1).any()
    c.old_logp = (c.old_logp + 2 * c.noise).astype(np.float32)
    grad_loss = np.array([1.0, 0.25, 2.0])
    for agg in ("token_mean", "seq_mean_token_mean"):
        ref = helpers.oracle_bwd(c, agg=agg, grad_loss=grad_loss)
        dc = DeviceCase(c, gpu_device)
        say(f"[odd] {cfg.name} padded={padded} agg={agg}: rows={c.st.n_tok}")
        fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip, agg=agg)
        gl = torch.from_numpy(grad_loss.astype(np.float32)).to(gpu_device)
        bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                          cfg.eps_clip, agg=agg, grad_loss=gl)
        torch.cuda.synchronize()
        assert api.error_word(fwd["workspace"]) == 0
        err = assert_logp_close(host(fwd["logp"]), ref["logp"], tol, "logp")
        assert np.array_equal(host(fwd["n_valid"]), ref["n_valid"])
        loss = host(fwd["loss"]).astype(np.float64)
        assert np.all(np.abs(loss - ref["loss"]) <= tol["loss_rel"] * np.abs(ref["loss"]) + 1e-5), (loss, ref["loss"])
        lo32, hi32 = orc.clip_thresholds(cfg.eps_clip, cfg.eps_clip)
        d = ref["logp"].astype(np.float32) - c.old_logp
        near = (np.abs(d - lo32) <= max(10 * err, 1e-6)) | (np.abs(d - hi32) <= max(10 * err, 1e-6))
        assert not near.any()
        assert np.array_equal(host(fwd["clip_mask"]), ref["clip_mask"])
        helpers.assert_grad_close(host(bwd["d_hidden"]), ref["d_hidden"], tol["grad_rel"], "d_hidden")
        assert np.all(host(bwd["d_hidden"])[ref["g"] == 0] == 0)
        for k in range(3):
            helpers.assert_grad_close(host(bwd["dW"][k]), ref["dW"][k], tol["grad_rel"], f"dW[{k}]")


@pytest.mark.gpu
def test_single_row_batch(gpu_device):
    cfg = replace(synth.CONFIGS["C1"], name="one-row", dtype="bf16", H=64, V=300, E=1, N=1, T=1, K=1, len_lo=1,
                  len_hi=1, forced_equal_groups=0)
    c = helpers.build_case(cfg, device=gpu_device)
    c.adv = np.array([0.7], np.float32)            # a singleton group has advantage 0; give the row a gradient
    ref = helpers.oracle_bwd(c)
    dc = DeviceCase(c, gpu_device)
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                      cfg.eps_clip)
    torch.cuda.synchronize()
    assert abs(float(fwd["logp"][0]) - ref["logp"][0]) <= 1e-2
    assert abs(float(fwd["loss"][0]) - ref["loss"][0]) <= 2e-2 * abs(ref["loss"][0]) + 1e-5
    helpers.assert_grad_close(host(bwd["d_hidden"]), ref["d_hidden"], 2e-2, "d_hidden")
    helpers.assert_grad_close(host(bwd["dW"][0]), ref["dW"][0], 2e-2, "dW")


@pytest.mark.gpu
def test_reproducible_and_independent_of_workspace_contents(gpu_device):
    """No float atomics anywhere: two runs give identical bits, also when the scratch memory starts
    out full of NaN patterns (every padded region the kernels read must be written by them first)."""
    cfg = mini_cfg("C3")
    c = helpers.build_case(cfg, device=gpu_device)
    dc = DeviceCase(c, gpu_device)

    def run():
        ga = api.at_grpo_group_advantage(dc.env_id, dc.agent_id, dc.turn_id, dc.reward, cfg.E, cfg.N, cfg.T)
        fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, ga["adv"], cfg.eps_clip, cfg.eps_clip)
        bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, ga["adv"], fwd["logp"], fwd["lse"],
                                          cfg.eps_clip, cfg.eps_clip)
        torch.cuda.synchronize()
        return [ga["adv"].clone(), ga["perm"].clone(), fwd["loss"].clone(), fwd["logp"].clone(), fwd["lse"].clone(),
                fwd["clip_mask"].clone(), bwd["d_hidden"].clone()] + [g.clone() for g in bwd["dW"]]

    say("[repro] first run")
    first = run()
    ws = api._workspace(1, gpu_device)
    ws.fill_(0xFF)
    say("[repro] second run on poisoned scratch")
    second = run()
    for a, b in zip(first, second):
        assert torch.equal(a, b)
    assert all(torch.isfinite(t.float()).all() for t in second)


# ---------------------------------------------------------------------------- several super-chunks per head
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_backward_across_several_super_chunks_matches_oracle_elementwise(gpu_device, dtype):
    """Each head receives more than two full super-chunks (32768 list positions each) of rows that
    carry gradient, plus a ragged last one, at a size the fp64 oracle still runs in full: dW is then
    accumulated across launches inside one call, d_hidden and logp rows come from every chunk, and
    everything is compared row by row and element by element.  V = 1001 leaves a ragged vocabulary
    tile; the second half of the test adds onto a random pre-filled dW."""
    H = 128 if dtype == "bf16" else 64
    cfg = replace(synth.CONFIGS["C3"], name=f"chunks-{dtype}", dtype=dtype, H=H, V=1001, n_heads=2, E=24, N=2, T=2,
                  K=8, len_lo=180, len_hi=280, reward_kind="uniform", forced_equal_groups=2,
                  seed=synth.BASE_SEED + 900)
    tol = tolerances(cfg)
    say(f"[chunks] building {cfg.name}: H={cfg.H} V={cfg.V}")
    c = helpers.build_case(cfg, device=gpu_device)
    grad_loss = np.array([1.0, 0.5])
    say(f"[chunks] oracle on {c.st.n_tok} rows")
    ref = helpers.oracle_bwd(c, grad_loss=grad_loss)
    per_head = [int(((ref["g"] != 0) & (c.head_of_tok == k)).sum()) for k in range(2)]
    say(f"[chunks] rows with gradient per head: {per_head}")
    assert min(per_head) > 2 * 32768 and all(n % 32768 != 0 for n in per_head)
    dc = DeviceCase(c, gpu_device)
    fwd = api.at_grpo_policy_loss_fwd(dc.batch(), dc.old_logp, dc.adv, cfg.eps_clip, cfg.eps_clip)
    torch.cuda.synchronize()
    assert api.error_word(fwd["workspace"]) == 0
    err = assert_logp_close(host(fwd["logp"]), ref["logp"], tol, "logp")
    assert_logp_close(host(fwd["lse"]), ref["lse"], tol, "lse")
    loss = host(fwd["loss"]).astype(np.float64)
    assert np.all(np.abs(loss - ref["loss"]) <= tol["loss_rel"] * np.abs(ref["loss"]) + 1e-5), (loss, ref["loss"])
    assert np.array_equal(host(fwd["n_valid"]), ref["n_valid"])
    # the backward is given the oracle's log-probs (rounded to fp32) so that both sides take the same
    # branch at every token, also next to a threshold: stage parity of S7 + S8
    logp_in = torch.from_numpy(ref["logp"].astype(np.float32)).to(gpu_device)
    lse_in = torch.from_numpy(ref["lse"].astype(np.float32)).to(gpu_device)
    gl = torch.from_numpy(grad_loss.astype(np.float32)).to(gpu_device)
    say("[chunks] backward")
    bwd = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, logp_in, lse_in, cfg.eps_clip, cfg.eps_clip,
                                      grad_loss=gl)
    torch.cuda.synchronize()
    assert api.error_word(bwd["workspace"]) == 0
    dH = host(bwd["d_hidden"]).astype(np.float64)
    assert np.all(dH[ref["g"] == 0] == 0)
    r = helpers.assert_grad_close(dH, ref["d_hidden"], tol["grad_rel"], "d_hidden")
    say(f"[chunks] d_hidden worst row {r[0]:.3e}, worst element {r[1]:.3e}, Frobenius {r[2]:.3e}")
    for k in range(2):
        r = helpers.assert_grad_close(host(bwd["dW"][k]), ref["dW"][k], tol["grad_rel"], f"dW[{k}]")
        say(f"[chunks] dW[{k}] worst row {r[0]:.3e}, worst element {r[1]:.3e}, Frobenius {r[2]:.3e}")
    # the chain as a caller runs it (forward's own outputs) lands on the same gradients
    chain = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                        cfg.eps_clip, grad_loss=gl)
    torch.cuda.synchronize()
    lo32, hi32 = orc.clip_thresholds(cfg.eps_clip, cfg.eps_clip)
    d = ref["logp"].astype(np.float32) - c.old_logp
    near = (np.abs(d - lo32) <= max(10 * err, 1e-6)) | (np.abs(d - hi32) <= max(10 * err, 1e-6))
    say(f"[chunks] {int(near.sum())} tokens next to a threshold")
    helpers.assert_grad_close(host(chain["d_hidden"]).astype(np.float64)[~near], ref["d_hidden"][~near],
                              tol["grad_rel"], "d_hidden (chain)")
    if not near.any():
        for k in range(2):
            helpers.assert_grad_close(host(chain["dW"][k]), ref["dW"][k], tol["grad_rel"], f"dW[{k}] (chain)")

    say("[chunks] accumulate onto a random pre-filled dW")
    gen = torch.Generator(device=gpu_device)
    gen.manual_seed(9)
    base = [torch.randn(g.shape, generator=gen, device=gpu_device) * g.abs().mean() for g in bwd["dW"]]
    before = [b.clone() for b in base]
    acc = api.at_grpo_policy_loss_bwd(dc.batch(), dc.old_logp, dc.adv, logp_in, lse_in, cfg.eps_clip, cfg.eps_clip,
                                      grad_loss=gl, dW=base, accumulate_dW=True)
    torch.cuda.synchronize()
    for k in range(2):
        added = host(acc["dW"][k]).astype(np.float64) - host(before[k]).astype(np.float64)
        helpers.assert_grad_close(added, ref["dW"][k], max(tol["grad_rel"], 1e-3), f"accumulated dW[{k}]")


# ---------------------------------------------------------------------------- mini-batches (App. C.1)
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_two_mini_batches_accumulate_into_one_update(gpu_device, dtype):
    """App. C.1 trains with a global batch of 128 prompts in mini-batches of 64: here a batch of 128
    responses is split into two halves of 64, each half's loss (its own token mean, weighted 1/2) is
    back-propagated with accumulate_dW on the second call, and one clipped Adam step follows.  The
    accumulated gradient and the stepped weights are compared with the oracle run the same way."""
    cfg = replace(synth.CONFIGS["C1"], name=f"minibatch-{dtype}", dtype=dtype, H=64, V=700, E=8, N=2, T=2, K=4,
                  len_lo=5, len_hi=40, reward_kind="uniform", forced_equal_groups=1, seed=synth.BASE_SEED + 64)
    assert cfg.n_resp == 128
    tol = tolerances(cfg)
    c = helpers.build_case(cfg, device=gpu_device)
    st = c.st
    dc = DeviceCase(c, gpu_device)
    half_w = np.array([0.5])
    hyper = dict(lr=1e-3, weight_decay=0.01, max_grad_norm=1.0)
    passed = {k: float(np.float32(v)) for k, v in dict(hyper, beta1=0.9, beta2=0.999, eps=1e-8).items()}

    dW_ref = np.zeros((cfg.V, cfg.H))
    dW_dev = [torch.empty((cfg.V, cfg.H), dtype=torch.float32, device=gpu_device).fill_(float("nan"))]
    losses, losses_ref = [], []
    for half in range(2):
        r0, r1 = 64 * half, 64 * (half + 1)
        t0, t1 = int(st.cu_seqlens[r0]), int(st.cu_seqlens[r1])
        cu_h = st.cu_seqlens[r0:r1 + 1] - t0
        ref = orc.policy_loss_bwd(c.hidden[t0:t1], c.W, c.token_id[t0:t1], None, cu_h, None, None,
                                  c.old_logp[t0:t1], c.adv[r0:r1], cfg.eps_clip, cfg.eps_clip, grad_loss=half_w)
        dW_ref += ref["dW"][0]
        losses_ref.append(ref["loss"][0])
        batch = api.Batch(dc.hidden[t0:t1].clone(), dc.W, dc.token_id[t0:t1].clone(),
                          torch.from_numpy(cu_h).to(gpu_device))
        old_h, adv_h = dc.old_logp[t0:t1].clone(), dc.adv[r0:r1].clone()
        say(f"[minibatch] half {half}: responses {r0}..{r1 - 1}, rows {t0}..{t1 - 1}")
        fwd = api.at_grpo_policy_loss_fwd(batch, old_h, adv_h, cfg.eps_clip, cfg.eps_clip)
        api.at_grpo_policy_loss_bwd(batch, old_h, adv_h, fwd["logp"], fwd["lse"], cfg.eps_clip,
                                    cfg.eps_clip, grad_loss=torch.from_numpy(half_w.astype(np.float32)).to(gpu_device),
                                    dW=dW_dev, accumulate_dW=(half == 1))
        torch.cuda.synchronize()
        losses.append(float(fwd["loss"][0]))
    assert np.allclose(losses, losses_ref, rtol=tol["loss_rel"], atol=1e-5)
    r = helpers.assert_grad_close(host(dW_dev[0]), dW_ref, tol["grad_rel"], "accumulated dW")
    say(f"[minibatch] accumulated dW worst row {r[0]:.3e}, worst element {r[1]:.3e}")
    # neither half alone is the answer
    assert helpers.rel_fro(host(dW_dev[0]), ref["dW"][0]) > 0.3

    # one clipped Adam step on the accumulated gradient
    if dtype == "bf16":
        master = [dc.W[0].float()]
        W = [dc.W[0].clone()]
        up = api.at_grpo_head_update(W, dW_dev, [torch.zeros_like(master[0])], [torch.zeros_like(master[0])], 1,
                                     W_master=master, **hyper)
        stepped = master[0]
    else:
        W = [dc.W[0].clone()]
        up = api.at_grpo_head_update(W, dW_dev, [torch.zeros_like(W[0])], [torch.zeros_like(W[0])], 1, **hyper)
        stepped = W[0]
    torch.cuda.synchronize()
    W0 = c.W[0].astype(np.float64)
    upd = orc.head_update([W0], [dW_ref], [np.zeros_like(W0)], [np.zeros_like(W0)], 1, **passed)
    assert np.isclose(float(up["grad_norm"][0]), upd["grad_norm"], rtol=tol["grad_rel"])
    move, move_ref = host(stepped).astype(np.float64) - W0, upd["W"][0] - W0
    # The first Adam step moves a weight by lr * g / (|g| + eps), i.e. by about lr * sign(g): it is compared
    # where the gradient element is not so small against its row that the bf16 rounding of dZ (about 1e-3 of
    # the row's rms) could turn its sign, and the rest may differ by at most the two steps a flipped sign costs.
    rms = np.linalg.norm(dW_ref, axis=1, keepdims=True) / np.sqrt(cfg.H)
    firm = np.abs(dW_ref) > (0.1 if dtype == "bf16" else 1e-3) * rms
    assert firm.mean() > 0.8
    assert np.allclose(move[firm], move_ref[firm], rtol=max(tol["grad_rel"], 1e-3), atol=1e-3 * passed["lr"])
    assert np.abs(move - move_ref).max() <= 2.1 * passed["lr"]
    assert helpers.rel_fro(move, move_ref) <= 0.1
    if dtype == "bf16":
        assert torch.equal(W[0], master[0].to(torch.bfloat16))
