"""Grouping at the sizes where the launch plan changes: one launch (key ranges), pools (partition by key range), and the
histogram pipeline for what neither takes.  Integers against the oracle in full; advantages and statistics on groups
the oracle handles one by one, within 1e-4 (fp32 sums of a few members)."""
import threading

import numpy as np
import pytest
import torch

from oracle import at_grpo_oracle as orc
from paper_2510_11062_amd import api
from tests.gpu_case import host
from tests.test_gpu_parity import say


def draw(E, N, T, sizes, seed):
    """sizes: members of every key, in key order."""
    rng = np.random.default_rng(seed)
    key = np.repeat(np.arange(E * N * T), sizes)[rng.permutation(int(np.sum(sizes)))]
    reward = (rng.integers(0, 9, size=key.size) / np.float32(8)).astype(np.float32)
    return (key // (N * T)).astype(np.int32), (key // T % N).astype(np.int32), (key % T).astype(np.int32), reward


CASES = {
    "range: most responses": (2048, 2, 4, lambda rng, n: np.full(n, 4)),
    "range: most keys": (8191, 2, 4, lambda rng, n: np.ones(n, int)),
    "range: more members than a list holds": (2, 1, 2, lambda rng, n: np.array([6000, 3, 4097, 700])),
    "range: 4097 responses": (241, 1, 1, lambda rng, n: np.full(n, 17)),
    "pool: fewest responses": (8193, 2, 2, lambda rng, n: np.full(n, 2)),
    "pool: keys missing, sizes up to 24": (3000, 2, 12, lambda rng, n: rng.integers(0, 25, n) * (rng.random(n) < 0.4)),
    "pool: the first with 512 bins": (49153, 2, 2, lambda rng, n: np.full(n, 4)),
    "pool: bins of fewer responses for their keys": (525000, 2, 1, lambda rng, n: 1 + (np.arange(n) % 2)),
    "histogram: as many keys as responses": (500000, 2, 1, lambda rng, n: np.ones(n, int)),
    "pool: one oversized bin": (5000, 2, 3, lambda rng, n: np.where(np.arange(n) == 777, 9000, 3)),
    # ids from a part of their extents: the work of one workgroup goes to all of them
    "range: one workgroup's keys, groups of 256": (65280, 1, 1, lambda rng, n: np.where(np.arange(n) < 256, 255, 0)),
    "range: one workgroup's keys, sizes up to 40": (20000, 1, 1, lambda rng, n: np.where(np.arange(n) < 700, rng.integers(0, 41, n), np.arange(n) % 9 == 0)),
    "range: all but two in the last workgroup's keys": (12000, 1, 1, lambda rng, n: np.where(np.arange(n) >= n - 90, 70, np.arange(n) < 2)),
    "pool: one bin, groups of 128": (524288, 1, 1, lambda rng, n: np.where(np.arange(n) < 1024, 128, 0)),
    "pool: the last bin, groups of 15 to 18": (262143, 1, 2, lambda rng, n: np.where(np.arange(n) >= n - 2000, rng.integers(15, 19, n), np.arange(n) % 8 == 0)),
    "pool: large bins among small ones": (3000, 2, 12, lambda rng, n: np.where(np.arange(n) // 2000 % 3 == 1, 24, rng.random(n) < 0.3)),
    "pool: large bins only": (6000, 2, 12, lambda rng, n: np.where(np.arange(n) < n // 16, 30, 0)),
    "pool: blocks sorted by bin": (150001, 1, 2, lambda rng, n: np.full(n, 8)),
    "histogram: few keys": (4, 1, 2, lambda rng, n: np.full(n, 8800)),
    "histogram: few responses, many keys": (40000, 1, 2, lambda rng, n: (rng.random(n) < 0.2).astype(int)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("mixed", [False, True], ids=["given", "mixed"])
@pytest.mark.parametrize("name", list(CASES))
def test_grouping_paths(gpu_device, name, mixed):
    E, N, T, sizes_of = CASES[name]
    rng = np.random.default_rng(len(name))
    env, agent, turn, reward = draw(E, N, T, sizes_of(rng, E * N * T), 11)
    R = env.size
    # some responses take no part: an id out of range, a reward that is not finite
    env = env.copy()
    env[R // 3] = E
    bad = np.array([0, R // 2])
    reward = reward.copy()
    reward[bad] = [np.inf, np.nan]
    kept = np.ones(R, bool)
    kept[[R // 3, *bad]] = False
    say(f"[grouping] {name} R={R} keys={E * N * T} mixed={mixed}")
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    ids = (dev(env), dev(agent), dev(turn))
    if mixed:
        loc = (np.arange(R) % 5 / np.float32(7)).astype(np.float32)
        out = api.at_grpo_group_advantage_mixed(*ids, dev(reward), dev(loc), 0.3, E, N, T)
        reward = orc.mix_rewards(reward, loc, 0.3)
        assert np.array_equal(host(out["reward"])[kept].view(np.uint32), reward[kept].view(np.uint32))
    else:
        out = api.at_grpo_group_advantage(*ids, dev(reward), E, N, T)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 3          # AT_GRPO_DATA_ID_RANGE | AT_GRPO_DATA_REWARD
    rows = np.nonzero(kept)[0]
    gid, G, offs, perm = orc.group_segments(orc.group_key(env[kept], agent[kept], turn[kept], N, T))
    gmax = min(R, E * N * T)
    assert int(out["n_groups"].item()) == G
    got = host(out["group_id"])
    assert np.array_equal(got[kept], gid) and np.all(got[~kept] == -1)
    seg = host(out["seg_offsets"])
    assert seg.size == gmax + 1 and np.array_equal(seg[:G + 1], offs) and np.all(seg[G + 1:] == 0)
    assert np.array_equal(host(out["perm"])[:rows.size], rows[perm]) and np.all(host(out["perm"])[rows.size:] == 0)
    pick = np.sort(np.random.default_rng(1).choice(G, size=min(G, 300), replace=False))
    members = np.concatenate([rows[perm[offs[g]:offs[g + 1]]] for g in pick])
    sub = np.repeat(np.arange(pick.size), [offs[g + 1] - offs[g] for g in pick])
    adv, mean, std = orc.group_advantage(reward[members], sub, pick.size)
    a = host(out["adv"]).astype(np.float64)
    assert np.all(a[~kept] == 0) and np.all(a[members][std[sub] == 0] == 0)
    assert np.allclose(a[members], adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[pick], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[pick], std, rtol=1e-4, atol=1e-7)
    assert np.all(host(out["group_mean"])[G:] == 0) and np.all(host(out["group_std"])[G:] == 0)
    if mixed:
        best = host(out["best"])
        assert np.all(best[G:] == -1)
        # ascending members: the first of the largest rewards
        want = [rows[perm[offs[g]:offs[g + 1]]][np.argmax(reward[rows[perm[offs[g]:offs[g + 1]]]])] for g in pick]
        assert np.array_equal(best[pick], want)


@pytest.mark.gpu
@pytest.mark.parametrize("over", ["team", "loc", "given"])
@pytest.mark.parametrize("shape", [(4, 2, 2, 4), (16, 2, 4, 8), (20, 3, 5, 10), (512, 2, 1, 4), (257, 2, 1, 8), (4096, 2, 2, 4),
                                   (1, 1, 2, 40000), (262144, 1, 1, 128, 1024), (65280, 1, 1, 200, 256),
                                   (300000, 1, 1, 8), (540000, 1, 1, 8)], ids=str)      # blocks sorted by bin: one round, more
def test_results_in_place(gpu_device, shape, over):
    """Mixed rewards over one of their parts, and advantages over the rewards they come from: bit for bit what separate
    arrays give, on every launch plan."""
    E, N, T, K, *used = shape                    # the first `used` keys, or all of them
    env, agent, turn, team = draw(E, N, T, np.where(np.arange(E * N * T) < (used or [E * N * T])[0], K, 0), 7)
    R, G = env.size, min(env.size, E * N * T)
    say(f"[grouping] in place over {over} {shape}")
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    ids = (dev(env), dev(agent), dev(turn))
    loc = (np.arange(R) % 5 / np.float32(7)).astype(np.float32)
    lib = api.load_library()
    if over == "given":
        ref = api.at_grpo_group_advantage(*ids, dev(team), E, N, T)
    else:
        ref = api.at_grpo_group_advantage_mixed(*ids, dev(team), dev(loc), 0.3, E, N, T)
    ws = ref["workspace"]
    n_groups = int(ref["n_groups"].item())
    got = api.group_advantage_outputs(R, G, gpu_device)
    best = torch.full((G,), -1, dtype=torch.int32, device=gpu_device)
    r_team, r_loc = dev(team), dev(loc)
    tail = lambda adv: [got["group_id"].data_ptr(), got["n_groups"].data_ptr(), got["seg_offsets"].data_ptr(),
                        got["perm"].data_ptr(), adv.data_ptr(), got["group_mean"].data_ptr(), got["group_std"].data_ptr()]
    head = [R, E, N, T, *(t.data_ptr() for t in ids)]
    scratch = [ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream]
    if over == "given":
        assert lib.at_grpo_group_advantage(*head, r_team.data_ptr(), 1e-6, 0, 0, *tail(r_team), *scratch) == 0
        got["adv"] = r_team
    else:
        reward = r_team if over == "team" else r_loc
        assert lib.at_grpo_group_advantage_mixed(*head, r_team.data_ptr(), r_loc.data_ptr(), 0.3, 1e-6, 0, 0, reward.data_ptr(),
                                                 *tail(got["adv"]), best.data_ptr(), *scratch) == 0
        got["reward"], got["best"] = reward, best
    torch.cuda.synchronize()
    for k in set(got) & set(ref) - {"workspace", "data_error"}:
        n = n_groups if k in ("group_mean", "group_std", "best") else None
        assert np.array_equal(host(got[k])[:n].view(np.uint32), host(ref[k])[:n].view(np.uint32)), k


@pytest.mark.gpu
@pytest.mark.parametrize("group_by", ["trajectory", "parallel"])
def test_pools_under_the_other_keys(gpu_device, group_by):
    E, N, T, C = 20000, 2, 3, 4
    rng = np.random.default_rng(5)
    R = 90001 if group_by == "trajectory" else 120003
    env, agent, turn, sample = (rng.integers(0, m, R).astype(np.int32) for m in (E, N, T, C))
    reward = (rng.integers(0, 9, size=R) / np.float32(8)).astype(np.float32)
    say(f"[grouping] pool by {group_by}")
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    out = api.at_grpo_group_advantage_keyed(group_by, dev(env), dev(agent), dev(turn), dev(reward), E, N, T, sample_id=dev(sample),
                                            n_sample=C)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    gid, G, offs, perm = orc.group_segments(orc.group_key_by(env, agent, turn, sample, N, T, C, group_by))
    adv, mean, std = orc.group_advantage(reward, gid, G)
    assert int(out["n_groups"].item()) == G
    assert np.array_equal(host(out["group_id"]), gid) and np.array_equal(host(out["perm"]), perm)
    assert np.array_equal(host(out["seg_offsets"])[:G + 1], offs) and np.all(host(out["seg_offsets"])[G + 1:] == 0)
    got = host(out["adv"]).astype(np.float64)
    assert np.all(got[std[gid] == 0] == 0) and np.allclose(got, adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[:G], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[:G], std, rtol=1e-4, atol=1e-7)


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["spread", "one part"])
@pytest.mark.parametrize("shape", [(8192, 1, 4, 3), (30000, 1, 2, 2), (5000, 1, 2, 3), (300000, 1, 2, 4)], ids=str)
def test_scratch_and_tails_without_fill(gpu_device, shape, where):
    """A caller with the least workspace (no room for the pool path) and one that does not ask for filled tails: group for group
    the same bits (sums are taken in ascending order everywhere), nothing written behind the last group."""
    E, N, T, K = shape
    sizes = np.full(E * N * T, K)
    if where == "one part":
        sizes = np.where(np.arange(E * N * T) < E * N * T // 8, 8 * K, 0)
    env, agent, turn, reward = draw(E, N, T, sizes, 3)
    R, keys = env.size, E * N * T
    say(f"[grouping] scratch and tails {shape} {where}")
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    ids, rew = (dev(env), dev(agent), dev(turn)), dev(reward)
    ref = api.at_grpo_group_advantage(*ids, rew, E, N, T)
    torch.cuda.synchronize()
    G = int(ref["n_groups"].item())
    up = lambda n: (4 * n + 255) // 256 * 256
    least = up(64) + 2 * up(keys) + 3 * up(R) + 2 * up(-(-keys // 2048))
    full = api.load_library().at_grpo_group_advantage_keyed_workspace_bytes(0, R, E, N, T, 1)
    assert full >= least
    for nbytes in (least, full):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device=gpu_device)
        got = api.group_advantage_outputs(R, keys, gpu_device)
        for k in ("seg_offsets", "perm", "group_mean", "group_std"):
            got[k].fill_(77)
        st = api.load_library().at_grpo_group_advantage(
            R, E, N, T, *(t.data_ptr() for t in ids), rew.data_ptr(), 1e-6, 0, 0, got["group_id"].data_ptr(), got["n_groups"].data_ptr(),
            got["seg_offsets"].data_ptr(), got["perm"].data_ptr(), got["adv"].data_ptr(), got["group_mean"].data_ptr(),
            got["group_std"].data_ptr(), ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        assert api.error_word(ws) == 0 and int(got["n_groups"].item()) == G
        for k, n in (("group_id", R), ("seg_offsets", G + 1), ("perm", R), ("adv", R), ("group_mean", G), ("group_std", G)):
            assert np.array_equal(host(got[k])[:n].view(np.uint32), host(ref[k])[:n].view(np.uint32)), k
            assert np.all(host(got[k])[n:] == 77), k


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(8192, 1, 4, 3, 8192 * 4), (262144, 1, 1, 128, 1024), (65280, 1, 1, 200, 256), (40, 2, 4, 8, 320)], ids=str)
def test_replays_on_other_inputs(gpu_device, shape):
    """A captured call replayed on other responses in the same arrays: spread over the bins, in one part of the extents, and back
    (whatever a pass leaves in the scratch must not reach the next)."""
    E, N, T, K, used = shape
    keys = np.arange(E * N * T)
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    batches = []
    for seed, sizes in enumerate([np.where(keys < used, K, 0), np.where(keys >= keys.size - used, K, 0), np.where(keys < used, K, 0)]):
        batches.append([dev(a) for a in draw(E, N, T, sizes, seed)])
    bufs = [torch.empty_like(a) for a in batches[0]]
    call = lambda: api.at_grpo_group_advantage(*bufs, E, N, T)
    for b, a in zip(bufs, batches[0]):
        b.copy_(a)
    call()
    torch.cuda.synchronize()
    say(f"[grouping] capture {shape}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for batch in batches:
        for b, a in zip(bufs, batch):
            b.copy_(a)
        ref = {k: v.clone() for k, v in call().items() if k != "workspace"}
        torch.cuda.synchronize()
        for k in ref:
            out[k].fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        for k in ref:
            assert torch.equal(out[k], ref[k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("n,order,crowded", [(2342913, "shuffled", 0), (4194304, "shuffled", 0), (4194305, "half in rollout order", 0),
                                             (2400001, "half in rollout order", 2048), (4300001, "shuffled", 2048)], ids=str)
def test_blocks_sorted_by_bin(gpu_device, n, order, crowded):
    """The largest pools: blocks of 16384 responses that lie in many bins are sorted by bin first.  One round of workgroups and more,
    a ragged last block, blocks in rollout order among them, every tenth response without a key, and keys so crowded that their bins
    exceed the LDS lists (blocks with members of those are not sorted)."""
    rng = np.random.default_rng(n + crowded)
    E, K = n // 8, 8
    key = np.arange(n) // K % E
    crowd = np.arange(n) >= n - 40000 if crowded else np.zeros(n, bool)
    key[crowd] = rng.integers(0, max(crowded, 1), int(crowd.sum()))
    shuffled = n - 60000 if crowded else n
    lo = shuffled // 2 if order.startswith("half") else 0
    key[lo:shuffled] = key[lo:shuffled][rng.permutation(shuffled - lo)]
    env = key.astype(np.int32)
    kept = rng.random(n) >= 0.1
    env[~kept] = np.where(np.arange(n)[~kept] % 2 == 0, E, -1)
    reward = (rng.integers(0, 9, size=n) / np.float32(8)).astype(np.float32)
    zero = np.zeros(n, np.int32)
    say(f"[grouping] sorted blocks n={n} {order} crowded={crowded}")
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    out = api.at_grpo_group_advantage(dev(env), dev(zero), dev(zero), dev(reward), E, 1, 1)
    torch.cuda.synchronize()
    rows = np.nonzero(kept)[0]
    gid, G, offs, perm = orc.group_segments(orc.group_key(env[kept], zero[kept], zero[kept], 1, 1))
    assert int(out["n_groups"].item()) == G
    got = host(out["group_id"])
    assert np.array_equal(got[kept], gid) and np.all(got[~kept] == -1)
    seg = host(out["seg_offsets"])
    assert np.array_equal(seg[:G + 1], offs) and np.all(seg[G + 1:] == 0)
    assert np.array_equal(host(out["perm"])[:rows.size], rows[perm]) and np.all(host(out["perm"])[rows.size:] == 0)
    # means of all groups in 64 bits, the oracle's results on 300 of them; fp32 sums of a group's members: within 1e-4, as above
    x = reward[kept].astype(np.float64)
    count = np.bincount(gid, minlength=G)
    mean = np.bincount(gid, x, G) / count
    pick = np.sort(rng.choice(G, size=300, replace=False))
    members = np.concatenate([perm[offs[g]:offs[g + 1]] for g in pick])
    sub = np.repeat(np.arange(pick.size), count[pick])
    adv, m, s = orc.group_advantage(reward[kept][members], sub, pick.size)
    a = host(out["adv"]).astype(np.float64)
    assert np.all(a[~kept] == 0)
    assert np.allclose(a[kept][members], adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[:G], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[pick], s, rtol=1e-4, atol=1e-7)
    # all responses: what their groups' own statistics give
    gm, gs = host(out["group_mean"]).astype(np.float64)[gid], host(out["group_std"]).astype(np.float64)[gid]
    want = np.where(gs > 0, (x - gm) / np.where(gs > 0, gs, 1), 0)
    assert np.allclose(a[kept], want, rtol=1e-4, atol=1e-5)


@pytest.mark.gpu
@pytest.mark.parametrize("group_by,E,R", [("trajectory", 600000, 2400011), ("parallel", 50000, 2400007), ("trajectory", 600000, 4300003)])
def test_sorted_blocks_under_the_other_keys(gpu_device, group_by, E, R):
    N, T, C = 2, 3, 4
    rng = np.random.default_rng(R)
    env, agent, turn, sample = (rng.integers(0, m, R).astype(np.int32) for m in (E, N, T, C))
    reward = (rng.integers(0, 9, size=R) / np.float32(8)).astype(np.float32)
    say(f"[grouping] sorted blocks by {group_by} R={R}")
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    out = api.at_grpo_group_advantage_keyed(group_by, dev(env), dev(agent), dev(turn), dev(reward), E, N, T, sample_id=dev(sample),
                                            n_sample=C)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 0
    gid, G, offs, perm = orc.group_segments(orc.group_key_by(env, agent, turn, sample, N, T, C, group_by))
    assert int(out["n_groups"].item()) == G
    assert np.array_equal(host(out["group_id"]), gid) and np.array_equal(host(out["perm"]), perm)
    assert np.array_equal(host(out["seg_offsets"])[:G + 1], offs) and np.all(host(out["seg_offsets"])[G + 1:] == 0)
    pick = np.sort(rng.choice(G, size=300, replace=False))
    members = np.concatenate([perm[offs[g]:offs[g + 1]] for g in pick])
    sub = np.repeat(np.arange(pick.size), [offs[g + 1] - offs[g] for g in pick])
    adv, mean, std = orc.group_advantage(reward[members], sub, pick.size)
    got = host(out["adv"]).astype(np.float64)[members]
    assert np.all(got[std[sub] == 0] == 0) and np.allclose(got, adv, rtol=1e-4, atol=1e-6)
    assert np.allclose(host(out["group_mean"])[pick], mean, rtol=1e-4, atol=1e-7)
    assert np.allclose(host(out["group_std"])[pick], std, rtol=1e-4, atol=1e-7)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2400001, 4300001])
def test_replays_from_shuffled_to_rollout_order(gpu_device, n):
    """A captured call whose blocks are sorted in one replay, are not in the next, and hold members of large bins in a third: what the
    places of a block mean changes, and nothing of one pass reaches the next."""
    E, rng = n // 8, np.random.default_rng(n)
    order = np.arange(n) // 8 % E
    shuffled = order[rng.permutation(n)]
    crowded = shuffled.copy()
    crowded[n // 3:n // 3 + 40000] = rng.integers(0, 2048, 40000)
    half = np.concatenate([order[:n // 2], shuffled[n // 2:]])
    dev = lambda a: torch.from_numpy(a).to(gpu_device)
    zero = torch.zeros(n, dtype=torch.int32, device=gpu_device)
    batches = [(dev(k.astype(np.int32)), dev((rng.integers(0, 9, size=n) / np.float32(8)).astype(np.float32)))
               for k in (shuffled, order, crowded, shuffled, half, order)]
    env, reward = torch.empty_like(batches[0][0]), torch.empty_like(batches[0][1])
    call = lambda: api.at_grpo_group_advantage(env, zero, zero, reward, E, 1, 1)
    env.copy_(batches[0][0])
    reward.copy_(batches[0][1])
    call()
    torch.cuda.synchronize()
    say(f"[grouping] capture of sorted blocks n={n}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call()
    for e, r in batches:
        env.copy_(e)
        reward.copy_(r)
        ref = {k: v.clone() for k, v in call().items() if k != "workspace"}
        torch.cuda.synchronize()
        key = e.long()
        assert int(ref["n_groups"].item()) == int(torch.unique(key).numel())
        assert torch.equal(ref["perm"].long(), torch.sort(key, stable=True).indices)
        for k in ref:
            out[k].fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        for k in ref:
            assert torch.equal(out[k], ref[k]), k


@pytest.mark.gpu
def test_pools_of_two_host_threads(gpu_device):
    """Two host threads, each with pools of its own size on its own stream: both kernels that need more LDS than a launch may ask
    for by itself, with 1536 bins in one thread and 2048 in the other.  Every call has its own results."""
    dev = gpu_device
    pools = []
    for n in (4300000, 8380000):
        gen = torch.Generator(device=dev).manual_seed(n)
        env = (torch.arange(n, device=dev, dtype=torch.int32) // 8)[torch.randperm(n, generator=gen, device=dev)].contiguous()
        zero = torch.zeros(n, dtype=torch.int32, device=dev)
        pools.append((env, zero, zero, torch.rand(n, generator=gen, device=dev), (n + 7) // 8, 1, 1))
    ref = [{k: v.clone() for k, v in api.at_grpo_group_advantage(*p).items() if k != "workspace"} for p in pools]
    torch.cuda.synchronize()
    say("[grouping] pools of two host threads")
    start, failed = threading.Barrier(2), []

    def work(i):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                start.wait()
                for _ in range(30):
                    out = api.at_grpo_group_advantage(*pools[i])
                    stream.synchronize()
                    assert api.error_word(out["workspace"]) == 0
                    failed.extend((i, k) for k in ref[i] if not torch.equal(out[k], ref[i][k]))
        except Exception as e:      # an assertion in another thread does not fail the test by itself
            failed.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["cpu ids", "cpu reward", "long ids", "double reward", "strided", "no local reward", "extents", "no ids"])
def test_refused_arguments(gpu_device, what):
    """Arguments that a grouping call refuses, plain and mixed, and a call behind the refusal."""
    ids = lambda: [torch.tensor([0, 0, 1, 1], dtype=torch.int32, device=gpu_device) for _ in range(3)]
    a, r, extents = ids(), torch.tensor([1.0, 0.0, 1.0, 1.0], device=gpu_device), (2, 2, 2)
    loc = torch.zeros_like(r)
    good = [t.clone() for t in a]
    if what == "cpu ids":
        a[1] = a[1].cpu()
    elif what == "cpu reward":
        r = r.cpu()
    elif what == "long ids":
        a[2] = a[2].long()
    elif what == "double reward":
        r = r.double()
    elif what == "strided":
        a[0] = a[0].repeat_interleave(2)[::2]
    elif what == "no local reward":
        loc = None
    elif what == "extents":
        extents = (0, 2, 2)
    else:
        a[0] = None
    with pytest.raises(api.AtGrpoError):
        api.at_grpo_group_advantage_mixed(*a, r, loc, 1.0, *extents)
    if what != "no local reward":
        with pytest.raises(api.AtGrpoError):
            api.at_grpo_group_advantage(*a, r, *extents)
    out = api.at_grpo_group_advantage(*good, torch.tensor([1.0, 0.0, 1.0, 1.0], device=gpu_device), 2, 2, 2, want_stats=False)
    assert list(out) == ["group_id", "n_groups", "seg_offsets", "perm", "adv", "group_mean", "group_std", "workspace"]
    assert out["group_mean"] is None and out["group_std"] is None
    assert out["group_id"].tolist() == [0, 0, 1, 1] and out["perm"].tolist() == [0, 1, 2, 3] and int(out["n_groups"]) == 2
    assert out["adv"].dtype == torch.float32 and out["adv"].device == gpu_device
