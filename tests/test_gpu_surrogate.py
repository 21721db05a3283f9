"""Surrogate and diagnostics on both sides of every switch of the lanes that share a response (16, 32, 64, 256), with tensors
that start anywhere, against the CPU oracle: flags and counts exact, sums within fp32's 1e-4 as in tests/test_gpu_parity.py
(here the mean of terms of both signs and size about 1, hence 1e-6 absolute)."""
import numpy as np
import pytest
import torch

from oracle import at_grpo_oracle as orc
from paper_2510_11062_amd import api
from tests.gpu_case import host
from tests.test_gpu_parity import say


SIZES = [(50, 59), (50, 60), (8192, 60), (8193, 60), (50, 159), (50, 160), (32768, 160), (32769, 160), (33000, 511), (50, 512),
         (512, 160), (513, 160)]


@pytest.mark.gpu
@pytest.mark.parametrize("n_resp,mean,shift", [(n, m, 0) for n, m in SIZES] + [(n, m, s) for n, m in SIZES if n < 9000 for s in (1, 3)])
def test_rows_per_team(gpu_device, n_resp, mean, shift):
    rng = np.random.default_rng(n_resp + mean)
    lengths = rng.integers(0, 2 * mean + 1, n_resp)
    lengths[0] += n_resp * mean - lengths.sum() if n_resp * mean > lengths.sum() else 0
    while lengths.sum() > n_resp * mean:                       # the mean decides, so it is met exactly
        at = rng.integers(0, n_resp, n_resp)
        over = lengths.sum() - n_resp * mean
        pick = np.unique(at[lengths[at] > 0])[:over]
        lengths[pick] -= 1
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    n, V, heads = int(cu[-1]), 1000, 3
    assert n == n_resp * mean
    say(f"[surrogate] {n_resp} responses of {mean} rows, shift {shift}")
    logp = (-12 * rng.random(n)).astype(np.float32)
    old = (logp + 0.2 * rng.standard_normal(n)).astype(np.float32)
    token = rng.integers(0, V, n).astype(np.int32)
    token[[7, n // 2, n - 1]] = [V, -1, V + 5]
    mask = (rng.random(n) < 0.9).astype(np.uint8)
    mask[7] = 1
    adv = rng.standard_normal(n_resp).astype(np.float32)
    adv[::5] = 0
    agent = rng.integers(0, 3, n_resp).astype(np.int32)
    head_of_agent = np.array([2, 0, 1], np.int32)

    def dev(a):
        t = torch.from_numpy(np.concatenate([a[:shift], a]) if shift else a).to(gpu_device)
        return t[shift:]

    batch = api.Batch(None, None, dev(token), torch.from_numpy(cu).to(gpu_device), dev(mask), dev(agent), dev(head_of_agent),
                      n_tok=n, V=V, n_heads=heads)
    good = np.where((token >= 0) & (token < V), mask, 0).astype(np.uint8)
    resp, head = orc.token_heads(n, cu, agent, head_of_agent)
    for agg in ("token_mean", "seq_mean_token_mean"):
        out = api.at_grpo_surrogate_from_logp(batch, dev(logp), dev(old), dev(adv), 0.2, 0.28, agg)
        torch.cuda.synchronize()
        assert api.error_word(out["workspace"]) == 4           # AT_GRPO_DATA_TOKEN_RANGE
        ref = orc.policy_loss_from_logp(logp, old, adv, good, head, resp, heads, 0.2, 0.28, agg)
        assert np.array_equal(host(out["clip_mask"]), ref[1]) and np.array_equal(host(out["n_valid"]), ref[2])
        loss = host(out["loss"]).astype(np.float64)
        assert np.all(np.abs(loss - ref[0]) <= 1e-4 * np.abs(ref[0]) + 1e-6), (loss, ref[0])
    counts, kl, ratio = orc.surrogate_diagnostics(logp, old, adv, good, head, resp, heads, 0.2, 0.28)
    out = api.at_grpo_surrogate_diagnostics(batch, dev(logp), dev(old), dev(adv), 0.2, 0.28)
    torch.cuda.synchronize()
    assert api.error_word(out["workspace"]) == 4
    assert np.array_equal(host(out["counts"]).astype(np.int64), counts)
    stats = host(out["stats"]).astype(np.float64)
    assert np.allclose(stats[:, 0], kl, rtol=1e-4, atol=1e-7) and np.allclose(stats[:, 1], ratio, rtol=1e-4, atol=0)


@pytest.mark.gpu
@pytest.mark.parametrize("n_resp,mean", [(512, 160), (513, 160), (100, 70), (300, 20), (100, 20)])
def test_data_errors_per_team(gpu_device, n_resp, mean):
    """Bounds, agents and tokens out of range: the error word, and everything else as if those rows were masked; then clean data on
    the same scratch memory, whose error word nothing clears beforehand.  256, 64, 32 and 16 lanes per response, and the surrogate by
    one workgroup."""
    rng = np.random.default_rng(n_resp * mean)
    cu = np.arange(n_resp + 1, dtype=np.int64) * mean
    n, V, heads = n_resp * mean, 1000, 3
    say(f"[surrogate] data errors, {n_resp} responses of {mean} rows")
    logp = (-12 * rng.random(n)).astype(np.float32)
    old = (logp + 0.2 * rng.standard_normal(n)).astype(np.float32)
    token = rng.integers(0, V, n).astype(np.int32)
    mask = (rng.random(n) < 0.9).astype(np.uint8)
    adv = rng.standard_normal(n_resp).astype(np.float32)
    agent = rng.integers(0, 3, n_resp).astype(np.int32)
    head_of_agent = np.array([2, 0, 1, 7], np.int32)           # a fourth agent without a head
    dev = lambda a: torch.from_numpy(a).to(gpu_device)

    def check(want, token, cu_given, agent_given, out_resp, bad_tok):
        batch = api.Batch(None, None, dev(token), dev(cu_given), dev(mask), dev(agent_given), dev(head_of_agent), n_tok=n, V=V, n_heads=heads)
        good = mask.copy()
        good[bad_tok] = 0
        resp, head = orc.token_heads(n, cu, agent, head_of_agent)
        good[np.isin(resp, out_resp)] = 0
        for agg in ("token_mean", "seq_mean_token_mean"):
            out = api.at_grpo_surrogate_from_logp(batch, dev(logp), dev(old), dev(adv), 0.2, 0.28, agg)
            torch.cuda.synchronize()
            assert api.error_word(out["workspace"]) == want
            ref = orc.policy_loss_from_logp(logp, old, adv, good, head, resp, heads, 0.2, 0.28, agg)
            has_bounds = np.repeat((np.diff(cu_given) >= 0) & (cu_given[:-1] >= 0) & (cu_given[1:] <= n), mean)
            assert np.array_equal(host(out["clip_mask"])[has_bounds], ref[1][has_bounds]) and np.array_equal(host(out["n_valid"]), ref[2])
            loss = host(out["loss"]).astype(np.float64)
            assert np.all(np.abs(loss - ref[0]) <= 1e-4 * np.abs(ref[0]) + 1e-6), (loss, ref[0])
        counts, kl, ratio = orc.surrogate_diagnostics(logp, old, adv, good, head, resp, heads, 0.2, 0.28)
        out = api.at_grpo_surrogate_diagnostics(batch, dev(logp), dev(old), dev(adv), 0.2, 0.28)
        torch.cuda.synchronize()
        assert api.error_word(out["workspace"]) == want
        assert np.array_equal(host(out["counts"]).astype(np.int64), counts)
        stats = host(out["stats"]).astype(np.float64)
        assert np.allclose(stats[:, 0], kl, rtol=1e-4, atol=1e-7) and np.allclose(stats[:, 1], ratio, rtol=1e-4, atol=0)

    k, last = n_resp // 3, n_resp - 1
    bad_cu, bad_agent, bad_token = cu.copy(), agent.copy(), token.copy()
    bad_cu[k], bad_cu[-1] = -1, n + 5                          # responses k - 1 and k lose their common bound, the last one its end
    bad_agent[[2, k + 2, last - 1]] = [-1, 4, 3]
    at = np.nonzero(mask[5 * mean:6 * mean])[0][:3] + 5 * mean
    bad_token[at] = [V, -1, 2 ** 31 - 1]
    check(8, token, bad_cu, agent, [k - 1, k, last], [])
    check(0, token, cu, agent, [], [])
    check(16, token, cu, bad_agent, [2, k + 2, last - 1], [])
    check(28, bad_token, bad_cu, bad_agent, [k - 1, k, last, 2, k + 2, last - 1], at)
    check(0, token, cu, agent, [], [])


@pytest.mark.gpu
@pytest.mark.parametrize("n_resp,mean", [(1, 9), (128, 20), (129, 20), (60, 68), (61, 68), (31, 130), (32, 130), (4, 1024), (3, 1025)])
@pytest.mark.parametrize("shift", [0, 1])
def test_one_workgroup(gpu_device, n_resp, mean, shift):
    """Both sides of where one workgroup computes the whole stage: two rounds of responses, 4096 rows, 1024 rows per response."""
    test_rows_per_team(gpu_device, n_resp, mean, shift)


@pytest.mark.gpu
@pytest.mark.parametrize("n_resp,rows", [(5, 3), (256, 20), (257, 20), (128, 100), (129, 100), (64, 256), (64, 257), (2, 8192), (2, 8193)])
@pytest.mark.parametrize("agg", ["token_mean", "seq_mean_token_mean"])
@pytest.mark.parametrize("bad_bounds", [False, True])
def test_fp32_step_equals_two_calls(gpu_device, n_resp, rows, agg, bad_bounds):
    """Where the loss is computed beside the backward's preparation and where it is not (four rounds of responses, 16384 rows), with
    tokens, an agent and bounds of responses out of range: the same bits as the two calls but for the loss, whose terms are added in
    another order (sums of up to 25700 fp32 terms of size about 1, in chains of 128 at most, 1e-6)."""
    gen = torch.Generator(device=gpu_device).manual_seed(n_resp * rows)
    n, H, V = n_resp * rows, 32, 200
    rand = lambda *s: torch.randn(*s, generator=gen, device=gpu_device)
    hidden, W = rand(n, H), [rand(V, H) * 0.1 for _ in range(2)]
    token = torch.randint(0, V, (n,), generator=gen, device=gpu_device, dtype=torch.int32)
    token[[1, n - 1]] = torch.tensor([V, -3], dtype=torch.int32, device=gpu_device)
    mask = (torch.rand(n, generator=gen, device=gpu_device) < 0.8).to(torch.uint8)
    mask[[1, n - 1]] = 1
    agent = (torch.arange(n_resp, device=gpu_device) % 2).to(torch.int32)
    agent[min(2, n_resp - 1)] = 7
    cu = torch.arange(n_resp + 1, device=gpu_device) * rows
    bounded = torch.ones(n, dtype=torch.bool, device=gpu_device)     # rows whose response has bounds: the others get no flags
    if bad_bounds:
        k = n_resp // 2
        if k > 3:                                                    # responses k - 1 and k lose their common bound
            cu[k] = -1
            bounded[(k - 1) * rows:(k + 1) * rows] = False
        if n_resp > 2:                                               # the last one its end
            cu[-1] = n + 5
            bounded[-rows:] = False
        else:                                                        # the first one its beginning
            cu[0] = -2
            bounded[:rows] = False
    batch = api.Batch(hidden, W, token, cu, mask, agent, torch.tensor([1, 0], dtype=torch.int32, device=gpu_device))
    old, adv = -5.3 + 0.2 * rand(n), rand(n_resp)
    if n_resp > 3:
        adv[3] = 0
    say(f"[surrogate] fp32 step of {n_resp} responses of {rows} rows, {agg}, {'bounds out of range' if bad_bounds else 'good bounds'}")
    one = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, 0.2, 0.2, agg)
    err = api.error_word(one["workspace"])
    one = {k: [x.clone() for x in v] if k == "dW" else v.clone() for k, v in one.items() if k != "workspace"}
    fwd = api.at_grpo_policy_loss_fwd(batch, old, adv, 0.2, 0.2, agg)
    # tokens (of two responses without bounds or agent nobody looks at them), agents, bounds
    assert api.error_word(fwd["workspace"]) == err == (16 | 8 if bad_bounds and n_resp == 2 else 4 | 16 | 8 * bad_bounds)
    bwd = api.at_grpo_policy_loss_bwd(batch, old, adv, fwd["logp"], fwd["lse"], 0.2, 0.2, agg)
    for k in ("logp", "lse", "n_valid"):
        assert torch.equal(one[k], fwd[k]), k
    assert torch.equal(one["clip_mask"][bounded], fwd["clip_mask"][bounded])
    assert torch.equal(one["d_hidden"], bwd["d_hidden"]) and all(torch.equal(a, b) for a, b in zip(one["dW"], bwd["dW"]))
    assert float((one["loss"] - fwd["loss"]).abs().max()) <= 1e-6


@pytest.mark.gpu
def test_loss_of_one_long_response_against_64_bits(gpu_device):
    """A step of one response of 16384 rows, whose loss one wavefront of the merged kernel adds up, 200 times.  What every order of
    addition shares (log-ratio and exp in fp32, the last sums, the division) comes to 4.2e-8 root mean square of the loss.  A chain of
    n additions in each of k lanes adds 2^-24 / sqrt(3) * sqrt(n / 3 / k): 1e-8 for the 64 of 256 sums, 4e-8 for the 256 of 64 sums."""
    n, H, V = 16384, 32, 200
    gen = torch.Generator(device=gpu_device).manual_seed(5)
    rand = lambda *s: torch.randn(*s, generator=gen, device=gpu_device)
    token = torch.randint(0, V, (n,), generator=gen, device=gpu_device, dtype=torch.int32)
    batch = api.Batch(rand(n, H), [rand(V, H) * 0.1], token, torch.tensor([0, n], device=gpu_device))
    logp = api.at_grpo_token_logprob(batch)["logp"]
    say("[surrogate] loss of one response of 16384 rows")
    lo, hi = np.float32(np.log1p(-0.2)), np.float32(np.log1p(0.2))
    errors = []
    for _ in range(200):
        old, adv = logp + 0.1 * rand(n), rand(1)
        out = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, 0.2, 0.2)
        d, A = out["logp"] - old, float(adv)                        # clipped or not is decided on the fp32 difference
        ratio = torch.exp(d.double())
        clipped = torch.where(d < float(lo), 0.8, torch.where(d > float(hi), 1.2, ratio))
        loss = -float(torch.minimum(ratio * A, clipped * A).mean())
        errors.append((float(out["loss"][0]) - loss) / loss)
    rms = float(np.sqrt(np.mean(np.square(errors))))
    assert rms < 5.2e-8, rms
