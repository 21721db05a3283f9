"""Logits launches of few tokens (streams of k-steps on narrow tiles), tiles cut in the last round, and rows without an
advantage on the list of the others, at the sizes where those rules switch, against plain torch in 64 bits.  Log-probabilities
and entropies are fp32 sums of up to 2048 exact products (2e-5 of values up to 12); the gradients carry two roundings to bf16
(2^-8 in the worst case: rows within 1e-2, the whole within 5e-3)."""
import math

import pytest
import torch

from paper_2510_11062_amd import api
from tests.test_gpu_parity import say

EPS = 0.2


def make(dev, lengths, adv, H, V, seed=1):
    gen = torch.Generator(device=dev).manual_seed(seed)
    n = sum(lengths)
    hidden = torch.randn(n, H, generator=gen, device=dev).bfloat16()
    W = (torch.randn(V, H, generator=gen, device=dev) * 0.02).bfloat16()
    y = torch.randint(0, V, (n,), generator=gen, device=dev, dtype=torch.int32)
    y[-1] = V - 1
    cu = torch.tensor([0] + list(lengths), device=dev).cumsum(0)
    z = hidden.double() @ W.double().T
    logp = torch.log_softmax(z, 1)
    drift = 0.05 * torch.randn(n, generator=gen, device=dev, dtype=torch.float64).clamp(-3, 3)
    old = (logp.gather(1, y.long()[:, None])[:, 0] + drift).float()
    adv = torch.tensor(adv, device=dev, dtype=torch.float32)
    return api.Batch(hidden, [W], y, cu), logp, old, adv


def reference(batch, logp, old, adv, lengths):
    """log-probabilities, entropies, and the gradients of Eq. (2) (token mean) of rows with an advantage"""
    p = logp.exp()
    lp = logp.gather(1, batch.token_id.long()[:, None])[:, 0]
    A = adv.double().repeat_interleave(torch.tensor(lengths, device=adv.device))
    d = lp - old.double()
    flat = (A == 0) | ((d > math.log1p(EPS)) & (A > 0)) | ((d < math.log1p(-EPS)) & (A < 0))
    g = torch.where(flat, torch.zeros_like(A), -A * d.clamp(max=50).exp() / len(A))
    dz = -g[:, None] * p
    dz[torch.arange(len(A), device=A.device), batch.token_id.long()] += g
    dz[flat] = 0
    return lp, -(p * logp).sum(1), dz @ batch.W[0].double(), dz.T @ batch.hidden.double()


def close(got, ref, what):
    got = got.double()
    assert bool(torch.isfinite(got).all()), what
    rows = (got - ref).norm(dim=1) / (ref.norm(dim=1) + 1e-2 * ref.norm() / math.sqrt(ref.shape[0]))
    assert float(rows.max()) <= 1e-2, (what, float(rows.max()))
    assert float((got - ref).norm() / ref.norm()) <= 5e-3, what


def check(batch, logp, old, adv, lengths, two_calls=True):
    lp, ent, dh, dw = reference(batch, logp, old, adv, lengths)
    out = api.at_grpo_token_entropy(batch)
    step = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, EPS, EPS)
    torch.cuda.synchronize()
    assert api.error_word(step["workspace"]) == 0
    for got in (out["logp"], step["logp"]):
        assert float((got.double() - lp).abs().max()) <= 2e-5
    assert float((out["entropy"].double() - ent).abs().max()) <= 2e-5
    close(step["d_hidden"], dh, "d_hidden, one pass")
    close(step["dW"][0], dw, "dW, one pass")
    if not two_calls:
        return
    back = api.at_grpo_policy_loss_bwd(batch, old, adv, out["logp"], out["lse"], EPS, EPS)
    close(back["d_hidden"], dh, "d_hidden, two calls")
    close(back["dW"][0], dw, "dW, two calls")


@pytest.mark.gpu
@pytest.mark.parametrize("n,H,V", [
    (1, 64, 128),           # one row, one k-step, one narrow tile
    (64, 64, 129),          # the widest of the narrowest; a tile of one vocabulary row
    (65, 192, 300),         # three k-steps in a ring of four; an odd number of narrow tiles
    (128, 2048, 1000),
    (129, 128, 70000),      # several tiles per workgroup, two k-steps each: requests run tiles ahead
    (192, 320, 33000),      # the last stream; 258 tiles on 256 workgroups
    (193, 320, 33000),      # 129 whole tiles: not cut
    (250, 64, 20000),       # 79 tiles: halves, the second with 122 tokens
    (256, 128, 16385),      # 65 tiles, one of a single vocabulary row: halves
    (300, 192, 8200),       # 66 tiles of two token tiles, the second one's second half empty: halves
    (450, 64, 5000),        # 40 tiles: quarters, the last one empty
    (700, 64, 30000),       # 354 tiles: a whole round and 98 in halves
])
def test_few_tokens(gpu_device, n, H, V):
    say(f"[few] n={n} H={H} V={V}")
    lengths = [n - n // 2] + ([n // 2] if n > 1 else [])
    check(*make(gpu_device, lengths, [1.0, -0.5][:len(lengths)], H, V), lengths)


@pytest.mark.gpu
@pytest.mark.parametrize("with_adv,without", [(1, 1), (100, 2048), (100, 2049), (700, 300), (64, 63), (64, 512), (64, 513), (700, 700),
                                              (700, 701), (1100, 1024), (1100, 1025)])
def test_rows_without_advantage(gpu_device, with_adv, without):
    """Up to 512 of them stand on the list of the others, up to 1024 where as many have an advantage; wherever they stand they get
    their log-probability and no gradient, also where their ratio overflows."""
    say(f"[few] {with_adv} rows with and {without} without an advantage")
    lengths = [without - without // 2, with_adv, without // 2]
    batch, logp, old, adv = make(gpu_device, lengths, [0.0, 0.7, 0.0], 128, 2000)
    old[:1] = -300.0
    check(batch, logp, old, adv, lengths, two_calls=False)


@pytest.mark.gpu
@pytest.mark.parametrize("without", [70, 2200])       # on the list of the others, and on one of their own
def test_rows_without_advantage_out_of_range(gpu_device, without):
    """Rows without an advantage whose exponentials leave their range (targets that are all but impossible) or whose hidden state is
    infinite: they get their own log-probability, and the others' results stay the same bits, which they do not where the
    launch is redone by the kernels that round softmax - onehot."""
    say(f"[few] {without} rows without an advantage, some of them out of range")
    a, b = without - 40, 40
    lengths = [a, 70, b]
    batch, logp, old, adv = make(gpu_device, lengths, [0.0, 0.7, 0.0], 128, 2000)
    _, _, dh, dw = reference(batch, logp, old, adv, lengths)
    clean = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, EPS, EPS)
    clean = {k: clean[k][0].clone() if k == "dW" else clean[k].clone() for k in ("logp", "d_hidden", "dW")}
    far, inf = [0, 7, a - 1, a + 70], [a + 75, a + 109]
    batch.hidden[far] *= 512
    z = batch.hidden[far].double() @ batch.W[0].double().T
    batch.token_id[far] = z.argmin(1).int()
    want = z.min(1).values - z.logsumexp(1)
    assert float(want.max()) < -100               # beyond e^-88 for certain
    batch.hidden[inf] = float("inf")
    step = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, EPS, EPS)
    torch.cuda.synchronize()
    close(step["d_hidden"], dh, "d_hidden")
    close(step["dW"][0], dw, "dW")
    assert torch.equal(step["d_hidden"], clean["d_hidden"]) and torch.equal(step["dW"][0], clean["dW"])
    rest = torch.ones(sum(lengths), dtype=torch.bool, device=gpu_device)
    rest[far + inf] = False
    assert torch.equal(step["logp"][rest], clean["logp"][rest])
    # logits of up to a few hundred: fp32 sums of 128 products
    assert float((step["logp"][far].double() - want).abs().max()) <= 4e-6 * float(z.abs().max())


@pytest.mark.gpu
def test_rows_of_both_kinds_out_of_range(gpu_device):
    """The launch is redone for a row with an advantage; the rows without one get their log-probability all the same."""
    say("[few] rows of both kinds out of range")
    lengths = [30, 70, 40]
    batch, logp, old, adv = make(gpu_device, lengths, [0.0, 0.7, 0.0], 128, 2000)
    far = [0, 29, 100, 110, 139]
    batch.hidden[far + [50]] *= 512
    z = batch.hidden.double() @ batch.W[0].double().T
    batch.token_id[far + [50]] = z[far + [50]].argmin(1).int()
    logp = torch.log_softmax(z, 1)
    old[50] = logp[50, batch.token_id[50].long()].float()
    lp, _, dh, dw = reference(batch, logp, old, adv, lengths)
    step = api.at_grpo_policy_loss_fwd_bwd(batch, old, adv, EPS, EPS)
    torch.cuda.synchronize()
    assert float((step["logp"].double() - lp).abs().max()) <= 4e-6 * float(z.abs().max())
    close(step["d_hidden"], dh, "d_hidden")
    close(step["dW"][0], dw, "dW")


@pytest.mark.gpu
@pytest.mark.parametrize("n,H,V", [(1, 2048, 65537), (65, 2048, 65537), (192, 2048, 65537), (130, 1024, 131200), (192, 2048, 65536)])
def test_weights_past_the_caches(gpu_device, n, H, V):
    """The first sizes of weights that the caches do not hold (and the last that they do): ragged vocabulary tiles and k-steps."""
    say(f"[few] weights past the caches n={n} H={H} V={V}")
    lengths = [n - n // 2] + ([n // 2] if n > 1 else [])
    check(*make(gpu_device, lengths, [1.0, -0.5][:len(lengths)], H, V), lengths)


@pytest.mark.gpu
@pytest.mark.parametrize("n,H,V", [
    (224, 64, 20000),       # one token tile of 224, 79 vocabulary tiles: halves of 112
    (225, 64, 1000),        # one of 256
    (257, 192, 8200),       # two of 160, 66 tiles in all: halves of 80
    (320, 64, 5000),        # 40 tiles: quarters of 40
    (321, 128, 3000),       # two of 192
    (384, 64, 20000),       # 158 tiles: not cut
    (385, 64, 33000),       # 258 tiles of 224: a whole round and two in quarters of 56
    (448, 64, 700),
    (449, 64, 700),         # two of 256
    (513, 128, 2100),       # three of 192
    (1120, 64, 1300),       # five of 224, all full
    (1568, 64, 520),        # the last size that is not in tiles of 256
    (1569, 64, 520),
])
def test_equal_token_tiles(gpu_device, n, H, V):
    """Also on a workspace full of NaN: rows behind the last tile are read by the contractions over tokens."""
    say(f"[few] equal token tiles n={n} H={H} V={V}")
    lengths = [n - n // 2, n // 2]
    case = make(gpu_device, lengths, [1.0, -0.5], H, V)
    check(*case, lengths)
    api.at_grpo_token_entropy(case[0])["workspace"].fill_(255)
    check(*case, lengths)
