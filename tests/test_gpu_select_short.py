"""Selection at the edges of its dispatch: prefix lengths around the number of positions a thread holds, budgets from one
token to nearly everything, scores that span many binades (an attention sink, cuts far below it, exact zeros) and ties
that do not fit the candidate list."""
import numpy as np
import pytest
import torch

from paper_2406_02069_amd import binding, synth
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(N, alpha, seed, scale=1.0, B=1, Hq=2, Hkv=2, d=64):
    g = torch.Generator(device=DEV).manual_seed(seed)
    Q = (torch.randn(B, Hq, alpha, d, generator=g, device=DEV) * scale).to(torch.bfloat16)
    K = torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    return Q, K, V


def _check(Q, K, V, k_l, pool, pw, lens=None):
    alpha = Q.shape[2]
    print("select", tuple(K.shape), alpha, k_l, pool, pw, lens, flush=True)
    ld = None if lens is None else torch.from_numpy(lens).to(DEV)
    out = binding.compress_layer(Q, K, V, k_l, pool, pw, seq_lens=ld, want_scores=True)
    torch.cuda.synchronize()
    return compare_layer(Q, K, V, k_l, alpha, pool, pw, lens, out)


@pytest.mark.parametrize("npre", [255, 256, 257, 4095, 4096, 4097, 8191, 8192, 8193, 16384, 16385, 32767, 32768, 32769])
def test_prefix_lengths_around_the_dispatch(npre):
    alpha = 8
    Q, K, V = _inputs(npre + alpha, alpha, seed=npre)
    for kk, pool, pw in ((1, synth.POOL_MAX, 7), (100, synth.POOL_AVG, 5), (min(npre - 1, 1500), synth.POOL_MAX, 3),
                         (npre - 1, synth.POOL_NONE, 1), (50, synth.POOL_MAX, 13), (50, synth.POOL_AVG, 63)):
        if 0 < kk < npre:
            _check(Q, K, V, alpha + kk, pool, pw)


@pytest.mark.parametrize("N", [3000, 12000, 30000])
@pytest.mark.parametrize("kk", [3, 700, 2500])
def test_scores_over_many_binades(N, kk):
    alpha = 4
    Q, K, V = _inputs(N, alpha, seed=N + kk, scale=6.0)      # cuts tens of binades below the largest score
    K[:, :, 0] *= 3
    _check(Q, K, V, alpha + kk, synth.POOL_MAX, 5)
    K[:, :, N // 8:] = -10 * Q[:, :, :1]                     # most scores are exact zeros in fp32
    out = binding.compress_layer(Q, K, V, alpha + kk, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    from oracle import pkv_oracle
    for g in range(2):                                       # selection exact on the device's own scores
        own = pkv_oracle.topk(out[4][0, g, :N - alpha].cpu().numpy().astype(np.float64), kk)
        np.testing.assert_array_equal(out[2][0, g, :kk].cpu().numpy(), own)


@pytest.mark.parametrize("N", [2000, 9000, 20000])
def test_equal_scores_beyond_the_list(N):
    alpha = 4
    Q, K, V = _inputs(N, alpha, seed=N)
    K[:] = K[:, :, :1]
    out = binding.compress_layer(Q, K, V, alpha + 600, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    assert out[2][0, 0, :600].tolist() == list(range(600))
    K[0, 0, N // 2] = (Q[0, 0].float().sum(dim=0) * 2).to(torch.bfloat16)      # one key above a plateau of equals
    out = binding.compress_layer(Q, K, V, alpha + 600, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    assert out[2][0, 0, :600].tolist() == list(range(599)) + [N // 2]


def test_many_units_of_ragged_lengths():
    alpha, N = 8, 20000
    Q, K, V = _inputs(N, alpha, seed=5, B=6)
    lens = np.array([20000, 8200, 8201, 4104, 300, 40], dtype=np.int32)
    _check(Q, K, V, 200, synth.POOL_MAX, 7, lens)


@pytest.mark.parametrize("N,kk,scale", [(520, 40, 0.02), (520, 200, 0.004), (4000, 300, 0.02), (1500, 90, 0.1)])
def test_many_units_rank_the_keys_of_one_bin(N, kk, scale):
    # scores so close together that the cut falls into a bin of up to some hundred keys, which are ranked against each other:
    # the waves read the bin while its keys are being counted
    alpha, B, Hkv = 8, 128, 16
    Q, K, V = _inputs(N, alpha, seed=N + kk, scale=scale, B=B, Hq=Hkv, Hkv=Hkv)
    print("select bins", N, kk, scale, flush=True)
    out = binding.compress_layer(Q, K, V, alpha + kk, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    order = torch.sort(out[4][:, :, :N - alpha], dim=2, descending=True, stable=True)[1][:, :, :kk]
    assert torch.equal(out[2][:, :, :kk].long(), order.sort(dim=2)[0])


@pytest.mark.parametrize("N", [520, 4000, 7900, 16100, 32500])
@pytest.mark.parametrize("share", [0.02, 0.3, 0.55, 0.97])
@pytest.mark.parametrize("kind", ["spread", "sharp", "flat", "zeros behind", "zeros between", "two values", "equal"])
def test_budgets_of_every_share_of_the_prefix(N, share, kind):
    # lists that do not fit, positive keys that are fewer than the budget or sit in few groups, cuts in the last bin,
    # bins of equal keys
    alpha, B, Hkv = 4, 2, 8
    Q, K, V = _inputs(N, alpha, seed=N, scale={"sharp": 8.0, "flat": 0.002}.get(kind, 1.0), B=B, Hq=Hkv, Hkv=Hkv)
    far = -30 * Q[:, :, :1]                                   # exact zeros
    if kind == "zeros behind":
        K[:, :, N // 8:] = far
    if kind == "zeros between":
        K[:, :, torch.arange(N, device=DEV) % 3 != 0] = far
    if kind == "two values":
        K[:, :, ::2] = K[:, :, :1]
        K[:, :, 1::2] = K[:, :, 1:2]
    if kind == "equal":
        K[:] = K[:, :, :1]
    kk = max(int(share * (N - alpha)), 1)
    print("select share", N, share, kind, flush=True)
    for pool, pw in ((synth.POOL_NONE, 1), (synth.POOL_MAX, 7)):
        out = binding.compress_layer(Q, K, V, alpha + kk, pool, pw, want_scores=True)
        torch.cuda.synchronize()
        order = torch.sort(out[4][:, :, :N - alpha], dim=2, descending=True, stable=True)[1][:, :, :kk]
        assert torch.equal(out[2][:, :, :kk].long(), order.sort(dim=2)[0])
