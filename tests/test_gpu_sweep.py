"""Scoring in two streaming launches for many query rows (G * alpha > 128) at the edges of its work split: rows around the
32-row tiles and the limit, lengths around a pass and a chunk, ragged batches, chunk counts that the workgroups do not
divide, references that do not fit, supplied denominators.  (Own denominators: the queries lie so far apart that the one-pass
kernel, which serves most of these shapes otherwise, does not take them; and lengths that it leaves to this one anyway.)"""
import numpy as np
import pytest
import torch

from oracle import pkv_oracle
from paper_2406_02069_amd import binding, synth
from tests import prefill_stub
from tests.parity import compare_layer, spread_queries
from tests.test_gpu_stream import precision_of_scores

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(B, Hq, Hkv, d, N, alpha, seed, scale=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    Q = (torch.randn(B, Hq, alpha, d, generator=g, device=DEV) * scale).to(torch.bfloat16)
    K = torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    return Q, K, V


def _taken(Q, K, k_l, seq_lens=False):
    """The kernel under test takes the call."""
    return binding.scoring_route(binding.make_desc(Q, K, k_l, synth.POOL_MAX, 7), seq_lens=seq_lens)[0] == "score_sweep"


def _check(Q, K, V, k_l, lens=None, pool=synth.POOL_MAX, pw=7):
    Q = spread_queries(Q)
    assert _taken(Q, K, k_l, lens is not None)
    print("sweep", tuple(Q.shape), tuple(K.shape), k_l, None if lens is None else lens.tolist()[:8], flush=True)
    ld = None if lens is None else torch.from_numpy(lens).to(DEV)
    out = binding.compress_layer(Q, K, V, k_l, pool, pw, seq_lens=ld, want_scores=True)
    torch.cuda.synchronize()
    return compare_layer(Q, K, V, k_l, Q.shape[2], pool, pw, lens, out)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha", [(3, 43), (4, 40), (7, 23), (5, 51), (8, 33), (7, 64), (8, 64)])
def test_rows(d, G, alpha):
    Hkv = 8
    N = 4100 if G * alpha <= 224 else 4096 if G * alpha <= 256 else 8192 if G * alpha == 512 else 8200   # (room for the statistics of the last chunk)
    Q, K, V = _inputs(1, Hkv * G, Hkv, d, N, alpha, seed=G * 100 + alpha + d)
    _check(Q, K, V, alpha + 60)


@pytest.mark.parametrize("N", [3600, 3647, 4031, 4095, 4096, 4097, 4128, 4159, 4160, 4161])
def test_lengths_around_a_pass(N):
    Q, K, V = _inputs(1, 32, 8, 128, N, 33, seed=N)
    _check(Q, K, V, 100)


def test_one_chunk_per_unit():
    Q, K, V = _inputs(8, 24, 8, 64, 512, 64, seed=3)
    _check(Q, K, V, 80)


@pytest.mark.parametrize("G,alpha,N", [(4, 40, 45057), (8, 32, 59000), (8, 64, 46100)])
def test_lengths_that_the_one_pass_kernel_leaves(G, alpha, N):
    Q, K, V = _inputs(1, 8 * G, 8, 128, N, alpha, seed=N)
    assert _taken(Q, K, alpha + 60)
    out = binding.compress_layer(Q, K, V, alpha + 60, synth.POOL_MAX, 7, want_scores=True)
    torch.cuda.synchronize()
    compare_layer(Q, K, V, alpha + 60, alpha, synth.POOL_MAX, 7, None, out)


def test_ragged_batch():
    alpha, N = 40, 4300
    lens = np.array([4300, 0, 39, 40, 41, 100, 552, 553, 4096, 1037], dtype=np.int32)
    Q, K, V = _inputs(len(lens), 8, 2, 128, N, alpha, seed=11)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")
    _check(Q, K, V, 60, lens)


def test_no_sequence_needs_scores():
    alpha, N = 40, 4300
    lens = np.full(4, 50, dtype=np.int32)
    Q, K, V = _inputs(4, 8, 2, 128, N, alpha, seed=12)
    _check(Q, K, V, 60, lens)


def test_many_layers_equal_one_call_per_layer():
    L, alpha, N = 7, 40, 4300
    data = [_inputs(2, 16, 4, 64, N, alpha, seed=500 + l) for l in range(L)]
    data = [(spread_queries(x[0]), x[1], x[2]) for x in data]
    assert _taken(data[0][0], data[0][1], 50, seq_lens=True)
    lens = torch.tensor([4300, 3100], dtype=torch.int32, device=DEV)
    ks = [N + 5, 50, 60, 70, 3500, 90, N]                     # layers and sequences kept whole among them
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], ks, synth.POOL_MAX, 7,
                                   seq_lens=lens, want_scores=True)
    torch.cuda.synchronize()
    for l in range(L):
        one = binding.compress_layer(*data[l], ks[l], synth.POOL_MAX, 7, seq_lens=lens, want_scores=True)
        torch.cuda.synchronize()
        for x, y in zip(outs[l], one):
            assert torch.equal(x, y), l
        if l in (1, 4):
            compare_layer(*data[l], ks[l], alpha, synth.POOL_MAX, 7, lens.cpu().numpy(), outs[l])


@pytest.mark.parametrize("G", [4, 8])
def test_references_that_do_not_fit(G):
    # some rows' logit of key 0 lies hundreds of binades below those of later keys: their chunks are formed again
    alpha, N, Hkv = 40, 8200, 8
    Q, K, V = _inputs(1, G * Hkv, Hkv, 128, N, alpha, seed=G, scale=0.5)
    for g in (0, 5):
        K[0, g, 700] = 40 * Q[0, g * G, 3]
        K[0, g, 0] = -20 * Q[0, g * G, 3]
    _check(Q, K, V, alpha + 30, pool=synth.POOL_NONE, pw=1)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha,N", [(5, 27, 4099), (8, 64, 8200)])
def test_supplied_denominators(d, G, alpha, N):
    Q, K, V = _inputs(2, G * 4, 4, d, N, alpha, seed=G + N)
    lens = np.array([N, N - 700], dtype=np.int32)
    lse = prefill_stub.window_lse(Q, K, lens)
    out = binding.compress_layers_lse([Q], [K], [V], [lse], [alpha + 50], synth.POOL_AVG, 5,
                                      seq_lens=torch.from_numpy(lens).to(DEV), want_scores=True)[0]
    torch.cuda.synchronize()
    ref = pkv_oracle.compress_layer(Q, K, V, alpha + 50, alpha, synth.POOL_AVG, 5, seq_lens=lens,
                                    lse=np.nan_to_num(lse.cpu().numpy(), nan=0.0))
    compare_layer(Q, K, V, alpha + 50, alpha, synth.POOL_AVG, 5, lens, out, ref=ref)


@pytest.mark.parametrize("d,G,alpha,N", [(64, 8, 17, 11300), (128, 8, 17, 11300), (128, 8, 64, 36000)])
def test_sixteen_waves_write_the_scores(d, G, alpha, N):
    # enough passes for sixteen waves, with chunks of which the last pass is partly empty; bit for bit what eight give
    L, Hkv = 12, 8
    data = [_inputs(1, G * Hkv, Hkv, d, N, alpha, seed=70 + l) for l in range(L)]
    data = [(spread_queries(x[0]), x[1], x[2]) for x in data]
    assert _taken(data[0][0], data[0][1], alpha + 20)
    ks = [alpha + 20 + 9 * l for l in range(L)]
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], ks, synth.POOL_AVG, 5,
                                   want_scores=True)
    torch.cuda.synchronize()
    for l in range(L):
        one = binding.compress_layer(*data[l], ks[l], synth.POOL_AVG, 5, want_scores=True)
        torch.cuda.synchronize()
        for x, y in zip(outs[l], one):
            assert torch.equal(x, y), l
    compare_layer(*data[3], ks[3], alpha, synth.POOL_AVG, 5, None, outs[3])


@pytest.mark.parametrize("d,G,alpha", [(64, 1, 5), (128, 4, 8), (128, 1, 32)])
def test_supplied_denominators_few_rows(d, G, alpha):
    # one layer against the oracle; a call with so many keys that another kernel takes it gives the same bits
    Hkv, N, L = 8, 5003, 2 + (4 << 20) // (8 * 5003)
    Q, K, V = _inputs(1, G * Hkv, Hkv, d, N, alpha, seed=G + alpha)
    lse = prefill_stub.window_lse(Q, K, None)
    one = binding.compress_layers_lse([Q], [K], [V], [lse], [alpha + 50], synth.POOL_MAX, 7, want_scores=True)[0]
    many = binding.compress_layers_lse([Q] * L, [K] * L, [V] * L, [lse] * L, [alpha + 50] * L, synth.POOL_MAX, 7,
                                       want_scores=True)
    torch.cuda.synchronize()
    ref = pkv_oracle.compress_layer(Q, K, V, alpha + 50, alpha, synth.POOL_MAX, 7, lse=lse.cpu().numpy())
    compare_layer(Q, K, V, alpha + 50, alpha, synth.POOL_MAX, 7, None, one, ref=ref)
    for l in (0, L // 2, L - 1):
        for x, y in zip(many[l], one):
            assert torch.equal(x, y), l


@pytest.mark.parametrize("Hq,Hkv,d,N,alpha", [(64, 8, 128, 8192, 32), (28, 4, 128, 20001, 40), (16, 4, 64, 16384, 64), (64, 8, 128, 16384, 64)])
def test_precision_of_the_normalisers(Hq, Hkv, d, N, alpha):
    # errors of single rows average out over this many; what is left is common to all rows: the rounding of kappa, 2^-25 of a
    # logit up to 10 binades from the mean, 10 ln 2 / 2^25 = 2.1e-7, and as much again for the normalisers
    assert precision_of_scores(Hq, Hkv, d, N, alpha, None, "score_sweep", spread_queries) < 4.2e-7


@pytest.mark.parametrize("finite", [[1, 700, 701, 2500, 4000], list(range(3000, 3200))])
def test_logits_of_minus_infinity(finite):
    # products that overflow to -inf but for a few keys whose logits are two hundred binades below 0
    G, alpha, Hkv, N, d = 4, 40, 8, 4300, 128
    Q, K, V = _inputs(1, G * Hkv, Hkv, d, N, alpha, seed=7)
    Q = Q.abs()
    low = (-15 - 0.05 * K[:, :, finite].float()).to(torch.bfloat16)
    K[:] = -3e38
    K[:, :, finite] = low
    K[:, :, N - alpha:] = -3e38
    _check(Q, K, V, alpha + 3, pool=synth.POOL_NONE, pw=1)
