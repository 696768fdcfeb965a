"""The one-pass scoring of up to 32 query rows per head takes 512 or 1024 keys at a time, by how many a call has: a layer's scores
are the same bit for bit either way, and right (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2406_02069_amd import binding, synth
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _same(Q, K, k, lens=None):
    B, Hkv, N = K.shape[:3]
    L = 256 // (B * Hkv * -(-N // 512)) + 1
    lens_dev = None if lens is None else torch.tensor(lens, dtype=torch.int32, device=DEV)
    one = binding.compress_layers([Q], [K], [K], [k], synth.POOL_NONE, 1, seq_lens=lens_dev, want_scores=True)[0]
    many = binding.compress_layers([Q] * L, [K] * L, [K] * L, [k] * L, synth.POOL_NONE, 1, seq_lens=lens_dev, want_scores=True)
    torch.cuda.synchronize()
    print("items", tuple(Q.shape), tuple(K.shape), "layers", L, flush=True)
    alpha = Q.shape[2]
    for out in (many[0], many[-1]):
        for b, n in enumerate(lens or [N] * B):
            if n > k:
                assert torch.equal(out[4][b, :, :n - alpha], one[4][b, :, :n - alpha])
                assert torch.equal(out[2][b], one[2][b])
    compare_layer(Q, K, K, k, alpha, synth.POOL_NONE, 1, None if lens is None else np.array(lens, dtype=np.int32), one)


def _inputs(B, Hq, Hkv, d, N, alpha, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    Q = torch.randn(B, Hq, alpha, d, generator=g, device=DEV).to(torch.bfloat16)
    return Q, torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)


# 8, 16, 17 and 32 rows; the first prompts of two words, of two items, of an odd number of words, the last split and the first whole
@pytest.mark.parametrize("G,alpha", [(1, 8), (2, 8), (1, 17), (4, 8)])
@pytest.mark.parametrize("d", [64, 128])
def test_items_of_either_size_give_the_same_scores(G, alpha, d):
    for N in (60, 512, 513, 1024, 1025, 1537, 4100, 8192, 8193):
        Q, K = _inputs(1, 2 * G, 2, d, N, alpha, N % 89)
        _same(Q, K, alpha + 20)


@pytest.mark.parametrize("G,alpha", [(1, 8), (4, 8)])
def test_items_of_a_ragged_batch(G, alpha):
    lens = [5000, 0, 513, 4609, 30, 1024]
    Q, K = _inputs(len(lens), 2 * G, 2, 128, 5000, alpha, 7)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")   # never read
    _same(Q, K, alpha + 20, lens)


@pytest.mark.parametrize("G,alpha", [(1, 8), (4, 8)])
def test_items_with_references_that_do_not_fit(G, alpha):
    # keys far above the sampled ones, in the first and in the second part of an item: such waves take references of their own
    for at in (100, 700, 3000):
        Q, K = _inputs(1, G, 1, 64, 4100, alpha, at)
        K[0, 0, at] = (Q[0, 0, 3].float() * 12).to(torch.bfloat16)
        _same(Q, K, alpha + 20)


# (16 sequences: a layer of them has more items than there are workgroups, a layer of one has not)
@pytest.mark.parametrize("G,alpha", [(1, 8), (2, 8), (4, 8)])
@pytest.mark.parametrize("N", [513, 2300, 8192])
def test_scores_do_not_depend_on_the_number_of_sequences(G, alpha, N):
    B, k = 16, alpha + 20
    Q, K = _inputs(B, 8 * G, 8, 128, N, alpha, N % 89)
    batch = binding.compress_layers([Q], [K], [K], [k], synth.POOL_NONE, 1, want_scores=True)[0]
    for b in (0, B - 1):
        one = binding.compress_layers([Q[b:b + 1]], [K[b:b + 1]], [K[b:b + 1]], [k], synth.POOL_NONE, 1, want_scores=True)[0]
        torch.cuda.synchronize()
        assert torch.equal(batch[4][b, :, :N - alpha], one[4][0, :, :N - alpha])
        assert torch.equal(batch[2][b], one[2][0])
    print("sequences", tuple(Q.shape), tuple(K.shape), flush=True)
