"""Scoring with the keys held in registers, at the 65 to 128 query rows that the one-pass kernel takes otherwise (the queries lie
too far apart for that one): rows around the row tiles, lengths around a part of a unit, ragged batches, both exchanges of the
softmax statistics, and lengths that the one-pass kernel leaves to this one anyway."""
import numpy as np
import pytest
import torch

from paper_2406_02069_amd import binding, synth
from tests.parity import compare_layer, spread_queries
from tests.test_gpu_stream import _inputs

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(Q, K, V, k_l, lens=None):
    desc = binding.make_desc(Q, K, k_l, synth.POOL_MAX, 7)
    assert binding.scoring_route(desc, seq_lens=lens is not None)[0] == "score_resident"
    print("resident", tuple(Q.shape), tuple(K.shape), k_l, None if lens is None else lens.tolist()[:8], flush=True)
    ld = None if lens is None else torch.from_numpy(lens).to(DEV)
    out = binding.compress_layer(Q, K, V, k_l, synth.POOL_MAX, 7, seq_lens=ld, want_scores=True)
    torch.cuda.synchronize()
    compare_layer(Q, K, V, k_l, Q.shape[2], synth.POOL_MAX, 7, lens, out)


@pytest.mark.parametrize("flags", [0, binding.FLAG_COUNTER_EXCHANGE])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha,N", [(5, 13, 2047), (3, 32, 2560), (48, 2, 4097), (2, 64, 2049), (4, 32, 9000)])
def test_rows(d, G, alpha, N, flags, monkeypatch):
    monkeypatch.setattr(binding, "DESC_FLAGS", flags)
    Q, K, V = _inputs(1, 3 * G, 3, d, N, alpha, seed=G + N)
    _check(spread_queries(Q), K, V, alpha + 60)


def test_ragged_batch():
    alpha, N = 32, 5000
    lens = np.array([5000, 0, 31, 32, 33, 100, 512, 513, 4097, 1037], dtype=np.int32)
    Q, K, V = _inputs(len(lens), 8, 2, 128, N, alpha, seed=5)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")
    _check(spread_queries(Q), K, V, 50, lens)


@pytest.mark.parametrize("G,alpha,N,ragged", [(4, 32, 60000, False), (3, 32, 131072, False), (4, 32, 140000, True)])
def test_lengths_that_the_one_pass_kernel_leaves(G, alpha, N, ragged):
    Q, K, V = _inputs(1, 2 * G, 2, 128, N, alpha, seed=N)
    _check(Q, K, V, alpha + 60, np.array([N - 3000], dtype=np.int32) if ragged else None)


def test_many_layers_equal_one_call_per_layer():
    L, alpha, N = 9, 32, 4300
    data = [_inputs(2, 16, 4, 64, N, alpha, seed=500 + l) for l in range(L)]
    data = [(spread_queries(x[0]), x[1], x[2]) for x in data]
    lens = torch.tensor([4300, 3100], dtype=torch.int32, device=DEV)
    ks = [40 + 9 * l for l in range(L)]
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], ks, synth.POOL_MAX, 7,
                                   seq_lens=lens, want_scores=True)
    torch.cuda.synchronize()
    for l in range(L):
        one = binding.compress_layer(*data[l], ks[l], synth.POOL_MAX, 7, seq_lens=lens, want_scores=True)
        torch.cuda.synchronize()
        for x, y in zip(outs[l], one):
            assert torch.equal(x, y), l
    compare_layer(*data[3], ks[3], alpha, synth.POOL_MAX, 7, lens.cpu().numpy(), outs[3])
