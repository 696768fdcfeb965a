"""Selection from prefixes beyond 32768 keys over several workgroups per head: candidates of every stretch first, the kept
set out of them.  Asking for the pooled scores makes one workgroup per head search all keys instead; that path is compared
with the oracle elsewhere, and both have to keep the same positions, whole numbers, bit for bit (needs an MI355X)."""
import numpy as np
import pytest
import torch

from oracle import pkv_oracle
from paper_2406_02069_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ALPHA, HKV, D = 8, 2, 64


def _inputs(N, B, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    Q = torch.randn(B, HKV, ALPHA, D, generator=g, device=DEV).to(torch.bfloat16)
    K = torch.randn(B, HKV, N, D, generator=g, device=DEV).to(torch.bfloat16)
    return Q, K


def _compare(Q, K, ks, pool, pw, lens=None):
    lens = None if lens is None else torch.tensor(lens, dtype=torch.int32, device=DEV)
    args = ([Q] * len(ks), [K] * len(ks), [K] * len(ks), list(ks), pool, pw)
    outs = binding.compress_layers(*args, seq_lens=lens)
    refs = binding.compress_layers(*args, seq_lens=lens, want_scores=True)
    torch.cuda.synchronize()
    for k, out, ref in zip(ks, outs, refs):
        print("stretches", tuple(K.shape), "k", k, "pool", pool, pw, flush=True)
        assert torch.equal(out[3], ref[3])
        for b, n in enumerate(ref[3].tolist()):
            assert torch.equal(out[2][b, :, :n], ref[2][b, :, :n])
            assert torch.equal(out[0][b, :, :n].view(torch.int16), ref[0][b, :, :n].view(torch.int16))
    return refs


# prefixes: the last that one workgroup takes, the first that is cut (3 stretches), 4, 5, 8, 16 and 17 stretches, full and not; kept:
# 1, few, many, the most that the shortest and the longest stretches take and one more, more than any takes
@pytest.mark.parametrize("npre", [32768, 32769, 65536, 65537, 131064, 16384 * 16, 16384 * 16 + 1])
@pytest.mark.parametrize("pool,pw", [(synth.POOL_NONE, 1), (synth.POOL_MAX, 7), (synth.POOL_AVG, 5), (synth.POOL_MAX, 63)])
def test_stretches_keep_what_one_workgroup_keeps(npre, pool, pw):
    Q, K = _inputs(npre + ALPHA, 1, npre % 997)
    count = -(-npre // 16384)
    last = npre - (count - 1) * (-(-npre // count) + 63 & ~63)
    _compare(Q, K, [ALPHA + k for k in (1, 96, 2016, last // 4, last // 4 + 1, 20000)], pool, pw)


def test_stretches_of_a_ragged_batch():
    lens = [100000, 32776, 32777, 45000, 9000, 0, 7, 200]
    Q, K = _inputs(100000, len(lens), 5)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")   # never read
    _compare(Q, K, [ALPHA + 120, ALPHA + 1], synth.POOL_AVG, 5, lens)


@pytest.mark.parametrize("pool,pw", [(synth.POOL_NONE, 1), (synth.POOL_MAX, 5)])
def test_stretches_with_equal_concentrated_and_vanishing_scores(pool, pw):
    N = 50000
    for what in ("all equal", "half equal", "equal at the edge", "one stretch", "vanishing", "few above zero"):
        Q, K = _inputs(N, 1, 11)
        q = Q.float().mean(2, keepdim=True)   # [1, HKV, 1, D], its direction raises a key's score
        if what == "all equal":
            K[:] = K[:, :, :1]
        elif what == "half equal":
            K[:, :, 7::2] = K[:, :, 7:8]
        elif what == "equal at the edge":    # ranks around the last kept one hold equal keys, in several stretches
            K[:, :, ::500] = (3 * q).to(torch.bfloat16)
        elif what == "one stretch":
            K[:, :, 9000:12000] += (2 * q).to(torch.bfloat16)
        elif what == "vanishing":            # exact zeros but for one stretch
            K[:, :, :40000] = (-1000 * q).to(torch.bfloat16)
        else:
            K[:] = (-1000 * q).to(torch.bfloat16)
            K[:, :, 100:150] = (3 * q).to(torch.bfloat16)
            K[:, :, -ALPHA:] = 0
        print(what, flush=True)
        _compare(Q, K, [ALPHA + 60, ALPHA + 600], pool, pw)


def test_stretches_against_the_oracle():
    N, k = 70001, ALPHA + 300
    Q, K = _inputs(N, 1, 3)
    ref = _compare(Q, K, [k], synth.POOL_AVG, 3)[0]
    pooled = ref[4].float().cpu().numpy()
    for h in range(HKV):
        want = pkv_oracle.topk(pooled[0, h, :N - ALPHA], k - ALPHA)
        assert np.array_equal(ref[2][0, h, :k - ALPHA].cpu().numpy(), want)
