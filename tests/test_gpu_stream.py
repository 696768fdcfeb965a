"""One-pass scoring for few query rows (G * alpha <= 64) at the edges of its work split: rows around the register groups,
lengths around the keys of an item, ragged batches whose sequences contribute unequal numbers of items, many items per
workgroup, more sequences than one launch's table holds, references that do not fit or overflow, precision, the end of the
workspace."""
import numpy as np
import pytest
import torch

from paper_2406_02069_amd import binding, synth
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(B, Hq, Hkv, d, N, alpha, seed, scale=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    Q = (torch.randn(B, Hq, alpha, d, generator=g, device=DEV) * scale).to(torch.bfloat16)
    K = torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    V = torch.randn(B, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    return Q, K, V


def _check(Q, K, V, k_l, lens=None, pool=synth.POOL_MAX, pw=7, kernel="score_stream"):
    assert binding.scoring_route(binding.make_desc(Q, K, k_l, pool, pw), seq_lens=lens is not None)[0] == kernel
    print(kernel, tuple(Q.shape), tuple(K.shape), k_l, None if lens is None else lens.tolist()[:8], flush=True)
    ld = None if lens is None else torch.from_numpy(lens).to(DEV)
    out = binding.compress_layer(Q, K, V, k_l, pool, pw, seq_lens=ld, want_scores=True)
    torch.cuda.synchronize()
    return compare_layer(Q, K, V, k_l, Q.shape[2], pool, pw, lens, out)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha", [(1, 1), (1, 5), (1, 8), (3, 3), (2, 8), (1, 17), (4, 8), (1, 33), (6, 8), (8, 8)])
def test_rows(d, G, alpha):
    Q, K, V = _inputs(1, 2 * G, 2, d, 2600, alpha, seed=G * 100 + alpha + d)
    _check(Q, K, V, alpha + 60)


@pytest.mark.parametrize("N", [9, 32, 33, 255, 511, 512, 513, 520, 1023, 1024, 1025, 1032, 2048, 2049, 4100])
@pytest.mark.parametrize("G", [1, 8])
def test_lengths_around_an_item(N, G):
    alpha = 8
    Q, K, V = _inputs(1, G, 1, 128, N, alpha, seed=N + G)
    _check(Q, K, V, min(alpha + 40, N - 1))


@pytest.mark.parametrize("G", [1, 4, 8])
def test_ragged_batch(G):
    alpha, N = 8, 5000
    lens = np.array([5000, 0, 7, 8, 9, 40, 1032, 1033, 4097, 513], dtype=np.int32)
    Q, K, V = _inputs(len(lens), 2 * G, 2, 128, N, alpha, seed=G)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")
    _check(Q, K, V, 40, lens)


def test_many_items_per_workgroup():
    # 40 layers x 16 heads x 4 items = 2560 items: ten per workgroup; equal to one call per layer, bit for bit
    L, alpha, N = 40, 8, 4000
    data = [_inputs(2, 8, 8, 64, N, alpha, seed=500 + l) for l in range(L)]
    lens = torch.tensor([4000, 3100], dtype=torch.int32, device=DEV)
    ks = [alpha + 3 + 5 * l for l in range(L)]
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], ks, synth.POOL_MAX, 7,
                                   seq_lens=lens, want_scores=True)
    torch.cuda.synchronize()
    for l in range(L):
        one = binding.compress_layer(*data[l], ks[l], synth.POOL_MAX, 7, seq_lens=lens, want_scores=True)
        torch.cuda.synchronize()
        for x, y in zip(outs[l], one):
            assert torch.equal(x, y), l


def test_more_sequences_than_one_launch_holds():
    L, B, alpha, N = 3, 1100, 4, 96                          # 2048 (layer, sequence) pairs per launch
    data = [_inputs(B, 1, 1, 64, N, alpha, seed=40 + l) for l in range(L)]
    lens = np.random.RandomState(3).randint(0, N + 1, size=B).astype(np.int32)
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], [20, 12, 7],
                                   synth.POOL_AVG, 3, seq_lens=torch.from_numpy(lens).to(DEV), want_scores=True)
    torch.cuda.synchronize()
    for l, k_l in enumerate((20, 12, 7)):
        compare_layer(*data[l], k_l, alpha, synth.POOL_AVG, 3, lens, outs[l])


@pytest.mark.parametrize("G", [2, 8])
def test_references_that_do_not_fit(G):
    # the first key of a wave's tiles lies hundreds of binades below a later one: its rows are recomputed
    alpha, N = 8, 3000
    Q, K, V = _inputs(1, G, 1, 128, N, alpha, seed=G, scale=0.5)
    K[0, 0, 700] = 40 * Q[0, 0, 3]
    K[0, 0, 0:2500:32] = -20 * Q[0, 0, 3]
    _check(Q, K, V, alpha + 30, pool=synth.POOL_NONE, pw=1)


def precision_of_scores(Hq, Hkv, d, N, alpha, sink, kernel, layout=lambda Q: Q):
    """Largest error of a KV head's un-pooled scores against 64 bits, 2-norm over the prefix, for queries that point largely
    the same way.  sink: key 0 as a multiple of that direction, None for a key like the others."""
    g = torch.Generator(device=DEV).manual_seed(N + alpha)
    base = torch.randn(1, Hkv, 1, d, generator=g, device=DEV)
    Q = 1.2 * base + 0.9 * torch.randn(1, Hkv, Hq // Hkv * alpha, d, generator=g, device=DEV)
    Q = Q.reshape(1, Hq, alpha, d).to(torch.bfloat16)
    K = torch.randn(1, Hkv, N, d, generator=g, device=DEV).to(torch.bfloat16)
    if sink is not None:
        K[:, :, 0] = (sink * base[:, :, 0]).to(torch.bfloat16)
    Q = layout(Q)
    assert binding.scoring_route(binding.make_desc(Q, K, alpha + 100, synth.POOL_NONE, 1))[0] == kernel
    out = binding.compress_layer(Q, K, K, alpha + 100, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    hidden = torch.ones(alpha, alpha, dtype=torch.bool, device=DEV).triu(1)
    worst = 0.0
    for h in range(Hkv):
        x = Q[0].reshape(Hkv, -1, d)[h].double() @ K[0, h].double().t().contiguous() / d ** 0.5
        x.view(-1, alpha, N)[:, :, N - alpha:].masked_fill_(hidden, -np.inf)
        want = x.softmax(dim=1).sum(dim=0)[:N - alpha] / (Hq // Hkv)
        worst = max(worst, float((out[4][0, h, :N - alpha].double() - want).norm() / want.norm()))
    return worst


@pytest.mark.parametrize("Hq,Hkv,d,N,alpha", [(32, 8, 128, 8192, 16), (32, 8, 128, 30000, 8), (8, 8, 64, 1024, 8), (16, 4, 64, 5000, 16)])
@pytest.mark.parametrize("sink", [None, 3, -4])
def test_precision_with_a_sink_above_or_below_the_other_keys(Hq, Hkv, d, N, alpha, sink):
    # bound: a logit of up to 2^5 binades carries half a unit in the last place, 2^-20, and so does its distance from the
    # reference; together 2^-19 ln 2 = 1.3e-6 in a score
    assert precision_of_scores(Hq, Hkv, d, N, alpha, sink, "score_stream") < 1.3e-6



def _along(G, alpha, binades, d, seed):
    """One KV head whose query rows all point the same way; key j's logit for each of them is about binades[j] ln 2."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    base = torch.randn(d, generator=g, device=DEV)
    base *= d ** 0.5 / base.norm()
    Q = (base + 0.02 * torch.randn(1, G, alpha, d, generator=g, device=DEV)).to(torch.bfloat16)
    x = torch.tensor(binades, device=DEV, dtype=torch.float32) * np.log(2)
    noise = 0.3 * torch.randn(len(binades), d, generator=g, device=DEV)
    K = ((x / d ** 0.5)[:, None] * base + noise).to(torch.bfloat16)[None, None].contiguous()
    return Q, K, torch.randn(1, 1, len(binades), d, generator=g, device=DEV).to(torch.bfloat16)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha", [(1, 8), (3, 5), (4, 8), (8, 8)])
@pytest.mark.parametrize("first,top", [(-70, 75), (-20, 50), (-5, 75), (-30, 90), (-60, 20)])
def test_normalisers_far_above_the_references(d, G, alpha, first, top):
    # in every row one key stands far above the others and above key 0: the scores of the other keys, down to 2^-100 of
    # it, are ordinary fp32 numbers, and equal keys in different waves and items get equal ones
    binades = np.random.RandomState(G + d).uniform(-25, 25, 4100)
    binades[0], binades[700] = first, top
    Q, K, V = _along(G, alpha, binades, d, seed=G)
    equal = [100, 701, 1500, 1800, 3999]
    K[0, 0, equal] = K[0, 0, 1500].clone()
    print("far", d, G, alpha, first, top, flush=True)
    out = binding.compress_layer(Q, K, V, alpha + 30, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    compare_layer(Q, K, V, alpha + 30, alpha, synth.POOL_NONE, 1, None, out)
    assert len(set(out[4][0, 0, equal].tolist())) == 1


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha", [(1, 8), (2, 8), (4, 8), (8, 8)])
@pytest.mark.parametrize("lo,hi", [(0, 1), (32, 64), (0, 600), (1024, 2048), (0, 3500), (500, 4000)])
def test_logits_of_minus_infinity(d, G, alpha, lo, hi):
    # products that overflow to -inf: single keys, whole waves and items of them, and all keys that the references come from
    Q, K, V = _inputs(1, G, 1, d, 4100, alpha, seed=G + hi)
    Q = Q.abs()
    K[:, :, lo:hi] = -3e38
    _check(Q, K, V, alpha + 30, pool=synth.POOL_NONE, pw=1)


@pytest.mark.parametrize("L,B,Hkv,G,alpha,N", [(1, 1, 1, 1, 8, 40), (1, 1, 8, 4, 8, 100), (32, 1, 8, 4, 8, 100), (40, 1, 8, 4, 8, 127),
                                               (40, 1, 8, 4, 8, 128), (33, 1, 8, 8, 8, 250), (33, 1, 8, 8, 8, 256), (3, 2, 8, 8, 8, 600),
                                               (33, 4, 16, 8, 8, 100), (2, 150, 16, 1, 8, 60)])
def test_nothing_is_written_behind_the_workspace(L, B, Hkv, G, alpha, N):
    data = [_inputs(B, G * Hkv, Hkv, 128, N, alpha, seed=900 + l) for l in range(L)]
    print("guard", L, B, Hkv, G, alpha, N, flush=True)
    call = binding.LayersCall([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], [alpha + 5] * L, synth.POOL_MAX, 7,
                              want_scores=True)
    need = binding.workspace_bytes(call.descs[0], L)
    guarded = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device=DEV)   # (the guard is this test's own memory)
    call.workspace = guarded[:need]
    outs = call.run()
    torch.cuda.synchronize()
    assert bool((guarded[need:] == 0x5A).all())
    compare_layer(*data[-1], alpha + 5, alpha, synth.POOL_MAX, 7, None, outs[-1])


@pytest.mark.parametrize("G,alpha,name", [(4, 8, "score_stream"), (4, 32, "score_lag"), (4, 64, "score_lag")])
def test_the_recorder_names_the_scoring_kernel(G, alpha, name):
    Q, K, V = _inputs(1, 8 * G, 8, 128, 8192, alpha, seed=1)
    call = binding.LayersCall([Q], [K], [V], [alpha + 20], synth.POOL_MAX, 7)
    events = binding.HipEvents(6)
    ids = binding.run_profiled(call, events)
    torch.cuda.synchronize()
    events.close()
    assert [binding.KERNEL_NAMES[i] for i in ids] == [name, "pool_select"]
    assert binding.scoring_route(call.descs[0])[0] == name
