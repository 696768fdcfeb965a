"""One-pass scoring, 64 rows at a time, probabilities two steps behind (33 .. 512 query rows) at the edges of its work split:
rows around the groups, lengths around the items, ragged batches, odd and even numbers of items and steps, layers kept whole,
references that do not fit or are -inf, precision, the end of the workspace, waits that are given up."""
import numpy as np
import pytest
import torch

from paper_2406_02069_amd import binding, synth
from tests.parity import compare_layer
from tests.test_gpu_stream import _along, _inputs, precision_of_scores
from tests.test_gpu_stream import _check as check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _taken(Q, K, k_l, seq_lens=False):
    """The kernel under test takes the call."""
    desc = binding.make_desc(Q, K, k_l, synth.POOL_MAX, 7, None)
    return binding.scoring_route(desc, seq_lens=seq_lens)[0] == "score_lag"


def _check(Q, K, V, k_l, lens=None, pool=synth.POOL_MAX, pw=7):
    return check(Q, K, V, k_l, lens, pool, pw, kernel="score_lag")


def _enough_heads(Q, K, V):
    """One head's data over so many heads that the kernel under test takes it at 64 rows and less."""
    n = 1 if Q.shape[1] * Q.shape[2] > 64 else -(-1280 // -(-K.shape[2] // 512))
    return Q.repeat(1, n, 1, 1), K.repeat(1, n, 1, 1), V.repeat(1, n, 1, 1)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,alpha", [(5, 13), (3, 32), (127, 1), (8, 16), (3, 43), (4, 48), (1, 64), (7, 28), (5, 51), (8, 32), (7, 37),
                                     (8, 40), (6, 64), (7, 56), (8, 64)])
def test_rows(d, G, alpha):
    # one to eight groups of rows, the last of them full or with a single row
    Hkv = 2 if G * alpha > 64 else 144
    Q, K, V = _inputs(1, Hkv * G, Hkv, d, 4111, alpha, seed=G * 100 + alpha + d)
    assert _taken(Q, K, alpha + 60)
    _check(Q, K, V, alpha + 60)


@pytest.mark.parametrize("N", [1024, 1025, 1055, 1056, 1057, 1535, 1536, 1537, 1567, 1568, 2047, 2048, 2049, 2560])
@pytest.mark.parametrize("G,alpha", [(4, 32), (2, 64)])
def test_lengths_around_an_item(N, G, alpha):
    Q, K, V = _inputs(1, 3 * G, 3, 128, N, alpha, seed=N + G)
    assert _taken(Q, K, alpha + 40)
    _check(Q, K, V, alpha + 40)


@pytest.mark.parametrize("d,G,alpha", [(64, 3, 40), (128, 4, 32), (128, 3, 51), (128, 8, 32), (64, 5, 64)])
def test_ragged_batch(d, G, alpha):
    # sequences without scores, of one key more than the window, and items that units share a workgroup's round with
    N = 6000
    lens = np.array([6000, 0, 7, alpha, alpha + 1, 100, 512, 513, 4097, 1037, 2048 + alpha, 2047 + alpha], dtype=np.int32)
    Q, K, V = _inputs(len(lens), 2 * G, 2, d, N, alpha, seed=G)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")
    assert _taken(Q, K, alpha + 20, seq_lens=True)
    _check(Q, K, V, alpha + 20, lens)


@pytest.mark.parametrize("d,Hkv,G,alpha,L,N", [(64, 16, 8, 8, 5, 33000), (128, 16, 4, 32, 9, 5000), (64, 16, 3, 50, 7, 6000), (128, 4, 8, 33, 6, 9000), (64, 40, 4, 64, 11, 4100)])
def test_many_items_per_workgroup_equal_one_call_per_layer(d, Hkv, G, alpha, L, N):
    # several rounds of items, units that straddle them, odd and even numbers of steps; layers kept whole among them
    data = [_inputs(1, G * Hkv, Hkv, d, N, alpha, seed=500 + l) for l in range(L)]
    ks = [alpha + 3 + 5 * l for l in range(L)]
    ks[1] = N
    ks[L - 1] = N + 7
    assert _taken(data[0][0], data[0][1], ks[0]) and _taken(data[0][0], data[0][1], ks[0], seq_lens=True)
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], ks, synth.POOL_MAX, 7,
                                   want_scores=True)
    full = torch.full((1,), N, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    for l in range(L):
        one = binding.compress_layer(*data[l], ks[l], synth.POOL_MAX, 7, seq_lens=full, want_scores=True)
        torch.cuda.synchronize()
        for x, y in zip(outs[l], one):
            assert torch.equal(x, y), l
    compare_layer(*data[0], ks[0], alpha, synth.POOL_MAX, 7, None, outs[0])


@pytest.mark.parametrize("d,B,Hkv,G,alpha,N", [(128, 12, 9, 2, 32, 6000), (64, 12, 20, 1, 50, 6000), (128, 9, 16, 8, 8, 16000)])
def test_ragged_batch_of_one_group(d, B, Hkv, G, alpha, N):
    # ... likewise with a new item at every step; workgroups with odd and with even numbers of items, 3 to 9 of them
    lens = np.array([N, 0, 7, alpha, alpha + 1, 513, N - 511, 4097, 2048 + alpha, N, 512, N - 1], dtype=np.int32)[:B]
    Q, K, V = _inputs(B, Hkv * G, Hkv, d, N, alpha, seed=G)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")
    _check(Q, K, V, alpha + 20, lens)


@pytest.mark.parametrize("G,alpha", [(1, 40), (4, 10), (4, 32), (4, 36)])
@pytest.mark.parametrize("Hkv", [3, 4])
def test_ragged_batch_of_long_sequences(Hkv, G, alpha):
    # units that may not lie in two rounds of the workgroups, two of them to a round (an odd one out among three), one to a round,
    # behind units that may; more layers than a launch has room for
    N = 131072 if G * alpha <= 128 else 65536
    lens = np.array([n for n in (45056, 45057, 7, 52224, 52225, 64513, 65536, 65537, 90113, 0, 600, 131072) if n <= N], dtype=np.int32)
    B, k, d = len(lens), alpha + 20, 64
    Q, K, V = _inputs(B, Hkv * G, Hkv, d, N, alpha, seed=G + Hkv)
    for b, n in enumerate(lens):
        K[b, :, n:] = float("nan")
    assert _taken(Q, K, k, seq_lens=True)
    L = 10
    outs = binding.compress_layers([Q] * L, [K] * L, [V] * L, [k] * L, synth.POOL_MAX, 7, seq_lens=torch.from_numpy(lens).to(DEV),
                                   want_scores=True)
    torch.cuda.synchronize()
    print("long", Hkv, G, alpha, flush=True)
    for out in outs[1:]:
        assert torch.equal(out[3], outs[0][3])
        for b, n in enumerate(lens):
            if n > k:
                assert torch.equal(out[4][b, :, :n - alpha], outs[0][4][b, :, :n - alpha])
                assert torch.equal(out[2][b], outs[0][2][b])
    some = [b for b in range(B) if lens[b] in (45057, 7, 65536, 90113)]
    compare_layer(Q[some], K[some], V[some], k, alpha, synth.POOL_MAX, 7, lens[some], tuple(x[some] for x in outs[0]))


@pytest.mark.parametrize("G,alpha", [(2, 32), (4, 32), (8, 24), (8, 64)])
@pytest.mark.parametrize("first,top", [(-70, 75), (-20, 50), (-5, 75), (-30, 90), (-60, 20)])
def test_normalisers_far_above_the_references(G, alpha, first, top):
    # in every row one key stands far above the others and above key 0, and above the keys the references come from: its sum is
    # kept apart or the unit is scored again, and equal keys in different waves and items get equal scores
    binades = np.random.RandomState(G + alpha).uniform(-25, 25, 4100)
    binades[0], binades[700] = first, top
    Q, K, V = _along(G, alpha, binades, 128, seed=G)
    equal = [100, 701, 1500, 1800, 3999]
    K[0, 0, equal] = K[0, 0, 1500].clone()
    Q, K, V = _enough_heads(Q, K, V)
    assert _taken(Q, K, alpha + 30)
    print("far", G, alpha, first, top, flush=True)
    out = binding.compress_layer(Q, K, V, alpha + 30, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    compare_layer(Q, K, V, alpha + 30, alpha, synth.POOL_NONE, 1, None, out)
    assert len(set(out[4][0, 0, equal].tolist())) == 1


def test_some_units_of_many_are_scored_again():
    # two of forty-eight heads in three of nine layers, in a launch whose workgroups have several items
    L, Hkv, G, alpha, N = 9, 16, 4, 32, 5000
    data = [_inputs(1, G * Hkv, Hkv, 128, N, alpha, seed=70 + l, scale=0.5) for l in range(L)]
    for l in (0, 4, 8):
        for g in (3, 15):
            data[l][1][0, g, 1234 + l] = 40 * data[l][0][0, g * G, 3]
    assert _taken(data[0][0], data[0][1], alpha + 30)
    outs = binding.compress_layers([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], [alpha + 30] * L,
                                   synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    for l in (0, 3, 8):
        compare_layer(*data[l], alpha + 30, alpha, synth.POOL_NONE, 1, None, outs[l])


@pytest.mark.parametrize("d,G,alpha", [(64, 4, 32), (128, 4, 32), (128, 5, 51), (64, 3, 20), (128, 1, 64)])
@pytest.mark.parametrize("lo,hi", [(0, 1), (0, 600), (1024, 2048), (0, 4000), (500, 5000)])
def test_logits_of_minus_infinity(d, G, alpha, lo, hi):
    # products that overflow to -inf: single keys, whole items, and all keys that the references come from
    Q, K, V = _inputs(1, G, 1, d, 5100, alpha, seed=G + hi)
    Q = Q.abs()
    K[:, :, lo:hi] = -3e38
    _check(*_enough_heads(Q, K, V), alpha + 30, pool=synth.POOL_NONE, pw=1)


@pytest.mark.parametrize("Hq,Hkv,d,N,alpha", [(64, 64, 128, 12000, 40), (32, 8, 128, 30000, 32), (16, 4, 64, 5000, 32), (64, 8, 128, 8192, 64)])
@pytest.mark.parametrize("sink", [None, 3, -4])
def test_precision_of_the_scores(Hq, Hkv, d, N, alpha, sink):
    # errors of single rows average out over this many; what is left is common to all rows: the rounding of kappa, 2^-25 of a
    # logit up to 10 binades from the mean, 10 ln 2 / 2^25 = 2.1e-7
    assert precision_of_scores(Hq, Hkv, d, N, alpha, sink, "score_lag") < 2.1e-7


@pytest.mark.parametrize("L,B,Hkv,G,alpha,N", [(1, 1, 1, 4, 32, 1024), (33, 1, 8, 2, 64, 1024), (3, 2, 8, 8, 24, 1537), (7, 1, 4, 8, 64, 4096)])
def test_nothing_is_written_behind_the_workspace(L, B, Hkv, G, alpha, N):
    data = [_inputs(B, G * Hkv, Hkv, 128, N, alpha, seed=900 + l) for l in range(L)]
    assert _taken(data[0][0], data[0][1], alpha + 5)
    call = binding.LayersCall([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], [alpha + 5] * L, synth.POOL_MAX, 7,
                              want_scores=True)
    need = binding.workspace_bytes(call.descs[0], L)
    guarded = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device=DEV)   # (the guard is this test's own memory)
    call.workspace = guarded[:need]
    outs = call.run()
    torch.cuda.synchronize()
    assert bool((guarded[need:] == 0x5A).all())
    compare_layer(*data[-1], alpha + 5, alpha, synth.POOL_MAX, 7, None, outs[-1])


@pytest.mark.parametrize("Hq,Hkv,alpha", [(16, 4, 32), (128, 64, 30), (8, 2, 64)])
def test_given_up_waits_are_reported(Hq, Hkv, alpha, monkeypatch):
    # forced from the host: no wait for other workgroups; the kernel runs to its end and the counts say so
    Q, K, V = _inputs(2, Hq, Hkv, 128, 5000, alpha, seed=1)
    monkeypatch.setattr(binding, "DESC_FLAGS", binding.FLAG_NO_WAIT)
    out = binding.compress_layer(Q, K, V, 80, synth.POOL_MAX, 7)
    torch.cuda.synchronize()
    assert out[3].tolist() == [-1, -1]
    monkeypatch.setattr(binding, "DESC_FLAGS", 0)
    _check(Q, K, V, 80)


@pytest.mark.parametrize("G,alpha", [(2, 32), (4, 32), (8, 24), (8, 64)])
@pytest.mark.parametrize("N", [4500, 5200])
@pytest.mark.parametrize("top", [12, 14, 22, 35, 42, 45, 60, 72, 75, 90, 101, 106])
def test_sums_that_are_counted_apart(G, alpha, top, N):
    # a key that many binades above all others, in one item or in several: sums beyond 2^13, 2^43 and 2^73 are kept in words of
    # their own (at 512 rows the shorter prompts have no third one), beyond 2^103 the unit is scored again
    for step in (N, 1100):
        binades = np.random.RandomState(top).uniform(-6, 0, N)
        binades[700::step] = top
        Q, K, V = _along(G, alpha, binades, 128, seed=top)
        Q, K, V = _enough_heads(Q, K, V)
        assert _taken(Q, K, alpha + 30)
        out = binding.compress_layer(Q, K, V, alpha + 30, synth.POOL_NONE, 1, want_scores=True)
        torch.cuda.synchronize()
        compare_layer(Q, K, V, alpha + 30, alpha, synth.POOL_NONE, 1, None, out)


@pytest.mark.parametrize("G,alpha", [(1, 64), (4, 32), (8, 64)])
@pytest.mark.parametrize("tops", [(10, 43, 73, 103), (30, 45, 44), (60, 74, 73.5), (99, 100, 70, 40, 10)])
def test_sums_in_several_words_add_up(G, alpha, tops):
    # items whose sums go to different words, about as large as each other at the borders between them
    binades = np.random.RandomState(len(tops)).uniform(-6, 0, 5200)
    for i, top in enumerate(tops):
        binades[300 + 900 * i] = top
    Q, K, V = _enough_heads(*_along(G, alpha, binades, 128, seed=7))
    assert _taken(Q, K, alpha + 30)
    out = binding.compress_layer(Q, K, V, alpha + 30, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    compare_layer(Q, K, V, alpha + 30, alpha, synth.POOL_NONE, 1, None, out)


@pytest.mark.parametrize("binades", [55, 75])
def test_a_key_far_above_the_others_in_every_unit_costs_little(binades):
    # (scoring such units again takes some fifteen times as long; reading the words for large sums a few per cent)
    G, alpha, N, Hkv, L = 4, 32, 16384, 8, 8
    data = [_inputs(1, G * Hkv, Hkv, 128, N, alpha, seed=l) for l in range(L)]
    for l, (Q, _, _) in enumerate(data):                      # queries of a head that point largely the same way
        base = torch.randn(1, Hkv, 1, 1, 128, generator=torch.Generator(device=DEV).manual_seed(90 + l), device=DEV)
        Q += (1.5 * base).expand(1, Hkv, G, 1, 128).reshape(1, Hkv * G, 1, 128).to(torch.bfloat16)

    def best(call):
        took = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            call.run()
            b.record()
            torch.cuda.synchronize()
            took.append(a.elapsed_time(b))
        return min(took)

    def call():
        return binding.LayersCall([x[0] for x in data], [x[1] for x in data], [x[2] for x in data], [alpha + 60] * L, synth.POOL_MAX, 7)

    assert _taken(data[0][0], data[0][1], alpha + 60)
    plain = best(call())
    for Q, K, _ in data:
        q = Q.view(1, Hkv, G * alpha, 128).float().mean(dim=2)
        K[:, :, 9000] = (q * (binades * np.log(2) * 128 ** 0.5 / q.square().sum(dim=2, keepdim=True))).to(torch.bfloat16)
    far = best(call())
    print("far", binades, plain, far, flush=True)
    assert far < 3 * plain


@pytest.mark.parametrize("Hkv,G,alpha,N", [(1, 4, 32, 32768), (1, 8, 64, 32768), (6, 4, 16, 65536), (1, 4, 32, 131072)])
def test_sums_far_below_the_reference_count(Hkv, G, alpha, N):
    # key 0 alone is the reference; every item of the others adds 2^-26 of it to the normaliser, 64 items 2^-20 = 9.5e-7, and
    # nobody's sum may be rounded away.  Bound of key 0's score: roundings of the normaliser, its reciprocal (1 ulp), the weight,
    # the sums over the rows (two per group of 64, five across the lanes), half an ulp each where not said otherwise;
    # and below 8e-7, half of what would be lost here (1.6e-6 and more)
    heads = [_along(G, alpha, np.where(np.arange(N) > 0, -35.0, 0.0), 128, seed=h) for h in range(Hkv)]
    Q, K, V = (torch.cat([x[i] for x in heads], dim=1).contiguous() for i in range(3))
    assert _taken(Q, K, alpha + 30)
    out = binding.compress_layer(Q, K, V, alpha + 30, synth.POOL_NONE, 1, want_scores=True)
    torch.cuda.synchronize()
    hidden = torch.ones(alpha, alpha, dtype=torch.bool, device=DEV).triu(1)
    bound = (1 + 2 + 1 + 2 * ((G * alpha + 63) // 64) + 5) * 2.0 ** -24
    for h in range(Hkv):
        x = Q[0].view(Hkv, -1, 128)[h].double() @ K[0, h].double().t().contiguous() / 128 ** 0.5
        x.view(-1, alpha, N)[:, :, N - alpha:].masked_fill_(hidden, -np.inf)
        rest = x[:, 1:].sub(x[:, :1]).exp().sum(dim=1)
        assert 0.5 * N / 512 * 2.0 ** -26 < float(rest.mean()) < 1.9 * N / 512 * 2.0 ** -26   # (else the inputs miss the point)
        want = float((1 / (1 + rest)).sum() / G)
        got = float(out[4][0, h, 0])
        print("sink", Hkv, G, alpha, N, (got - want) / want, bound, flush=True)
        assert abs(got - want) < min(bound, 8e-7) * want
