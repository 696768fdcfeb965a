"""Scoring by estimates (G * alpha > 64, 16k keys and more, 3 or 4 million in the call, no scores asked for): kept sets against the CPU oracle and against
the kernel that scores every key, at the edges of the work split; and the calls that are handed on to that kernel: estimates
that are no use, sums that do not fit, more keys near the cut than there is room for, layers whose scores are asked for."""
import numpy as np
import pytest
import torch

from oracle import pkv_oracle
from paper_2406_02069_amd import binding, synth
from tests.parity import compare_layer

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NONE, MAX, AVG = synth.POOL_NONE, synth.POOL_MAX, synth.POOL_AVG


def _inputs(B, G, Hkv, d, N, alpha, seed, spread=0.9):
    """Window queries that point largely the same way, key 0 an attention sink."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    base = torch.randn(B, Hkv, 1, 1, d, generator=g, device=DEV)
    Q = (1.2 * base + spread * torch.randn(B, Hkv, G, alpha, d, generator=g, device=DEV)).reshape(B, Hkv * G, alpha, d)
    K, V = (torch.randn(B, Hkv, N, d, generator=g, device=DEV) for _ in range(2))
    K[:, :, 0] *= 6
    return Q.to(torch.bfloat16), K.to(torch.bfloat16), V.to(torch.bfloat16)


def _run(Qs, Ks, Vs, ks, pool, pw, lens=None, scores=False):
    """The call over the layers, repeated until it is large enough to be taken; and of the first ones, per layer, sequence and
    head, what became of it: 0 scored by estimates; handed on: 1 no use, 2 failed, 4 too few take part."""
    L = len(Ks)
    n = -(-(6 << 20) // (L * Ks[0].shape[0] * Ks[0].shape[1] * Ks[0].shape[2]))
    Qs, Ks, Vs, ks = Qs * n, Ks * n, Vs * n, ks * n
    ld = None if lens is None else torch.from_numpy(np.asarray(lens, np.int32)).to(DEV)
    call = binding.LayersCall(Qs, Ks, Vs, ks, pool, pw, seq_lens=ld, want_scores=scores)
    call.run()
    torch.cuda.synchronize()
    B, Hkv = Ks[0].shape[:2]
    flags = call.workspace[8:8 + 4 * len(Ks) * B * Hkv].view(torch.int32).cpu().numpy().reshape(len(Ks), B, Hkv)
    for l in range(L, len(Ks)):
        assert np.array_equal(flags[l], flags[l % L])
        for i in range(4):
            assert torch.equal(call.outputs[l][i], call.outputs[l % L][i])
    assert np.isin(flags, (0, 1, 2, 4, 5)).all()
    return call, flags[:L]


def _sifted(flags):
    """Per layer and sequence: scored by estimates, but for a quarter of the heads at most, which are not tried."""
    return (4 * (flags & 1).sum(-1) <= flags.shape[-1]) & ((flags & 6) == 0).all(-1)


def _same(a, b):
    """Same kept sets and rows, ties and all: the scores of the two kernels are the same to the bit."""
    for x, y in zip(a[:4], b[:4]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d,G,alpha,N,pool,pw,k", [
    (128, 4, 17, 16384, AVG, 5, 17 + 60),      # a third row tile; the shortest buffer
    (128, 4, 32, 16417, MAX, 7, 32 + 1),       # one key to keep; a last pass of one key
    (128, 8, 64, 16640, NONE, 1, 64 + 120),    # all rows that fit, many kept
    (64, 8, 16, 16500, AVG, 17, 16 + 60),      # the widest pooling window
    (64, 7, 37, 16500, MAX, 3, 37),            # nothing to choose; rows that fill no tile
    (128, 5, 33, 17000, AVG, 3, 33 + 120),
])
def test_against_the_oracle(d, G, alpha, N, pool, pw, k):
    print("sift", d, G, alpha, N, pool, pw, k, flush=True)
    Q, K, V = _inputs(1, G, 8, d, N, alpha, seed=N + G)
    call, flags = _run([Q], [K], [V], [k], pool, pw)
    assert _sifted(flags).all()
    compare_layer(Q, K, V, k, alpha, pool, pw, None, call.outputs[0])
    rec = binding.attention_recall(call)[0].cpu().numpy()
    idx = call.outputs[0][2].cpu().numpy()
    for g in (0, 7):
        want = pkv_oracle.attention_recall(Q[0, g * G:(g + 1) * G], K[0, g], idx[0, g])
        assert abs(rec[0, g] - want) <= 1e-5  # (sums of 16k fp32 terms of at most 1)


@pytest.mark.parametrize("N", [32768, 33000, 65536, 131072])
@pytest.mark.parametrize("pool,pw", [(AVG, 5), (MAX, 13)])
def test_against_every_key_scored(N, pool, pw):
    print("sift", N, pool, pw, flush=True)
    alpha, G, ks = 32, 4, [32 + 20, 32 + 250]
    data = [_inputs(1, G, 8, 128, N, alpha, seed=N + l) for l in range(2)]
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, ks, pool, pw)
    assert _sifted(flags).all()
    full, other = _run(Qs, Ks, Vs, ks, pool, pw, scores=True)
    assert np.all(other == 1)
    for l in range(2):
        _same(call.outputs[l], full.outputs[l])


@pytest.mark.parametrize("G,million", [(4, 4), (5, 3)])
def test_fewest_keys(G, million):
    """From 4 million keys in a call on, 3 million with more than 128 rows: the same kept sets with a layer less, which the sifting
    kernels have no part in."""
    alpha, N = 32, 32768
    Q, K, V = _inputs(1, G, 8, 128, N, alpha, seed=G)
    L = (million << 20) // (8 * N)
    print("sift fewest keys", G, L, flush=True)
    outs = []
    for n in (L, L - 1):
        call = binding.LayersCall([Q] * n, [K] * n, [V] * n, [alpha + 60] * n, AVG, 5)
        events = binding.HipEvents(5 * n + 1)
        ids = [binding.KERNEL_NAMES[i] for i in binding.run_profiled(call, events)]
        torch.cuda.synchronize()
        events.close()
        assert ids == (["score_sift"] if n == L else []) + ["score_lag", "pool_select"]
        if n == L:
            flags = call.workspace[8:8 + 4 * n * 8].view(torch.int32).cpu().numpy().reshape(n, 1, 8)
            assert _sifted(flags).all()
        outs.append(call.outputs[n - 1])
    _same(*outs)


@pytest.mark.parametrize("d,G,alpha", [(128, 4, 32), (64, 4, 21), (128, 5, 40)])
def test_token_major_layout(d, G, alpha):
    """Keys and queries of a token beside one another, heads inside: rows d * heads apart."""
    print("sift token-major", d, G, alpha, flush=True)
    data = _inputs(2, G, 8, d, 16401, alpha, seed=d + G)
    strided = [x.transpose(1, 2).contiguous().transpose(1, 2) for x in data]
    assert strided[1].stride(2) == 8 * d
    (a, flags), (b, same) = (_run([x[0]], [x[1]], [x[2]], [alpha + 40], AVG, 5) for x in (data, strided))
    assert _sifted(flags).all() and np.array_equal(flags, same)
    _same(a.outputs[0], b.outputs[0])


def test_ragged_batch():
    B, G, alpha, N, k = 5, 4, 32, 20000, 100
    lens = [20000, 4000, 90, 16401, 12289]   # two that are too short for it, one of them kept whole
    Q, K, V = _inputs(B, G, 8, 128, N, alpha, seed=5)
    for b in range(B):
        K[b, :, lens[b]:] = float("nan")
        V[b, :, lens[b]:] = float("nan")
    call, flags = _run([Q], [K], [V], [k], AVG, 5, lens)
    print(flags[0], flush=True)
    assert _sifted(flags)[0].tolist() == [True, False, True, True, True]
    compare_layer(Q, K, V, k, alpha, AVG, 5, np.asarray(lens, np.int32), call.outputs[0])


@pytest.mark.parametrize("G,alpha,pool,pw", [(8, 64, MAX, 7), (4, 32, NONE, 1), (4, 32, AVG, 5)])
def test_sink_does_not_hide_that_many_keys_lie_near_the_cut(G, alpha, pool, pw):
    """Queries without a common direction and a sink that all of them see: no layer is tried."""
    print("sift sink", G, alpha, pool, flush=True)
    Q, K, V = _inputs(1, G, 8, 128, 16384, alpha, seed=G)
    Q = torch.randn_like(Q.float()).to(torch.bfloat16)
    K[0, :, 0] = 0.5 * Q.float().reshape(8, G * alpha, 128).sum(1).to(torch.bfloat16)
    call, flags = _run([Q], [K], [V], [alpha + 60], pool, pw)
    print(flags, flush=True)
    assert not _sifted(flags).any() and (flags & 2 == 0).all()
    compare_layer(Q, K, V, alpha + 60, alpha, pool, pw, None, call.outputs[0])


def test_handed_on():
    """Queries without a common direction (any key may be kept), keys far above the estimates, many keys at the cut, scores
    asked for: the kernel that scores every key takes these, among others that it does not."""
    alpha, G, N, k, L = 32, 4, 16384, 100, 5
    data = [list(_inputs(1, G, 8, 128, N, alpha, seed=50 + l)) for l in range(L)]
    data[1][0] = torch.randn_like(data[1][0].float()).to(torch.bfloat16)
    data[2][1][0, 3, 7001] = 4 * data[2][0][0, 13, 5]           # one head's normaliser is far above its estimate
    data[3][1][0, 2, 9000:15000] = data[3][1][0, 2, 9000] * 0 + 0.9 * data[3][0][0, 9, 0]  # 6000 equal keys at the top
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [k] * L, MAX, 7)
    print(flags[:, 0], flush=True)
    assert _sifted(flags)[:, 0].tolist() == [True, False, False, False, True] and flags[2, 0, 3] & 2 and flags[3, 0, 2] & 2
    full, _ = _run(Qs, Ks, Vs, [k] * L, MAX, 7, scores=True)
    for l in range(L):
        _same(call.outputs[l], full.outputs[l])
    a, b = (torch.stack(binding.attention_recall(c)).cpu().numpy() for c in (call, full))
    assert np.abs(a - b).max() <= 1e-5


@pytest.mark.parametrize("B,Hkv,tried", [(64, 7, False), (255, 1, False), (51, 5, True), (254, 1, True)])
def test_many_heads_of_128_items(B, Hkv, tried):
    """A layer whose heads' rounds do not fit a launch of the kernel that takes what is handed on (rounds of 256 workgroups, two heads
    of a sequence each: 254 fit) is scored by that kernel alone, every key; otherwise all of it may be handed on.  Queries without a
    common direction; keys and values of all sequences are the same memory."""
    N, alpha, G, k = 65536, 32, 4, 100
    print("sift many heads", B, Hkv, flush=True)
    g = torch.Generator(device=DEV).manual_seed(B)
    Q = torch.randn(B, Hkv * G, alpha, 64, generator=g, device=DEV).to(torch.bfloat16)
    K, V = (torch.randn(1, Hkv, N, 64, generator=g, device=DEV).to(torch.bfloat16).expand(B, -1, -1, -1) for _ in range(2))
    call = binding.LayersCall([Q], [K], [V], [k], MAX, 7)
    assert binding.scoring_route(call.descs[0], kept_only=True)[0] == ("score_sift" if tried else "score_lag")
    call.workspace.fill_(0x7F)  # (what an earlier call left there counts for nothing)
    call.run()
    torch.cuda.synchronize()
    if tried:
        flags = call.workspace[8:8 + 4 * B * Hkv].view(torch.int32).cpu().numpy().reshape(B, Hkv)
        assert _sifted(flags).mean() < 0.1  # (nearly all are handed on)
    for b in (0, B // 2, B - 1):  # one sequence alone: no estimates
        alone = binding.compress_layer(Q[b:b + 1], K[b:b + 1], V[b:b + 1], k, MAX, 7)
        for i in range(3):
            assert torch.equal(call.outputs[0][i][b:b + 1], alone[i])
    assert (call.outputs[0][3] == k).all()


@pytest.mark.parametrize("d,G,alpha", [(128, 4, 32), (128, 5, 40), (64, 4, 21)])
def test_large_sums_are_held(d, G, alpha):
    """Keys that one query sees above all others (a needle), by 2^20, 2^53, 2^78: the sums go to further words, the heads are not
    handed on for them, and the kept sets are those of the kernel that scores every key."""
    N, k, unit = 16500, alpha + 60, 1.4426950408889634 / d ** 0.5
    print("sift large sums", d, G, alpha, flush=True)
    data = [list(_inputs(1, G, 8, d, N, alpha, seed=20 + l)) for l in range(3)]
    for (Q, K, V), above in zip(data, (20, 53, 78)):
        for g in range(8):
            q = Q[0, g * G:(g + 1) * G].float().reshape(-1, d)
            row = q[alpha + 5 + g]
            own = row - q.mean(0)  # what it does not share with the others
            top = (K[0, g].float() @ row).max().item() * unit
            K[0, g, 2000 + 1500 * g] = ((above + top) / ((row @ own).item() * unit) * own).to(torch.bfloat16)
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [k] * 3, AVG, 5)
    print(flags[:, 0], flush=True)
    # every layer is tried; a head may be handed on all the same (the strongest keys are seen by many other queries, too)
    assert (4 * (flags & 1).sum(-1) <= 8).all() and ((flags & 2) != 0).sum() <= 3
    full, _ = _run(Qs, Ks, Vs, [k] * 3, AVG, 5, scores=True)
    for l in range(3):
        _same(call.outputs[l], full.outputs[l])
    a, b = (torch.stack(binding.attention_recall(c)).cpu().numpy() for c in (call, full))
    assert np.abs(a - b).max() <= 1e-5


def _scored_again(call, flags):
    """Per unit of the call's scoring layers: whether the kernel that scores every key has added sums of it."""
    d, L = call.descs[0], len(flags)
    need = binding.load().pkv_workspace_bytes(call.descs, call.L)
    at = need - binding.scoring_route(d, call.L)[2]
    groups = -(-(d.Hq // d.Hkv * d.alpha) // 64)
    words = call.workspace[at:at + L * d.B * d.Hkv * groups * 2048].view(torch.int64).view(L, d.B, d.Hkv, groups, 8, 32)
    return (words[..., :8] != 0).flatten(3).any(-1).cpu().numpy()  # (eight rows' sums, further words, references, maxima)


def test_a_head_that_fails_is_handed_on_alone():
    alpha, G, N, k = 32, 4, 32768, 100
    data = [list(_inputs(1, G, 8, 128, N, alpha, seed=70 + l)) for l in range(2)]
    data[1][1][0, 3, 7001] = 4 * data[1][0][0, 13, 5]           # one head's normalisers are far above their estimates
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [k] * 2, MAX, 7)
    print(flags[:, 0], flush=True)
    want = np.zeros((2, 1, 8), bool)
    want[1, 0, 3] = True
    assert np.array_equal(flags != 0, want) and np.array_equal(_scored_again(call, flags), want)
    full, _ = _run(Qs, Ks, Vs, [k] * 2, MAX, 7, scores=True)
    for l in range(2):
        _same(call.outputs[l], full.outputs[l])
    a, b = (torch.stack(binding.attention_recall(c)).cpu().numpy() for c in (call, full))
    assert np.abs(a - b).max() <= 1e-5


@pytest.mark.parametrize("B,N,G,d", [(3, 20000, 4, 64), (2, 65536, 4, 64), (1, 131072, 4, 128), (3, 16500, 9, 128)])
def test_some_heads_are_handed_on(B, N, G, d):
    """Single heads of several sequences, of units that are dealt one after the other and of units with rounds of their own (128 and
    256 items), of an odd number of heads, beside a layer of which all are handed on."""
    alpha, k, Hkv = 32, 100, 5
    print("sift some heads", B, N, G, d, flush=True)
    data = [list(_inputs(B, G, Hkv, d, N, alpha, seed=80 + l)) for l in range(3)]
    bad = [(l, b, g) for l in (0, 2) for b in range(B) for g in range(Hkv) if (l + b + g) % 3 == 0 and b != 1]
    for l, b, g in bad:
        data[l][1][b, g, 4001 + g] = 6 * data[l][0][b, g * G + 1, 5]
    data[1][0] = torch.randn_like(data[1][0].float()).to(torch.bfloat16)
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [k] * 3, MAX, 7)
    print(flags.tolist(), flush=True)
    for l, b, g in bad:
        assert flags[l, b, g] & 2
    assert not _sifted(flags)[1].any() and ((flags[[0, 2]] & 3) == 0).sum() >= 10 * B - len(bad) - 2
    full, _ = _run(Qs, Ks, Vs, [k] * 3, MAX, 7, scores=True)
    for l in range(3):
        _same(call.outputs[l], full.outputs[l])


def test_too_few_take_part():
    """4.5 million keys in the call, 1.5 million of heads that would be sifted: nothing is, and every key is scored."""
    alpha, G, N, k = 32, 4, 16384, 100
    data = [list(_inputs(1, G, 8, 128, N, alpha, seed=90 + l)) for l in range(3)]
    for l in (0, 1):
        data[l][0] = torch.randn_like(data[l][0].float()).to(torch.bfloat16)
    Qs, Ks, Vs = ([data[l % 3][i] for l in range(36)] for i in range(3))
    call = binding.LayersCall(Qs, Ks, Vs, [k] * 36, MAX, 7)
    call.run()
    torch.cuda.synchronize()
    flags = call.workspace[8:8 + 4 * 36 * 8].view(torch.int32).cpu().numpy().reshape(36, 1, 8)
    print(flags[:3, 0], flush=True)
    assert (flags & 4).all() and not (flags & 2).any() and _scored_again(call, flags).all()
    full = binding.LayersCall(Qs, Ks, Vs, [k] * 36, MAX, 7, want_scores=True)
    full.run()
    for l in range(36):
        _same(call.outputs[l], full.outputs[l])
    for a, b in zip(binding.attention_recall(call), binding.attention_recall(full)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("G,alpha,d", [(4, 32, 128), (4, 21, 64), (10, 40, 128)])
def test_hopeless_head_among_others(G, alpha, d):
    """Two heads of eight whose queries have no common direction are not tried, the others are."""
    N, k = 16500, alpha + 60
    print("sift hopeless heads", G, alpha, d, flush=True)
    Q, K, V = _inputs(1, G, 8, d, N, alpha, seed=G + alpha)
    for g in (2, 7):
        Q[0, g * G:(g + 1) * G] = torch.randn_like(Q[0, g * G:(g + 1) * G].float()).to(torch.bfloat16)
    call, flags = _run([Q], [K], [V], [k], MAX, 7)
    print(flags[0, 0], flush=True)
    assert flags[0, 0].tolist() == [0, 0, 1, 0, 0, 0, 0, 1]
    full, _ = _run([Q], [K], [V], [k], MAX, 7, scores=True)
    _same(call.outputs[0], full.outputs[0])


@pytest.mark.parametrize("pool,pw,strength,scale", [(AVG, 5, 1.2, 0.8), (MAX, 7, 1.2, 0.8), (MAX, 7, 0.6, 0.0), (AVG, 5, 0.7, 0.0)])
def test_most_heads_pass(pool, pw, strength, scale):
    """Key channels of unequal scales (LogNormal(0, scale)), which set the rows' weights apart from their estimates, and queries with a weak
    common direction: most heads pass their check, and all kept sets are those of the kernel that scores every key."""
    alpha, G, N, L = 32, 4, 32768, 4
    print("sift most heads", pool, pw, strength, scale, flush=True)
    data = []
    for l in range(L):
        Q, K, V = _inputs(1, G, 8, 128, N, alpha, seed=110 + l)
        g = torch.Generator(device=DEV).manual_seed(7 + l)
        base = torch.randn(1, 8, 1, 1, 128, generator=g, device=DEV)
        Q = (strength * base + 0.9 * torch.randn(1, 8, G, alpha, 128, generator=g, device=DEV)).reshape(Q.shape).to(torch.bfloat16)
        K *= torch.exp(scale * torch.randn(1, 8, 1, 128, generator=g, device=DEV)).to(torch.bfloat16)
        data.append((Q, K, V))
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [alpha + 96] * L, pool, pw)
    print(flags[:, 0], flush=True)
    assert (4 * (flags & 1).sum(-1) <= 8).all() and ((flags & 2) != 0).sum() <= 8 * L // 3
    full, _ = _run(Qs, Ks, Vs, [alpha + 96] * L, pool, pw, scores=True)
    for l in range(L):
        _same(call.outputs[l], full.outputs[l])


def _as_bits(out):
    return [t.view(torch.int16) if t.dtype == torch.bfloat16 else t for t in out[:4]]


@pytest.mark.parametrize("G", [4, 6])
def test_nan_and_infinities(G):
    """NaN, +inf and -inf in keys and queries that count: heads that see them are handed on or selected as with every key scored."""
    alpha, N, k = 32, 16500, 100
    nan, inf = float("nan"), float("inf")
    data = [_inputs(1, G, 8, 128, N, alpha, seed=130 + l) for l in range(3)]
    (_, K, _), (Q1, K1, _), (Q2, _, _) = data
    K[0, 0, 5000, 3] = nan
    K[0, 1, 5000, 3] = inf
    K[0, 2, 5000] = -inf
    K[0, 3, N - 2, 7] = nan           # in the window
    K1[0, 4, 0, 7] = inf              # among the references' keys
    Q1[0, 5 * G, 3, 2] = nan
    Q2[0, 6 * G + 1, 31, 2] = inf
    print("sift nan", G, flush=True)
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run_bits(Qs, Ks, Vs, [k] * 3, MAX, 7)
    print(flags[:, 0], flush=True)
    full, _ = _run_bits(Qs, Ks, Vs, [k] * 3, MAX, 7, scores=True)
    for l in range(3):
        for x, y in zip(_as_bits(call.outputs[l]), _as_bits(full.outputs[l])):
            assert torch.equal(x, y)
    odd = np.zeros((3, 1, 8), bool)
    odd[0, 0, :4] = odd[1, 0, 4:6] = odd[2, 0, 6] = True
    assert np.array_equal(flags != 0, odd)


def _run_bits(Qs, Ks, Vs, ks, pool, pw, scores=False):
    """As _run, whose comparison of repeated layers does not hold for NaN: fewer repeats of more layers, none compared."""
    n = -(-(6 << 20) // (len(Ks) * Ks[0].shape[1] * Ks[0].shape[2]))
    call = binding.LayersCall(Qs * n, Ks * n, Vs * n, ks * n, pool, pw, want_scores=scores)
    call.run()
    torch.cuda.synchronize()
    Hkv = Ks[0].shape[1]
    flags = call.workspace[8:8 + 4 * len(Ks) * n * Hkv].view(torch.int32).cpu().numpy().reshape(len(Ks) * n, 1, Hkv)
    return call, flags[:len(Ks)]


def test_more_layers_than_a_launch_takes():
    """110 layers, 96 to a launch of the sifting kernels, four kept whole among them, some handed on by each launch."""
    alpha, G, N, L = 32, 4, 16384, 110
    data = [list(_inputs(1, G, 8, 64, N, alpha, seed=140 + l)) for l in range(5)]
    data[1][0] = torch.randn_like(data[1][0].float()).to(torch.bfloat16)
    data[2][1][0, 3, 7001] = 6 * data[2][0][0, 13, 5]
    Qs, Ks, Vs = ([data[l % 5][i] for l in range(L)] for i in range(3))
    ks = [N + 5 if l in (7, 50, 97, 109) else alpha + 20 + l for l in range(L)]
    calls = []
    for scores in (False, True):
        call = binding.LayersCall(Qs, Ks, Vs, ks, MAX, 7, want_scores=scores)
        call.workspace.fill_(0x7F)
        call.run()
        torch.cuda.synchronize()
        calls.append(call)
    flags = calls[0].workspace[8:8 + 4 * L * 8].view(torch.int32).cpu().numpy().reshape(L, 1, 8)
    scoring = [l for l in range(L) if ks[l] < N]
    print("sift many layers", flags[95:100, 0], flush=True)
    for l in scoring:
        # (14 layers are too few for a launch of their own: all of them are handed on)
        assert flags[l, 0, 0] in (0, 1) if l < scoring[96] else flags[l, 0, 0] & 4
        assert l % 5 != 1 or (flags[l, 0] & 1).sum() > 2
    assert flags[2, 0, 3] & 2 and flags[92, 0, 3] & 2
    for l in range(L):
        _same(calls[0].outputs[l], calls[1].outputs[l])
    for a, b in zip(*(binding.attention_recall(c) for c in calls)):
        assert (a - b).abs().max().item() <= 1e-5


def test_several_launches_of_what_is_handed_on():
    """100 sequences of one head with 128 items each: two layers to a launch of the kernel that takes the rest, five layers; keys and values
    of all sequences are the same memory."""
    B, N, alpha, G, L = 100, 65536, 32, 4, 5
    g = torch.Generator(device=DEV).manual_seed(150)
    K, V = (torch.randn(1, 1, N, 64, generator=g, device=DEV).to(torch.bfloat16).expand(B, -1, -1, -1) for _ in range(2))
    Qs = [torch.randn(B, G, alpha, 64, generator=g, device=DEV).to(torch.bfloat16) for _ in range(L)]
    for l in (0, 1, 3, 4):  # layers of which most is sifted
        Qs[l] = (1.2 * torch.randn(B, 1, 1, 64, generator=g, device=DEV) + 0.9 * Qs[l].float()).to(torch.bfloat16)
    ks = [alpha + 60 + l for l in range(L)]
    call = binding.LayersCall(Qs, [K] * L, [V] * L, ks, MAX, 7)
    events = binding.HipEvents(5 * L + 1)
    ids = [binding.KERNEL_NAMES[i] for i in binding.run_profiled(call, events)]
    torch.cuda.synchronize()
    events.close()
    assert ids[:4] == ["score_sift"] + ["score_lag"] * 3
    flags = call.workspace[8:8 + 4 * L * B].view(torch.int32).cpu().numpy().reshape(L, B, 1)
    share = _sifted(flags).mean(-1)
    print("sift several launches", share, flush=True)
    assert min(share[l] for l in (0, 1, 3, 4)) > 0.5 and share[2] < 0.2
    full = binding.LayersCall(Qs, [K] * L, [V] * L, ks, MAX, 7, want_scores=True)
    full.run()
    for l in range(L):
        _same(call.outputs[l], full.outputs[l])


@pytest.mark.parametrize("flat,taken", [(1, True), (3, True), (4, True), (5, False)])
def test_heads_object_one_by_one(flat, taken):
    """Some heads of every layer without a common direction of their queries: these alone are handed on, or all where they are more
    than half."""
    alpha, G, N, k, L = 32, 4, 32768, 100, 2
    data = [list(_inputs(1, G, 8, 128, N, alpha, seed=160 + l)) for l in range(L)]
    for x in data:
        x[0][0, :flat * G] = torch.randn_like(x[0][0, :flat * G].float()).to(torch.bfloat16)
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [k] * L, MAX, 7)
    print("sift flat heads", flat, flags[:, 0].tolist(), flush=True)
    want = np.zeros((L, 1, 8), np.int32) + (0 if taken else 4)
    want[:, :, :flat] |= 1
    assert np.array_equal(flags, want) and np.array_equal(_scored_again(call, flags), want != 0)
    full, _ = _run(Qs, Ks, Vs, [k] * L, MAX, 7, scores=True)
    for l in range(L):
        _same(call.outputs[l], full.outputs[l])


@pytest.mark.parametrize("at", [3, 20, 63])
@pytest.mark.parametrize("d,G,alpha,pool,pw", [(128, 4, 32, AVG, 5), (64, 6, 32, MAX, 7)])
def test_second_sink(at, d, G, alpha, pool, pw):
    """A key among the first 64 that all queries see far above the others: it counts in the weights, and heads pass their check; queries
    without a common direction are seen to have none all the same."""
    N, k = 32768, alpha + 60
    print("sift second sink", at, d, G, pool, flush=True)
    data = [list(_inputs(1, G, 8, d, N, alpha, seed=170 + l)) for l in range(2)]
    data[1][0] = torch.randn_like(data[1][0].float()).to(torch.bfloat16)
    for l, (Q, K, V) in enumerate(data):
        q = Q[0].float().view(8, G * alpha, d)
        K[0, :, at] = ((2.0 if l == 0 else 0.5 * G * alpha) * q.mean(1)).to(torch.bfloat16)
    Qs, Ks, Vs = ([x[i] for x in data] for i in range(3))
    call, flags = _run(Qs, Ks, Vs, [k] * 2, pool, pw)
    print(flags[:, 0].tolist(), flush=True)
    assert (flags[0] & 3 == 0).all() and (flags[1] & 1 != 0).all()
    full, _ = _run(Qs, Ks, Vs, [k] * 2, pool, pw, scores=True)
    for l in range(2):
        _same(call.outputs[l], full.outputs[l])


@pytest.mark.parametrize("G,fit,taken,ragged", [(6, 12, True, False), (6, 11, False, False), (4, 16, True, False), (4, 15, False, False),
                                                (4, 24, True, True), (4, 23, False, True)])
def test_layers_that_keep_many(G, fit, taken, ragged):
    """Layers of 8 x 16k keys, most of which keep more than a 43rd of their keys: the others are sifted from 1.5 million keys on with more than
    128 rows, from 2 million with 128, with sequence lengths from 3 million, those are not asked."""
    alpha, N, L = 32, 16384, 2 * fit + 8
    lens = torch.full((1,), N, dtype=torch.int32, device="cuda") if ragged else None
    data = [_inputs(1, G, 8, 64, N, alpha, seed=190 + l) for l in range(2)]
    Qs, Ks, Vs = ([data[l % 2][i] for l in range(L)] for i in range(3))
    ks = [alpha + (380 if l % 2 == 0 and l // 2 < fit else 381) for l in range(L)]   # 380 * 43 <= 16352 < 381 * 43
    print("sift large budgets", G, fit, ragged, flush=True)
    calls = []
    for scores in (False, True):
        call = binding.LayersCall(Qs, Ks, Vs, ks, MAX, 7, seq_lens=lens, want_scores=scores)
        events = binding.HipEvents(5 * L + 1)
        ids = [binding.KERNEL_NAMES[i] for i in binding.run_profiled(call, events)] if not scores else call.run()
        torch.cuda.synchronize()
        events.close()
        assert scores or ("score_sift" in ids) == taken
        calls.append(call)
    if taken:
        flags = calls[0].workspace[8:8 + 4 * L * 8].view(torch.int32).cpu().numpy().reshape(L, 1, 8)
        want = np.array([0 if k == alpha + 380 else 1 for k in ks])[:, None, None] + np.zeros((1, 1, 8), np.int64)
        assert np.array_equal(flags, want) and np.array_equal(_scored_again(calls[0], flags), want != 0)
    for l in range(L):
        _same(calls[0].outputs[l], calls[1].outputs[l])
    for a, b in zip(*(binding.attention_recall(c) for c in calls)):
        assert (a - b).abs().max().item() <= 1e-5
