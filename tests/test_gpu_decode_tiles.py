"""Decoding attention at the edges of its work split: group sizes of every padded width, row counts around the tiles of
a wave and the ranges of a workgroup, page sizes that are no power of two, and logits that climb along the cache so that
the running reference exponent has to be moved again and again."""
import numpy as np
import pytest
import torch

from paper_2406_02069_amd import binding
from tests.test_gpu_decode import DEV, _cmp, _rand

pytestmark = pytest.mark.gpu


def _climbing(q, Ks, Hq, Hkv, top):
    """Adds to key j a share of the group's first query such that its logit climbs to about `top` at the last row."""
    B, _, k_cap, d = Ks.shape
    q0 = q.view(B, Hkv, Hq // Hkv, d)[:, :, 0].float()
    step = top * np.sqrt(d) * torch.arange(k_cap, device=DEV) / max(k_cap - 1, 1)
    return (Ks.float() + step[None, None, :, None] * (q0 / q0.square().sum(-1, keepdim=True))[:, :, None]).to(torch.bfloat16)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,k_cap,top", [(1, 17, 0), (2, 15, 0), (3, 33, 0), (4, 16, 0), (5, 31, 0), (7, 257, 0), (8, 65, 0),
                                          (4, 700, 90), (8, 700, 90), (1, 1025, 60), (2, 769, 60), (6, 1537, 90)])
def test_groups_tiles_and_climbing_logits(d, G, k_cap, top):
    B, Hkv = 2, 2
    q, Ks, Vs = _rand(B, G * Hkv, Hkv, d, k_cap, seed=31 * G + k_cap + d)
    if top:
        Ks = _climbing(q, Ks, G * Hkv, Hkv, top)
    count = np.array([k_cap, max(k_cap - 13, 1)], dtype=np.int32)
    Ks[1, :, count[1]:] = float("nan")
    Vs[1, :, count[1]:] = float("nan")
    print("decode tiles", d, G, k_cap, top, flush=True)
    out, lse = binding.decode_attention(q, Ks, Vs, torch.from_numpy(count).to(DEV), want_lse=True)
    both = binding.decode_attention_layers([q, q], [Ks, Ks], [Vs, Vs], [torch.from_numpy(count).to(DEV)] * 2, want_lse=True)
    torch.cuda.synchronize()
    Kc, Vc = Ks.clone(), Vs.clone()
    Kc[1, :, count[1]:] = 0
    Vc[1, :, count[1]:] = 0
    for o, s in ((out, lse), both[0], both[1]):
        assert not torch.isnan(o).any()
        _cmp(o, s, Kc, Vc, q, count)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,lo,hi", [(1, 0, 32), (2, 0, 40), (4, 0, 300), (8, 0, 700), (4, 100, 600), (8, 0, 1499)])
def test_logits_of_minus_infinity(d, G, lo, hi):
    # products that overflow to -inf in the first tiles of a wave, of a whole range, and in all rows but the last ones
    B, Hkv, k_cap = 2, 2, 1600
    q, Ks, Vs = _rand(B, G * Hkv, Hkv, d, k_cap, seed=G + hi)
    q = q.abs()
    Ks[:, 0, lo:hi] = -3e38
    count = np.array([k_cap, 1500], dtype=np.int32)
    print("decode -inf", d, G, lo, hi, flush=True)
    out, lse = binding.decode_attention(q, Ks, Vs, torch.from_numpy(count).to(DEV), want_lse=True)
    torch.cuda.synchronize()
    _cmp(out, lse, Ks, Vs, q, count)


@pytest.mark.parametrize("page_size,k_cap", [(1, 40), (3, 100), (5, 333), (100, 999), (4095, 1300), (5000, 70)])
def test_page_sizes(page_size, k_cap):
    B, Hq, Hkv, d = 2, 8, 2, 128
    q, Ks, Vs = _rand(B, Hq, Hkv, d, k_cap, seed=page_size)
    per = (k_cap + page_size - 1) // page_size
    table = torch.from_numpy(np.random.RandomState(page_size).permutation(B * per).astype(np.int32).reshape(B, per)).to(DEV)
    pools = []
    for x in (Ks, Vs):
        p = torch.full((B * per, Hkv, page_size, d), float("nan"), dtype=torch.bfloat16, device=DEV)
        for b in range(B):
            for i in range(per):
                rows = x[b, :, i * page_size:(i + 1) * page_size]
                p[int(table[b, i]), :, :rows.shape[1]] = rows
        pools.append(p)
    count = np.array([k_cap, k_cap - 7], dtype=np.int32)
    print("decode pages", page_size, k_cap, flush=True)
    out, lse = binding.decode_attention(q, pools[0], pools[1], torch.from_numpy(count).to(DEV), block_table=table,
                                        k_cap=k_cap, want_lse=True)
    torch.cuda.synchronize()
    assert not torch.isnan(out).any()
    _cmp(out, lse, Ks, Vs, q, count)


@pytest.mark.parametrize("page_size", [0, 7])
@pytest.mark.parametrize("B,G,Hkv,d,k_cap", [
    (4, 4, 8, 128, 64), (4, 4, 8, 128, 63),      # 128 workgroups for the columns, the fewest rows; one range each
    (3, 3, 11, 128, 200),                        # a head too many
    (2, 1, 16, 128, 128), (2, 1, 16, 128, 127),  # single queries need twice the rows
    (1, 8, 2, 128, 768), (1, 8, 2, 128, 769),    # one range; several, merged
    (4, 2, 16, 64, 65), (1, 5, 3, 64, 1536),
])
def test_columns_of_few_heads(B, G, Hkv, d, k_cap, page_size):
    q, Ks, Vs = _rand(B, G * Hkv, Hkv, d, k_cap, seed=k_cap + B)
    count = np.array([k_cap, k_cap - 1, 5, 0][:B], dtype=np.int32)
    print("decode columns", B, G, Hkv, d, k_cap, page_size, flush=True)
    K, V, kw = Ks, Vs, {}
    if page_size:
        per = (k_cap + page_size - 1) // page_size
        table = np.random.RandomState(k_cap).permutation(B * per).astype(np.int32).reshape(B, per)
        K, V = (torch.zeros(B * per, Hkv, page_size, d, dtype=torch.bfloat16, device=DEV) for _ in range(2))
        for b in range(B):
            for i in range(per):
                n = min(page_size, k_cap - i * page_size)
                for pool, x in ((K, Ks), (V, Vs)):
                    pool[int(table[b, i]), :, :n] = x[b, :, i * page_size:i * page_size + n]
        kw = {"block_table": torch.from_numpy(table).to(DEV), "k_cap": k_cap}
    out, lse = binding.decode_attention(q, K, V, torch.from_numpy(count).to(DEV), want_lse=True, **kw)
    torch.cuda.synchronize()
    _cmp(out, lse, Ks, Vs, q, count)
