"""The work that users of this library have it do, as measurable cases.

Two kinds of case, told apart by "entry":

  compress  "layer"   one pkv_compress_layer call: a prefill that compresses every layer as soon as it is done
            "layers"  one pkv_compress_layers call for all layers of a request batch; with "lse" the softmax
                      denominators come from the prefill's attention kernel (pkv_compress_layers_lse), with "page" the
                      kept rows go into page pools (pkv_compress_layers_paged)
  decode    "decode"         one new query per sequence over every layer's compacted cache, one pkv_decode_attention
                             call per layer, as a decoder makes them
            "decode_layers"  the same for the caches of all layers in one pkv_decode_attention_layers call

Shapes are the configurations of the benchmark and of the tests (head geometries, 1k to 128k contexts, windows of 8 to
64 queries, cache sizes of 64 to 2048 per layer under a pyramid of ratio 20, ragged batches) and points between them.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2406_02069_amd import binding

DEV = "cuda:0"


# ---------------------------------------------------------------- cases

def _compress(name, entry, B, L, Hq, Hkv, d, N, alpha, avg, pool=1, pool_w=7, ragged_min=0, lse=False, page=0):
    return {"name": name, "entry": entry, "B": B, "L": L, "Hq": Hq, "Hkv": Hkv, "d": d, "N": N, "alpha": alpha,
            "avg": avg, "pool": pool, "pool_w": pool_w, "ragged_min": ragged_min, "lse": lse, "page": page}


def _decode(name, entry, B, L, Hq, Hkv, d, alpha, avg, page=0):
    return {"name": name, "entry": entry, "B": B, "L": L, "Hq": Hq, "Hkv": Hkv, "d": d, "alpha": alpha, "avg": avg,
            "page": page}


def listed():
    return [
        # one layer of a small multi-head model with a short prompt: nothing but launches and latency
        _compress("layer-mha-1k", "layer", 1, 1, 8, 8, 64, 1024, 8, 128),
        # one layer of a grouped-query model right behind its prefill, an ordinary prompt
        _compress("layer-8k", "layer", 1, 1, 32, 8, 128, 8192, 8, 128),
        # all layers of one request: ordinary prompt, few window queries
        _compress("step-8k", "layers", 1, 32, 32, 8, 128, 8192, 8, 128),
        # the benchmark's headline: long prompt, 32 window queries, average pooling
        _compress("step-32k", "layers", 1, 32, 32, 8, 128, 32768, 32, 128, pool=2, pool_w=5),
        # a ragged batch of requests, as a serving engine hands over
        _compress("batch-ragged-16k", "layers", 8, 32, 32, 8, 128, 16384, 16, 256, ragged_min=8192),
        # a large model: 80 layers, 8 query heads per key head, 64 window queries
        _compress("step-80-layers-32k", "layers", 1, 80, 64, 8, 128, 32768, 64, 128),
        # multi-head attention at a long context: few query rows per head, many heads
        _compress("step-mha-32k", "layers", 1, 8, 32, 32, 128, 32768, 8, 128),
        # the longest context
        _compress("step-128k", "layers", 1, 32, 32, 8, 128, 131072, 32, 128, pool=2, pool_w=5),
        # denominators supplied by the prefill kernel, a large cache, kept rows straight into 16-slot pages; odd length
        _compress("lse-paged-24001", "layers", 1, 32, 32, 8, 128, 24001, 32, 2048, pool=2, pool_w=5, lse=True, page=16),
        # decoding, one call per layer as the model goes up its layers: a single request, a medium cache
        _decode("decode-per-layer", "decode", 1, 32, 32, 8, 128, 32, 512),
        # decoding for a batch over large compact caches, all layers in one call
        _decode("decode-layers-batch", "decode_layers", 8, 32, 32, 8, 128, 32, 2048),
        # decoding for a few requests over paged caches, all layers in one call
        _decode("decode-layers-paged", "decode_layers", 3, 32, 32, 8, 128, 16, 700, page=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    heads = rng.choice([(8, 8, 64), (16, 4, 64), (32, 8, 128), (32, 8, 128), (28, 4, 128), (64, 8, 128), (32, 32, 128)])
    Hq, Hkv, d = heads
    alpha = rng.choice([8, 16, 32, 64, rng.randint(8, 64)])
    L = _log_int(rng, 2, 48)
    if rng.random() < 0.3:
        entry = rng.choice(["decode", "decode_layers"])
        c = _decode("", entry, _log_int(rng, 1, 12), min(L, 32), Hq, Hkv, d, alpha,
                    max(_log_int(rng, 64, 2048), alpha + 16), rng.choice([0, 0, 16, 64]))
        # no more rows than the largest listed decoding case reads
        while c["B"] > 1 and c["B"] * c["L"] * c["Hkv"] * c["avg"] * d > 8 * 32 * 8 * 2048 * 128:
            c["B"] -= 1
    else:
        entry = rng.choice(["layer", "layers", "layers"])
        B = rng.choice([1, 1, 1, 2, rng.randint(3, 8)])
        N = _log_int(rng, 700, 131072)
        avg = min(max(_log_int(rng, 64, 2048), alpha + 16), N // 3)
        pool, pool_w = rng.choice([(1, 7), (2, 5), (1, 5), (2, 3), (1, 13)])
        c = _compress("", entry, B, 1 if entry == "layer" else L, Hq, Hkv, d, N, alpha, max(avg, alpha + 1), pool, pool_w,
                      ragged_min=N // 2 if B > 1 and rng.random() < 0.7 else 0)
        if entry == "layers":
            c["lse"] = rng.random() < 0.3
            c["page"] = rng.choice([0, 0, 0, 16, 32])
        # no more keys and no more matrix work than the largest listed case
        while c["L"] > 1 and (c["L"] * B * Hkv * N * d > 80 * 8 * 32768 * 128 or
                              c["L"] * B * Hq * alpha * N * d > 80 * 64 * 64 * 32768 * 128):
            c["L"] -= 1
        while c["B"] > 1 and c["B"] * Hkv * N * d > 80 * 8 * 32768 * 128:
            c["B"] -= 1
    del c["name"]
    return c


def _budgets(c):
    if c["entry"] == "layer":
        return [c["avg"]]
    return binding.budgets(c["L"], c["avg"], 20, c["alpha"])


def _lengths(c):
    """Valid lengths of the sequences: evenly spread over [ragged_min, N] (prepare deals them out in random order)."""
    if not c["ragged_min"]:
        return [c["N"]] * c["B"]
    return [int(round(c["ragged_min"] + (c["N"] - c["ragged_min"]) * (i + 0.5) / c["B"])) for i in range(c["B"])]


# ---------------------------------------------------------------- inputs

def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.bfloat16)


def _window_and_keys(gen, c):
    """Window queries, keys and values of one layer.  The queries of a window point largely the same way (they are
    neighbouring tokens of one instruction), so that a key's score varies over orders of magnitude, as it does in a
    trained model; key channels have unequal scales, and key 0 is an attention sink."""
    B, Hq, Hkv, d, N, alpha = (c[k] for k in ("B", "Hq", "Hkv", "d", "N", "alpha"))
    base = _normal(gen, B, Hkv, 1, 1, d).float()
    Q = 1.2 * base + 0.9 * torch.randn(B, Hkv, Hq // Hkv, alpha, d, generator=gen, device=DEV)
    K = _normal(gen, B, Hkv, N, d)
    K *= torch.exp(0.3 * torch.randn(1, Hkv, 1, d, generator=gen, device=DEV)).to(torch.bfloat16)
    K[:, :, 0, :] *= 6
    V = _normal(gen, B, Hkv, N, d)
    return Q.reshape(B, Hq, alpha, d).to(torch.bfloat16), K, V


def _denominators(Q, K, lens):
    """Natural-log softmax denominators of the window queries, fp32 [B, Hq, alpha]: what an attention kernel keeps."""
    B, Hq, alpha, d = Q.shape
    Hkv = K.shape[1]
    out = torch.empty(B, Hq, alpha, device=DEV)
    causal = torch.ones(alpha, alpha, dtype=torch.bool, device=DEV).triu(1)
    for b in range(B):
        n = lens[b]
        for g in range(Hkv):
            h0, h1 = g * (Hq // Hkv), (g + 1) * (Hq // Hkv)
            q = Q[b, h0:h1].reshape(-1, d).float()
            x = (q @ K[b, g, :n].float().t().contiguous()) / math.sqrt(d)
            x = x.view(h1 - h0, alpha, n)
            x[:, :, n - alpha:].masked_fill_(causal, -math.inf)
            out[b, h0:h1] = torch.logsumexp(x, dim=2)
    return out


def _pointers(tensors):
    return (ctypes.c_void_p * len(tensors))(*[t.data_ptr() for t in tensors])


def _prepare_compress(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(1_000_003 * (seed % (1 << 40)) + 7)
    rs = np.random.RandomState(seed % (1 << 32))
    B, Hkv, d, N, page = c["B"], c["Hkv"], c["d"], c["N"], c["page"]
    ks = _budgets(c)
    L = len(ks)
    lens = [_lengths(c)[i] for i in rs.permutation(B)]
    layers = [_window_and_keys(gen, c) for _ in range(L)]
    Q, K, V = ([x[i] for x in layers] for i in range(3))
    lens_dev = torch.tensor(lens, dtype=torch.int32, device=DEV) if c["ragged_min"] else None
    caps = [min(k, N) for k in ks]
    s = {"entry": c["entry"], "inputs": (Q, K, V, lens_dev), "k": ks, "pool": c["pool"], "pool_w": c["pool_w"]}
    # the compacted caches of all layers lie in one block of memory each for K and V, positions and counts likewise
    idx = torch.full((sum(B * Hkv * k for k in caps),), -1, dtype=torch.int32, device=DEV)
    count = torch.zeros(L, B, dtype=torch.int32, device=DEV)
    if page:
        max_pages = max((k + page - 1) // page for k in caps)
        pool_shape = (B * max_pages, Hkv, page, d)
        kc, vc = (torch.zeros(L, *pool_shape, dtype=torch.bfloat16, device=DEV) for _ in range(2))
        K_out, V_out = list(kc), list(vc)
        tables = [torch.from_numpy(rs.permutation(B * max_pages).astype(np.int32).reshape(B, max_pages)).to(DEV)
                  for _ in range(L)]
        s["paged"] = binding.PagedDesc(page, B * max_pages, max_pages, 0)
        s["tables"] = tables
    else:
        rows = B * Hkv * sum(caps)
        kc, vc = (torch.zeros(rows * d, dtype=torch.bfloat16, device=DEV) for _ in range(2))
        K_out, V_out, at = [], [], 0
        for k in caps:
            n = B * Hkv * k * d
            K_out.append(kc[at:at + n].view(B, Hkv, k, d))
            V_out.append(vc[at:at + n].view(B, Hkv, k, d))
            at += n
    idx_out, at = [], 0
    for k in caps:
        idx_out.append(idx[at:at + B * Hkv * k].view(B, Hkv, k))
        at += B * Hkv * k
    # kept rows are bit copies: they are handed out as 16-bit words
    s["result"] = {"k": kc.view(torch.int16), "v": vc.view(torch.int16), "idx": idx, "count": count}
    descs = (binding.LayerDesc * L)(*[binding.make_desc(Q[l], K[l], ks[l], c["pool"], c["pool_w"],
                                                        None if page else K_out[l]) for l in range(L)])
    s["workspace"] = binding.alloc_workspace(descs[0], DEV, L)
    if c["entry"] == "layer":
        s["outputs"] = (K_out[0], V_out[0], idx_out[0], count[0], None)
        return s
    s["L"], s["descs"] = L, descs
    s["in_ptrs"] = [_pointers(t) for t in (Q, K, V)]
    s["out_ptrs"] = [_pointers(t) for t in (K_out, V_out)]
    s["idx_ptrs"] = [_pointers(idx_out), _pointers(list(count))]
    s["lens_ptr"] = None if lens_dev is None else lens_dev.data_ptr()
    s["lse_ptrs"] = s["table_ptrs"] = None
    if c["lse"]:
        s["lse"] = [_denominators(Q[l], K[l], lens) for l in range(L)]
        s["lse_ptrs"] = _pointers(s["lse"])
    if page:
        s["table_ptrs"] = _pointers(s["tables"])
    return s


def _prepare_decode(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(1_000_003 * (seed % (1 << 40)) + 11)
    rs = np.random.RandomState(seed % (1 << 32))
    B, Hq, Hkv, d, page = c["B"], c["Hq"], c["Hkv"], c["d"], c["page"]
    ks = _budgets(c)
    L = len(ks)
    s = {"entry": c["entry"], "k": ks, "tables": None}
    s["q"] = [1.5 * _normal(gen, B, Hq, d) for _ in range(L)]
    s["count"] = [torch.full((B,), k, dtype=torch.int32, device=DEV) for k in ks]
    if page:
        need = [B * ((k + page - 1) // page) for k in ks]
        shapes = [(n, Hkv, page, d) for n in need]
        s["tables"] = [torch.from_numpy(rs.permutation(n).astype(np.int32).reshape(B, n // B)).to(DEV) for n in need]
    else:
        shapes = [(B, Hkv, k, d) for k in ks]
    s["K"] = [_normal(gen, *sh) for sh in shapes]
    s["V"] = [_normal(gen, *sh) for sh in shapes]
    if c["entry"] == "decode_layers":
        s["call"] = binding.DecodeLayersCall(s["q"], s["K"], s["V"], s["count"], block_tables=s["tables"],
                                             k_caps=ks if page else None)
        return s
    s["out"] = torch.zeros(L, B, Hq, d, dtype=torch.float32, device=DEV)
    s["outs"] = list(s["out"])
    s["workspace"] = torch.empty(B * Hkv * 16 * (8 * d + 16) * 4, dtype=torch.uint8, device=DEV)
    return s


def prepare(case, seed):
    return _prepare_decode(case, seed) if case["entry"].startswith("decode") else _prepare_compress(case, seed)


# ---------------------------------------------------------------- one pass

def run(s):
    entry = s["entry"]
    if entry == "layer":
        Q, K, V, lens = s["inputs"]
        binding.compress_layer(Q[0], K[0], V[0], s["k"][0], s["pool"], s["pool_w"], seq_lens=lens, outputs=s["outputs"],
                               workspace=s["workspace"])
        return s["result"]
    if entry == "layers":
        lib = binding.load()
        ws = s["workspace"]
        tail = (None, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
        if s["table_ptrs"] is not None:
            rc = lib.pkv_compress_layers_paged(s["L"], s["descs"], *s["in_ptrs"], s["lse_ptrs"], s["lens_ptr"],
                                               ctypes.byref(s["paged"]), *s["out_ptrs"], s["table_ptrs"],
                                               *s["idx_ptrs"], *tail)
        elif s["lse_ptrs"] is not None:
            rc = lib.pkv_compress_layers_lse(s["L"], s["descs"], *s["in_ptrs"], s["lse_ptrs"], s["lens_ptr"],
                                             *s["out_ptrs"], *s["idx_ptrs"], *tail)
        else:
            rc = lib.pkv_compress_layers(s["L"], s["descs"], *s["in_ptrs"], s["lens_ptr"], *s["out_ptrs"],
                                         *s["idx_ptrs"], *tail)
        if rc != binding.OK:
            raise binding.PkvError(rc, "pkv_compress_layers")
        return s["result"]
    if entry == "decode":
        for l, k in enumerate(s["k"]):
            table = None if s["tables"] is None else s["tables"][l]
            binding.decode_attention(s["q"][l], s["K"][l], s["V"][l], s["count"][l], block_table=table,
                                     k_cap=k if table is not None else None, out=s["outs"][l],
                                     workspace=s["workspace"])
        return s["out"]
    return [o[0] for o in s["call"].run()]


# ---------------------------------------------------------------- accounting

def work(case):
    c = case
    ks = _budgets(c)
    B, Hq, Hkv, d, alpha = c["B"], c["Hq"], c["Hkv"], c["d"], c["alpha"]
    if c["entry"].startswith("decode"):
        rows = B * Hkv * sum(ks)                       # kept K and V rows read once; queries in, results out
        return {"bytes": 2 * rows * d * 2 + len(ks) * B * Hq * d * (2 + 4), "flops": 4.0 * (Hq // Hkv) * rows * d}
    lens = _lengths(c)
    out = {"bytes": 0, "flops": 0.0}
    for k in ks:
        scored = sum(n for n in lens if n > k)         # every key of the others is read once and scored once
        kept = sum(min(k, n) for n in lens)            # kept K and V rows read and written, their positions written
        out["bytes"] += Hkv * scored * d * 2 + B * Hq * alpha * (d * 2 + (4 if c["lse"] else 0)) + \
            kept * Hkv * (4 * d * 2 + 4)
        out["flops"] += 2.0 * Hq * alpha * d * scored
    return out


def tolerance(case):
    if case["entry"].startswith("decode"):
        return {"rel": 1e-5, "max": 1e-4}              # bf16 inputs, fp32 sums and results
    # Positions, counts and bit copies of rows.  Scores are fp32: where two keys at the cut agree to the last bits
    # another order of the sums may keep the other one, and the rows between the two move by one place.
    return {"rel": 0.0, "differ": 0.01}
