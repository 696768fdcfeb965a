// Window scoring for more than 64 query rows per KV head where only the kept set is asked for (Sec. 4.2.2, Eq. Al, Eq. att_score
// and the top-k behind it) on MI355X: estimated scores of all keys, exact ones of the few that can be kept.
//
// A key's score s_i = sum_r w_r p_ri (p: un-normalised probabilities, w_r = 1 / (G z_r)) needs the normalisers z_r, which are known only
// after all keys of the head have been seen.  The other kernels wait for them, with the keys or the probabilities on the chip, or form
// everything twice.  Here nothing waits: K streams through once, and with it go the normalisers and the estimates
// e_i = sum_r o_r p_ri with weights o_r from a sample of the keys.  Behind it the largest ratio rho = max_r w_r / o_r is known,
// and s_i <= rho e_i for every key.  So the keys (with pooling: the windows) with e_i >= tau are listed and scored exactly, and
// where the kept number of them reaches rho tau, no other key can be among the kept: the estimates of the others stay where they
// are, all below, and the selection finds the kept set among all of them.  tau is a guess (from the largest estimates, less what
// the weights differ); whether it was low enough is checked, never assumed.
//
// Handed on to the lagging one-pass kernel, which scores all keys: heads whose estimates are no use (seen beforehand: scores spread
// little where queries have no common direction), all of a launch where these are many, heads whose sums fit no word, whose list
// does not fit an eighth of the keys, or that fail the check.  Sums and scores come about exactly as in that kernel (same
// references, same order of additions), so that the kept sets are the same to the bit whoever scores.
//
// Four launches: sift_prepare_kernel (references, weights o_r from the first 64 keys and 512 or 1024 others: the median of eight groups'
// sums, so that a rare large key does not spoil them), score_sift_few_kernel or score_sift_many_kernel (the pass over K), sift_list_kernel (a workgroup per head: tau and the list),
// sift_exact_kernel (256 listed keys at a time; the last workgroup of a head makes the check and selects the kept set among the few
// places that reach the bound, so that the selection kernel only copies their rows).
//
// The pass over K: 256 persistent workgroups of 512 threads.  A wave holds 32 keys as matrix operands and passes over all query rows with
// them, the next two tiles of keys under way; up to 128 rows lie in the registers of every wave, more in LDS.  One product's matrix
// instructions are issued between the exponentials of the one before.  A barrier per 512 keys, for the sums.  Workgroups take stretches
// of items of equal length; no workgroup waits for another.
//
// What bounds it: vector instructions and HBM, and the clock the chip holds under this load, at 128 rows (32 layers x 8 heads x 32k
// keys 432 us, 5.0 TB/s, in the median of 60 launches behind one another, 425 at the least; 470 .. 480 in shorter series; the lagging
// kernel 622 .. 655), power at 512 rows (80 layers 3.2 ms at 1.8 GHz; 4.3: two key tiles per
// query fragment, sixteen waves, or products and exponentials of two waves in turn by barriers change the clock, 1.80 .. 1.94 GHz, and
// the time to 3.2 .. 3.5).  A launch begins with 12 us until the first product.  The kernels around it are chains of latencies:
// 26, 26 and 33 us for 256 heads of 32k keys (the selection kernel, which takes 27 otherwise, is left with 11).
#include <type_traits>

#include "pkv_internal.h"
#include "pkv_select_parts.h"
#include "pkv_tile.h"

namespace pkv {
namespace {

constexpr int kW = 8, kT = kW * 64;   // waves and threads of the kernel that reads K
constexpr int kPass = 32 * kW;        // keys of a pass
constexpr u64 kZLarge = 1ull << 63, kZBad = 1ull << 62;  // an item's sum lies in a further word; fits none
constexpr int kBlockRows = 128, kBlockTiles = kBlockRows / 32;  // query rows that lie in LDS at a time, but for the pass over K
constexpr int kSiftParts = 8;  // workgroups per unit there

// A unit's place: layer entry, sequence, head, valid length.
struct Unit {
  int l, b, g, n;
};
__device__ __forceinline__ int valid_length(const SiftArgs& a, int b) {
  if (!a.seq_lens) return a.N;
  const int n = a.seq_lens[b];
  return n < 0 ? 0 : (n > a.N ? a.N : n);
}
__device__ __forceinline__ Unit unit_of(const SiftArgs& a, int u) {
  const int BH = a.B * a.Hkv, l = (int)((u64)(uint32_t)(u + 1) * a.bh_magic >> 32), bg = u - l * BH, b = (int)((u64)(uint32_t)(bg + 1) * a.hkv_magic >> 32);
  return {l, b, bg - b * a.Hkv, valid_length(a, b)};
}
// Whether the heads of a (layer, sequence) of length n are asked at all: not where scores are wanted or many of the keys are kept.
__device__ __forceinline__ bool asked(const SiftArgs& a, int l, int n) {
  const int npre = n - a.alpha, kk = a.layer[l].k_l - a.alpha;
  return (a.scored[l >> 5] >> (l & 31) & 1) == 0 && npre >= kSiftMinKeys && (int64_t)kk * a.min_share <= npre;
}
__device__ __forceinline__ const int32_t* flags_of(const SiftArgs& a, int l, int b) {
  return a.flags + (size_t)a.layer[l].slot * a.B * a.Hkv + (size_t)b * a.Hkv;
}
__device__ __forceinline__ const uint16_t* keys_of(const SiftArgs& a, const Unit& p) {
  return a.layer[p.l].K + (size_t)p.b * a.kv_sb + (size_t)p.g * a.kv_sh;
}
__device__ __forceinline__ const uint16_t* queries_of(const SiftArgs& a, const Unit& p) {
  return a.layer[p.l].Q + (size_t)p.b * a.q_sb + (size_t)(p.g * a.G) * a.q_sh;
}
// Row r of 32 as matrix operand, from memory: lane (l32, hf) holds elements 16 ks + 8 hf of its row.
template <int KS>
__device__ __forceinline__ void load_rows(bf16x8 (&f)[KS], const uint16_t* row, int hf) {
  const char* p = reinterpret_cast<const char*>(row) + 16 * hf;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) f[ks] = as_frag(*reinterpret_cast<const u32x4*>(p + 32 * ks));
}

// ROWS rows of D elements on their way into LDS: rows of D / 8 + 1 sixteen-byte slots there (bank-free).
template <int D, int ROWS>
struct RowBlock {
  static constexpr int SEG = D / 8, PITCH = SEG + 1, PER = ROWS * SEG / kT, SLOTS = ROWS * PITCH;
  u32x4 v[PER];
  template <class Row>
  __device__ __forceinline__ void request(int row0, Row row) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int j = (int)threadIdx.x + i * kT;
      v[i] = *reinterpret_cast<const u32x4*>(row(row0 + j / SEG) + 8 * (j % SEG));
    }
  }
  __device__ __forceinline__ void commit(u32x4* s_q) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int j = (int)threadIdx.x + i * kT;
      s_q[j / SEG * PITCH + j % SEG] = v[i];
    }
  }
};
__device__ __forceinline__ const uint16_t* query_row_of(const SiftArgs& a, const uint16_t* Q, int row) {  // (rows behind the last repeat it)
  row = min(row, a.R - 1);
  const int hh = (int)(__umul24(row, a.alpha_magic) >> 16);
  return Q + (uint32_t)(hh * (int)a.q_sh + (row - hh * a.alpha) * (int)a.q_st);
}
// Logits of 32 keys (rows) and the 32 queries from `row` on of such a block.
template <int KS>
__device__ __forceinline__ f32x16 product_of(const u32x4* s_k, int key, const u32x4* s_q, int row, int hf) {
  const u32x4 *k = s_k + key * (2 * KS + 1) + hf, *q = s_q + row * (2 * KS + 1) + hf;
  f32x16 x = {};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) x = PKV_MFMA32(as_frag(k[2 * ks]), as_frag(q[2 * ks]), x);
  __builtin_amdgcn_sched_barrier(0);  // (one product's operands at a time)
  return x;
}
template <int KS>
__device__ __forceinline__ f32x16 product(const bf16x8 (&k)[KS], const u32x4* s_q, int row, int hf) {
  const u32x4* q = s_q + row * (2 * KS + 1) + hf;
  f32x16 x = {};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) x = PKV_MFMA32(k[ks], as_frag(q[2 * ks]), x);
  __builtin_amdgcn_sched_barrier(0);  // (one product's operands at a time)
  return x;
}

// Sums over the lower 32 lanes and over all of them (the same in all lanes).
__device__ __forceinline__ float2 wave_sums(float v) {
#define PKV_DPP_ADD(ctrl, rows) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rows, 0xF, false))
  PKV_DPP_ADD(0x111, 0xF);  // as wave_max_lane63
  PKV_DPP_ADD(0x112, 0xF);
  PKV_DPP_ADD(0x114, 0xF);
  PKV_DPP_ADD(0x118, 0xF);
  PKV_DPP_ADD(0x142, 0xA);
  PKV_DPP_ADD(0x143, 0xC);
#undef PKV_DPP_ADD
  return make_float2(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 31)), __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63)));
}

// ---- estimates of the normalisers of 128 rows of a unit; with its first rows, whether it is worth it ----
// Where it is not, that is seen from the 64 keys of the references, and the sample is left out (256 units of 128 rows 31 -> 10 us).  It is
// requested behind that: in front of it, it held the references' keys up and cost more than its latency does here (29 -> 26 us where it is used).
// What bounds it: latencies, and the address units, which take a fragment's 32 rows one by one.  So queries and the keys that
// several waves multiply come through LDS (256 units of 128 rows 31 -> 26 us, 640 of 512 rows 154 -> 98 when this was made, 111 with the
// first 64 keys and the question, against 64 rows per workgroup and every key as fragments from memory).
template <int D>
__global__ __launch_bounds__(kT, 4) void sift_prepare_kernel(const SiftArgs a, int clear_err) {
  constexpr int KS = D / 16;
  using QB = RowBlock<D, kBlockRows>;
  __shared__ u32x4 s_q[QB::SLOTS], s_k[QB::SLOTS];  // queries; 64 keys for the references and 64 of the window, then the first 64
  __shared__ float s_m[kBlockRows], s_part[kW][kBlockRows], s_win[2][kBlockRows], s_first[2][kBlockRows], s_score[64 * kBlockTiles];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blocks = (a.Rs + kBlockRows - 1) / kBlockRows, u = blockIdx.x / blocks, row0 = kBlockRows * (blockIdx.x - u * blocks);
  const int rows = min(kBlockRows, a.Rs - row0), ntile = rows / 32;
  if (blockIdx.x == 0 && tid == 0 && clear_err) a.err[0] = a.err[1] = 0;
  const Unit p = unit_of(a, u);
  const bool whole = a.layer[p.l].k_l >= p.n;
  const int npre = whole ? 1 : p.n - a.alpha;
  const bool ask = !whole && asked(a, p.l, p.n);
  const uint16_t* Q = queries_of(a, p);
  const uint16_t* K = keys_of(a, p);
  bf16x8 kf[2][KS];
  QB qb, kb;
  RowBlock<D, 64> fb;
  // The sample: wave w's group of keys is spread evenly over the prefix in runs of eight neighbours, four to a tile.
  auto sample = [&](int tile, bf16x8 (&f)[KS]) {
    const uint32_t run = (uint32_t)((4 * tile + (l32 >> 3)) * kW + wave);
    load_rows(f, K + (size_t)min((int)((uint32_t)npre * run >> a.sample_shift) + (l32 & 7), npre - 1) * a.kv_st, hf);
  };
  if (!whole) {
    // references: the largest logit of 64 keys, eight neighbours each at eight places, key 0 among them
    kb.request(0, [&](int i) { return K + (size_t)(i < 64 ? min((int)((uint32_t)npre * (uint32_t)(i >> 3) >> 3) + (i & 7), npre - 1) : min(npre + i - 64, p.n - 1)) * a.kv_st; });
    qb.request(row0, [&](int row) { return query_row_of(a, Q, row); });
    fb.request(0, [&](int i) { return K + (size_t)min(i, npre - 1) * a.kv_st; });
  }
  // the words of the kernel that takes the other sequences
  const size_t group0 = (size_t)u * a.groups + row0 / 64;
  u64* words = a.words + group0 * (kLagGroupBytes / 8);
  if (tid < rows * (kLagGroupBytes / 512) && ((tid & 31) < kLagRefs || (tid & 31) >= kLagMax)) words[tid] = 0;
  if (a.words4 && tid < rows) a.words4[group0 * (kLagGroupBytes4 / 8) + tid] = 0;
  int32_t* flag = a.flags + (size_t)a.layer[p.l].slot * a.B * a.Hkv + (size_t)p.b * a.Hkv + p.g;
  if (row0 == 0 && tid == 0) a.done[u] = a.total[u] = 0;
  if (whole) {
    if (row0 == 0 && tid == 0) *flag = 0;
    return;
  }
  kb.commit(s_k);
  qb.commit(s_q);
  lds_barrier();
  const int half = wave & 1, rt = wave >> 1;  // of the reference and window keys: the tile; of the rows
  f32x16 x, xw;  // logits of the wave's keys of the references and of the window
  if (rt < ntile) {
    x = product_of<KS>(s_k, 32 * half + l32, s_q, 32 * rt + l32, hf);
    float m = x[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) m = fmaxf(m, x[v]);
    m = both_halves<true>(m) * a.kappa;
    if (hf == 0) s_part[half][32 * rt + l32] = m;
    xw = product_of<KS>(s_k, 64 + 32 * half + l32, s_q, 32 * rt + l32, hf);
  }
  lds_barrier();
  fb.commit(s_k);
  if (tid < rows) {
    const float m = fmaxf(s_part[0][tid], s_part[1][tid]);
    s_m[tid] = m;
    reinterpret_cast<float*>(words)[lag_half_word(kLagRefs, tid)] = m;
  }
  lds_barrier();
  if (rt < ntile) {
    const int lim = min(row0 + 32 * rt + l32, a.R - 1) % a.alpha - 32 * half - 4 * hf;  // last window key the lane's query sees
    const float nm = -s_m[32 * rt + l32];
    float y = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) y += mrow0(v) > lim ? 0.f : fast_exp2(__builtin_fmaf(xw[v], a.kappa, nm));
    y = both_halves<false>(y);
    if (hf == 0) s_win[half][32 * rt + l32] = y;
    // Hopeless ones are seen from the references' keys, before the sample is looked at: the scores of 24 or 32 of them, with weights
    // from themselves, spread little.  (The first eight, where sinks lie, do not count.)
    y = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      x[v] = fast_exp2(__builtin_fmaf(x[v], a.kappa, nm));
      y += v < 4 && half == 0 ? 0.f : x[v];
    }
    const float o = row0 + 32 * rt + l32 < a.R ? __builtin_amdgcn_rcpf(both_halves<false>(y)) : 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] *= o;
    s_score[64 * rt + 32 * half + transpose_key(lane)] = transpose_sum(x, lane);
  }
  lds_barrier();
  {
    float e = 0.f;
    for (int i = 0; i < ntile; ++i) e += s_score[64 * i + lane];
    const float y = lane < 8 ? 0.f : fast_log2(fmaxf(e, 0x1p-100f));
    const float2 sum = wave_sums(y);
    const float off = lane < 8 ? 0.f : y - (lane < 32 ? sum.x * (1.f / 24.f) : (sum.y - sum.x) * (1.f / 32.f));
    // (a block that is not the unit's first does not decide; that it leaves is rarer, and void weights have the head handed on)
    const float least = row0 == 0 ? a.min_spread : 0.75f * a.min_spread;
    if (!ask || !(wave_sums(off * off).y >= 54.f * least * least)) {  // (the same in all waves)
      if (tid < rows) a.omega[(size_t)u * a.Rs + row0 + tid] = 0.f;
      if (row0 == 0 && tid == 0) *flag = kSiftObjects;
      return;
    }
    if (row0 == 0 && tid == 0) *flag = 0;
  }
  sample(0, kf[0]);
  sample(1, kf[1]);
  if (rt < ntile) {
    // the first 64 keys, which count themselves: sinks lie there, and the sample would miss them (one at key 20 that all rows see, 32
    // layers x 8 heads x 32k keys, 128 rows: the weights of every head lay apart, and the call took 1245 us, now 542; this takes 2)
    const float nm = -s_m[32 * rt + l32];
    float y0 = 0.f, y1 = 0.f;
    x = product_of<KS>(s_k, 32 * half + l32, s_q, 32 * rt + l32, hf);
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      y0 += fast_exp2(__builtin_fmaf(x[v], a.kappa, nm));
      y1 += fast_exp2(__builtin_fmaf(x[v + 1], a.kappa, nm));
    }
    y0 = both_halves<false>(y0 + y1);
    if (hf == 0) s_first[half][32 * rt + l32] = y0;
  }
  float z[kBlockTiles] = {};
#pragma unroll 1
  for (int tile = 0; tile < a.sample_tiles; tile += 2) {
    if (tile > 0) {
      sample(tile, kf[0]);
      sample(tile + 1, kf[1]);
    }
#pragma unroll
    for (int q = 0; q < kBlockTiles; ++q) {
      if (q >= ntile) continue;  // (uniform)
      const float nm = -s_m[32 * q + l32];
      float z0 = 0.f, z1 = 0.f;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const f32x16 x = product(kf[i], s_q, 32 * q + l32, hf);
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          z0 += fast_exp2(__builtin_fmaf(x[v], a.kappa, nm));
          z1 += fast_exp2(__builtin_fmaf(x[v + 1], a.kappa, nm));
        }
      }
      z[q] += z0 + z1;
    }
  }
#pragma unroll
  for (int q = 0; q < kBlockTiles; ++q) {
    const float y = both_halves<false>(z[q]);
    if (hf == 0) s_part[wave][32 * q + l32] = y;
  }
  lds_barrier();
  if (tid < rows) {
    // half the sum of the two middle ones of the groups: a rare large key does not count
    float v[kW], mid = 0.f;
#pragma unroll
    for (int w = 0; w < kW; ++w) v[w] = s_part[w][tid];
#pragma unroll
    for (int w = 0; w < kW; ++w) {
      int rank = 0;
#pragma unroll
      for (int x = 0; x < kW; ++x) rank += (v[x] < v[w] || (v[x] == v[w] && x < w)) ? 1 : 0;
      if (rank == kW / 2 - 1 || rank == kW / 2) mid += v[w];
    }
    const float window = s_win[0][tid] + s_win[1][tid];
    const float sum = __builtin_fmaf(mid, (float)(npre - 64) / (float)(64 * a.sample_tiles), s_first[0][tid] + s_first[1][tid]) + window;
    a.window[(size_t)u * a.Rs + row0 + tid] = window;
    const float o = row0 + tid < a.R ? a.inv_G / sum : 0.f;
    a.omega[(size_t)u * a.Rs + row0 + tid] = o;
    a.zsum[(size_t)u * a.Rs + row0 + tid] = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) a.zlarge[((size_t)u * 3 + i) * a.Rs + row0 + tid] = 0;
  }
}

// ---- the pass over K ----
// A pass of a workgroup (all fields wave-uniform): keys from `key` on of unit u.
struct Pass {
  int u, n, key, left;  // left: items of this workgroup behind this one
  const uint16_t* K;
};
__device__ __forceinline__ float* scores_of(const SiftArgs& a, int u) {
  const Unit x = unit_of(a, u);
  return a.raw + ((size_t)a.layer[x.l].slot * a.B * a.Hkv + (size_t)x.b * a.Hkv + x.g) * a.N;
}
// Keys and length of unit p.u; false: the unit is not sifted.
__device__ __forceinline__ bool open_unit(const SiftArgs& a, Pass& p, bool known) {
  const Unit x = unit_of(a, p.u);
  p.n = x.n;
  p.K = keys_of(a, x);
  return known || (a.layer[x.l].k_l < x.n && (flags_of(a, x.l, x.b)[x.g] & kSiftObjects) == 0);
}
// The pass after p, of KEYS keys; false if there is none (p is then a pass over the unit's first key alone).
template <int KEYS>
__device__ __forceinline__ bool advance(const SiftArgs& a, Pass& p) {
  p.key += KEYS;
  if (p.key % kLagKeys != 0 && p.key < p.n) return true;
  if (p.left == 0) {
    p.key = 0;
    p.n = 1;
    return false;
  }
  --p.left;
  if (p.key >= p.n) {
    do ++p.u;
    while (!open_unit(a, p, false));  // (there is one: an item is left)
    p.key = 0;
  }
  return true;
}
// The workgroup's first pass; false if it has none.  wsum: 2 kW + 2 words of LDS, read before the next barrier.
__device__ __forceinline__ bool first_pass(const SiftArgs& a, Pass& p, int* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // wsum: [kW] sums of the waves, [kW], [kW + 1] the first item's place; [kW] sums of the waves over all that were asked
  int* const wall = wsum + kW + 2;
  const int E = a.L * a.B;
  int lo = 0, hi = 0, u0 = 0, c0 = 0;
  int c = 0, parts = 0, before = 0;
  for (int round = 0; round < 2; ++round) {  // how many items there are; then who owns the first one
    int run = 0, all = 0;
    for (int e0 = 0; e0 < E; e0 += kT) {
      const int e = e0 + tid;
      if (round == 0 || E > kT) {  // (else the first round's are still there)
        int items = 0;
        c = parts = 0;
        if (e < E) {
          const int l = e / a.B, b = e - l * a.B, n = valid_length(a, b);
          parts = a.layer[l].k_l < n ? (n + kLagKeys - 1) / kLagKeys : 0;
          c = sift_heads<false>(flags_of(a, l, b), a.Hkv, kSiftObjects) * parts;
          items = asked(a, l, n) ? a.Hkv * parts : 0;
        }
        const int v = (int)wave_inclusive_sum((uint32_t)c), y = (int)wave_inclusive_sum((uint32_t)items);
        lds_barrier();
        if (lane == 63) {
          wsum[wave] = v;
          wall[wave] = y;
        }
        lds_barrier();
        before = run + v - c;
#pragma unroll
        for (int w = 0; w < kW; ++w) {
          before += w < wave ? wsum[w] : 0;
          run += wsum[w];
          all += wall[w];
        }
      }
      if (round == 1 && lo >= before && lo < before + c) {
        const int rem = lo - before, k = rem / parts, l = e / a.B;
        wsum[kW] = e * a.Hkv + sift_head<false>(flags_of(a, l, e - l * a.B), a.Hkv, kSiftObjects, k);
        wsum[kW + 1] = rem - k * parts;
      }
    }
    if (round == 0) {
      // Where little takes part (the same in all workgroups) the launches behind this one cost more than is gained, and heads that
      // barely take part gain little.  1 .. 5 heads of 8 without a common direction, 32 layers x 32k keys, 128 rows, max pooling, us: without
      // estimates 678, with them whatever takes part 567, 591, 613, 653, 663, handed on altogether 690; 24 layers, 512 rows 1316: 1085, 1159,
      // 1219, 1281, 1382 and 1345.  Average pooling, a common direction of 0.45 (half of the heads take part): 675: 724, 697; 1320: 1531, 1404.
      if (run < a.min_items || 2 * run < all) {
        for (int u = (int)blockIdx.x * kT + tid; u < a.L * a.B * a.Hkv; u += (int)gridDim.x * kT) {
          const Unit x = unit_of(a, u);
          a.flags[(size_t)a.layer[x.l].slot * a.B * a.Hkv + (size_t)x.b * a.Hkv + x.g] |= kSiftTooFew;  // (others may read it now, but another bit)
        }
        return false;
      }
      lo = (int)((int64_t)blockIdx.x * run / gridDim.x);
      hi = (int)((int64_t)(blockIdx.x + 1) * run / gridDim.x);
    }
  }
  lds_barrier();
  p.left = hi - lo;
  if (p.left == 0) return false;
  u0 = __builtin_amdgcn_readfirstlane(wsum[kW]);
  c0 = __builtin_amdgcn_readfirstlane(wsum[kW + 1]);
  --p.left;
  p.u = u0;
  p.key = c0 * kLagKeys;
  (void)open_unit(a, p, true);
  return true;
}

// A row's sum over an item: into what the workgroup adds up of the unit, or, where it is large, into a further word.
__device__ __forceinline__ void add_item(const SiftArgs& a, int u, int row, float z, u64& sum) {
  if (__builtin_expect(z <= kSumLimit, 1)) {
    sum += fixed_point(z, kSumUnits);
  } else if (z <= kSumLimit4) {
    const int i = z <= kSumLimit2 ? 0 : z <= kSumLimit3 ? 1 : 2;
    const u64 y = fixed_point(z, z <= kSumLimit2 ? kSumUnits2 : z <= kSumLimit3 ? kSumUnits3 : kSumUnits4);
    (void)__hip_atomic_fetch_add(a.zlarge + ((size_t)u * 3 + i) * a.Rs + row, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    sum |= kZLarge;
  } else {
    sum |= kZBad;
  }
}
// ... over a workgroup's items of the unit.
__device__ __forceinline__ void add_sum(const SiftArgs& a, int u, int row, u64 sum) {
  u64* z = a.zsum + (size_t)u * a.Rs + row;
  constexpr u64 marks = kZLarge | kZBad;
  if (sum & marks) (void)__hip_atomic_fetch_or(z, sum & marks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  (void)__hip_atomic_fetch_add(z, sum & ~marks, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 65 to 128 rows: they lie in the registers of every wave as matrix operands (but for the last row tile's, for which there are none
// left), and K comes through LDS.  A wave requests its tile two passes ahead, whole rows at a time and past the registers, and reads
// each fragment once, behind the last product that needs its predecessor.  Against queries in LDS and keys requested as operands a
// pass reads 16 KB of LDS per wave instead of 32 and has a fifth fewer vector instructions (407 are counted for 32 keys x 128 rows): both
// in one series, 32 layers x 8 heads x 32k keys 450 -> 412 us, x 128k 1853 -> 1700.
template <int D>
struct FewRows {
  static constexpr int ROWS = 128, TILES = ROWS / 32;
  static constexpr int SEG = D / 8, TILE = 32 * SEG;   // sixteen-byte slots of a key and of a wave's tile
  static constexpr int PER = 64 / SEG, LOADS = TILE / 64;  // keys of a request, requests of a tile
  static constexpr int QROWS = 64, QPITCH = SEG + 1;   // queries on their way into the registers
  static constexpr size_t kLds = (size_t)(2 * kW * TILE + QROWS * QPITCH) * 16 + ROWS * 8 + 3 * kW * ROWS * 4;
};
static_assert(FewRows<128>::kLds <= 160 * 1024, "one workgroup per compute unit");

template <int D>
__global__ __launch_bounds__(kT, 2) void score_sift_few_kernel(const SiftArgs a) {
  using F = FewRows<D>;
  constexpr int KS = D / 16, SEG = F::SEG, NRT = F::TILES;
  constexpr int TPM = 16 / KS;  // logits per lane handled between two matrix instructions
  extern __shared__ u32x4 smem[];
  u32x4* s_q = smem + 2 * kW * F::TILE;
  float2* s_r = reinterpret_cast<float2*>(s_q + F::QROWS * F::QPITCH);  // [ROWS] minus the reference, estimated weight
  float* s_z = reinterpret_cast<float*>(s_r + F::ROWS);                  // [2][kW][ROWS] sums by wave, in turn

  float* s_end = s_z + 2 * kW * F::ROWS;                                 // [kW][ROWS] a wave's sums behind a unit's end

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  u32x4* s_k = smem + wave * 2 * F::TILE;  // [2][32] keys, slot s of key i at s ^ (i % SEG) (bank-free)
  const uint32_t s_k_at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)s_k);

  Pass cur;
  if (!first_pass(a, cur, reinterpret_cast<int*>(s_z))) return;

  // Requests the wave's tile of a pass.  Keys at or beyond n are replaced by the last one.  Nothing of the buffer is being read.
  auto request = [&](const Pass& p, auto BUF) __attribute__((always_inline)) {
    const uint32_t stride = (uint32_t)a.kv_st * 2u;
    const int ln = fresh(lane), row = ln / SEG;
    const uint32_t seg16 = (uint32_t)((ln % SEG) ^ row) * 16u;
    const int key0 = min(p.key + 32 * wave, p.n - 1), last = p.n - 1 - key0;
    const char* base = reinterpret_cast<const char*>(p.K) + (uint64_t)(uint32_t)key0 * stride;
    uint32_t to0 = s_k_at;
    asm volatile("" : "+s"(to0));  // (not one register for each request all through the loop)
    auto go = [&](int j, const char* from, uint32_t row_at) __attribute__((always_inline)) {
      const uint32_t to = to0 + (uint32_t)(decltype(BUF)::value * F::TILE + 64 * j) * 16u;
      const uint32_t at = row_at + (seg16 ^ (F::PER * j & (SEG - 1)) * 16u);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(to), "v"(at), "s"(from) : "memory");
    };
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (__builtin_expect(last >= 31, 1)) {
      const uint32_t row_at = __umul24(row, stride);
#pragma unroll
      for (int j = 0; j < F::LOADS; ++j) go(j, base + (uint64_t)(F::PER * j) * stride, row_at);
    } else {
#pragma unroll
      for (int j = 0; j < F::LOADS; ++j) go(j, base, __umul24((uint32_t)min(F::PER * j + row, last), stride));
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the tile before the one requested last is there
  auto arrived = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(F::LOADS) : "memory");
  };
  typedef const __attribute__((address_space(3))) u32x4* lds_slots;
  const uint32_t k_lane = s_k_at + (uint32_t)((lane & 31) * SEG + ((lane >> 5) ^ (lane & (SEG - 1)))) * 16u;
  auto key_frag = [&](auto BUF, int ks) __attribute__((always_inline)) {
    return as_frag(reinterpret_cast<lds_slots>((uint32_t)fresh((int)k_lane) ^ (32u * ks))[decltype(BUF)::value * F::TILE]);
  };

  bf16x8 q[NRT - 1][KS], ql[3], kc[KS];  // queries but for the last row tile's, and a part of those
  float2 ref[NRT];
  float z[NRT] = {};
  f32x16 fin, out;  // products of even and of odd row tiles
  float* raw;  // the unit's scores
  // Queries, references and estimates of a unit.
  auto stage = [&](const Pass& p) __attribute__((always_inline)) {
    const uint16_t* Q = queries_of(a, unit_of(a, p.u));
    raw = scores_of(a, p.u);
    constexpr int N = F::QROWS * SEG / kT;
    const int tid = fresh(threadIdx.x), l32 = tid & 31, hf = tid >> 5 & 1;
    if (tid < F::ROWS)
      s_r[tid] = make_float2(-reinterpret_cast<const float*>(a.words + (size_t)p.u * a.groups * (kLagGroupBytes / 8))[lag_half_word(kLagRefs, tid)],
                             a.omega[(size_t)p.u * a.Rs + tid]);
#pragma unroll
    for (int h = 0; h < F::ROWS / F::QROWS; ++h) {
      u32x4 v[N];
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int j = tid + i * kT;
        v[i] = *reinterpret_cast<const u32x4*>(query_row_of(a, Q, F::QROWS * h + j / SEG) + 8 * (j % SEG));
      }
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int j = tid + i * kT;
        s_q[j / SEG * F::QPITCH + j % SEG] = v[i];
      }
      lds_barrier();
#pragma unroll
      for (int rt = 0; rt < F::QROWS / 32; ++rt)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          if (F::QROWS / 32 * h + rt < NRT - 1) q[F::QROWS / 32 * h + rt][ks] = as_frag(s_q[(32 * rt + l32) * F::QPITCH + 2 * ks + hf]);
      if (h == 0)
#pragma unroll
        for (int rt = 0; rt < NRT; ++rt) ref[rt] = s_r[32 * rt + l32];
      if (h == 0) lds_barrier();
    }
  };
  const u32x4* q_lane = s_q + (F::QROWS - 32 + (lane & 31)) * F::QPITCH + (lane >> 5);
  auto last_q = [&](int ks) __attribute__((always_inline)) {
    return as_frag(q_lane[2 * ks]);
  };
  auto prime = [&]() __attribute__((always_inline)) {  // the first product of a pass
    fin = f32x16{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fin = PKV_MFMA32(kc[ks], q[0][ks], fin);
  };

  int zbuf = 0;  // table in use
  u64 sum = 0;   // of the thread's row over the unit's items so far
  Pass nxt = cur;
  bool has_next = advance<kPass>(a, nxt);
  // One pass over the keys in kc; those of the next pass are on their way into the other buffer, those of the one after it are
  // requested into this one, which has been read.
  auto pass = [&](auto BUF) __attribute__((always_inline)) {
    using Other = std::integral_constant<int, 1 - decltype(BUF)::value>;
    Pass nx2 = nxt;
    const bool has_nx2 = has_next && advance<kPass>(a, nx2);
    request(nx2, BUF);
    const int wkey = cur.key + 32 * wave, npre = cur.n - a.alpha;
    f32x16 t;
    const bool ends = wkey + 32 > npre;  // the tile reaches into the causal window or beyond the end
    if (__builtin_expect(ends, 0)) {
      // sums without what a query does not see
      const int ln = fresh(lane), l32 = ln & 31, hf = ln >> 5;
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        const int lim = npre + (32 * rt + l32) % a.alpha - wkey - 4 * hf;  // last key the lane's query sees
        float z0 = 0.f, z1 = 0.f;
        f32x16 x = {};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x = PKV_MFMA32(kc[ks], rt < NRT - 1 ? q[min(rt, NRT - 2)][ks] : last_q(ks), x);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float y = mrow0(v) > lim ? 0.f : fast_exp2(__builtin_fmaf(x[v], a.kappa, ref[rt].x));
          if (v & 1) z1 += y;
          else z0 += y;
        }
        s_end[wave * F::ROWS + 32 * rt + l32] = z[rt] + both_halves<false>(z0 + z1);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // Product of row tile rt + 1 (behind the last one: of the next pass's keys and row tile 0) goes into `nx` while `fi`, that of row
    // tile rt, turns into exponentials.
    auto step = [&](auto RT, const f32x16& fi, f32x16& nx) __attribute__((always_inline)) {
      constexpr int rt = decltype(RT)::value;
      if constexpr (rt == NRT - 2) arrived();
      float z0 = 0.f, z1 = 0.f;
      nx = f32x16{};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if constexpr (rt == NRT - 2) {
          nx = PKV_MFMA32(kc[ks], ql[ks % 3], nx);
          if (ks + 2 < KS) ql[(ks + 2) % 3] = last_q(ks + 2);
          kc[ks] = key_frag(Other{}, ks);
        } else {
          nx = PKV_MFMA32(kc[ks], q[(rt + 1) % NRT][ks], nx);
          if (rt == NRT - 3 && ks >= KS - 2) ql[ks - KS + 2] = last_q(ks - KS + 2);
        }
        float x[TPM];
#pragma unroll
        for (int j = 0; j < TPM; ++j) x[j] = __builtin_fmaf(fi[TPM * ks + j], a.kappa, ref[rt].x);
#pragma unroll
        for (int j = 0; j < TPM; ++j) x[j] = fast_exp2(x[j]);
#pragma unroll
        for (int j = 0; j < TPM; ++j) {
          t[TPM * ks + j] = rt == 0 ? x[j] * ref[rt].y : __builtin_fmaf(x[j], ref[rt].y, t[TPM * ks + j]);
          if (j & 1) z1 += x[j];
          else z0 += x[j];
          asm volatile("" : "+v"(t[TPM * ks + j]));
        }
        asm volatile("" : "+v"(z0), "+v"(z1));
        __builtin_amdgcn_sched_barrier(0);
      }
      z[rt] += both_halves<false>(z0 + z1);  // (the sums of an item come about as in the kernel that scores the other sequences)
    };
    step(std::integral_constant<int, 0>{}, fin, out);
    step(std::integral_constant<int, 1>{}, out, fin);
    step(std::integral_constant<int, 2>{}, fin, out);
    step(std::integral_constant<int, 3>{}, out, fin);
    if (__builtin_expect(ends, 0)) {
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) z[rt] = s_end[wave * F::ROWS + 32 * rt + (fresh(lane) & 31)];
    }
    {
      const int ln = fresh(lane), key = wkey + transpose_key(ln);
      const float s = transpose_sum(t, ln);
      if (key < npre && (ln & 1) == 0) raw[key] = s;
    }
    const bool unit_ends = !has_next || nxt.u != cur.u;
    if (unit_ends || nxt.key % kLagKeys == 0) {  // the item's sums
      const int tid = fresh(threadIdx.x), l32 = tid & 31, hf = tid >> 5 & 1;
      float* z_lane = s_z + (zbuf * kW + wave) * F::ROWS + l32;
#pragma unroll
      for (int rt = 0; rt < NRT; ++rt) {
        if (hf == 0) z_lane[32 * rt] = z[rt];
        z[rt] = 0.f;
      }
      lds_barrier();
      if (tid < a.R) {
        const float* z8 = s_z + zbuf * kW * F::ROWS + tid;
        float w[kW];
#pragma unroll
        for (int i = 0; i < kW; ++i) w[i] = z8[i * F::ROWS];
        add_item(a, cur.u, tid, ((w[0] + w[1]) + (w[2] + w[3])) + ((w[4] + w[5]) + (w[6] + w[7])), sum);
      }
      zbuf ^= 1;  // (the table is written again behind the next item's barrier)
    }
    if (unit_ends) {
      const int tid = fresh(threadIdx.x);
      if (tid < a.R) add_sum(a, cur.u, tid, sum);
      sum = 0;
      if (has_next) {
        stage(nxt);
        prime();
      }
    }
    const bool more = has_next;
    cur = nxt;
    nxt = nx2;
    has_next = has_nx2;
    return more;
  };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  request(cur, B0{});
  request(nxt, B1{});
  stage(cur);
  arrived();
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kc[ks] = key_frag(B0{}, ks);
  prime();
#pragma unroll 1
  for (;;) {
    if (!pass(B0{})) break;
    if (!pass(B1{})) break;
  }
  // (requests of the pass that is not there: LDS belongs to the workgroup until they are through)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int D>
constexpr size_t sift_lds(int Rs) {
  // queries with a row pitch of D / 8 + 1 sixteen-byte slots (bank-free), references and estimates, sums by wave
  return (size_t)Rs * ((D / 8 + 1) * 16 + 8 + 4 * kW * sift_zbufs(Rs));
}
static_assert(sift_lds<128>(kResidentMaxRows) <= 160 * 1024 && sift_lds<128>(384) <= 160 * 1024, "one workgroup per compute unit");

// More than 128 rows: they lie in LDS.
template <int D>
__global__ __launch_bounds__(kT, 2) void score_sift_many_kernel(const SiftArgs a) {
  constexpr int KS = D / 16, SEG = D / 8, PITCH = SEG + 1;
  constexpr int TPM = 16 / KS;  // logits per lane handled between two matrix instructions
  extern __shared__ u32x4 smem[];
  u32x4* s_q = smem;
  float2* s_r = reinterpret_cast<float2*>(s_q + a.Rs * PITCH);  // [Rs] minus the reference, estimated weight
  float* s_z = reinterpret_cast<float*>(s_r + a.Rs);            // [zbufs][kW][Rs]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int nrt = a.Rs / 32;  // (even, six at least)

  Pass cur;
  if (!first_pass(a, cur, reinterpret_cast<int*>(smem))) return;
  float* raw;  // the unit's scores
  // Queries, references and estimates of a unit into LDS.  Barriers around it are the caller's.
  auto stage = [&](const Pass& p) {
    const uint16_t* Q = queries_of(a, unit_of(a, p.u));
    raw = scores_of(a, p.u);
    const int seg = tid & (SEG - 1);
    float2 ref = make_float2(0.f, 0.f);
    if (tid < a.Rs) {
      ref.x = -reinterpret_cast<const float*>(a.words + (size_t)p.u * a.groups * (kLagGroupBytes / 8))[lag_half_word(kLagRefs, tid)];
      ref.y = a.omega[(size_t)p.u * a.Rs + tid];
    }
    for (int row0 = tid / SEG; row0 < a.Rs; row0 += 4 * (kT / SEG)) {
      u32x4 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const u32x4*>(query_row_of(a, Q, row0 + j * (kT / SEG)) + 8 * seg);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = row0 + j * (kT / SEG);
        if (row < a.Rs) s_q[row * PITCH + seg] = v[j];
      }
    }
    if (tid < a.Rs) s_r[tid] = ref;
  };
  // Keys of a wave's tile as matrix operand.  Keys at or beyond n are replaced by the last one.
  bf16x8 b0[KS], b1[KS], b2[KS];
  auto issue_k = [&](const Pass& p, bf16x8 (&f)[KS]) {
    const int ln = fresh(lane);
    const int key = min(p.key + 32 * wave + (ln & 31), p.n - 1);
    const char* rowp = reinterpret_cast<const char*>(p.K) + 16 * (ln >> 5) + (uint32_t)key * ((uint32_t)a.kv_st * 2u);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = as_frag(*reinterpret_cast<const u32x4*>(rowp + 32 * ks));
    __builtin_amdgcn_sched_barrier(0);
  };
  const u32x4* q_lane = s_q + l32 * PITCH + hf;
  auto q_frag = [&](int rt, int ks) { return as_frag(q_lane[32 * rt * PITCH + 2 * ks]); };
  float* z_lane = s_z + wave * a.Rs + l32;

  bf16x8 qf[4];
  f32x16 fin, out;  // products of even and of odd row tiles
  bool first = true;  // pass of an item
  int zbuf = 0;       // table in use
  u64 sum = 0;        // of the thread's row over the unit's items so far
  auto prime = [&](const bf16x8 (&kc)[KS]) {  // the first product of a pass
    fin = f32x16{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fin = PKV_MFMA32(kc[ks], q_frag(0, ks), fin);
#pragma unroll
    for (int s = 0; s < 3; ++s) qf[s] = q_frag(1, s);
  };
  Pass nxt = cur;
  bool has_next = advance<kPass>(a, nxt);
  // One pass over the keys in kc; those of the next pass are in kn, those of the one after it are requested into kp.
  auto pass = [&](bf16x8 (&kc)[KS], bf16x8 (&kn)[KS], bf16x8 (&kp)[KS]) {
    Pass nx2 = nxt;
    const bool has_nx2 = has_next && advance<kPass>(a, nx2);
    issue_k(nx2, kp);
    const int wkey = cur.key + 32 * wave, npre = cur.n - a.alpha;
    f32x16 t;
    float* zp = z_lane + zbuf * kW * a.Rs;
    // (the sums of an item come about as in the kernel that scores the other sequences)
    auto z_before = [&](int rt) { return first ? 0.f : zp[32 * rt]; };
    auto set_z = [&](int rt, float z) {
      if (hf == 0) zp[32 * rt] = z;
    };
    if (__builtin_expect(wkey + 32 > npre, 0)) {
      // the tile reaches into the causal window or beyond the end
      t = f32x16{};
#pragma unroll 1
      for (int rt = 0; rt < nrt; ++rt) {
        const float2 ref = s_r[32 * rt + l32];
        const float before = z_before(rt);
        const int lim = npre + (32 * rt + l32) % a.alpha - wkey - 4 * hf;  // last key the lane's query sees
        float z0 = 0.f, z1 = 0.f;
        f32x16 x = {};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) x = PKV_MFMA32(kc[ks], q_frag(rt, ks), x);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float y = mrow0(v) > lim ? 0.f : fast_exp2(__builtin_fmaf(x[v], a.kappa, ref.x));
          if (v & 1) z1 += y;
          else z0 += y;
          t[v] = __builtin_fmaf(y, ref.y, t[v]);
        }
        set_z(rt, both_halves<false>(z0 + z1) + before);
      }
      if (has_next && nxt.u == cur.u) prime(kn);
    } else {
      // Product of row tile rt + 1 (LAST: of the next pass's keys and row tile 0) goes into `nx` while `fi`, that of row
      // tile rt, turns into exponentials.
      float2 ref_next = s_r[l32];
      auto step = [&](auto FIRST, auto LAST, int rt, const f32x16& fi, f32x16& nx) {
        constexpr bool start = decltype(FIRST)::value, last = decltype(LAST)::value;
        const int mul = last ? 0 : rt + 1, then = last ? 1 : rt + 2 < nrt ? rt + 2 : 0;
        // (what the next step needs at its beginning, and this one at its end)
        const float2 ref = ref_next;
        if (!last) ref_next = s_r[32 * (rt + 1) + l32];
        const float before = z_before(rt);
        float z0 = 0.f, z1 = 0.f;
        nx = f32x16{};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          // fragment 3 ahead: of this product, or of the next one
          if (ks + 3 < KS) qf[(ks + 3) & 3] = q_frag(mul, ks + 3);
          else qf[(ks + 3) & 3] = q_frag(then, ks + 3 - KS);
          nx = PKV_MFMA32(last ? kn[ks] : kc[ks], qf[ks & 3], nx);
          float x[TPM];
#pragma unroll
          for (int j = 0; j < TPM; ++j) x[j] = __builtin_fmaf(fi[TPM * ks + j], a.kappa, ref.x);
#pragma unroll
          for (int j = 0; j < TPM; ++j) x[j] = fast_exp2(x[j]);
#pragma unroll
          for (int j = 0; j < TPM; ++j) {
            t[TPM * ks + j] = start ? x[j] * ref.y : __builtin_fmaf(x[j], ref.y, t[TPM * ks + j]);
            if (j & 1) z1 += x[j];
            else z0 += x[j];
            asm volatile("" : "+v"(t[TPM * ks + j]));
          }
          asm volatile("" : "+v"(z0), "+v"(z1));
          __builtin_amdgcn_sched_barrier(0);
        }
        set_z(rt, before + both_halves<false>(z0 + z1));
      };
      using Y = std::true_type;
      using N = std::false_type;
      step(Y{}, N{}, 0, fin, out);
      step(N{}, N{}, 1, out, fin);
#pragma unroll 1
      for (int rt = 2; rt + 2 < nrt; rt += 2) {
        step(N{}, N{}, rt, fin, out);
        step(N{}, N{}, rt + 1, out, fin);
      }
      step(N{}, N{}, nrt - 2, fin, out);
      step(N{}, Y{}, nrt - 1, out, fin);
    }
    {
      const int ln = fresh(lane), key = wkey + transpose_key(ln);
      const float s = transpose_sum(t, ln);
      if (key < npre && (ln & 1) == 0) raw[key] = s;
    }
    const bool unit_ends = !has_next || nxt.u != cur.u;
    first = unit_ends || nxt.key % kLagKeys == 0;
    if (first) {  // the item's sums
      lds_barrier();
      if (tid < a.R) {
        const float* z8 = s_z + zbuf * kW * a.Rs + tid;
        float z[kW];
#pragma unroll
        for (int w = 0; w < kW; ++w) z[w] = z8[w * a.Rs];
        add_item(a, cur.u, tid, ((z[0] + z[1]) + (z[2] + z[3])) + ((z[4] + z[5]) + (z[6] + z[7])), sum);
      }
      if (a.zbufs == 2) zbuf ^= 1;  // (the table is written again behind the next item's barrier)
      else lds_barrier();
    }
    if (unit_ends) {
      if (tid < a.R) add_sum(a, cur.u, tid, sum);
      sum = 0;
      if (has_next) {  // (every wave is done with the unit's queries: the barrier above)
        stage(nxt);
        lds_barrier();
        prime(kn);
      }
    }
    const bool more = has_next;
    cur = nxt;
    nxt = nx2;
    has_next = has_nx2;
    return more;
  };
  issue_k(cur, b0);
  issue_k(nxt, b1);
  lds_barrier();  // (the first item's place has been read)
  stage(cur);
  lds_barrier();
  prime(b0);
#pragma unroll 1
  for (;;) {
    if (!pass(b0, b1, b2)) break;
    if (!pass(b1, b2, b0)) break;
    if (!pass(b2, b0, b1)) break;
  }
}

// ---- the keys that can be kept ----
// The row's weight 1 / (G z), the other kernel's to the bit; 0 where its sum is not usable.
__device__ __forceinline__ float weight_of(const SiftArgs& a, int u, int row, u64 w) {
  if (__builtin_expect((w & kZLarge) != 0 && (w & kZBad) == 0, 0)) {
    const u64* large = a.zlarge + (size_t)u * 3 * a.Rs + row;
    return __builtin_amdgcn_rcpf(sum_of_words(as_float(w & ~kZLarge), large[0], large[a.Rs], large[2 * a.Rs])) * a.inv_G;
  }
  return (w & kZBad) != 0 || w < 1024ull ? 0.f : __builtin_amdgcn_rcpf(as_float(w)) * (kSumUnits * a.inv_G);
}

__global__ __launch_bounds__(NT, 8) void sift_list_kernel(const SiftArgs a) {
  extern __shared__ uint32_t smem_u[];  // [N / 8] the largest of every four, upper 16 bits | [N / 32] a bit per key
  __shared__ __attribute__((aligned(16))) uint32_t hist[HIST];
  __shared__ uint32_t scan[2 * NW], sel[4];
  __shared__ float s_red[5][NW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int u = blockIdx.x;
  const Unit p = unit_of(a, u);
  if (a.layer[p.l].k_l >= p.n || flags_of(a, p.l, p.b)[p.g] != 0) return;
  const int npre = p.n - a.alpha, kk = a.layer[p.l].k_l - a.alpha;
  const size_t place = (size_t)a.layer[p.l].slot * a.B * a.Hkv + (size_t)p.b * a.Hkv + p.g;
  float* raw = a.raw + place * a.N;
  const int ngroup4 = (npre + 3) / 4, nwords = (npre + 31) / 32;
  uint16_t* gmax = reinterpret_cast<uint16_t*>(smem_u);
  uint32_t* bitmap = smem_u + (a.N + 7) / 8;
  const bool is_avg = a.pool == PKV_POOL_AVG;
  const int r = a.pool == PKV_POOL_NONE ? 0 : (a.pool_w - 1) / 2;
  const float inv_w = 1.f / (float)a.pool_w;
  // no list: the kernel behind the next one scores the head
  auto fail = [&]() {
    if (tid == 0) a.flags[place] = kSiftFailed;
  };

  // rows: the largest and the mean ratio of the weight to its estimate
  const u64 word = tid < a.R ? a.zsum[(size_t)u * a.Rs + tid] : 0ull;
  const float omega = tid < a.R ? a.omega[(size_t)u * a.Rs + tid] : 1.f;
  const float row_window = tid < a.R ? a.window[(size_t)u * a.Rs + tid] : 0.f;
  // the pooled score of the middle one, M scores on each side at hand
  auto pooled_of = [&](const float* x, int at, auto M) __attribute__((always_inline)) {
    float acc = x[at];
#pragma unroll
    for (int o = 1; o <= decltype(M)::value; ++o) {
      if (o > r) break;  // (uniform)
      acc = is_avg ? acc + (x[at - o] + x[at + o]) : fmaxf(acc, fmaxf(x[at - o], x[at + o]));
    }
    return is_avg ? acc * inv_w : acc;
  };
  // the pooled scores of positions q .. q + 3, from the scores around them (P: 4-score pieces on each side)
  auto pooled4 = [&](auto PP, int q) __attribute__((always_inline)) {
    constexpr int P = decltype(PP)::value;
    float x[4 + 8 * P];
    if (q >= 4 * P && q + 4 + 4 * P <= npre) {
#pragma unroll
      for (int i = 0; i < 1 + 2 * P; ++i) {
        const f32x4 v = *reinterpret_cast<const f32x4_u*>(raw + q + 4 * (i - P));
#pragma unroll
        for (int c = 0; c < 4; ++c) x[4 * i + c] = v[c];
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4 + 8 * P; ++i) x[i] = q + i - 4 * P >= 0 && q + i - 4 * P < npre ? raw[q + i - 4 * P] : 0.f;
    }
    f32x4 y;
#pragma unroll
    for (int c = 0; c < 4; ++c) y[c] = P > 0 ? pooled_of(x, 4 * P + c, std::integral_constant<int, 4 * P>{}) : x[c];
    return y;
  };
  reinterpret_cast<uint2*>(hist)[tid] = make_uint2(0u, 0u);
  for (int i = tid; i < nwords; i += NT) bitmap[i] = 0u;
  // ---- A. the largest estimated pooled score of every four neighbours ----
  uint32_t kmax = 0u;
  auto note = [&](int i, const f32x4& y) {
    uint32_t m = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) m = max(m, 4 * i + c < npre ? __float_as_uint(y[c]) : 0u);
    kmax = max(kmax, m);
    gmax[i] = (uint16_t)(m >> 16);
  };
  if (r <= 4) {
    // A wave takes 256 neighbouring groups at a time, lane l those from l on, 64 apart: what lies beside a lane's four scores is
    // with its neighbours, but for the first and the last lane's.  The next 256 are under way.
    auto quad = [&](int q) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (q >= 0 && q + 4 <= npre) v = *reinterpret_cast<const f32x4_u*>(raw + q);
      else if (q >= 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (q + c < npre) v[c] = raw[q + c];
      }
      return v;
    };
    struct Batch {
      f32x4 v[4], e;
    };
    auto load = [&](int g0) {
      Batch x;
#pragma unroll
      for (int j = 0; j < 4; ++j) x.v[j] = quad(4 * (g0 + 64 * j + lane));
      x.e = f32x4{0.f, 0.f, 0.f, 0.f};
      if (r > 0 && (lane == 0 || lane == 63)) x.e = quad(lane == 0 ? 4 * g0 - 4 : 4 * (g0 + 256));
      return x;
    };
#define PKV_DPP(old, src, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src), ctrl, 0xF, 0xF, false))
    auto work = [&](int g0, const Batch& x) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        f32x4 y = x.v[j];
        if (r > 0) {
          float at[12];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const float first = j == 0 ? x.e[c] : PKV_DPP(0.f, x.v[j == 0 ? 0 : j - 1][c], 0x13C);  // wave_ror:1
            const float last = j == 3 ? x.e[c] : PKV_DPP(0.f, x.v[j == 3 ? 3 : j + 1][c], 0x134);   // wave_rol:1
            at[c] = PKV_DPP(first, x.v[j][c], 0x138);     // wave_shr:1
            at[4 + c] = x.v[j][c];
            at[8 + c] = PKV_DPP(last, x.v[j][c], 0x130);  // wave_shl:1
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) y[c] = pooled_of(at, 4 + c, std::integral_constant<int, 4>{});
        }
        if (g0 + 64 * j + lane < ngroup4) note(g0 + 64 * j + lane, y);
      }
    };
#undef PKV_DPP
    Batch one = load(256 * wave), two;
    for (int g0 = 256 * wave; g0 < ngroup4; g0 += 512 * NW) {  // (uniform within the wave)
      two = load(g0 + 256 * NW);
      work(g0, one);
      one = load(g0 + 512 * NW);
      work(g0 + 256 * NW, two);
    }
  } else {
    for (int i = tid; i < ngroup4; i += NT) note(i, pooled4(std::integral_constant<int, 2>{}, 4 * i));
  }
  {
    const float weight = tid < a.R ? weight_of(a, u, tid, word) : 0.f, ratio = weight / omega;
    // (a ratio that is not a number has the largest bits of all; it is seen below)
    const float mx = __int_as_float(__builtin_amdgcn_readlane((int)wave_max_lane63(__float_as_uint(ratio)), 63));
    const float sm = wave_sums(ratio).y, sq = wave_sums(ratio * ratio).y, wn = wave_sums(row_window * weight).y;
    const bool bad = __any(tid < a.R && !(ratio > 0.f && ratio < INFINITY));
    kmax = row_max_lane15(kmax);
    const uint32_t m = min(min((uint32_t)__builtin_amdgcn_readlane((int)kmax, 15), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 31)),
                           min((uint32_t)__builtin_amdgcn_readlane((int)kmax, 47), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 63)));
    if (lane == 0) {
      s_red[0][wave] = mx;
      s_red[1][wave] = sm;
      s_red[2][wave] = bad ? 1.f : 0.f;
      s_red[3][wave] = wn;
      s_red[4][wave] = sq;
      scan[wave] = m;
    }
  }
  __syncthreads();
  float rmax = 1.f, mean = 0.f, square = 0.f, anybad = 0.f, window = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    rmax = fmaxf(rmax, s_red[0][w]);
    mean += s_red[1][w];
    anybad += s_red[2][w];
    window += s_red[3][w];
    square += s_red[4][w];
  }
  auto uniform = [](float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); };
  rmax = uniform(rmax);
  window = uniform(window);
  mean = uniform(mean / (float)a.R);
  const float apart = uniform(__builtin_sqrtf(fmaxf(square / (float)a.R - mean * mean, 0.f)) / mean);
  if (anybad != 0.f) {
    fail();
    return;
  }
  uint32_t total = 0u;
  float bound = 0.f;
  if (kk > 0) {  // (uniform)
    // ---- B. what about kk positions reach, and the estimates down to which a key can be kept then ----
    const KeyBins<HIST> bins{(uint32_t)__builtin_amdgcn_readlane((int)row_max_lane15(scan[lane & 15]), 15)};
    // (those four binades and more below the reference, nearly all, only if the others are not enough)
    const uint32_t low = bins.ref > (4u << 23) ? bins.ref - (4u << 23) : 0u;
    for (int i = tid; i < ngroup4; i += NT) {
      const uint32_t m = (uint32_t)gmax[i] << 16;
      if (m != 0u && m >= low) atomicAdd(&hist[bins.of(m)], 1u);
    }
    __syncthreads();
    // (a pooling window's largest score fills 4 w / (w + 3) places of a group it reaches, on average; whether this was enough
    // is seen at the end)
    const uint32_t want = min((uint32_t)kk, (uint32_t)((float)(kk * (2 * r + 4)) * (kSiftRank / (float)(8 * r + 4))) + 4u);
    if (find_bin(hist, want, scan + NW, sel) < want) {  // (uniform; it leaves the bins cleared)
      for (int i = tid; i < ngroup4; i += NT) {
        const uint32_t m = (uint32_t)gmax[i] << 16;
        if (m != 0u) atomicAdd(&hist[bins.of(m)], 1u);
      }
      __syncthreads();
      if (find_bin(hist, want, scan + NW, sel) < want) {
        fail();
        return;
      }
    }
    const float edge = __uint_as_float(bins.lower_edge(__builtin_amdgcn_readfirstlane(sel[0])));
    // (less where the ratios lie apart, as far as there is room for what is listed then: about four keys per group)
    float slack = kSiftSlack;
    for (float less = fminf(kSiftApart * fmaxf(apart - kSiftApartFrom, 0.f), 4.f); less > 0.f; less = less > 0.25f ? less * (1.f / 3.f) : 0.f) {
      const float lower = kSiftSlack * fast_exp2(-less);
      const uint32_t low16 = __float_as_uint(edge * fminf(1.f, lower * mean / rmax)) >> 16;
      uint32_t cnt = 0u, groups;
      for (int i = tid; i < ngroup4; i += NT) cnt += gmax[i] >= low16 ? 1u : 0u;
      cnt = wave_inclusive_sum(cnt);
      if (lane == 63) scan[wave] = cnt;
      __syncthreads();
      (void)sum_before(scan, wave, groups);
      __syncthreads();
      if (4u * groups <= (uint32_t)sift_list(a.N)) {  // (uniform)
        slack = lower;
        break;
      }
    }
    const float tau = edge * fminf(1.f, slack * mean / rmax);
    bound = tau * rmax * (1.f + 0x1p-9f);
    if (!(tau > 0x1p-60f) || !(bound < 0x1p100f)) {
      fail();
      return;
    }
    // ---- C. the positions whose scores can matter: the windows of the pooled scores from tau on ----
    const uint32_t tau16 = __float_as_uint(tau) >> 16;
    uint16_t* hit = reinterpret_cast<uint16_t*>(hist);  // groups that reach it, in any order
    if (tid == 0) sel[3] = 0u;
    __syncthreads();
    for (int i = tid; i < ngroup4; i += NT)
      if (gmax[i] >= tau16) {
        const uint32_t at = atomicAdd(&sel[3], 1u);
        if (at < 2u * HIST) hit[at] = (uint16_t)i;
      }
    __syncthreads();
    const int hits = (int)sel[3];
    if (hits > 2 * HIST) {
      fail();
      return;
    }
    for (int h = tid; h < hits; h += NT) {
      const int q = 4 * (int)hit[h];
      // from the first to the last of the four that reaches it (max: by its own score)
      const f32x4 y = !is_avg || r == 0 ? pooled4(std::integral_constant<int, 0>{}, q) : r <= 4 ? pooled4(std::integral_constant<int, 1>{}, q) : pooled4(std::integral_constant<int, 2>{}, q);
      int first = 4, last = -1;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (q + c < npre && __float_as_uint(y[c]) >> 16 >= tau16) {
          first = min(first, c);
          last = c;
        }
      if (last < 0) continue;  // (its window's largest lies in another group)
      const int lo = q + first - r;
      int hi = q + last + 1 + r;
      hi = min(hi, npre);
      for (int x = max(lo, 0); x < hi;) {
        const int e = min((x | 31) + 1, hi);
        atomicOr(&bitmap[x >> 5], (e - x == 32 ? 0xFFFFFFFFu : ((1u << (e - x)) - 1u)) << (x & 31));
        x = e;
      }
    }
    __syncthreads();
    uint32_t bits[kSiftMaxKeys / 32 / NT], cnt = 0u;
#pragma unroll
    for (int j = 0; j < kSiftMaxKeys / 32 / NT; ++j) {
      const int w = tid * (kSiftMaxKeys / 32 / NT) + j;
      bits[j] = w < nwords ? bitmap[w] : 0u;
      cnt += (uint32_t)__popc(bits[j]);
    }
    const uint32_t incl = wave_inclusive_sum(cnt);
    if (lane == 63) scan[wave] = incl;
    __syncthreads();
    uint32_t at = sum_before(scan, wave, total) + incl - cnt;
    if (total > (uint32_t)sift_list(a.N)) {
      fail();
      return;
    }
    uint32_t* list = a.list + (size_t)u * sift_list(a.N);
#pragma unroll
    for (int j = 0; j < kSiftMaxKeys / 32 / NT; ++j)
      for (uint32_t b = bits[j]; b != 0u; b &= b - 1u) list[at++] = 32u * (uint32_t)(tid * (kSiftMaxKeys / 32 / NT) + j) + (uint32_t)__ffs((int)b) - 1u;
  }
  if (kk == 0) {
    for (int t = tid; t < a.alpha; t += NT) a.layer[p.l].idx[((size_t)p.b * a.Hkv + p.g) * a.alpha + t] = npre + t;
  }
  if (tid == 0) {
    a.total[u] = (int)total;
    a.bound[u] = bound;
    raw[npre] = (float)a.alpha - window;  // the attention to the prefix, behind the scores: for the recall of the kept set
  }
}

// ---- their exact scores ----
// Workgroup x takes the parts x / units, x / units + kSiftParts, ... of unit x % units.
template <int D>
__global__ __launch_bounds__(kT, 4) void sift_exact_kernel(const SiftArgs a, int units) {
  constexpr int KS = D / 16;
  using QB = RowBlock<D, kBlockRows>;
  static_assert(kSiftJob == 32 * kW, "a tile per wave");
  constexpr int kView = 4 * kT, kEdge = 32;  // keys of the list that are looked at at a time, and around them
  constexpr int kReach = 6144;               // places that reach the bound, at most
  constexpr int kWords = 2 * (kView + 2 * kEdge) + 2 * kReach;
  constexpr int kSlots = 2 * QB::SLOTS > kWords / 4 ? 2 * QB::SLOTS : kWords / 4;
  static_assert(kSiftMaxPoolW <= 17, "eight keys on each side");
  static_assert(kWords % 4 == 0 && kEdge % 4 == 0 && kSlots * 16 + 6 * 1024 <= 80 * 1024, "two workgroups per compute unit");
  __shared__ u32x4 s_q[kSlots];
  __shared__ float2 s_r[kResidentMaxRows];  // minus the reference, weight
  __shared__ uint32_t s_scan[2 * kW], s_sel[4];
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part0 = blockIdx.x / units, u = blockIdx.x - part0 * units;
  const uint32_t* list = a.list + (size_t)u * sift_list(a.N);
  uint32_t q = list[min(part0 * kSiftJob + 32 * wave + l32, sift_list(a.N) - 1)];  // (not one of the list's, perhaps)
  const int total = a.total[u];
  const float bound = a.bound[u];
  if (part0 * kSiftJob >= total) return;
  const Unit p = unit_of(a, u);
  const int npre = p.n - a.alpha, kk = a.layer[p.l].k_l - a.alpha;
  const size_t place = (size_t)a.layer[p.l].slot * a.B * a.Hkv + (size_t)p.b * a.Hkv + p.g;
  float* raw = a.raw + place * a.N;
  const uint16_t* Q = queries_of(a, p);
  const uint16_t* K = keys_of(a, p);
  const int jobs = (total + kSiftJob - 1) / kSiftJob;
  QB qb;
  auto row_at = [&](int row) { return query_row_of(a, Q, row); };
  if (tid < a.Rs) {
    const float m = reinterpret_cast<const float*>(a.words + (size_t)u * a.groups * (kLagGroupBytes / 8))[lag_half_word(kLagRefs, tid)];
    s_r[tid] = make_float2(-m, tid < a.R ? weight_of(a, u, tid, a.zsum[(size_t)u * a.Rs + tid]) : 0.f);
  }
#pragma unroll 1
  for (int part = part0; part < jobs; part += kSiftParts) {
    qb.request(0, row_at);
    const int e = part * kSiftJob + 32 * wave + l32;
    const bool mine = part * kSiftJob + 32 * wave < total;  // (uniform within the wave)
    if (part != part0) q = list[min(e, total - 1)];
    const int pos = e < total ? (int)q : 0;
    bf16x8 kf[KS];
    load_rows(kf, K + (size_t)pos * a.kv_st, hf);
    f32x16 t = {};
    int buf = 0;
#pragma unroll 1
    for (int row0 = 0; row0 < a.Rs; row0 += kBlockRows, buf ^= 1) {
      const int ntile = min(kBlockTiles, (a.Rs - row0) / 32);
      qb.commit(s_q + buf * QB::SLOTS);
      __syncthreads();
      if (row0 + kBlockRows < a.Rs) qb.request(row0 + kBlockRows, row_at);
      if (mine) {
        // (products, exponentials and sums as in the kernel that scores every key, so that the scores are its to the bit)
#pragma unroll 1
        for (int rt = 0; rt < ntile; ++rt) {
          const f32x16 x = product(kf, s_q + buf * QB::SLOTS, 32 * rt + l32, hf);
          const float2 ref = s_r[row0 + 32 * rt + l32];
#pragma unroll
          for (int v = 0; v < 16; ++v) t[v] = __builtin_fmaf(fast_exp2(__builtin_fmaf(x[v], a.kappa, ref.x)), ref.y, t[v]);
        }
      }
    }
    const float s = transpose_sum(t, lane);
    const int es = part * kSiftJob + 32 * wave + transpose_key(lane);
    const int ps = __shfl(pos, transpose_key(lane));
    if ((lane & 1) == 0 && es < total)  // (another workgroup may look at it before the kernel ends)
      __hip_atomic_store(raw + ps, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_s_waitcnt(0);  // the scores are on their way no more when the job counts as done
    __syncthreads();
    if (tid == 0) s_last = __hip_atomic_fetch_add(a.done + u, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == jobs - 1 ? 1 : 0;
    __syncthreads();
    if (s_last == 0) continue;
    // ---- the unit's last job: the places whose pooled score reaches the bound, in order.  If they are enough, the kept ones
    // are among them, and nothing outside the list is ----
    uint32_t* lpos = reinterpret_cast<uint32_t*>(s_q) + kEdge;  // [-kEdge, kView + kEdge)
    float* exact = reinterpret_cast<float*>(lpos + kView + 2 * kEdge);
    uint32_t* qpos = reinterpret_cast<uint32_t*>(s_q) + 2 * (kView + 2 * kEdge);
    uint32_t* qkey = qpos + kReach;
    const bool is_avg = a.pool == PKV_POOL_AVG;
    const int r = a.pool == PKV_POOL_NONE ? 0 : (a.pool_w - 1) / 2;
    const float inv_w = 1.f / (float)a.pool_w;
    // sums over the threads before a thread and over all of them (x: the thread's, ends with the scratch free)
    auto scan = [&](uint32_t x, uint32_t& total) {
      const uint32_t incl = wave_inclusive_sum(x);
      if (lane == 63) s_scan[wave] = incl;
      lds_barrier();
      uint32_t before = incl - x;
      total = 0u;
#pragma unroll
      for (int w = 0; w < kW; ++w) {
        before += w < wave ? s_scan[w] : 0u;
        total += s_scan[w];
      }
      lds_barrier();
      return before;
    };
    uint32_t reach = 0u;
    bool odd = false;
#pragma unroll 1
    for (int i0 = 0; i0 < total; i0 += kView) {
      for (int i = tid - kEdge; i < kView + kEdge; i += kT) {  // (what is not there lies far away)
        const bool there = i0 + i >= 0 && i0 + i < total;
        const uint32_t at = there ? list[i0 + i] : i < 0 ? 0u - 1024u : 1u << 30;
        float y = 0.f;
        if (there) y = __hip_atomic_load(raw + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        lpos[i] = at;
        exact[i] = y;
        odd = odd || !(y < INFINITY);
      }
      lds_barrier();
      // a thread takes four neighbours and what is listed around them
      int P[20];
      float E[20];
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(lpos + 4 * tid - 8 + 4 * i);
        const f32x4 y = *reinterpret_cast<const f32x4*>(exact + 4 * tid - 8 + 4 * i);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          P[4 * i + c] = (int)x[c];
          E[4 * i + c] = y[c];
        }
      }
      uint32_t key[4], mine4 = 0u;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int at = P[8 + c];
        float y = is_avg ? 0.f : E[8 + c];
        int found = 0;
#pragma unroll
        for (int d = -8; d <= 8; ++d) {
          if (d < -r || d > r) continue;  // (uniform)
          const int o = P[8 + c + d] - at;
          const bool in = o >= -r && o <= r;
          found += in ? 1 : 0;
          y = is_avg ? y + (in ? E[8 + c + d] : 0.f) : in ? fmaxf(y, E[8 + c + d]) : y;
        }
        y = is_avg ? y * inv_w : y;
        const bool whole = !is_avg || found == min(r, at) + min(r, npre - 1 - at) + 1;  // (else the window is not listed whole)
        key[c] = i0 + 4 * tid + c < total && whole && y >= bound ? __float_as_uint(y) : 0u;
        mine4 += key[c] != 0u ? 1u : 0u;
      }
      uint32_t all;
      uint32_t to = reach + scan(mine4, all);
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (key[c] != 0u) {
          if (to < (uint32_t)kReach) {
            qpos[to] = (uint32_t)P[8 + c];
            qkey[to] = key[c];
          }
          ++to;
        }
      reach += all;
      lds_barrier();
    }
    if (__any(odd) && lane == 0) s_scan[kW + wave] = 1u;
    else if (lane == 0) s_scan[kW + wave] = 0u;
    lds_barrier();
    uint32_t bad = reach < (uint32_t)kk || reach > (uint32_t)kReach ? 1u : 0u;
#pragma unroll
    for (int w = 0; w < kW; ++w) bad |= s_scan[kW + w];
    if (bad != 0u) {
      if (tid == 0) a.flags[place] = kSiftFailed;
      return;  // (no part of the unit is left)
    }
    // ---- the kk-th largest of them: bins of equal width between the smallest and the largest, as long as more than 64 are in its bin ----
    uint32_t* hist = reinterpret_cast<uint32_t*>(s_q);  // [1024] (the list is done with)
    uint32_t lo = __float_as_uint(bound), hi = 0u, need = (uint32_t)kk, open = reach;
    for (uint32_t i = tid; i < reach; i += kT) hi = max(hi, qkey[i]);
    hi = (uint32_t)__builtin_amdgcn_readlane((int)wave_max_lane63(hi), 63);
    if (lane == 0) s_scan[wave] = hi;
    lds_barrier();
#pragma unroll
    for (int w = 0; w < kW; ++w) hi = max(hi, s_scan[w]);
    lds_barrier();
    while (need != open && open > 64u && lo != hi) {
      const int bits = 32 - __clz((int)(hi - lo)), sh = bits > 10 ? bits - 10 : 0;
      reinterpret_cast<uint2*>(hist)[tid] = make_uint2(0u, 0u);
      lds_barrier();
      for (uint32_t i = tid; i < reach; i += kT)
        if (qkey[i] >= lo && qkey[i] <= hi) atomicAdd(&hist[(hi - qkey[i]) >> sh], 1u);
      lds_barrier();
      const uint2 h = reinterpret_cast<uint2*>(hist)[tid];
      uint32_t all;
      const uint32_t before = scan(h.x + h.y, all);
      const bool in0 = before < need && before + h.x >= need, in1 = before + h.x < need && before + h.x + h.y >= need;
      if (in0 || in1) {
        s_sel[0] = (uint32_t)(2 * tid + (in1 ? 1 : 0));
        s_sel[1] = in1 ? before + h.x : before;
        s_sel[2] = in1 ? h.y : h.x;
      }
      lds_barrier();
      need -= s_sel[1];
      open = s_sel[2];
      hi -= s_sel[0] << sh;
      if (((hi - lo) >> sh) != 0u) lo = hi - (1u << sh) + 1u;
      lds_barrier();
    }
    uint32_t T = need == open ? lo - 1u : lo;  // (all of the bin are kept, or all are equal)
    if (need != open && lo != hi) {
      if (tid == 0) s_sel[3] = 0u;
      lds_barrier();
      for (uint32_t i = tid; i < reach; i += kT)
        if (qkey[i] >= lo && qkey[i] <= hi) hist[atomicAdd(&s_sel[3], 1u)] = qkey[i];
      lds_barrier();
      if (wave == 0) {
        const uint32_t d = lane < (int)open ? hist[lane] : 0u;
        uint32_t above = 0u, from = 0u;
        for (int j = 0; j < (int)open; ++j) {
          const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)d, j);
          above += x > d ? 1u : 0u;
          from += x >= d ? 1u : 0u;
        }
        if (lane < (int)open && above < need && need <= from) s_sel[0] = d;
      }
      lds_barrier();
      T = s_sel[0];
    }
    // ---- the kept positions in order, equal ones the lowest first; behind them the window ----
    int32_t* idx = a.layer[p.l].idx + ((size_t)p.b * a.Hkv + p.g) * (size_t)(kk + a.alpha);
    const uint32_t run = (reach + kT - 1) / kT, i0 = min(tid * run, reach), i1 = min(i0 + run, reach);
    uint32_t gt = 0u, eq = 0u, all_gt, all_eq;
    for (uint32_t i = i0; i < i1; ++i) {
      gt += qkey[i] > T ? 1u : 0u;
      eq += qkey[i] == T ? 1u : 0u;
    }
    gt = scan(gt, all_gt);
    eq = scan(eq, all_eq);
    const uint32_t need_eq = (uint32_t)kk - all_gt;
    for (uint32_t i = i0; i < i1; ++i) {
      if (qkey[i] > T) {
        idx[gt + min(eq, need_eq)] = (int)qpos[i];
        ++gt;
      } else if (qkey[i] == T) {
        if (eq < need_eq) idx[gt + eq] = (int)qpos[i];
        ++eq;
      }
    }
    for (int t = tid; t < a.alpha; t += kT) idx[kk + t] = npre + t;
    return;
  }
}

template <int D>
hipError_t launch_sift(const SiftArgs& a, bool clear_err, hipStream_t s) {
  static bool attr_set[kMaxDevices];
  constexpr size_t list_lds = (size_t)(kSiftMaxKeys + kMaxAlpha) / 2 + kSiftMaxKeys / 8 + 64;
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {  // raise the dynamic LDS limits once per device (idempotent; no allocation)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(score_sift_few_kernel<D>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)FewRows<D>::kLds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(score_sift_many_kernel<D>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)sift_lds<D>(kResidentMaxRows));
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(sift_list_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)list_lds);
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  const int units = a.L * a.B * a.Hkv;
  hipLaunchKernelGGL((sift_prepare_kernel<D>), dim3(units * ((a.Rs + kBlockRows - 1) / kBlockRows)), dim3(kT), 0, s, a, clear_err ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.Rs == FewRows<D>::ROWS) hipLaunchKernelGGL((score_sift_few_kernel<D>), dim3(a.grid), dim3(kT), FewRows<D>::kLds, s, a);
  else hipLaunchKernelGGL((score_sift_many_kernel<D>), dim3(a.grid), dim3(kT), sift_lds<D>(a.Rs), s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t lds = (size_t)((a.N + 7) / 8 + (a.N + 31) / 32) * 4;
  hipLaunchKernelGGL(sift_list_kernel, dim3(units), dim3(NT), lds, s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sift_exact_kernel<D>), dim3(units * kSiftParts), dim3(kT), 0, s, a, units);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_sift(const SiftArgs& a, bool clear_err, hipStream_t s) {
  if (a.d == 128) return launch_sift<128>(a, clear_err, s);
  if (a.d == 64) return launch_sift<64>(a, clear_err, s);
  return hipErrorInvalidValue;
}

}  // namespace pkv
