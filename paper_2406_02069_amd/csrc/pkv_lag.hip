// Window scoring in one pass over K for 33 .. 512 query rows per KV head (G * alpha; Sec. 4.2.2, Eq. Al and Eq. att_score) on
// MI355X: the probabilities wait on the chip for the normalisers, 64 rows at a time.
//
// The score of a key needs the softmax normaliser of every window query, which is known only after all keys of the head have
// been seen.  The kernels that keep the keys, or read them twice, form every product and every exponential twice.  Here the
// un-normalised probabilities p = exp2(kappa q.k - m) (m: a reference exponent of the row, the same for all keys of the unit)
// are what waits:  s_i = (1 / G) sum_r p_ri / z_r,  z_r = sum_i p_ri.  That is one multiply-add per logit; K is read and
// multiplied once.
//
// Work split.  An item is 512 keys of one unit (layer, sequence, KV head).  256 persistent workgroups of 512 threads, one per
// compute unit (all of its LDS, 256 registers per lane), take the items in turn, item j workgroup j % 256.  A wave holds its 64
// keys as matrix operands through all groups of 64 rows of the item: a step is one group.  What waits does not grow with the
// rows, so that 512 rows are scored like 64: with all rows of an item at once p of 128 rows x 512 keys would take what
// registers and LDS hold together, and one of 256 keys starts as many exchanges for half the products.
//
// Per step a workgroup multiplies its keys with the group's queries (product rows = keys, columns = queries, so that a lane owns
// a query and its sum is a plain one), turns the logits into p, and puts them in the place of the p of two steps before (in
// registers and in LDS in turn), which are weighted with 1 / (G z) and summed over the rows on the way.  Behind the item's last
// group the sums go over the lanes once.
//
// The exchange.  References are common to a unit, so the items' sums can be added in memory: as integers (the order does not
// show), with the number of items that have been added in the same word.  One atomic add per row and item, one load per row a
// step later; nobody folds, and nothing but 2 KB per unit and group has to be cleared.  Among 128 workgroups beside a stream of
// keys this takes half the time of storing the sums, folding and storing the normalisers (3.3 against 5.4 us per round with one
// round's slack, 2.7 against 3.8 with two).
//
// A sum beyond 2^103 times its reference (2^73 in units of less than 640 keys per group of rows; or undefined) does not fit:
// the unit is scored again at the launch's end, from memory and with exact maxima, which is slow.
//
// What bounds it: at 64 rows HBM (32 layers of 32k keys 599 -> 487 us whole call, against the one-pass kernel that waits for an
// exchange of all items' statistics), beyond them no pipe alone: at 128 rows a step takes 11 350 clk (5.1 us), in which vector
// instructions issue for 4 570, the LDS is busy for 2 350 and the matrix pipe for 2 050, one after the other for the most part
// with two waves per SIMD, and waves wait for 43 % of the time; its keys alone take 2.8 us from HBM.  128 rows, 32 layers of
// 32k keys 773 -> 672 us, 512 rows, 80 layers 5435 -> 4385, against the kernels that form everything twice.
//
// Every wait is bounded by wall-clock time (a workgroup that has waited too long raises the error word and carries on), so the
// grid always drains.
#include <type_traits>

#include "pkv_internal.h"
#include "pkv_tile.h"

namespace pkv {
namespace {

constexpr int kW = 8;  // waves per workgroup
constexpr int kT = kW * 64;

__device__ __forceinline__ u64 ld64(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t ld32(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void add64(u64* p, u64 v) { (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Words of a unit in the workspace, 256 bytes for eight rows: their sums, two further words each for large sums, references
// (floats) and exact maxima (ordered integers).  (An exchange among 128 workgroups takes 2.3 us with eight rows' sums to 256
// bytes and 4.3 us with the sums in one piece: the adds to a memory channel come one after the other.)  A third word for large
// sums per row lies behind the words of all units, where there is room for it (from 640 keys per group of 64 rows on).
// A sum is a 64-bit integer that the items add to: bits 0 .. 51 the sum of p in units of 2^-30 (2^-34 at the second
// attempt, which uses the first word for large sums), bits 52 .. 61 the items that have been added (in the group's first row
// also those whose maxima are in), bit 62 an item whose sum does not fit, bit 63 one that is counted in a word for large sums: up
// to 2^13, 2^43, 2^73 and 2^103, in units 2^-24 of what the word before holds.  That is rare but has to cost little.  A key
// far above the sampled ones for every row of every unit, 32 layers of 32k keys, 128 rows: 660 us without, 739 with one 20 binades
// above, 774 at 55 (10 100 where the unit is scored again); 8 layers, 512 rows: 540, 633 and 654 (10 250).  What remains is one
// read of these words per step, for which everything under way is waited for.
// (One key alone adds 1 to a row's sum, so half a unit of each of 256 items is at most 2^-23 of it: as much as two roundings of
// a float.  In units of 2^-24 the sums of items far below the reference were lost: 64 items of 2^-26 each 9.5e-7 of the
// normaliser, 256 items 3.8e-6.)
constexpr int kSums = 0, kSums2 = 8, kSums3 = 16, kRefs = kLagRefs, kMax = kLagMax;  // places in a block, in 64-bit words
__device__ __forceinline__ uint32_t word_of(int which, int row) { return (uint32_t)(which + (row >> 3) * 32 + (row & 7)); }
__device__ __forceinline__ uint32_t half_word_of(int which, int row) { return lag_half_word(which, row); }
constexpr u64 kOne = 1ull << 52, kBad = 1ull << 62, kBig = 1ull << 63;
constexpr float kUnits = kSumUnits, kUnits2 = kSumUnits2, kUnits3 = kSumUnits3, kUnits4 = kSumUnits4;
constexpr float kLimit = kSumLimit, kLimit2 = kSumLimit2, kLimit3 = kSumLimit3, kLimit4 = kSumLimit4;

// An item's sum of a row, at the first and at the second attempt.  What does not fit is marked first, so that whoever finds
// the item counted sees it.  word4(): the row's last word for large sums, or null.
template <class F>
__device__ __forceinline__ void add_sum(u64* word, float z, F word4) {
  u64 add = kOne;
  if (__builtin_expect(!(z <= kLimit), 0)) {
    u64* big = z <= kLimit2 ? word + (kSums2 - kSums) : z <= kLimit3 ? word + (kSums3 - kSums) : z <= kLimit4 ? word4() : nullptr;
    u64 seen = 0;
    if (big) seen = __hip_atomic_fetch_add(big, fixed_point(z, z <= kLimit2 ? kUnits2 : z <= kLimit3 ? kUnits3 : kUnits4), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" : "+v"(seen));
    seen = __hip_atomic_fetch_or(word, big ? kBig : kBad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" : "+v"(seen));
  } else {
    add += fixed_point(z, kUnits);
  }
  add64(word, add);
}
__device__ __forceinline__ void add_sum_again(u64* word, float z) {
  u64 add = kOne;
  if (z <= 0x1p10f) {
    add += fixed_point(z, 0x1p34f);
  } else {
    u64 seen = __hip_atomic_fetch_or(word, kBad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" : "+v"(seen));
  }
  add64(word, add);
}
// sum, and 1 / sum, times scale
__device__ __forceinline__ float sum_of(u64 w) { return as_float(w & (kOne - 1)); }
__device__ __forceinline__ float inverse(u64 w, float scale) { return __builtin_amdgcn_rcpf(sum_of(w)) * scale; }

// A step handles 64 query rows (a group: two row tiles) of an item's 512 keys (two key tiles per wave).
template <int D>
struct LagShape {
  static constexpr int KS = D / 16, SEG = D / 8, ROWS = 64, KI = 32 * kW * 2;
  static constexpr int PITCH = SEG + 1;  // of Q in LDS, in 16-byte slots (bank-free); the last one holds the row's reference
  static constexpr int PQ = 15;          // 16-byte slots per lane of a group that waits in LDS (of 16, one does not fit)
  static constexpr int P_SLOTS = kW * PQ * 64, Q_SLOTS = ROWS * PITCH;
  static constexpr int NQ = ROWS * SEG / kT;  // 16-byte loads per thread for a group's queries
  static constexpr size_t LDS = (size_t)(P_SLOTS + 2 * Q_SLOTS) * 16 + (size_t)2 * kW * ROWS * 4 + (size_t)kLagItems * 8 + 8;
  static_assert(LDS <= 160 * 1024, "one workgroup per compute unit");
  static_assert((size_t)P_SLOTS * 16 >= (size_t)(kStreamUnits + 1 + kW) * 4, "prefix table fits");
};

// MODE: groups of 64 rows per item: 1, 2, 3 (any odd number from there on) or 4 (any even number).
template <int D, int MODE>
__global__ __launch_bounds__(kT, 2) void score_lag_kernel(const LagArgs a) {
  using S = LagShape<D>;
  constexpr int KS = S::KS, SEG = S::SEG, ROWS = S::ROWS, KI = S::KI, NQ = S::NQ, PQ = S::PQ, PITCH = S::PITCH;
  constexpr int TPM = 16 / KS;  // logits per lane handled between two matrix instructions
  extern __shared__ u32x4 smem[];
  u32x4* s_q = smem + S::P_SLOTS;                                 // [2][ROWS][PITCH] queries of a group, used in turn
  float* s_z = reinterpret_cast<float*>(s_q + 2 * S::Q_SLOTS);    // [2][kW][ROWS] sums by wave, used in turn
  uint2* s_item = reinterpret_cast<uint2*>(s_z + 2 * kW * ROWS);  // [kLagItems] (unit, part << 20 | keys)
  u64** s_words4 = reinterpret_cast<u64**>(s_item + kLagItems);   // a.words4 (kept in a register it would cost the loop one)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int BH = a.B * a.Hkv, NG = MODE < 3 ? MODE : a.groups;
  const uint32_t unit_words = (uint32_t)NG * (ROWS / 8 * 32);  // of 64 bits
  // head and window position of a unit's row
  auto head_of = [&](int row) { return (int)(__umul24((uint32_t)row, a.alpha_magic) >> 16); };

  if (tid == 0) *s_words4 = a.words4;
  // ---- the items of this workgroup ----
  int nmine;
  if (a.uniform) {  // every unit has N keys to score
    const int total = a.L * BH * a.parts;
    nmine = min((total - (int)blockIdx.x + kStreamGrid - 1) / kStreamGrid, kLagItems);
    if (tid < nmine) {
      const int j = tid * kStreamGrid + (int)blockIdx.x, u = j / a.parts;
      s_item[tid] = make_uint2((uint32_t)u, (uint32_t)(j - u * a.parts) << 20 | (uint32_t)a.N);
    }
    __syncthreads();
  } else {
    // A round is one item per workgroup.  Units that may lie in two rounds are dealt one after the other; behind them each
    // sequence of others starts a round of its own, as many units to a round as fit.  Heads that are scored take no part.  (All of them one after the other, 4
    // sequences of 0.8 .. 1 of 64k keys x 2 layers: 96 rows 497 -> 432 us, 128 rows 500 -> 446, 256 rows 680 -> 586.)
    int* pre = reinterpret_cast<int*>(smem);  // [E + 1] before (layer, sequence) e: items of the former, rounds of the latter << 20
    const int E = a.L * a.B;
    int* wsum = pre + kStreamUnits + 1;
    auto flags_of = [&](int e) {
      const int l = e / a.B;
      return a.flags + ((size_t)a.layer[l].slot * a.B + (e - l * a.B)) * a.Hkv;
    };
    auto heads = [&](int e) { return a.flags ? sift_heads<true>(flags_of(e), a.Hkv, kSiftLeft) : a.Hkv; };
    auto length = [&](int b) {
      int n = a.N;
      if (a.seq_lens) {
        n = a.seq_lens[b];
        n = n < 0 ? 0 : (n > a.N ? a.N : n);
      }
      return n;
    };
    int run = 0;
    for (int e0 = 0; e0 < E; e0 += kT) {
      const int e = e0 + tid;
      int c = 0;
      if (e < E) {
        const int l = e / a.B, n = length(e - l * a.B), parts = (n + KI - 1) / KI;
        if (a.layer[l].k_l < n) {  // (whole sequence kept: no scores needed)
          const int left = heads(e);
          if (lag_unit_straddles(parts, MODE)) c = left * parts;
          else {
            const int q = kStreamGrid / parts;  // (the host admits no unit of more items than workgroups)
            c = ((left + q - 1) / q) << 20;
          }
        }
      }
      int v = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(v, o);
        if (lane >= o) v += x;
      }
      __syncthreads();
      if (lane == 63) wsum[wave] = v;
      __syncthreads();
      int before = run;
#pragma unroll
      for (int w = 0; w < kW; ++w) {
        before += w < wave ? wsum[w] : 0;
        run += wsum[w];
      }
      if (e < E) pre[e] = before + v - c;
    }
    if (tid == 0) pre[E] = run;
    __syncthreads();
    const int shorts = run & 0xFFFFF, rounds0 = (shorts + kStreamGrid - 1) / kStreamGrid, rounds = rounds0 + (run >> 20);
    uint2 it = make_uint2(0u, 0u);
    bool mine = false;
    if (tid < min(rounds, kLagItems)) {  // (the host admits only launches that fit)
      const int w = (int)blockIdx.x;
      const bool is_short = tid < rounds0;
      const int shift = is_short ? 0 : 20, j = is_short ? tid * kStreamGrid + w : tid - rounds0;
      auto at = [&](int e) { return (pre[e] >> shift) & (is_short ? 0xFFFFF : 0xFFF); };
      if (!is_short || j < shorts) {
        int lo = 0, hi = E;  // at(lo) <= j < at(hi)
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (at(mid) <= j) lo = mid;
          else hi = mid;
        }
        const int rem = j - at(lo), n = length(lo % a.B), parts = (n + KI - 1) / KI;
        const int at_unit = is_short ? rem : w, k = at_unit / parts, left = heads(lo);
        int g = k;
        mine = true;
        if (!is_short) {
          const int q = kStreamGrid / parts;
          g += rem * q;
          mine = k < q && g < left;
        }
        if (mine && left < a.Hkv) g = sift_head<true>(flags_of(lo), a.Hkv, kSiftLeft, g);
        it = make_uint2((uint32_t)(lo * a.Hkv + g), (uint32_t)(at_unit - k * parts) << 20 | (uint32_t)n);
      }
    }
    const u64 held = __ballot(mine);
    if (lane == 0) wsum[wave] = __popcll(held);
    __syncthreads();
    int at = __popcll(held & ((1ull << lane) - 1ull));
    nmine = 0;
#pragma unroll
    for (int w = 0; w < kW; ++w) {
      at += w < wave ? wsum[w] : 0;
      nmine += wsum[w];
    }
    if (mine) s_item[at] = it;
    __syncthreads();
  }
  if (nmine == 0) return;

  // One item as this workgroup sees it (all fields wave-uniform).
  struct Item {
    int u, part, n;
    const uint16_t* Q;
    const uint16_t* K;
    float* raw;
  };
  auto item = [&](int i) {
    const uint2 e = s_item[i];
    Item d;
    d.u = __builtin_amdgcn_readfirstlane((int)e.x) & 0x7FFFFFFF;
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.y);
    d.part = (int)(w >> 20);
    d.n = (int)(w & 0xFFFFFu);
    const int l = (int)(((u64)(uint32_t)(d.u + 1) * a.bh_magic) >> 32), bg = d.u - l * BH;
    const int b = (int)(((u64)(uint32_t)(bg + 1) * a.hkv_magic) >> 32), g = bg - b * a.Hkv;
    d.Q = a.layer[l].Q + (size_t)b * a.q_sb + (size_t)(g * a.G) * a.q_sh;
    d.K = a.layer[l].K + (size_t)b * a.kv_sb + (size_t)g * a.kv_sh;
    d.raw = a.raw + (size_t)(a.layer[l].slot * BH + bg) * a.N;
    return d;
  };
  auto tile_key = [&](const Item& d, int t) { return d.part * KI + (t * kW + wave) * 32; };
  auto nparts = [&](const Item& d) { return a.uniform ? a.parts : (d.n + KI - 1) / KI; };

  // Keys of the wave's tile t as matrix operand: lane (row l32, half hf) holds elements 16 ks + 8 hf of its key.  Keys at
  // or beyond n are replaced by the last one.
  bf16x8 kf[2][KS];
  auto issue_k = [&](const Item& d, int t, bf16x8 (&f)[KS]) {
    const int ln = fresh(lane);
    const uint32_t key = (uint32_t)min(tile_key(d, t) + (ln & 31), d.n - 1);
    const char* rowp = reinterpret_cast<const char*>(d.K) + (key * ((uint32_t)a.kv_st * 2u) + 16u * (uint32_t)(ln >> 5));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = as_frag(*reinterpret_cast<const u32x4*>(rowp + 32 * ks));
    __builtin_amdgcn_sched_barrier(0);
  };
  // Queries and references of a group: requested into registers, written to LDS later.
  u32x4 qv[NQ];
  float mv;
  constexpr int RPT = kT / SEG;  // rows between a thread's loads
  auto request_q = [&](const Item& d, int h) {
    const uint32_t td = (uint32_t)fresh(tid);
    mv = reinterpret_cast<const float*>(a.words + (size_t)d.u * unit_words)[half_word_of(kRefs, 64 * h + (td & (ROWS - 1)))];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int row = min(64 * h + (int)(td / SEG) + i * RPT, a.R - 1);  // (rows behind the last repeat it; their weights are zero)
      const int hh = head_of(row), t = row - __umul24(hh, a.alpha);
      const uint32_t off = (__umul24(hh, (int)a.q_sh) + __umul24(t, (int)a.q_st)) * 2u + 16u * (td % SEG);
      qv[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(d.Q) + off);
    }
  };
  auto commit_q = [&](int buf) {
    const uint32_t td = (uint32_t)fresh(tid);
    u32x4* q = s_q + buf * S::Q_SLOTS + td / SEG * PITCH + td % SEG;
#pragma unroll
    for (int i = 0; i < NQ; ++i) q[i * RPT * PITCH] = qv[i];
    if (td < (uint32_t)ROWS) *reinterpret_cast<float*>(s_q + buf * S::Q_SLOTS + td * PITCH + SEG) = mv;
  };
  const u32x4* q_lane = s_q + l32 * PITCH + hf;
  auto q_frag = [&](int buf, int rt, int ks) { return as_frag(q_lane[buf * S::Q_SLOTS + 32 * rt * PITCH + 2 * ks]); };
  auto ref_of = [&](int buf, int rt) { return *reinterpret_cast<const float*>(s_q + buf * S::Q_SLOTS + (32 * rt + l32) * PITCH + SEG); };

  auto waited_too_long = [&](int& spins, long long& t0) -> bool {
    if (a.wait_ticks == 0) return true;
    if (spins++ == 0) {
      t0 = wall_clock64();
      return false;
    }
    if ((spins & 15) != 0) return false;
    return wall_clock64() - t0 > (long long)a.wait_ticks ||
           __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
  };
  auto give_up = [&]() { __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };

  auto word4_of = [&](int u, int h, int row) {
    u64* w = *s_words4;
    return w ? w + ((uint32_t)(u * NG + h) * ROWS + (uint32_t)row) : nullptr;
  };
  // Sum of a lane's row of a group, as it is now.
  u64 sum;
  auto request_sum = [&](int u, int h, int which) { sum = ld64(a.words + (size_t)u * unit_words + word_of(which, 64 * h + lane)); };
  // ... when all items have been added: the rows' weights 1 / (G z), of rows l32 and 32 + l32.  Returns whether some item's
  // sum did not fit (the same in all waves and workgroups).
  auto weights = [&](int u, int h, int np, int which, float scale, float (&w)[2], bool armed) -> bool {
    const uint32_t need = a.wait_ticks == 0 && np > 1 ? 0x400u : (uint32_t)np;
    auto missing = [&]() { return armed & (((uint32_t)(sum >> 52) & 0x3FFu) < need); };
    if (__builtin_expect(__any(missing()), 0)) {  // (a test of its own: inside a loop it would wait for all that is under way)
      int spins = 0;
      long long t0 = 0;
      do {
        if (waited_too_long(spins, t0)) {
          give_up();
          break;
        }
        request_sum(u, h, which);
      } while (__any(missing()));
    }
    const int top = (int)(sum >> 32);
    float x = inverse(sum, scale);
    if (__builtin_expect(which == kSums && __any(armed & (top < 0)), 0)) {
      const u64* w2 = a.words + (size_t)u * unit_words + word_of(kSums2, 64 * h + lane);
      const u64 b2 = ld64(w2), b3 = ld64(w2 + (kSums3 - kSums2)), b4 = *s_words4 ? ld64(word4_of(u, h, lane)) : 0ull;
      const float z = sum_of_words(sum_of(sum), b2, b3, b4);
      if (top < 0) x = __builtin_amdgcn_rcpf(z) * (scale * (1.f / kUnits));
    }
    if ((top & 0x40000000) != 0) x = __builtin_nanf("");
    const uint32_t mine = __float_as_uint(64 * h + lane < a.R ? x : 0.f);
    const u32x2 both = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(mine, mine, false, false));
    w[0] = __uint_as_float(both[0]);
    w[1] = __uint_as_float(both[1]);
    return armed & __any((top & 0x40000000) != 0);
  };

  // Where p waits: groups with an even number in registers, the others in LDS (but for four registers).
  float pr[4][16];
  f32x4 p_last = {};
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) pr[j][v] = 0.f;
  u32x4* p_lane = smem + (size_t)wave * (PQ * 64) + lane;
  // (Keys without a score write into the unit's first place behind the prefix, which nobody reads: a store under a condition
  // would make the waits for keys that follow allow for either way.)
  auto write_score = [&](const Item& d, int t, float s) {
    const int ln = fresh(lane);
    d.raw[min(tile_key(d, t) + transpose_key(ln), d.n - a.alpha)] = s;
  };
  auto mark = [&](bool bad, int i) {
    if (__builtin_expect(bad, 0) && lane == 0) atomicOr(&s_item[i].x, 0x80000000u);
  };

  // The waits for what is under way allow for both ways into the loop: what is requested in front of it is as many requests
  // apart as in it.  They do not count the atomic adds, which stand under a condition, and so reach one request too far: a
  // spare one lies behind the sums and returns with them.
  uint32_t spare[2] = {};
  auto spare_load = [&](int u, int par) {
    asm volatile("" ::"v"(spare[par]));
    spare[par] = ld32(reinterpret_cast<const uint32_t*>(a.words + (size_t)u * unit_words));
    __builtin_amdgcn_sched_barrier(0);
  };
  // Steps: group h of item i.  Behind the last item the requests go to the unit's key 0 alone.
  struct Step {
    Item d;
    int i, h;
  };
  auto after = [&](const Step& s) {
    Step n = s;
    if (MODE > 1 && s.h + 1 < NG) {
      ++n.h;
    } else {
      n.h = 0;
      n.i = s.i + 1;
      n.d = item(min(n.i, nmine - 1));
      if (n.i >= nmine) { n.d.part = 0; n.d.n = 1; }
    }
    return n;
  };
  Step cur = {item(0), 0, 0}, nx1 = after(cur), nx2 = after(nx1), old1 = cur, old = cur;
  auto pad_store = [&]() {
    __hip_atomic_store(cur.d.raw + min(tile_key(cur.d, 0) + l32, cur.d.n - a.alpha), 0.f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_sched_barrier(0);
  };
  request_q(cur.d, 0);
  commit_q(0);
  request_q(nx1.d, nx1.h);
  issue_k(cur.d, 0, kf[0]);
  pad_store();
  issue_k(cur.d, 1, kf[1]);
  pad_store();
  request_sum(cur.d.u, 0, kSums);
  spare_load(cur.d.u, 1);
  lds_barrier();

  // Sums of the step before: a wave looks after 8 rows, a lane adds those of two waves.
  auto publish = [&](int buf, int u, int h, bool armed) {
    const int ln = fresh(lane);
    const float* zp = s_z + buf * kW * ROWS + (ln >> 4) * 2 * ROWS + wave * (ROWS / kW) + (ln & (ROWS / kW - 1));
    const float y = zp[0] + zp[ROWS];
    const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(y), __float_as_uint(y), false, false));
    const float z = both_halves<false>(__uint_as_float(r[0]) + __uint_as_float(r[1]));
    if (ln < ROWS / kW && armed)
      add_sum(a.words + (size_t)u * unit_words + word_of(kSums, 64 * h + wave * (ROWS / kW) + ln), z,
              [&]() { return word4_of(u, h, wave * (ROWS / kW) + ln); });
  };
  f32x16 t[2] = {};  // scores of the item that has waited: a lane's rows of the groups so far, by key

  // Step cur (parity PAR) takes the place of the step two before.  LAST: the item's last group; the next item's keys follow.
  // (MODE 3: any group; whether it is the last one is seen here.)
  auto step = [&](auto PAR, auto LAST, int n) {
    constexpr int par = decltype(PAR)::value;
    constexpr bool last = decltype(LAST)::value;
    const int npre = cur.d.n - a.alpha;
    f32x16 T[2];
    bf16x8 qf[3];
    f32x4 po[2];
    float w[2];
    // Tiles in the order (key tile, row tile).  Tile j is multiplied while tile j - 1 turns into probabilities, which take the
    // place of those that have waited; these, weighted, are summed over the rows in t.
    auto frag_at = [&](int s) { return q_frag(par, (s / KS) & 1, s % KS); };  // fragment of step s = KS * tile + ks
    qf[0] = frag_at(0);
    qf[1] = frag_at(1);
    auto products = [&](auto J) {
      constexpr int j = decltype(J)::value;
      constexpr int jc = j < 1 ? 0 : j - 1, tc = jc >> 1, rc = jc & 1;
      constexpr bool mul = j < 4, probs = j > 0;
      f32x16& nx = T[j & 1];
      f32x16& cu = T[(j + 1) & 1];
      float nref = 0.f, z0 = 0.f, z1 = 0.f;
      auto old_p = [&](int q) {  // 16 bytes of the p that has waited
        if constexpr (par == 1 && probs)
          po[q & 1] = 4 * jc + q < PQ ? __builtin_bit_cast(f32x4, p_lane[64 * (4 * jc + q)]) : p_last;
      };
      if constexpr (probs) {
        nref = -ref_of(par, rc);
        old_p(0);
      }
      if constexpr (mul) nx = f32x16{};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if constexpr (mul) {
          const int s = j * KS + ks;
          if (s + 2 < 4 * KS) qf[(s + 2) % 3] = frag_at(s + 2);
          nx = PKV_MFMA32(kf[j >> 1][ks], qf[s % 3], nx);
        }
        if constexpr (probs) {
          float x[TPM];
#pragma unroll
          for (int e = 0; e < TPM; ++e) x[e] = __builtin_fmaf(cu[TPM * ks + e], a.kappa, nref);
          if ((TPM * ks) % 4 == 0 && TPM * ks / 4 < 3) old_p(TPM * ks / 4 + 1);
#pragma unroll
          for (int e = 0; e < TPM; ++e) {
            const int v = TPM * ks + e;
            const float o = par == 0 ? pr[jc][v] : po[(v / 4) & 1][v & 3];
            t[tc][v] = rc == 0 && (MODE == 1 || (MODE == 2 && par == 0)) ? o * w[rc] : __builtin_fmaf(o, w[rc], t[tc][v]);
            x[e] = fast_exp2(x[e]);
          }
#pragma unroll
          for (int e = 0; e < TPM; ++e) {
            const int v = TPM * ks + e;
            if constexpr (par == 0) pr[jc][v] = x[e];
            else cu[v] = x[e];
            if (e & 1) z1 += x[e];
            else z0 += x[e];
            asm volatile("" : "+v"(t[tc][v]));  // (formed here: put off, the sums would keep what they are formed of alive)
          }
          asm volatile("" : "+v"(z0), "+v"(z1));
          if constexpr (par == 1) {
            const int v = TPM * (ks + 1);
            if (v % 4 == 0) {
              const f32x4 xq = {cu[v - 4], cu[v - 3], cu[v - 2], cu[v - 1]};
              if (4 * jc + v / 4 - 1 < PQ) p_lane[64 * (4 * jc + v / 4 - 1)] = __builtin_bit_cast(u32x4, xq);
              else p_last = xq;
            }
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (probs) {
        if (__builtin_expect(tile_key(cur.d, tc) + 32 > npre, 0)) {  // the tile reaches into the causal window or beyond the end
          const int ln = fresh(lane), row = 64 * cur.h + 32 * rc + (ln & 31);
          const int lim = npre + row - head_of(row) * a.alpha - tile_key(cur.d, tc) - 4 * (ln >> 5);  // last key the lane's query sees
          z0 = z1 = 0.f;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            f32x4 x;
            const bool in_lds = 4 * jc + q < PQ;
            if (par == 0) x = f32x4{pr[jc][4 * q], pr[jc][4 * q + 1], pr[jc][4 * q + 2], pr[jc][4 * q + 3]};
            else x = in_lds ? __builtin_bit_cast(f32x4, p_lane[64 * (in_lds ? 4 * jc + q : 0)]) : p_last;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              x[c] = mrow0(4 * q + c) > lim ? 0.f : x[c];
              if (c & 1) z1 += x[c];
              else z0 += x[c];
              if (par == 0) pr[jc][4 * q + c] = x[c];
            }
            if (par == 1) {
              if (in_lds) p_lane[64 * (in_lds ? 4 * jc + q : 0)] = __builtin_bit_cast(u32x4, x);
              else p_last = x;
            }
          }
        }
        const float z = both_halves<false>(z0 + z1);
        float* zp = s_z + (par * kW + wave) * ROWS + 32 * rc + l32;
        if (tc == 0) *zp = z;
        else *zp += z;
        if constexpr (rc == 1) {
          if constexpr (MODE % 2 == 1 || par == 1)
            if (MODE < 3 || old.h == NG - 1) write_score(old.d, tc, transpose_sum(t[tc], fresh(lane)));
        }
      }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    if ((MODE == 3 || (MODE == 4 && par == 0)) && old.h == 0) t[0] = t[1] = f32x16{};
    // (the waves of a SIMD come to the barrier at about the same time: the younger one leads through three of the five tiles)
    if (wave >= kW / 2) __builtin_amdgcn_s_setprio(1);
    products(I0{});
    publish(par ^ 1, old1.d.u, old1.h, n > 0);
    // (in front of the first two steps there is nothing: their scores are written later, over what is written here)
    mark(weights(old.d.u, old.h, nparts(old.d), kSums, kUnits * a.inv_G, w, n >= 2), old.i);
    products(I1{});
    commit_q(par ^ 1);
    request_q(nx2.d, nx2.h);
    if constexpr (last) issue_k(nx1.d, 0, kf[0]);
    products(I2{});
    __builtin_amdgcn_s_setprio(0);
    products(I3{});
    if constexpr (last) issue_k(nx1.d, 1, kf[1]);
    if constexpr (MODE == 3)
      if (cur.h == NG - 1) {  // (both tiles under one condition: the waits count them together)
        issue_k(nx1.d, 0, kf[0]);
        issue_k(nx1.d, 1, kf[1]);
      }
    products(I4{});
    request_sum(old1.d.u, old1.h, kSums);  // (read at the next step)
    spare_load(old1.d.u, par);
    old = old1;
    old1 = cur;
    cur = nx1;
    nx1 = nx2;
    nx2 = after(nx2);
    lds_barrier();  // the group's sums and the next one's queries are there; nobody reads this one's any more
  };
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  const int steps = nmine * NG;
#pragma unroll 1
  for (int n = 0; n < steps; n += 2) {  // (one way out of the loop: behind an odd number of steps comes one without an item)
    if constexpr (MODE == 4) {
#pragma unroll 1
      for (int h = 2; h < NG; h += 2, n += 2) {
        step(P0{}, std::false_type{}, n);
        step(P1{}, std::false_type{}, n + 1);
      }
    }
    step(P0{}, std::integral_constant<bool, MODE == 1>{}, n);
    step(P1{}, std::integral_constant<bool, MODE != 3>{}, n + 1);
  }
  // ---- the last two steps ----
  auto finish = [&](auto PAR, const Step& s) {
    constexpr int par = decltype(PAR)::value;
    float w[2];
    request_sum(s.d.u, s.h, kSums);
    mark(weights(s.d.u, s.h, nparts(s.d), kSums, kUnits * a.inv_G, w, true), s.i);
#pragma unroll
    for (int tc = 0; tc < 2; ++tc) {
      if (s.h == 0) t[tc] = f32x16{};
#pragma unroll
      for (int rt = 0; rt < 2; ++rt)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int j = tc * 2 + rt;
          const bool in_lds = 4 * j + q < PQ;
          f32x4 o;
          if (par == 0) o = f32x4{pr[j][4 * q], pr[j][4 * q + 1], pr[j][4 * q + 2], pr[j][4 * q + 3]};
          else o = in_lds ? __builtin_bit_cast(f32x4, p_lane[64 * (in_lds ? 4 * j + q : 0)]) : p_last;
#pragma unroll
          for (int c = 0; c < 4; ++c) t[tc][4 * q + c] = __builtin_fmaf(o[c], w[rt], t[tc][4 * q + c]);
        }
      if (s.h == NG - 1) write_score(s.d, tc, transpose_sum(t[tc], fresh(lane)));
    }
  };
  if ((steps & 1) == 0) {
    publish(1, old1.d.u, old1.h, true);
    finish(P0{}, old);
    finish(P1{}, old1);
  } else {
    finish(P0{}, old);
  }

  // ---- rare: units with an item whose sum did not fit (a key a hundred binades above the sampled ones, or a reference of
  // -inf) are scored again, from memory and relative to the exact maxima, which their items exchange first ----
  lds_barrier();
  float ps[2] = {0.f, 0.f};  // scores over the groups so far
  // p of (key tile t, row tile rt of group h) relative to the references in LDS (maxima: the logits themselves, hidden ones
  // -inf); queries from memory
  auto again = [&](const Item& d, int t, int h, int rt, const bf16x8 (&f)[KS], bool maxima) {
    const int row = 64 * h + 32 * rt + l32, r = min(row, a.R - 1), hh = head_of(r);
    const char* q_row = reinterpret_cast<const char*>(d.Q) + ((uint32_t)(hh * (int)a.q_sh + (r - hh * a.alpha) * (int)a.q_st) * 2u + 16u * (uint32_t)hf);
    f32x16 x = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) x = PKV_MFMA32(f[ks], as_frag(*reinterpret_cast<const u32x4*>(q_row + 32 * ks)), x);
    const float m = ref_of(0, rt);
    const int lim = d.n - a.alpha + row - head_of(row) * a.alpha - tile_key(d, t) - 4 * hf;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const bool hidden = mrow0(v) > lim;
      if (maxima) x[v] = hidden ? -INFINITY : x[v] * a.kappa;
      else x[v] = hidden ? 0.f : fast_exp2(__builtin_fmaf(x[v], a.kappa, -m));
    }
    return x;
  };
#pragma unroll 1
  for (int i0 = 0; i0 < nmine; ++i0) {
    if ((__builtin_amdgcn_readfirstlane((int)s_item[i0].x) >> 31) == 0) continue;
    const Item d = item(i0);
    const int np = nparts(d);
    u64* words = a.words + (size_t)d.u * unit_words;
#pragma unroll 1
    for (int h = 0; h < NG; ++h)
#pragma unroll 1
      for (int round = 0; round < 3; ++round) {  // maxima; sums; scores
        float w[2];
        if (round == 1) {
          int spins = 0;
          long long t0 = 0;
          while (a.wait_ticks == 0 || (int)((uint32_t)(ld64(words + word_of(kSums, 64 * h)) >> 52) & 0x3FFu) < 2 * np)
            if (waited_too_long(spins, t0)) {
              give_up();
              break;
            }
          if (tid < ROWS) {
            const uint32_t o = ld32(reinterpret_cast<const uint32_t*>(words) + half_word_of(kMax, 64 * h + tid));
            const float m = __uint_as_float((o & 0x80000000u) ? o & 0x7FFFFFFFu : ~o);
            *reinterpret_cast<float*>(s_q + tid * PITCH + SEG) = o == 0u || m == -INFINITY ? 0.f : m;
          }
          lds_barrier();
        } else if (round == 2) {
          sum = 0;
          (void)weights(d.u, h, np, kSums2, 0x1p34f * a.inv_G, w, true);
        }
#pragma unroll 1
        for (int t = 0; t < 2; ++t) {
          issue_k(d, t, kf[0]);
          f32x16 s = {};
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) {
            const f32x16 x = again(d, t, h, rt, kf[0], round == 0);
            float r = round == 0 ? -INFINITY : 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              r = round == 0 ? fmaxf(r, x[v]) : r + x[v];
              if (round == 2) s[v] = __builtin_fmaf(x[v], w[rt], s[v]);
            }
            r = round == 0 ? both_halves<true>(r) : both_halves<false>(r);
            float* zp = s_z + wave * ROWS + 32 * rt + l32;
            const float before = *zp;
            if (t > 0) r = round == 0 ? fmaxf(r, before) : r + before;
            *zp = r;
          }
          if (round == 2) {
            const float s1 = transpose_sum(s, fresh(lane));
            const float all = h == 0 ? s1 : (t == 0 ? ps[0] : ps[1]) + s1;
            if (t == 0) ps[0] = all;
            else ps[1] = all;
            write_score(d, t, all);
          }
        }
        lds_barrier();
        if (tid < ROWS && round < 2) {
          float r = round == 0 ? -INFINITY : 0.f;
#pragma unroll
          for (int v = 0; v < kW; ++v) r = round == 0 ? fmaxf(r, s_z[v * ROWS + tid]) : r + s_z[v * ROWS + tid];
          if (round == 0) {
            const uint32_t o = __float_as_uint(r);
            (void)__hip_atomic_fetch_max(reinterpret_cast<uint32_t*>(words) + half_word_of(kMax, 64 * h + tid), (o & 0x80000000u) ? ~o : o | 0x80000000u,
                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          } else {
            add_sum_again(words + word_of(kSums2, 64 * h + tid), r);
          }
        }
        // (the words for these sums may hold what the first attempt put there; every item has been counted, and so has its
        // part of that.  Who still reads it has seen the mark and scores its item again.)
        if (round == 0 && d.part == 0 && tid < ROWS)
          __hip_atomic_store(words + word_of(kSums2, 64 * h + tid), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (round == 0) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // (the maxima before the count)
        __syncthreads();
        if (round == 0 && tid == 0) add64(words + word_of(kSums, 64 * h), kOne);
      }
  }
}

// Clears the words of a unit's group of 64 rows and forms its references: per row the largest logit of 64 keys, eight
// neighbours each at eight places spread evenly over the prefix, key 0 among them.  (One product per wave, so that memory is waited for once.)
template <int D>
__global__ __launch_bounds__(256) void lag_prepare_kernel(const LagArgs a, int clear_err) {
  constexpr int KS = D / 16;
  __shared__ float s_max[2][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l32 = lane & 31, hf = lane >> 5;
  const int h = blockIdx.x % a.groups, u = blockIdx.x / a.groups, BH = a.B * a.Hkv;
  const int l = u / BH, bg = u - l * BH, b = bg / a.Hkv, g = bg - b * a.Hkv;
  if (blockIdx.x == 0 && clear_err && tid < 2) a.err[tid] = 0;
  u64* words = a.words + (size_t)blockIdx.x * 256;
  if ((tid & 31) < kRefs || (tid & 31) >= kMax) words[tid] = 0;
  if (a.words4 && tid < 64) a.words4[(size_t)blockIdx.x * 64 + tid] = 0;
  if (a.flags && h == 0 && tid == 0) a.flags[(size_t)a.layer[l].slot * BH + bg] = kSiftObjects;  // (not sifted)
  int n = a.N;
  if (a.seq_lens) {
    n = a.seq_lens[b];
    n = n < 0 ? 0 : (n > a.N ? a.N : n);
  }
  if (a.layer[l].k_l >= n) return;
  const int rt = wave & 1, share = wave >> 1;
  const int row = min(64 * h + 32 * rt + l32, a.R - 1), hh = (int)(__umul24(row, a.alpha_magic) >> 16), t = row - hh * a.alpha;
  const char* q_row = reinterpret_cast<const char*>(a.layer[l].Q + (size_t)b * a.q_sb + (size_t)(g * a.G + hh) * a.q_sh + t * a.q_st) + 16 * hf;
  const uint32_t npre = (uint32_t)(n - a.alpha), key = min((npre * (uint32_t)(4 * share + (l32 >> 3)) >> 3) + (uint32_t)(l32 & 7), npre - 1);
  const char* k_row = reinterpret_cast<const char*>(a.layer[l].K + (size_t)b * a.kv_sb + (size_t)g * a.kv_sh) + (key * ((uint32_t)a.kv_st * 2u) + 16u * (uint32_t)hf);
  bf16x8 qf[KS], kf[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    qf[ks] = as_frag(*reinterpret_cast<const u32x4*>(q_row + 32 * ks));
    kf[ks] = as_frag(*reinterpret_cast<const u32x4*>(k_row + 32 * ks));
  }
  f32x16 x = {};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) x = PKV_MFMA32(kf[ks], qf[ks], x);
  float m = x[0];
#pragma unroll
  for (int v = 1; v < 16; ++v) m = fmaxf(m, x[v]);
  s_max[share][32 * rt + l32] = both_halves<true>(m) * a.kappa;
  __syncthreads();
  if (tid < 64)
    reinterpret_cast<float*>(words)[half_word_of(kRefs, tid)] = fmaxf(s_max[0][tid], s_max[1][tid]);
}

template <int D, int MODE>
hipError_t launch_lag(const LagArgs& a, bool clear_err, bool prepared, hipStream_t s) {
  using S = LagShape<D>;
  static bool attr_set[kMaxDevices];
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {  // raise the dynamic LDS limit once per device (idempotent; no allocation)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(score_lag_kernel<D, MODE>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  if (!prepared) {
    hipLaunchKernelGGL((lag_prepare_kernel<D>), dim3(a.L * a.B * a.Hkv * a.groups), dim3(256), 0, s, a, clear_err ? 1 : 0);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((score_lag_kernel<D, MODE>), dim3(a.grid), dim3(kT), S::LDS, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_lag(const LagArgs& a, bool clear_err, bool prepared, hipStream_t s) {
#define PKV_CASE(DD)                                                   \
  if (a.d == DD) {                                                     \
    if (a.groups == 1) return launch_lag<DD, 1>(a, clear_err, prepared, s);      \
    if (a.groups == 2) return launch_lag<DD, 2>(a, clear_err, prepared, s);      \
    if (a.groups % 2 == 0) return launch_lag<DD, 4>(a, clear_err, prepared, s);  \
    return launch_lag<DD, 3>(a, clear_err, prepared, s);                         \
  }
  PKV_CASE(128) PKV_CASE(64)
#undef PKV_CASE
  return hipErrorInvalidValue;
}

}  // namespace pkv
