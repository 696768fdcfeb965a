// Window scoring in one pass over K for few query rows per KV head (G * alpha <= 64; Sec. 4.2.2, Eq. Al and Eq.
// att_score) on MI355X.
//
// The score of a key needs the softmax normaliser of every window query, which is known only after all keys of the
// head have been seen.  With few query rows the un-normalised probabilities p = exp2(kappa q.k - m) of a key (m: a
// reference exponent of the row) take less room than the key itself, so they, and not the keys, are what waits for
// the normalisers:  s_i = sum_r p_ri exp2(m_r - c_r)  is one multiply-add per logit, K is multiplied once, and the
// registers of a key are free for the next one as soon as it has been multiplied.
//
// Work split.  An item is KI = 256 * TPW keys of one unit (layer, sequence, KV head): 512, or 1024 for up to 32 rows.  256 persistent workgroups of 512
// threads, one per compute unit (all of its LDS, 256 registers per lane), take the items in turn: item j belongs to
// workgroup j % 256.  Sequences of a ragged batch contribute the items they have, one after the other without gaps.
//
// Per item a workgroup
//   1. multiplies its keys with the unit's queries (rows = queries in registers, columns = keys; wave w takes the 32-key
//      tiles w, w + 8, ... of the item, loaded straight into operand layout, KB tiles ahead, across item boundaries),
//      turns the logits into p relative to the row's reference and keeps them in registers; sums over the keys give
//      the item's statistics (reference, sum) per row, published for the unit's other items (a word per row, or one for each of
//      the item's halves, so that items of 512 and of 1024 keys publish the same);
//   2. finishes the item BEFORE: the statistics of all items of its unit, which have had nearly the time of a whole item
//      to arrive, are read (8 bytes per row and item: a few per cent of the keys' traffic) and folded into the
//      normalisers; its p, moved to LDS meanwhile, are weighted and summed over the rows; one score per key is written
//      (already divided by G).
// A word of statistics carries a mark, the sign bit of the sum, and so announces itself (agent-scope relaxed atomics, cleared
// before the launch).  Every item has words of its own, written once: a workgroup that starts late or falls behind, however
// far, finds what it waits for.  They are requested a tile before they are used, in front of the keys requested at that
// place: a wave's loads return in order, so a probe issued behind keys would hold the wave until those have arrived.  (For
// the same reason there is one hop and not two, fold by one item and hand over: each hop costs a tile's time.)
// The reference of a row is its largest logit of four keys of the unit, the sink at position 0 among them: the same for all
// keys, so that equal keys get equal scores, bit for bit, and near enough to the terms that count, so that x - m loses little
// to its rounding.  (With key 0 alone the scores of a head whose key 0 lies 30 binades below the others were 2.2e-6 off those
// of 64 bits, now 0.1e-6; with the normaliser's own rounding taken out of the weights too, usual heads 0.5e-6 -> 0.1e-6,
// the register-resident kernel 0.6e-6.)
// A row whose reference was too far below its logits (sum beyond 2^100) is summed up once more by its wave with the exact
// maximum, from memory, and the items of such a unit are scored again at the end of the launch (rare: a key that stands 93
// binades above the four; such a launch takes up to three times as long).
//
// What bounds it: HBM for many units.  Measured against the register-resident kernel, which keeps the keys and multiplies
// them twice (one scoring launch, by the profiler): 256 units of 8k keys, 32 rows 146 -> 112 us; 256 of 32k, 8 rows 535
// -> 389 us (5.5 TB/s); ragged batch, 2048 units of 8k .. 16k, 64 rows 2.22 -> 1.67 ms (4.2 TB/s; an item of 512 keys
// takes 6 - 8 us, of which the hop between the workgroups is not always covered).  One unit or a few: the latency of the
// keys, one hop and two barriers; one layer of 8 heads with 8k keys 17.9 -> 16.5 us,
// with items of half the size and no more statistics requested than there are, whole calls 26.6 -> 23.0.
//
// Every wait is bounded by wall-clock time (a workgroup that has waited too long raises the error word and carries on),
// so the grid always drains.
#include <type_traits>

#include "pkv_internal.h"
#include "pkv_lds.h"

namespace pkv {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned long long u64;

constexpr int kW = 8;             // waves per workgroup
constexpr int kT = kW * 64;

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x2 as_pair(uint32_t u) { return __builtin_bit_cast(bf16x2, u); }
__device__ __forceinline__ bf16x8 as_frag(u32x4 u) { return __builtin_bit_cast(bf16x8, u); }
// A value the compiler must treat as new: lane constants derived from it are recomputed where they are used instead of
// being kept (and spilled) across the whole item loop.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
// LDS traffic of one wave to its own region needs ordering only inside the wave.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}
__device__ __forceinline__ void st64(u64* p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ u64 ld64(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void merge_stats(float& m, float& z, float m2, float z2) {
  const float M = fmaxf(m, m2);
  const float Ms = (M == -INFINITY) ? 0.f : M;
  z = z * fast_exp2(m - Ms) + z2 * fast_exp2(m2 - Ms);
  m = M;
}
// Maximum over the 32 lanes of a wave half, valid in its last lane.
__device__ __forceinline__ float half_max(float x) {
#define PKV_STEP(ctrl, rows) \
  x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(-INFINITY), __float_as_int(x), ctrl, rows, 0xF, false)));
  PKV_STEP(0x111, 0xF)  // row_shr:1, 2, 4, 8: the last lane of every row of 16 holds the row's result
  PKV_STEP(0x112, 0xF)
  PKV_STEP(0x114, 0xF)
  PKV_STEP(0x118, 0xF)
  PKV_STEP(0x142, 0xA)  // row_bcast:15 into rows 1 and 3
#undef PKV_STEP
  return x;
}
// Sums of a and of b over the 32 lanes of a wave half: a's in the last lane of the half's first row of 16, b's of its second.
__device__ __forceinline__ float half_sums(float a, float b) {
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false));
  float x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
#define PKV_STEP(ctrl) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xF, 0xF, true))
  PKV_STEP(0x111);  // row_shr:1, 2, 4, 8
  PKV_STEP(0x112);
  PKV_STEP(0x114);
  PKV_STEP(0x118);
#undef PKV_STEP
  return x;
}
// x summed over the two halves of the wave, in every lane.
__device__ __forceinline__ float both_halves(float x) {
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// NV: registers of a 32x32 product that hold real rows (register v of half h: row 8 (v / 4) + 4 h + v % 4), 4 per 8
// rows; RT: 32-row tiles of queries; TPW: 32-key tiles of an item per wave, summed up in SUB parts, a word of statistics
// each; NPL: loads of
// statistics made ahead per thread.
template <int D, int NV, int RT, int TPW, int SUB, int NPL>
struct StreamShape {
  static constexpr int KS = D / 16, SEG = D / 8, PITCH = SEG + 1;  // (row pitch of Q in LDS: 16-byte slots, bank-free)
  static constexpr int KI = 32 * kW * TPW;                         // keys per item
  static constexpr int WR = NV == 16 ? 32 * RT : 16;               // rows of a statistics word's place
  static constexpr int KB = D == 128 ? 2 : TPW;                    // tiles in flight per wave
  static constexpr int ROWS = 32 * RT;
  static constexpr int PPL = kT / (32 * RT);                       // items whose statistics one load per thread covers
  static constexpr int P_SLOTS = kW * TPW * RT * (NV / 4) * 64;    // 16-byte slots of the pending p
  static constexpr int Q_SLOTS = ROWS * PITCH;
  static constexpr size_t LDS = (size_t)(P_SLOTS + Q_SLOTS) * 16 + (size_t)kW * ROWS * (3 * SUB + 3) * 4 + (size_t)ROWS * 2 * 4 +
                                (size_t)kStreamItems * 8;
  static_assert(LDS <= 160 * 1024, "one workgroup per compute unit");
  static_assert((size_t)(P_SLOTS + Q_SLOTS) * 16 >= (size_t)(kStreamUnits + 1 + kW) * 4, "prefix table fits");
};

template <int D, int NV, int RT, int TPW, int SUB, int NPL>
__global__ __launch_bounds__(kT, 2) void score_stream_kernel(const StreamArgs a) {
  using S = StreamShape<D, NV, RT, TPW, SUB, NPL>;
  constexpr int TPS = TPW / SUB, WR = S::WR;
  constexpr int KS = S::KS, SEG = S::SEG, PITCH = S::PITCH, KI = S::KI, KB = S::KB, ROWS = S::ROWS, PPL = S::PPL;
  constexpr int NQ = ROWS * SEG / kT > 0 ? ROWS * SEG / kT : 1;  // 16-byte loads per thread for a unit's queries
  constexpr int G4 = NV / 4;
  extern __shared__ u32x4 smem[];
  u32x4* s_q = smem + S::P_SLOTS;
  float* s_m = reinterpret_cast<float*>(s_q + S::Q_SLOTS);  // [2][SUB][kW][ROWS] references by wave, of this item and the next
  float* s_z = s_m + 2 * SUB * kW * ROWS;                   // [SUB][kW][ROWS] sums of this item
  float* s_w = s_z + SUB * kW * ROWS;                       // [kW][ROWS] references, then weights of the pending item
  float2* s_f = reinterpret_cast<float2*>(s_w + kW * ROWS);  // [kW][ROWS] statistics of its unit, by wave
  int* s_t = reinterpret_cast<int*>(s_f + kW * ROWS);       // [ROWS] window position of a row
  int* s_off = s_t + ROWS;                                  // [ROWS] byte offset of a row of Q
  uint2* s_item = reinterpret_cast<uint2*>(s_off + ROWS);   // [kStreamItems] (waves to score it again << 24 | unit, part << 20 | keys)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int BH = a.B * a.Hkv;

  // ---- the items of this workgroup ----
  int nmine;
  if (tid < ROWS) {
    const int r = min(tid, a.R - 1);  // (rows behind the last repeat it; their weights are zero)
    const int hh = r / a.alpha, t = r - hh * a.alpha;
    s_t[tid] = t;
    s_off[tid] = (int)(hh * a.q_sh + t * a.q_st) * 2;
  }
  if (a.uniform) {  // every unit has N keys to score
    const int parts = (a.N + KI - 1) / KI, total = a.L * BH * parts;
    nmine = min((total - (int)blockIdx.x + kStreamGrid - 1) / kStreamGrid, kStreamItems);
    if (tid < nmine) {
      const int j = tid * kStreamGrid + (int)blockIdx.x, u = j / parts;
      s_item[tid] = make_uint2((uint32_t)u, (uint32_t)(j - u * parts) << 20 | (uint32_t)a.N);
    }
    __syncthreads();
  } else {
    int* pre = reinterpret_cast<int*>(smem);  // [E + 1] items before (layer, sequence) e
    const int E = a.L * a.B;
    int* wsum = pre + kStreamUnits + 1;
    int run = 0;
    for (int e0 = 0; e0 < E; e0 += kT) {
      const int e = e0 + tid;
      int c = 0;
      if (e < E) {
        const int l = e / a.B, b = e - l * a.B;
        int n = a.N;
        if (a.seq_lens) {
          n = a.seq_lens[b];
          n = n < 0 ? 0 : (n > a.N ? a.N : n);
        }
        c = a.layer[l].k_l < n ? a.Hkv * ((n + KI - 1) / KI) : 0;  // (whole sequence kept: no scores needed)
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
    nmine = run > (int)blockIdx.x ? (run - (int)blockIdx.x + kStreamGrid - 1) / kStreamGrid : 0;
    nmine = min(nmine, kStreamItems);  // (the host admits only launches that fit)
    for (int k = tid; k < nmine; k += kT) {
      const int j = k * kStreamGrid + (int)blockIdx.x;
      int lo = 0, hi = E;  // pre[lo] <= j < pre[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (pre[mid] <= j) lo = mid;
        else hi = mid;
      }
      const int rem = j - pre[lo], parts = (pre[lo + 1] - pre[lo]) / a.Hkv;
      const int g = rem / parts, part = rem - g * parts, b = lo % a.B;
      int n = a.N;
      if (a.seq_lens) {
        n = a.seq_lens[b];
        n = n < 0 ? 0 : (n > a.N ? a.N : n);
      }
      s_item[k] = make_uint2((uint32_t)(lo * a.Hkv + g), (uint32_t)part << 20 | (uint32_t)n);
    }
    __syncthreads();
  }
  if (nmine == 0) return;

  // One item as this workgroup sees it (all fields wave-uniform).
  struct Item {
    int u, part, n, start;
    const uint16_t* Q;
    const uint16_t* K;
  };
  auto item = [&](int i) {
    const uint2 e = s_item[i];
    Item d;
    d.u = __builtin_amdgcn_readfirstlane((int)e.x) & 0xFFFFFF;
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)e.y);
    d.part = (int)(w >> 20);
    d.n = (int)(w & 0xFFFFFu);
    d.start = i * kStreamGrid + (int)blockIdx.x - d.part;  // the unit's first item
    const int l = d.u / BH, bg = d.u - l * BH;
    const int b = bg / a.Hkv, g = bg - b * a.Hkv;
    d.Q = a.layer[l].Q + (size_t)b * a.q_sb + (size_t)(g * a.G) * a.q_sh;
    d.K = a.layer[l].K + (size_t)b * a.kv_sb + (size_t)g * a.kv_sh;
    return d;
  };
  auto tile_key = [&](const Item& d, int t) { return d.part * KI + (t * kW + wave) * 32; };
  auto nwords = [&](const Item& d) { return (d.n + KI / SUB - 1) / (KI / SUB); };  // of a unit, per row

  // Keys of the wave's tile t as matrix operand: lane (column l32, half hf) holds elements 16 ks + 8 hf of its key.
  // Keys at or beyond n are replaced by the last one.
  bf16x8 kf[KB][KS];
  auto issue_k = [&](const Item& d, int t, bf16x8 (&f)[KS]) {
    const int ln = fresh(lane);
    const int key = min(tile_key(d, t) + (ln & 31), d.n - 1);
    const char* rowp = reinterpret_cast<const char*>(d.K) + 16 * (ln >> 5) + (uint32_t)key * ((uint32_t)a.kv_st * 2u);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) f[ks] = as_frag(*reinterpret_cast<const u32x4*>(rowp + 32 * ks));
    __builtin_amdgcn_sched_barrier(0);
  };
  // A unit's queries and four sampled keys (spread evenly over the prefix, key 0 among them; sixteen lanes carry one):
  // requested into registers, written to LDS later.  The lanes that carry a row of Q come to see the same segments of each
  // key, so the row's logits of these keys, and with them its reference, are formed on the way.
  u32x4 qv[NQ], kv;
  auto request_q = [&](const Item& d) {
    const int td = fresh(tid);
    const uint32_t key = (uint32_t)max(d.n - a.alpha, 0) * (uint32_t)((td & 63) >> 4) >> 2;
    kv = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(d.K) + 16 * (td & (SEG - 1)) + key * ((uint32_t)a.kv_st * 2u));
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int c = td + kT * i, row = c / SEG, seg = c - row * SEG;
      qv[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(d.Q) + seg * 16 + (uint32_t)s_off[min(row, ROWS - 1)]);
    }
  };
  auto commit_q = [&](int mbuf) {
    const int td = fresh(tid);
    float ref[NQ][4];  // [row][key]
#pragma unroll
    for (int i = 0; i < NQ; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) ref[i][j] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // the key of each row of sixteen lanes, in all lanes
      const u32x2 h = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(kv[e], kv[e], false, false));
      const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false));
      const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false));
      const uint32_t k[4] = {lo[0], lo[1], hi[0], hi[1]};
#pragma unroll
      for (int i = 0; i < NQ; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) ref[i][j] = __builtin_amdgcn_fdot2_f32_bf16(as_pair(qv[i][e]), as_pair(k[j]), ref[i][j], false);
    }
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int c = td + kT * i, row = c / SEG, seg = c - row * SEG;
      if (row < ROWS) s_q[row * PITCH + seg] = qv[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float& dot = ref[i][j];
        // over the row's 16 or 8 lanes, in all of them
#define PKV_ADD(ctrl) dot += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(dot), ctrl, 0xF, 0xF, true))
        PKV_ADD(0xB1);                 // quad_perm 1,0,3,2
        PKV_ADD(0x4E);                 // quad_perm 2,3,0,1
        PKV_ADD(0x141);                // row_half_mirror: the other quad of 8 lanes
        if (SEG == 16) PKV_ADD(0x140); // row_mirror: the other half of 16 lanes
#undef PKV_ADD
      }
      const float m = fmaxf(fmaxf(ref[i][0], ref[i][1]), fmaxf(ref[i][2], ref[i][3])) * a.kappa;
#pragma unroll
      for (int sb = 0; sb < SUB; ++sb)
        if (row < ROWS && seg < kW) s_m[((mbuf * SUB + sb) * kW + seg) * ROWS + row] = m;  // (a table per wave and word)
    }
  };
  const u32x4* q_lane = s_q + l32 * PITCH + hf;
  auto product = [&](const bf16x8 (&f)[KS], int rt) {
    f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(q_lane[32 * rt * PITCH + 2 * ks]), f[ks], acc, 0, 0, 0);
    return acc;
  };

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
  // row r of statistics word j; the mark that it is there
  auto stat_word = [&](int j, int r) { return a.stats + (uint32_t)(j * WR + r); };
  constexpr u64 kThere = 1ull << 63;

  // Statistics of a unit: thread = (row, every PPL-th word).
  u64 sv[NPL];
  auto request_stats = [&](const Item& d, int np) {
    const int ln = fresh(lane);
    const int srow = min(ln & (ROWS - 1), a.R - 1), sitem = wave * (64 / ROWS) + ln / ROWS;
#pragma unroll
    for (int k = 0; k < NPL; ++k) sv[k] = ld64(stat_word(d.start * SUB + min(sitem + k * PPL, np - 1), srow));
  };
  // ... folded over the thread's items (those not there yet are waited for) and left in LDS
  auto fold_stats = [&](const Item& d, int np) {
    const int ln = fresh(lane);
    const int srow = min(ln & (ROWS - 1), a.R - 1), sitem = wave * (64 / ROWS) + ln / ROWS;
    float m = -INFINITY, z = 0.f;
    auto arrived = [&](int q, u64 w) -> u64 {
      if ((w & kThere) == 0) {
        int spins = 0;
        long long t0 = 0;
        for (;;) {
          w = ld64(stat_word(d.start * SUB + q, srow));
          if ((w & kThere) != 0) break;
          __builtin_amdgcn_s_sleep(1);
          if (waited_too_long(spins, t0)) {
            __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
          }
        }
      }
      return w;
    };
    // (the largest reference first, so that the exponentials do not wait for each other)
#pragma unroll
    for (int k = 0; k < NPL; ++k)
      if (sitem + k * PPL < np) {
        sv[k] = arrived(sitem + k * PPL, sv[k]);
        m = fmaxf(m, __uint_as_float((uint32_t)sv[k]));
      }
    const float ms = (m == -INFINITY) ? 0.f : m;
#pragma unroll
    for (int k = 0; k < NPL; ++k)
      if (sitem + k * PPL < np)
        z = __builtin_fmaf(__uint_as_float((uint32_t)(sv[k] >> 32) & 0x7FFFFFFFu), fast_exp2(__uint_as_float((uint32_t)sv[k]) - ms), z);
    for (int q = sitem + NPL * PPL; q < np; q += PPL) {
      const u64 w = arrived(q, ld64(stat_word(d.start * SUB + q, srow)));
      merge_stats(m, z, __uint_as_float((uint32_t)w), __uint_as_float((uint32_t)(w >> 32) & 0x7FFFFFFFu));
    }
    if (ROWS == 32) {
      const float m2 = __shfl_xor(m, 32), z2 = __shfl_xor(z, 32);
      merge_stats(m, z, m2, z2);
    }
    if (ln < ROWS) s_f[wave * ROWS + ln] = make_float2(m, z);
  };

  // Pending item (the one before): its p in LDS, waiting for normalisers.
  Item pend;
  pend.u = -1;
  pend.part = 0; pend.n = 1; pend.start = 0; pend.Q = nullptr; pend.K = nullptr;
  u32x4* p_wave = smem + (size_t)wave * (TPW * RT * G4 * 64);  // slot [t][rt][v / 4][lane]
  // Scores of the pending item (the workgroup's item i): weights exp2(m - mu) / (G zu) per row, p weighted and summed over
  // the rows.  Where some wave of the unit had to take a reference of its own (mu > m; in that wave s_w holds -inf),
  // exp2(m - mu) may vanish before the products do, and equal keys of different waves would get different scores: every wave
  // of the unit scores the item again at the end.
  bool again = false;
  auto finish = [&](const Item& d, int i) {
    const int lane = fresh(tid & 63), l32 = lane & 31, hf = lane >> 5;
    const u32x4* p_lane = p_wave + lane;
    bool differ = false;
    if (lane < ROWS) {
      float2 f[kW];
      float mu = -INFINITY, zu = 0.f;
#pragma unroll
      for (int w = 0; w < kW; ++w) {
        f[w] = s_f[w * ROWS + lane];
        mu = fmaxf(mu, f[w].x);
      }
#pragma unroll
      for (int w = 0; w < kW; ++w) zu = __builtin_fmaf(f[w].y, fast_exp2(f[w].x - mu), zu);
      const float m = s_w[wave * ROWS + lane];
      // (not exp2(m - c), c = mu + log2 zu: nothing is lost to the rounding of c)
      s_w[wave * ROWS + lane] = lane < a.R ? fast_exp2(m - mu) * __builtin_amdgcn_rcpf(zu) * a.inv_G : 0.f;
      differ = lane < a.R && !(m == mu);
    }
    if (__builtin_expect(__any(differ), 0)) {
      again = true;
      if (lane == 0) atomicOr(&s_item[i].x, 0x1000000u << wave);
    }
    wave_lds_fence();
    f32x4 w[RT][G4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int q = 0; q < G4; ++q) w[rt][q] = *reinterpret_cast<const f32x4*>(s_w + wave * ROWS + 32 * rt + 8 * q + 4 * hf);
    float* raw = a.raw + (size_t)d.u * a.N;
    const int npre = d.n - a.alpha;
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < G4; ++q) {
          const f32x4 p = __builtin_bit_cast(f32x4, p_lane[((t * RT + rt) * G4 + q) * 64]);
          s0 = __builtin_fmaf(p[0], w[rt][q][0], s0);
          s1 = __builtin_fmaf(p[1], w[rt][q][1], s1);
          s0 = __builtin_fmaf(p[2], w[rt][q][2], s0);
          s1 = __builtin_fmaf(p[3], w[rt][q][3], s1);
        }
      const float s = both_halves(s0 + s1);
      // (both halves of the wave hold the score; keys without one write into the unit's first place behind the prefix,
      // which nobody reads: a store under a condition would make the waits for keys that follow allow for either way in)
      raw[min(tile_key(d, t) + l32, npre)] = s;
    }
  };

  Item cur = item(0);
  request_q(cur);
#pragma unroll
  for (int t = 0; t < KB; ++t) issue_k(cur, t, kf[t]);
  commit_q(0);
  lds_barrier();

  for (int i = 0; i < nmine; ++i) {
    Item nxt = item(i + 1 < nmine ? i + 1 : i);
    if (i + 1 == nmine) {  // behind the last item: the requests go to the unit's key 0 alone
      nxt.part = 0;
      nxt.n = 1;
    }
    const int np_pend = nwords(pend);
    const int npre = cur.n - a.alpha;
    const int mbuf = i & 1;
    float* m_tab = s_m + (mbuf * SUB * kW + wave) * ROWS;  // (a word's: kW * ROWS further)
    f32x4 p[TPW][RT][G4];
    // the row tile's references, from the wave's table in LDS (two row tiles' would not fit the registers)
    auto load_m = [&](int sb, int rt, f32x4 (&m)[G4]) {
#pragma unroll
      for (int q = 0; q < G4; ++q) m[q] = *reinterpret_cast<const f32x4*>(m_tab + sb * kW * ROWS + 32 * rt + 8 * q + 4 * hf);
    };
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int key0 = tile_key(cur, t);
      const bool masked = key0 + 32 > npre;         // the tile reaches into the causal window or beyond the end
      f32x16 acc[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = product(kf[t % KB], rt);
      // (these come before the keys requested here: loads return in order, and waits under conditions stay exact)
      if (t == 0) request_q(nxt);
      if (t == TPW - 2) request_stats(pend, np_pend);
      if (t + KB < TPW) issue_k(cur, t + KB, kf[t % KB]);
      else if (t < TPW - 1) issue_k(nxt, t + KB - TPW, kf[t % KB]);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        f32x4 m[G4];
        load_m(0, rt, m);  // (both parts' are the unit's so far)
#pragma unroll
        for (int q = 0; q < G4; ++q)
#pragma unroll
          for (int c = 0; c < 4; ++c) p[t][rt][q][c] = fast_exp2(__builtin_fmaf(acc[rt][4 * q + c], a.kappa, -m[q][c]));
      }
      if (masked) {  // keys the row's query does not see
        const int over = key0 + l32 - npre;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int q = 0; q < G4; ++q) {
            const i32x4 tt = *reinterpret_cast<const i32x4*>(s_t + 32 * rt + 8 * q + 4 * hf);
#pragma unroll
            for (int c = 0; c < 4; ++c) p[t][rt][q][c] = over > tt[c] ? 0.f : p[t][rt][q][c];
          }
      }
    }
    // ---- the item's statistics ----
    // (two sums share a register: those of the two parts, or of neighbouring rows of four)
    constexpr int NZ = SUB == 2 ? G4 : (G4 + 1) / 2;
    static_assert(SUB == 1 || SUB == 2, "pairs");
    f32x4 z[RT][NZ];
    auto sum_up = [&]() -> uint32_t {  // sums (bit 4 (NZ rt + q) + c, in the lane that holds it) whose reference does not fit
      uint32_t bad = 0u;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < NZ; ++q) {
          const int qa = SUB == 2 ? q : 2 * q, qb = SUB == 2 ? q : (2 * q + 1 < G4 ? 2 * q + 1 : 2 * q), tb = SUB == 2 ? TPS : 0;
          f32x4 za = p[0][rt][qa], zb = p[tb][rt][qb];
#pragma unroll
          for (int t = 1; t < TPS; ++t) {
            za += p[t][rt][qa];
            zb += p[tb + t][rt][qb];
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            z[rt][q][c] = half_sums(za[c], zb[c]);
            // (keys far below the reference vanish, as they should: a sampled key alone contributes 1 to the unit's sum)
            bad |= ((lane & 15) == 15 && !(z[rt][q][c] <= 0x1p100f)) ? 1u << (4 * (NZ * rt + q) + c) : 0u;
          }
        }
      return bad;
    };
    uint32_t bad = sum_up();
    bool own = false;  // (lane = row) the wave has a reference of its own
    if (__builtin_expect(__any(bad != 0u) && tile_key(cur, 0) < cur.n, 0)) {
      const uint32_t bad_before = __shfl_xor(bad, 16);  // (in the last lane of a half: of the half's first row of lanes)
#pragma unroll
      for (int sb = 0; sb < SUB; ++sb) {
        if (tile_key(cur, TPS * sb) >= cur.n) continue;
        const float unit_ref = m_tab[sb * kW * ROWS + (lane & (ROWS - 1))];
        // rare: a reference that does not fit (the sum is beyond 2^100 or, with one of -inf, undefined): for such a row the
        // exact maximum over the wave's keys (-inf if there is nothing to add up), then p once more
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          f32x4 mx[G4];
#pragma unroll
          for (int q = 0; q < G4; ++q) mx[q] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
          for (int pass = 0; pass < 2; ++pass) {
            f32x4 m[G4];
            load_m(sb, rt, m);
#pragma unroll
            for (int q = 0; q < G4; ++q)
#pragma unroll
              for (int c = 0; c < 4; ++c) m[q][c] = m[q][c] == -INFINITY ? 0.f : m[q][c];
#pragma unroll
            for (int t = TPS * sb; t < TPS * (sb + 1); ++t) {
              bf16x8 f[KS];
              issue_k(cur, t, f);
              const f32x16 acc = product(f, rt);
              const int over = tile_key(cur, t) + l32 - npre;
#pragma unroll
              for (int q = 0; q < G4; ++q) {
                const i32x4 tt = *reinterpret_cast<const i32x4*>(s_t + 32 * rt + 8 * q + 4 * hf);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  const float y = acc[4 * q + c];
                  if (pass == 0) mx[q][c] = fmaxf(mx[q][c], over > tt[c] ? -INFINITY : y * a.kappa);
                  else p[t][rt][q][c] = over > tt[c] ? 0.f : fast_exp2(__builtin_fmaf(y, a.kappa, -m[q][c]));
                }
              }
            }
            if (pass == 0) {
#pragma unroll
              for (int q = 0; q < G4; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  const float x = half_max(mx[q][c]);
                  const bool second = SUB == 2 ? sb == 1 : (q & 1) == 1 || G4 == 1;
                  if (l32 == 31 && ((second ? bad : bad_before) >> (4 * (NZ * rt + (SUB == 2 ? q : q / 2)) + c) & 1u)) m_tab[sb * kW * ROWS + 32 * rt + 8 * q + 4 * hf + c] = x;
                }
              wave_lds_fence();
            }
          }
        }
        own = own || m_tab[sb * kW * ROWS + (lane & (ROWS - 1))] != unit_ref;
      }
      (void)sum_up();
    }
    if (pend.u >= 0) fold_stats(pend, np_pend);
    if ((lane & 15) == 15) {
      const int second = lane >> 4 & 1;
      float* zt = s_z + wave * ROWS + 4 * hf + second * (SUB == 2 ? kW * ROWS : G4 == 1 ? 0 : 8);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < NZ; ++q) *reinterpret_cast<f32x4*>(zt + 32 * rt + (SUB == 2 ? 8 : 16) * q) = z[rt][q];
    }
    lds_barrier();  // every wave is done with this unit's queries; the waves' statistics are there
    if (tid < ROWS * SUB) {
      const int sb = tid / ROWS, row = tid & (ROWS - 1);
      const float* mt = s_m + ((mbuf * SUB + sb) * kW) * ROWS + row;
      const float* zt = s_z + sb * kW * ROWS + row;
      float mm = -INFINITY, zz = 0.f;
#pragma unroll
      for (int w = 0; w < kW; ++w) mm = fmaxf(mm, mt[w * ROWS]);
      const float ms = mm == -INFINITY ? 0.f : mm;
#pragma unroll
      for (int w = 0; w < kW; ++w) zz = __builtin_fmaf(zt[w * ROWS], fast_exp2(mt[w * ROWS] - ms), zz);
      if (WR == ROWS || row < WR)
        st64(stat_word((cur.start + cur.part) * SUB + sb, row), kThere | (u64)__float_as_uint(zz) << 32 | __float_as_uint(mm));
    }
    commit_q(mbuf ^ 1);
    issue_k(nxt, KB - 1, kf[(TPW - 1) % KB]);  // (behind the statistics, which others wait for)
    // ---- the item before ----
    if (pend.u >= 0) finish(pend, i - 1);
    if (lane < ROWS) s_w[wave * ROWS + lane] = own ? -INFINITY : m_tab[lane];
#pragma unroll
    for (int t = 0; t < TPW; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int q = 0; q < G4; ++q) p_wave[((t * RT + rt) * G4 + q) * 64 + lane] = __builtin_bit_cast(u32x4, p[t][rt][q]);
    pend = cur;
    cur = nxt;
    lds_barrier();  // the next unit's queries are in place
  }
  request_stats(pend, nwords(pend));
  fold_stats(pend, nwords(pend));
  lds_barrier();
  finish(pend, nmine - 1);

  // ---- rare: items to score again, from memory and relative to the largest reference of the unit; every wave its own
  // tiles ----
  if (__builtin_expect(!again, 1)) return;
  float* ref_tab = reinterpret_cast<float*>(p_wave);  // [ROWS] references, [ROWS] weights
  static_assert((size_t)TPW * RT * G4 * 64 * 16 >= (size_t)ROWS * 8, "tables fit");
#pragma unroll 1
  for (int i = 0; i < nmine; ++i) {
    if ((__builtin_amdgcn_readfirstlane((int)s_item[i].x) >> (24 + wave) & 1) == 0) continue;
    const Item d = item(i);
    const int np = nwords(d), npre = d.n - a.alpha;
    if (lane < ROWS) {
      float m = -INFINITY, z = 0.f;
      for (int q = 0; q < np; ++q) {  // (all there: the item has been finished before)
        const u64 w = ld64(stat_word(d.start * SUB + q, min(lane, a.R - 1)));
        merge_stats(m, z, __uint_as_float((uint32_t)w), __uint_as_float((uint32_t)(w >> 32) & 0x7FFFFFFFu));
      }
      ref_tab[lane] = m;
      ref_tab[ROWS + lane] = lane < a.R ? __builtin_amdgcn_rcpf(z) * a.inv_G : 0.f;
    }
    wave_lds_fence();
    float* raw = a.raw + (size_t)d.u * a.N;
#pragma unroll 1
    for (int t = 0; t < TPW; ++t) {
      bf16x8 f[KS];
      issue_k(d, t, f);
      const int over = tile_key(d, t) + l32 - npre;
      float s = 0.f;
#pragma unroll 1
      for (int rt = 0; rt < RT; ++rt) {
        const char* q_row = reinterpret_cast<const char*>(d.Q) + 16 * hf + (uint32_t)s_off[32 * rt + l32];
        f32x16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(*reinterpret_cast<const u32x4*>(q_row + 32 * ks)), f[ks], acc, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < G4; ++q) {
          const i32x4 tt = *reinterpret_cast<const i32x4*>(s_t + 32 * rt + 8 * q + 4 * hf);
          const f32x4 m = *reinterpret_cast<const f32x4*>(ref_tab + 32 * rt + 8 * q + 4 * hf);
          const f32x4 w = *reinterpret_cast<const f32x4*>(ref_tab + ROWS + 32 * rt + 8 * q + 4 * hf);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            s = __builtin_fmaf(over > tt[e] ? 0.f : fast_exp2(__builtin_fmaf(acc[4 * q + e], a.kappa, -m[e])), w[e], s);
        }
      }
      raw[min(tile_key(d, t) + l32, npre)] = both_halves(s);
    }
    wave_lds_fence();
  }
}

// Clears n 16-byte slots at p and the error word.
__global__ __launch_bounds__(256) void clear_kernel(u32x4* p, int n, int32_t* err) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = u32x4{0u, 0u, 0u, 0u};
  if (err && i < 2) err[i] = 0;
}

template <int D, int NV, int RT, int TPW, int SUB, int NPL>
hipError_t launch_stream(const StreamArgs& a, hipStream_t s) {
  using S = StreamShape<D, NV, RT, TPW, SUB, NPL>;
  static bool attr_set[kMaxDevices];
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {  // raise the dynamic LDS limit once per device (idempotent; no allocation)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(score_stream_kernel<D, NV, RT, TPW, SUB, NPL>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)S::LDS);
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  hipLaunchKernelGGL((score_stream_kernel<D, NV, RT, TPW, SUB, NPL>), dim3(a.grid), dim3(kT), S::LDS, s, a);
  return hipGetLastError();
}

// A thread loads no more words of statistics ahead than the unit's number calls for: the loads pass the caches by, and four,
// most of them of the unit's last word again, cost a launch of 32 layers of 8 x 8k keys, 32 rows, 2 %, of one layer 6 %.
template <int D, int NV>
hipError_t launch_rows32(const StreamArgs& a, hipStream_t s) {
  if (a.item_keys == 512) return launch_stream<D, NV, 1, 2, 1, 1>(a, s);          // (up to 8192 keys: 16 words)
  if (a.words_per_item == 2) return launch_stream<D, NV, 1, 4, 2, 1>(a, s);       // (likewise)
  if (a.N <= 16384) return launch_stream<D, NV, 1, 4, 1, 1>(a, s);
  return a.N <= 32768 ? launch_stream<D, NV, 1, 4, 1, 2>(a, s) : launch_stream<D, NV, 1, 4, 1, 4>(a, s);
}
template <int D>
hipError_t launch_rows64(const StreamArgs& a, hipStream_t s) {
  if (a.N <= 4096) return launch_stream<D, 16, 2, 2, 1, 1>(a, s);
  return a.N <= 8192 ? launch_stream<D, 16, 2, 2, 1, 2>(a, s) : launch_stream<D, 16, 2, 2, 1, 4>(a, s);
}

}  // namespace

hipError_t launch_score_stream(const StreamArgs& a, bool clear_err, hipStream_t s) {
  const int n16 = a.items * a.words_per_item * a.word_rows / 2;  // 64-bit words, two per slot
  hipLaunchKernelGGL(clear_kernel, dim3((n16 + 255) / 256), dim3(256), 0, s, reinterpret_cast<u32x4*>(a.stats), n16,
                     clear_err ? a.err : nullptr);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
#define PKV_CASE(DD)                                             \
  if (a.d == DD) {                                               \
    if (a.R <= 8) return launch_rows32<DD, 4>(a, s);             \
    if (a.R <= 16) return launch_rows32<DD, 8>(a, s);            \
    if (a.R <= 32) return launch_rows32<DD, 16>(a, s);           \
    if (a.R <= 64) return launch_rows64<DD>(a, s);             \
  }
  PKV_CASE(128) PKV_CASE(64)
#undef PKV_CASE
  return hipErrorInvalidValue;
}

}  // namespace pkv
