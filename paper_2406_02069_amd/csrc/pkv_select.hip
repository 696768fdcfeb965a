// Group mean, 1-D pooling and per-head top-k selection (Sec. 4.2.2: pooling of the window scores, then
// the k^l - alpha highest-scoring prefix tokens per head; the alpha instruction tokens are always kept).
//
// One 1024-thread workgroup per unit (layer x sequence x KV head); all layers of a call run in one
// launch.  The fp32 bit patterns of the pooled scores are the selection keys (scores are >= 0, so unsigned order =
// numeric order).
//
// Prefixes of up to 32768 keys (select_short): every thread holds PER keys in registers.
//   A. pooled[i] = pool_w-wide max / average of the un-pooled scores, prefix only.  All loads are issued at once, four
//      neighbouring positions per thread and load; the neighbours of a thread's four come out of an LDS copy.
//   B. the kk-th largest key T.  (1) Of every group of up to PER / 4 keys of a thread the largest is counted in a
//      histogram over the distance from a typical large key: the bin in which the count reaches kk bounds T from below (kk
//      groups hold a key that large), with one LDS addition per group instead of one per key.  (2) The keys at or
//      above the bound, a small multiple of kk, move to a list in LDS, in position order.  (3) A histogram of the list
//      finds T's bin; (4) the few keys in that bin are ranked against each other.  For more than a quarter of the
//      prefix, where the list does not fit (many equal scores) or there are not enough groups with a positive key, the
//      histograms go over all keys.
//   C. ordered emission, from the list where there is one: keys > T and the lowest positions with key == T, in ascending order, followed
//      by the window positions.
// What bounds it: the latency of some fifteen steps between barriers, 0.6 - 1.4 us each, beside the loads (5.8 of 19 us
// for 256 units of 32k keys); the work over all keys (one maximum and one comparison each) is short.  Measured with the
// copy of the kept rows, by the profiler, against a search of T over all keys one bit per round: one unit of 1k keys
// 15.2 -> 9.0 us, 8 units of 8k 18.2 -> 11.4, 256 units of 8k 28 -> 19, of 32k 48 -> 27, 2048 units of 8k .. 16k
// 215 -> 128 (its 0.55 GB of kept rows take 112 us at the rate of a large copy).
// Longer prefixes are cut into stretches of up to 16384 keys, a workgroup each, which list the keys that can be among the
// largest (select_stretch_kernel); the unit's workgroup finds the kept ones among the listed (select_merge).  Where a
// stretch cannot list them (more than a quarter of it kept, very many equal scores) or pooled scores are asked for, one workgroup
// does it alone (select_long): it pools through LDS in tiles of 16384 positions (all loads of a tile in flight at once),
// keeps its keys in the pooled array in global memory and uses a radix select with LDS histograms, digits of up to
// 11 bits below the leading bits that all keys share (read off the largest and the smallest key).
// All counters are integers and the emission is ordered, so the result does not depend on scheduling.
#include <type_traits>

#include "pkv_internal.h"
#include "pkv_select_parts.h"

namespace pkv {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int TL = 16384;          // pooling tile of long prefixes (outputs per iteration)
constexpr int kLdsKeys = 32768;    // prefix lengths up to this keep their keys in registers
constexpr uint32_t kOpen = 512u;   // keys of a bin that are ranked against each other

// A wave-uniform value the compiler must treat as new: the lane masks of comparisons with it are formed where they are
// used instead of being kept (and spilled), 32 pairs of scalar registers, from an earlier use.
__device__ __forceinline__ int fresh(int v) {
  v = __builtin_amdgcn_readfirstlane(v);
  asm volatile("" : "+s"(v));
  return v;
}

// Number of set bits of m below this lane.
__device__ __forceinline__ uint32_t bits_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Inclusive scan over the workgroup, thread order.  `scratch` holds NW entries.
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t v, uint32_t* scratch, uint32_t* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  v = wave_inclusive_sum(v);
  __syncthreads();  // scratch may still be read from a previous use
  if (lane == 63) scratch[wave] = v;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint32_t s = scratch[w];
    if (w < wave) base += s;
    tot += s;
  }
  *total = tot;
  return v + base;
}


// A longer prefix, by one workgroup.
__device__ __forceinline__ void select_long(const float* raw, int nrb, size_t rb_stride, float inv_G, float* pooled, int32_t* idx, int npre, int kk, int alpha, int pool,
                                            int pool_w, uint32_t* lkeys, uint32_t* hist,
                                            uint32_t* scan32, uint32_t* sel) {
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const uint32_t* gkeys = reinterpret_cast<const uint32_t*>(pooled);

  // ---- A. group mean + pooling ----
  const int r = (pool == PKV_POOL_NONE) ? 0 : (pool_w - 1) / 2;
  const bool is_max = pool == PKV_POOL_MAX;
  const float inv_w = 1.0f / (float)pool_w;
  uint32_t gmax = 0u, gmin = 0xFFFFFFFFu;  // long prefixes: largest and smallest key this thread has produced
  // long prefixes: largest key of every group of 64 positions, in LDS behind the pooling tile (if they fit)
  constexpr int kGrpOff = 16512, kGrpCap = kLdsKeys - kGrpOff;
  static_assert(kGrpOff >= TL + 2 * (kMaxPoolW / 2), "group maxima lie behind the tile");
  uint32_t* grp = lkeys + kGrpOff;
  const int ngrp = (npre + 63) >> 6;
  const bool use_grp = ngrp <= kGrpCap;
  // fn(gi) for every group gi of [g_lo, g_hi), ascending, whose largest key is at least `bound`: 64 groups are
  // tested at a time, one per lane, and the wave then walks the set bits (all arguments wave-uniform)
  auto for_groups_at_least = [&](int g_lo, int g_hi, uint32_t bound, auto fn) {
    for (int g0 = g_lo; g0 < g_hi; g0 += 64) {
      const int gl = g0 + lane;
      unsigned long long m = __ballot(gl < g_hi && grp[gl] >= bound);
      while (m) {
        const int bsel = __ffsll((long long)m) - 1;
        m &= m - 1;
        fn(g0 + bsel);
      }
    }
  };
  {
    // Long prefix: tiles of TL outputs go through LDS, every load of a tile in flight at once; the pooled values
    // are the keys, kept in global memory.  On the way the largest and the smallest key are noted, and the largest
    // key of every group of 64 consecutive positions (kept in LDS behind the tile): later passes skip the groups
    // that cannot hold a key they look for, which is nearly all of them.
    float* lsc = reinterpret_cast<float*>(lkeys);
    constexpr int PT = TL / NT;  // outputs per thread and tile; one more load covers the 2 r halo positions
    static_assert(TL + 2 * (kMaxPoolW / 2) <= (PT + 1) * NT && TL + 2 * (kMaxPoolW / 2) <= kLdsKeys, "tile fits");
    float v[PT + 1];
    // the tile's scores (with the halo of r positions on both sides) into registers
    auto request_tile = [&](int t0) {
#pragma unroll
      for (int j = 0; j <= PT; ++j) {
        const int e = tid + NT * j, i = t0 - r + e;
        v[j] = 0.f;
        if (e < TL + 2 * r && i >= 0 && i < npre) v[j] = raw[i];
      }
      if (nrb > 1) {  // (kept apart: a loop of unknown length behind every load would make each wait for its own)
#pragma unroll
        for (int j = 0; j <= PT; ++j) {
          const int e = tid + NT * j, i = t0 - r + e;
          if (e < TL + 2 * r && i >= 0 && i < npre)
            for (int q = 1; q < nrb; ++q) v[j] += raw[q * rb_stride + i];
        }
      }
    };
    request_tile(0);
    for (int t0 = 0; t0 < npre; t0 += TL) {
      uint32_t wmax[PT];
#pragma unroll
      for (int j = 0; j <= PT; ++j) {
        const int e = tid + NT * j, i = t0 - r + e;
        if (e < TL + 2 * r) lsc[e] = (i >= 0 && i < npre) ? v[j] * inv_G : (is_max ? -INFINITY : 0.f);
      }
      lds_barrier();
      if (t0 + TL < npre) request_tile(t0 + TL);  // travels while this tile is pooled
      // window of 2 RR + 1 tile entries from the output's own slot on, in ascending position order; RR < 0: the
      // half-width is known at run time only.  (A compile-time width lets the LDS reads of all outputs of a thread
      // go out together instead of one dependent chain after the other.)
      auto pool_tile = [&](auto RR) {
        constexpr int R = decltype(RR)::value;
        const int w2 = R >= 0 ? 2 * R : 2 * r;
        constexpr int HB = 8;  // outputs worked on together (register budget)
#pragma unroll
        for (int j0 = 0; j0 < PT; j0 += HB) {
          float acc[HB];
#pragma unroll
          for (int j = 0; j < HB; ++j) acc[j] = lsc[tid + NT * (j0 + j)];
          if (R >= 0) {
#pragma unroll
            for (int u = 1; u <= (R >= 0 ? 2 * R : 0); ++u)
#pragma unroll
              for (int j = 0; j < HB; ++j) {
                const float x = lsc[tid + NT * (j0 + j) + u];
                acc[j] = is_max ? fmaxf(acc[j], x) : acc[j] + x;
              }
          } else {
            for (int u = 1; u <= w2; ++u)
#pragma unroll
              for (int j = 0; j < HB; ++j) {
                const float x = lsc[tid + NT * (j0 + j) + u];
                acc[j] = is_max ? fmaxf(acc[j], x) : acc[j] + x;
              }
          }
#pragma unroll
          for (int j = 0; j < HB; ++j) {
            const int i = t0 + tid + NT * (j0 + j);
            wmax[j0 + j] = 0u;
            if (i < npre) {
              const float y = (!is_max && w2 > 0) ? acc[j] * inv_w : acc[j];
              pooled[i] = y;
              wmax[j0 + j] = __float_as_uint(y);
              gmax = max(gmax, wmax[j0 + j]);
              gmin = min(gmin, wmax[j0 + j]);
            }
          }
        }
      };
      using std::integral_constant;
      if (r == 0) pool_tile(integral_constant<int, 0>{});
      else if (r == 1) pool_tile(integral_constant<int, 1>{});
      else if (r == 2) pool_tile(integral_constant<int, 2>{});
      else if (r == 3) pool_tile(integral_constant<int, 3>{});
      else pool_tile(integral_constant<int, -1>{});
      if (use_grp) {  // the 64 lanes of a wave hold 64 consecutive positions
#pragma unroll
        for (int j = 0; j < PT; ++j) {
          const uint32_t m = wave_max_lane63(wmax[j]);
          const int gi = (t0 + NT * j) / 64 + wave;
          if (lane == 63 && gi < ngrp) grp[gi] = m;
        }
      }
      lds_barrier();  // (the tile is rewritten next; the pooled values are read only after the loop)
    }
    __syncthreads();  // the keys in global memory and the group maxima are complete
  }

  if (kk > 0) {
    // ---- B. the kk-th largest key ----
    uint32_t prefix = 0;
    uint32_t remaining = (uint32_t)kk;
    {
      // Keys in global memory: radix select.  The leading bits that all keys share are T's as well and are read off
      // the largest and the smallest key; below them digits of up to 11 bits, most significant first, each with an
      // LDS histogram over the keys that agree with the digits decided so far.  (Starting at the first bit in which
      // keys differ also spreads the first digit over many bins: scores span a few binades, and a digit made of
      // sign and exponent bits would send nearly every key to the same few counters.)  Every thread has its 16
      // loads of a round in flight before it counts.
#pragma unroll
      for (int sft = 32; sft > 0; sft >>= 1) {
        gmax = max(gmax, (uint32_t)__shfl_xor((int)gmax, sft));
        gmin = min(gmin, (uint32_t)__shfl_xor((int)gmin, sft));
      }
      if (lane == 0) {
        scan32[wave] = gmax;
        scan32[NW + wave] = gmin;
      }
      __syncthreads();
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        gmax = max(gmax, scan32[w]);
        gmin = min(gmin, scan32[NW + w]);
      }
      __syncthreads();
      const uint32_t diff = gmax ^ gmin;
      int top = (diff == 0u) ? 0 : 32 - __clz((int)diff);  // undecided low bits
      prefix = (top >= 32) ? 0u : (gmax >> top) << top;
      constexpr int NB = 16;  // keys per thread and round
      bool first_level = true;
      while (top > 0) {
        const int nb = min(11, top), shift = top - nb;
        const uint32_t dmask = (1u << nb) - 1u;
        for (int e = tid; e < HIST; e += NT) hist[e] = 0;
        __syncthreads();
        if (use_grp && !first_level) {
          // an open key is at least `prefix` (its decided bits, zeros below): only groups whose largest key reaches
          // that can hold one
          const int gw = (ngrp + NW - 1) / NW;  // groups per wave
          for_groups_at_least(wave * gw, min(wave * gw + gw, ngrp), prefix, [&](int gi) {
            const int i = 64 * gi + lane;
            const uint32_t key = i < npre ? gkeys[i] : 0u;
            if (i < npre && (key >> top) == (prefix >> top)) atomicAdd(&hist[(key >> shift) & dmask], 1u);
          });
        } else {
          for (int i0 = 0; i0 < npre; i0 += NB * NT) {
            uint32_t key[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              const int i = i0 + tid + NT * j;
              key[j] = i < npre ? gkeys[i] : 0u;
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              const int i = i0 + tid + NT * j;
              const bool open = top >= 32 || (key[j] >> top) == (prefix >> top);
              if (i < npre && open) atomicAdd(&hist[(key[j] >> shift) & dmask], 1u);
            }
          }
        }
        first_level = false;
        __syncthreads();
        // thread t owns bins 2t, 2t+1; suffix sums over the bins owned by higher threads
        const uint32_t h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
        uint32_t total;
        const uint32_t incl = block_inclusive_scan(h0 + h1, scan32, &total);
        uint32_t above = total - incl;
        if (above < remaining && above + h1 >= remaining) {
          sel[0] = (uint32_t)(2 * tid + 1);
          sel[1] = above;
        }
        above += h1;
        if (above < remaining && above + h0 >= remaining) {
          sel[0] = (uint32_t)(2 * tid);
          sel[1] = above;
        }
        __syncthreads();
        prefix |= sel[0] << shift;
        remaining -= sel[1];
        top = shift;
        __syncthreads();
      }
    }
    const uint32_t T = prefix;           // bit pattern of the kk-th largest pooled score

    // ---- C. ordered emission ----
    {
      // every wave owns a contiguous range of positions; two passes over its keys (count, then emit).  With the
      // group maxima at hand only the groups that hold a key >= T are read; else eight groups of 64 positions per
      // round with their loads in flight together.
      constexpr int NE = 8;
      const int cw = ((npre + NW - 1) / NW + 63) & ~63;  // positions per wave, multiple of 64
      const int w0 = min(wave * cw, npre), w1 = min(w0 + cw, npre);
      uint32_t cgt = 0, ceq = 0;
      if (use_grp) {
        for_groups_at_least(w0 >> 6, w0 < w1 ? (w1 + 63) >> 6 : w0 >> 6, T, [&](int gi) {
          const int i = 64 * gi + lane;
          const uint32_t key = i < w1 ? gkeys[i] : 0u;
          cgt += __popcll(__ballot(i < w1 && key > T));
          ceq += __popcll(__ballot(i < w1 && key == T));
        });
      } else {
        for (int base = w0; base < w1; base += 64 * NE) {
          uint32_t key[NE];
#pragma unroll
          for (int j = 0; j < NE; ++j) {
            const int i = base + 64 * j + lane;
            key[j] = i < w1 ? gkeys[i] : 0u;
          }
#pragma unroll
          for (int j = 0; j < NE; ++j) {
            const int i = base + 64 * j + lane;
            cgt += __popcll(__ballot(i < w1 && key[j] > T));
            ceq += __popcll(__ballot(i < w1 && key[j] == T));
          }
        }
      }
      __syncthreads();
      if (lane == 0) {
        hist[wave] = cgt;
        hist[NW + wave] = ceq;
      }
      __syncthreads();
      uint32_t gt_before = 0, eq_before = 0, gt_total = 0;
      for (int w = 0; w < NW; ++w) {
        gt_total += hist[w];
        if (w < wave) {
          gt_before += hist[w];
          eq_before += hist[NW + w];
        }
      }
      const uint32_t need_eq = (uint32_t)kk - gt_total;  // keys equal to T to take, lowest positions first (>= 1)
      const unsigned long long lt_mask = (1ull << lane) - 1ull;
      // the 64 positions from `base` on, their keys in `key`: kept ones go to their ranks
      auto emit64 = [&](int base, uint32_t key) {
        const int i = base + lane;
        const bool gt = i < w1 && key > T, eq = i < w1 && key == T;
        const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
        if ((bgt | beq) == 0) return;
        const uint32_t gtb = gt_before + __popcll(bgt & lt_mask);
        const uint32_t eqb = eq_before + __popcll(beq & lt_mask);
        if (gt) idx[gtb + min(eqb, need_eq)] = i;
        if (eq && eqb < need_eq) idx[gtb + eqb] = i;
        gt_before += __popcll(bgt);
        eq_before += __popcll(beq);
      };
      if (use_grp) {
        for_groups_at_least(w0 >> 6, w0 < w1 ? (w1 + 63) >> 6 : w0 >> 6, T, [&](int gi) {
          const int i = 64 * gi + lane;
          emit64(64 * gi, i < w1 ? gkeys[i] : 0u);
        });
      } else {
        for (int base = w0; base < w1; base += 64 * NE) {
          uint32_t key[NE];
#pragma unroll
          for (int j = 0; j < NE; ++j) {
            const int i = base + 64 * j + lane;
            key[j] = i < w1 ? gkeys[i] : 0u;
          }
#pragma unroll
          for (int j = 0; j < NE; ++j) emit64(base + 64 * j, key[j]);
        }
      }
    }
  }
  for (int t = tid; t < alpha; t += NT) idx[kk + t] = npre + t;
}


// The need-th largest of the n_open distances in hist (entries behind the last are 0), plus lo: every distance counts those
// above it and those not below it.  Needs n_open <= NT.
__device__ __forceinline__ uint32_t rank_open(const uint32_t* hist, uint32_t n_open, uint32_t need, uint32_t lo, uint32_t* sel) {
  lds_barrier();
  if (threadIdx.x < n_open) {
    const uint32_t d = hist[threadIdx.x];
    uint32_t above = 0u, from = 0u;
    for (uint32_t j = 0; j < n_open; j += 4) {
      const u32x4 q = *reinterpret_cast<const u32x4*>(hist + j);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        above += q[c] > d ? 1u : 0u;
        from += q[c] >= d ? 1u : 0u;
      }
    }
    if (above < need && need <= from) sel[1] = lo + d;
  }
  lds_barrier();
  return __builtin_amdgcn_readfirstlane(sel[1]);
}

// A prefix of at most 1024 * PER keys.  Wave w owns positions [w * 64 * PER, (w + 1) * 64 * PER), lane l of it the four
// from 256 * jj + 4 * l on, for every jj.  Returns true when the kept prefix positions are left in LDS (`keep`, kk
// ascending entries), false when they have been written to idx instead.
template <int PER, int PMAX>
__device__ __forceinline__ bool select_short(const SelectBatchArgs& a, const float* raw, size_t rb_stride, float* pooled,
                                             int32_t* idx, int npre, int kk, uint32_t* area, uint32_t* hist,
                                             uint32_t* scan, uint32_t* sel, uint16_t* keep) {
  constexpr int NJ = PER / 4;
  constexpr int CW = 64 * PER;
  constexpr uint32_t kCap = PMAX * 512;  // entries of the list (key, position) and of `keep`: 8 bytes each of `area`
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w0 = wave * CW;
  const int p0 = w0 + 4 * lane;
  const int r = (a.pool == PKV_POOL_NONE) ? 0 : (a.pool_w - 1) / 2;
  const bool is_max = a.pool == PKV_POOL_MAX;

  // ---- A. group mean + pooling ----
  Scores<NJ> s;
  f32x4* v = s.v;
  int lim = npre - p0;  // the thread's position 256 * jj + c exists iff 256 * jj + c < lim
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) {
    const int g0 = w0 + 256 * jj, p = p0 + 256 * jj;  // first position of the wave's 256, of the thread's four
    v[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (g0 + 256 <= npre) v[jj] = *reinterpret_cast<const f32x4_u*>(raw + p);
    else if (g0 < npre) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (256 * jj + c < lim) v[jj][c] = raw[p + c];
    }
  }
  for (int q = 1; q < a.nrb; ++q) {
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (256 * jj + c < lim) v[jj][c] += raw[q * rb_stride + p0 + 256 * jj + c];
  }
  reinterpret_cast<uint2*>(hist)[tid] = make_uint2(0u, 0u);
  if (tid == 0) sel[3] = 0u;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) v[jj] *= a.inv_G;
  if (r > 0) {
    float* lsc = reinterpret_cast<float*>(area) + kPad;
    lim = fresh(npre) - p0;
    const float neutral = is_max ? -INFINITY : 0.f;
    if (tid < kPad) {
      lsc[tid - kPad] = neutral;
      lsc[NT * PER + tid] = neutral;
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const int g0 = w0 + 256 * jj, p = p0 + 256 * jj;
      if (g0 < npre + kPad) {
        f32x4 t = v[jj];
        if (g0 + 256 > npre) {
#pragma unroll
          for (int c = 0; c < 4; ++c) t[c] = 256 * jj + c < lim ? t[c] : neutral;
        }
        *reinterpret_cast<f32x4*>(lsc + p) = t;
      }
    }
    lds_barrier();
    s = pool_lds(lsc, p0, w0, npre, r, is_max, a.pool_w, s);
  }
  uint32_t key[NJ][4];  // 0: no such position
  lim = fresh(npre) - p0;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
    for (int c = 0; c < 4; ++c) key[jj][c] = 256 * jj + c < lim ? __float_as_uint(v[jj][c]) : 0u;
  if (pooled) {
    lim = fresh(npre) - p0;
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (256 * jj + c < lim) pooled[p0 + 256 * jj + c] = v[jj][c];
  }
  if (kk == 0) return true;

  // ---- B. the kk-th largest key ----
  uint32_t kmax = 0u;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
    for (int c = 0; c < 4; ++c) kmax = max(kmax, key[jj][c]);
  // A reference below the few outstanding keys (an attention sink stands many binades above all others): in every wave
  // the smallest of the largest keys of its four rows of 16 lanes, and the largest of these over the waves.
  kmax = row_max_lane15(kmax);
  {
    const uint32_t m = min(min((uint32_t)__builtin_amdgcn_readlane((int)kmax, 15), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 31)),
                           min((uint32_t)__builtin_amdgcn_readlane((int)kmax, 47), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 63)));
    if (lane == 0) scan[wave] = m;
  }
  lds_barrier();  // (also: every thread is done with the scores in `area`)
  const uint32_t ref = (uint32_t)__builtin_amdgcn_readlane((int)row_max_lane15(scan[lane & 15]), 15);

  uint32_t* lkey = area;                                         // [kCap]
  uint16_t* lpos = reinterpret_cast<uint16_t*>(area + kCap);      // [kCap]; `keep` lies behind it
  // groups of gs keys (a power of two, at most NJ): at least twice as many groups as keys to select, so that the bound
  // is not much below T.  A group's keys lie 256 positions apart: neighbours share a pooling window.
  int gs = 1;
  while (2 * gs <= NJ && 4 * gs * kk <= npre) gs *= 2;
  const KeyBins<HIST> bins{ref};
  auto bin_of = [&](uint32_t k) { return bins.of(k); };
  auto lower_edge = [&](uint32_t bin) { return bins.lower_edge(bin); };
  auto upper_edge = [&](uint32_t bin) { return bins.upper_edge(bin); };
  uint32_t n_list = 0u, T = 0u, lo = 0u, hi = 0u, need = (uint32_t)kk, n_open = 0u;  // (T's bin: edges, rank in it, keys)
  bool ok = false, have_bin = false;
  // The list pays for small shares of the prefix.  256 units of 32k keys, with and without it: kk = 0.02 of the prefix 22 and
  // 30 us, 0.1 27 and 32, 0.2 32 and 34, 0.3 38 and 37, 0.5 42 and 39; of 8k keys 15 and 16, 13 and 14, 14 and 14, 16 and 15,
  // 17 and 15.
  if (4 * kk <= npre) {  // (uniform)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      uint32_t m = 0u;
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj) {
        m = max(m, key[jj][c]);
        if (((jj + 1) & (gs - 1)) == 0) {  // uniform
          if (m != 0u) atomicAdd(&hist[bin_of(m)], 1u);
          m = 0u;
        }
      }
    }
    lds_barrier();
    if (find_bin(hist, (uint32_t)kk, scan + NW, sel) >= (uint32_t)kk) {
      // the keys at or above the bound: counted per wave, then listed in position order
      const uint32_t bound = lower_edge(__builtin_amdgcn_readfirstlane(sel[0]));
      uint32_t cnt = 0u;
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
        for (int c = 0; c < 4; ++c) cnt += (uint32_t)__popcll(__ballot(key[jj][c] >= bound));
      if (lane == 0) scan[wave] = cnt;
      lds_barrier();
      uint32_t base = sum_before(scan, wave, n_list);
      ok = n_list <= kCap;  // (uniform)
      if (ok && cnt != 0u) {
        const uint32_t bnd = (uint32_t)fresh((int)bound);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
          unsigned long long b[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) b[c] = __ballot(key[jj][c] >= bnd);
          if ((b[0] | b[1] | b[2] | b[3]) == 0ull) continue;
          uint32_t at = base + bits_below(b[0]) + bits_below(b[1]) + bits_below(b[2]) + bits_below(b[3]);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if (key[jj][c] >= bnd) {
              lkey[at] = key[jj][c];
              lpos[at] = (uint16_t)(p0 + 256 * jj + c);
              ++at;
            }
          }
          base += (uint32_t)(__popcll(b[0]) + __popcll(b[1]) + __popcll(b[2]) + __popcll(b[3]));
        }
      }
    }
  }
  if (ok) {
    lds_barrier();  // the list is complete
    for (uint32_t i = tid; i < n_list; i += NT) atomicAdd(&hist[bin_of(lkey[i])], 1u);
    lds_barrier();
    (void)find_bin(hist, (uint32_t)kk, scan + NW, sel);  // (there is such a bin: the list holds at least kk keys)
    const uint32_t bin = __builtin_amdgcn_readfirstlane(sel[0]);
    need = (uint32_t)kk - __builtin_amdgcn_readfirstlane(sel[1]);
    n_open = __builtin_amdgcn_readfirstlane(sel[2]);
    lo = lower_edge(bin);
    if (need == n_open) {
      T = lo - 1u;  // the whole bin is kept
    } else if (n_open <= kOpen) {
      // the bin's keys, as distances from its edge, in hist (cleared by find_bin); their order does not matter.  They are
      // counted in sel[3], which nothing else uses: other waves may still be reading the bin from sel[0].
      for (uint32_t i = tid; i < n_list; i += NT) {
        const uint32_t k = lkey[i];
        if (bin_of(k) == bin) hist[atomicAdd(&sel[3], 1u)] = k - lo;
      }
      T = rank_open(hist, n_open, need, lo, sel);
    } else {
      hi = upper_edge(bin);
      have_bin = true;
      ok = false;
    }
  }
  if (ok) {
    // ---- C. ordered emission from the list, wave w its w-th stretch ----
    const uint32_t seg = ((n_list + NW - 1) / NW + 63u) & ~63u;
    const uint32_t e0 = min(wave * seg, n_list), e1 = min(e0 + seg, n_list);
    uint32_t cgt = 0u, ceq = 0u;
    for (uint32_t i0 = e0; i0 < e1; i0 += 64) {
      const uint32_t k = i0 + lane < e1 ? lkey[i0 + lane] : 0u;
      cgt += (uint32_t)__popcll(__ballot(k > T));
      ceq += (uint32_t)__popcll(__ballot(k == T && i0 + lane < e1));
    }
    if (lane == 0) {
      scan[wave] = cgt;
      scan[NW + wave] = ceq;
    }
    lds_barrier();
    uint32_t gt_total, eq_total;
    uint32_t gt_before = sum_before(scan, wave, gt_total), eq_before = sum_before(scan + NW, wave, eq_total);
    const uint32_t need_eq = (uint32_t)kk - gt_total;
    for (uint32_t i0 = e0; i0 < e1; i0 += 64) {
      const bool in = i0 + lane < e1;
      const uint32_t k = in ? lkey[i0 + lane] : 0u;
      const bool gt = k > T, eq = in && k == T;
      const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
      const uint32_t gtb = gt_before + bits_below(bgt), eqb = eq_before + bits_below(beq);
      if (gt) keep[gtb + min(eqb, need_eq)] = lpos[i0 + lane];
      if (eq && eqb < need_eq) keep[gtb + eqb] = lpos[i0 + lane];
      gt_before += (uint32_t)__popcll(bgt);
      eq_before += (uint32_t)__popcll(beq);
    }
    lds_barrier();
    return true;
  }

  // ---- without a list: histograms over all keys, the first one as above, the next ones over the keys of the bin found, in
  // 2048 parts, until few keys are left in it or all of them are equal.  A thread adds up runs of keys of one bin (pooling
  // windows share their largest score) before it touches the histogram.  Keys of 0 are counted nowhere: if the others are
  // fewer than kk, T is 0.  Measured against a search of T over all keys, one bit per round: 256 units of 32k keys, kk = 0.6
  // or 0.95 of the prefix, 58 - 61 -> 40 us; 7 / 8 of the scores exact zeros, kk = 0.6, 77 -> 37 us ----
  auto count_keys = [&](auto is_open, auto bin_fn) {
    uint32_t run_bin = 0u, run = 0u;
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const uint32_t k = key[jj][c];
        if (is_open(k)) {
          const uint32_t bin = bin_fn(k);
          if (bin != run_bin) {
            if (run != 0u) atomicAdd(&hist[run_bin], run);
            run_bin = bin;
            run = 0u;
          }
          ++run;
        }
      }
    if (run != 0u) atomicAdd(&hist[run_bin], run);
    lds_barrier();
  };
  if (!have_bin) {
    count_keys([](uint32_t k) { return k != 0u; }, bin_of);
    have_bin = find_bin(hist, need, scan + NW, sel) >= need;
    if (have_bin) {
      const uint32_t bin = __builtin_amdgcn_readfirstlane(sel[0]);
      need -= __builtin_amdgcn_readfirstlane(sel[1]);
      n_open = __builtin_amdgcn_readfirstlane(sel[2]);
      lo = lower_edge(bin);
      hi = upper_edge(bin);
    }
  }
  if (have_bin) {
    while (need != n_open && n_open > kOpen && lo != hi) {
      const int bits = 32 - __clz((int)(hi - lo)), part = bits > 11 ? bits - 11 : 0;
      count_keys([&](uint32_t k) { return k >= lo && k <= hi; }, [&](uint32_t k) { return (hi - k) >> part; });
      (void)find_bin(hist, need, scan + NW, sel);
      const uint32_t bin = __builtin_amdgcn_readfirstlane(sel[0]);
      need -= __builtin_amdgcn_readfirstlane(sel[1]);
      n_open = __builtin_amdgcn_readfirstlane(sel[2]);
      hi -= bin << part;
      if (((hi - lo) >> part) != 0u) lo = hi - (1u << part) + 1u;
    }
    if (need == n_open) {
      T = lo - 1u;
    } else if (lo == hi) {
      T = lo;
    } else {
#pragma unroll
      for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          if (key[jj][c] >= lo && key[jj][c] <= hi) hist[atomicAdd(&sel[3], 1u)] = key[jj][c] - lo;
      T = rank_open(hist, n_open, need, lo, sel);
    }
  }
  uint32_t cgt = 0u, ceq = 0u;
  lim = fresh(npre) - p0;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      cgt += (uint32_t)__popcll(__ballot(key[jj][c] > T));
      ceq += (uint32_t)__popcll(__ballot(key[jj][c] == T && 256 * jj + c < lim));
    }
  __syncthreads();
  if (lane == 0) {
    scan[wave] = cgt;
    scan[NW + wave] = ceq;
  }
  __syncthreads();
  uint32_t gt_total, eq_total;
  uint32_t gt_before = sum_before(scan, wave, gt_total), eq_before = sum_before(scan + NW, wave, eq_total);
  const uint32_t need_eq = (uint32_t)kk - gt_total;  // keys equal to T to take, lowest positions first
  lim = fresh(npre) - p0;
  T = (uint32_t)fresh((int)T);
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) {
    unsigned long long bg[4], be[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      bg[c] = __ballot(key[jj][c] > T);
      be[c] = __ballot(key[jj][c] == T && 256 * jj + c < lim);
    }
    uint32_t gtb = gt_before, eqb = eq_before;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      gtb += bits_below(bg[c]);
      eqb += bits_below(be[c]);
      gt_before += (uint32_t)__popcll(bg[c]);
      eq_before += (uint32_t)__popcll(be[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int i = p0 + 256 * jj + c;
      if (key[jj][c] > T) {
        idx[gtb + min(eqb, need_eq)] = i;
        ++gtb;
      } else if (key[jj][c] == T && 256 * jj + c < lim) {
        if (eqb < need_eq) idx[gtb + eqb] = i;
        ++eqb;
      }
    }
  }
  return false;
}

// The kept rows' K and V of a unit, pos(j) the position of row j (-1: unused slot, the row is cleared).
template <class Pos>
__device__ __forceinline__ void gather_unit(const GatherBatchArgs& ga, const GatherLayer& gl, int b, int g, Pos pos) {
  const int sh = ga.d == 128 ? 4 : 3;  // 16 or 8 lanes per row
  const int total = gl.k_cap << sh;
  // four row segments per thread and round, each stage (positions, rows, stores) issued for all four before the
  // next one
  constexpr int NB = 4;
  const size_t head_off = (size_t)b * ga.kv_sb + (size_t)g * ga.kv_sh;
  const size_t out_off = (size_t)b * gl.o_sb + (size_t)g * gl.o_sh;
  for (int t0 = threadIdx.x; t0 < total; t0 += NB * NT) {
    int src[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int t = t0 + u * NT;
      src[u] = t < total ? pos(t >> sh) : -1;
    }
    u32x4 kv[NB], vv[NB];
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int seg = (t0 + u * NT) & ((1 << sh) - 1);
      kv[u] = u32x4{0u, 0u, 0u, 0u};
      vv[u] = kv[u];
      if ((uint32_t)src[u] < (uint32_t)ga.N) {  // nothing outside [0, N) is dereferenced
        const size_t off = head_off + (size_t)src[u] * ga.kv_st + seg * 8;
        kv[u] = *reinterpret_cast<const u32x4*>(gl.K + off);
        vv[u] = *reinterpret_cast<const u32x4*>(gl.V + off);
      }
    }
#pragma unroll
    for (int u = 0; u < NB; ++u) {
      const int t = t0 + u * NT;
      if (t < total) {
        const size_t o = out_off + (size_t)(t >> sh) * gl.o_st + (t & ((1 << sh) - 1)) * 8;
        *reinterpret_cast<u32x4*>(gl.K_out + o) = kv[u];
        *reinterpret_cast<u32x4*>(gl.V_out + o) = vv[u];
      }
    }
  }
}

// ---- prefixes beyond 32768 keys, first step: candidates ----
// The prefix is cut into stretches of nearly equal length, a workgroup each.  A workgroup pools its stretch and lists the
// keys that can be among the unit's kk largest: those at or above a bound that at least kk keys of the stretch reach.  The
// lists (keys, positions within the stretch, their number, the bound and the reference of the bins) lie in the unit's
// array for pooled scores, at the stretch's own place.  The kk largest of the unit are found among the listed keys then
// (select_merge).  What bounds it: for few units the latency of a dozen steps between barriers, twice (17 and 14 us); for
// many some 25 vector operations per key beside the read of the scores (256 units of 128k keys: 80 us, 26 of them the read
// alone).  Measured against one workgroup per unit, whole calls: one layer of 8 units of 128k keys 190 -> 138 us, of 50k
// 119 -> 88, 4 layers of 100k keys, 1024 kept, 441 -> 386, 32 layers of 128k 3222 -> 3207.  Stretches of 8192 keys by 256
// threads: 137, 88, 386; 16 layers of 60k keys 442 instead of 436, 8 of 40k 376 instead of 369.
constexpr int kMaxStretches = 64;       // a lane of a wave each
constexpr int kStretchThreads = 512;
constexpr int kStretch = 16384;         // keys a workgroup holds in registers
constexpr int kStretchWords = kStretch + 2 * kPad;
constexpr int kStretchBins = 1024;
constexpr uint32_t kNoList = 0xFFFFFFFFu;
struct Stretches {
  int count, len;  // count 0: the unit is left to select_long; the last stretch may be shorter
};
// A stretch must hold four keys per key to select, for the bound to be worth its while, and no pooled scores may be asked
// for (they would lie where the lists do).
__host__ __device__ inline int stretch_count(int npre) { return (npre + kStretch - 1) / kStretch; }
__device__ __forceinline__ Stretches stretches(int npre, int kk, bool listed, bool write_pooled) {
  if (!listed || write_pooled || kk <= 0 || npre <= kLdsKeys) return {0, 0};
  const int p = stretch_count(npre);
  if (p > kMaxStretches) return {0, 0};
  const int len = ((npre + p - 1) / p + 63) & ~63;
  const int last = npre - (p - 1) * len;
  return {last >= 64 && 4 * kk <= last ? p : 0, len};
}

__global__ __launch_bounds__(kStretchThreads, 4) void select_stretch_kernel(const SelectBatchArgs a) {
  constexpr int NTA = kStretchThreads, NJ = kStretch / (4 * NTA), CW = 64 * 4 * NJ, NWA = NTA / 64, OWN = kStretchBins / NTA;
  extern __shared__ uint32_t area[];  // kStretchWords entries
  __shared__ uint32_t hist[kStretchBins];
  __shared__ uint32_t scan[2 * NWA];
  __shared__ uint32_t sel[1];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int BH = a.B * a.Hkv;
  const int l = (int)blockIdx.y / BH;
  const int bg = (int)blockIdx.y - l * BH;
  const SelectLayer& ly = a.layer[l];
  int n = a.N;
  if (a.seq_lens) {
    n = a.seq_lens[bg / a.Hkv];
    n = n < 0 ? 0 : (n > a.N ? a.N : n);
  }
  if (ly.k_l >= n) return;
  if (a.flags && a.flags[(size_t)l * BH + bg] == 0) return;  // (the kept set is there)
  const int npre = n - a.alpha, kk = ly.k_l - a.alpha;
  const Stretches st = stretches(npre, kk, a.listed != 0, ly.write_pooled != 0);
  if ((int)blockIdx.x >= st.count) return;
  const int t0 = (int)blockIdx.x * st.len;
  const int len = min(st.len, npre - t0);       // keys of the stretch
  const int have = min(len + kPad, npre - t0);  // scores behind its first one that are looked at
  const size_t rb_stride = (size_t)BH * a.N;
  const float* raw = a.raw + ((size_t)l * a.nrb * BH + bg) * a.N + t0;
  uint32_t* out = reinterpret_cast<uint32_t*>(ly.pooled) + (size_t)bg * a.N + t0;

  // ---- group mean + pooling (as select_short has it) ----
  const int w0 = wave * CW, p0 = w0 + 4 * lane;
  const int r = (a.pool == PKV_POOL_NONE) ? 0 : (a.pool_w - 1) / 2;
  const bool is_max = a.pool == PKV_POOL_MAX;
  Scores<NJ> s;
  f32x4* v = s.v;
  int lim = have - p0;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) {
    const int g0 = w0 + 256 * jj, p = p0 + 256 * jj;
    v[jj] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (g0 + 256 <= have) v[jj] = *reinterpret_cast<const f32x4_u*>(raw + p);
    else if (g0 < have) {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (256 * jj + c < lim) v[jj][c] = raw[p + c];
    }
  }
  // the scores around them: 32 before the stretch, 32 behind the last position of any thread
  const float neutral = is_max ? -INFINITY : 0.f;
  const int pe = tid < kPad ? tid - kPad : kStretch + tid - kPad;
  const bool edge = tid < 2 * kPad && t0 + pe >= 0 && pe < have;
  float ve = edge ? raw[pe] : 0.f;
  for (int q = 1; q < a.nrb; ++q) {
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (256 * jj + c < lim) v[jj][c] += raw[q * rb_stride + p0 + 256 * jj + c];
    if (edge) ve += raw[q * rb_stride + pe];
  }
#pragma unroll
  for (int u = 0; u < OWN; ++u) hist[tid + NTA * u] = 0u;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) v[jj] *= a.inv_G;
  if (r > 0) {
    float* lsc = reinterpret_cast<float*>(area) + kPad;
    if (tid < 2 * kPad) lsc[pe] = edge ? ve * a.inv_G : neutral;
    lim = fresh(have) - p0;
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const int g0 = w0 + 256 * jj, p = p0 + 256 * jj;
      if (g0 < len + kPad) {
        f32x4 t = v[jj];
        if (g0 + 256 > have) {
#pragma unroll
          for (int c = 0; c < 4; ++c) t[c] = 256 * jj + c < lim ? t[c] : neutral;
        }
        *reinterpret_cast<f32x4*>(lsc + p) = t;
      }
    }
    lds_barrier();
    s = pool_lds(lsc, p0, w0, len, r, is_max, a.pool_w, s);
  }
  uint32_t key[NJ][4];  // 0: no such position
  lim = fresh(len) - p0;
  uint32_t kmax = 0u;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      key[jj][c] = 256 * jj + c < lim ? __float_as_uint(v[jj][c]) : 0u;
      kmax = max(kmax, key[jj][c]);
    }

  // ---- the bound: reference, histogram over the largest of every group, the bin in which kk is reached ----
  kmax = row_max_lane15(kmax);
  {
    const uint32_t m = min(min((uint32_t)__builtin_amdgcn_readlane((int)kmax, 15), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 31)),
                           min((uint32_t)__builtin_amdgcn_readlane((int)kmax, 47), (uint32_t)__builtin_amdgcn_readlane((int)kmax, 63)));
    if (lane == 0) scan[wave] = m;
  }
  if (tid == 0) sel[0] = kNoList;
  lds_barrier();  // (also: the histogram is cleared)
  KeyBins<kStretchBins> bins{0u};
#pragma unroll
  for (int w = 0; w < NWA; ++w) bins.ref = max(bins.ref, scan[w]);
  bins.ref = __builtin_amdgcn_readfirstlane(bins.ref);
  // groups of gs of a thread's keys, at least twice as many as keys to select
  int gs = 1;
  while (gs < 4 * NJ && 4 * gs * kk <= len) gs *= 2;
  uint32_t m = 0u;
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      m = max(m, key[jj][c]);
      if (((NJ * c + jj + 1) & (gs - 1)) == 0) {  // uniform
        if (m != 0u) atomicAdd(&hist[bins.of(m)], 1u);
        m = 0u;
      }
    }
  lds_barrier();
  {
    uint32_t h[OWN], sum = 0u;  // thread t owns bins OWN * t ..
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      h[u] = hist[OWN * tid + u];
      sum += h[u];
    }
    const uint32_t incl = wave_inclusive_sum(sum);
    if (lane == 63) scan[NWA + wave] = incl;
    lds_barrier();
    uint32_t at = incl - sum;
    for (int w = 0; w < wave; ++w) at += scan[NWA + w];
#pragma unroll
    for (int u = 0; u < OWN; ++u) {
      if (at < (uint32_t)kk && at + h[u] >= (uint32_t)kk) sel[0] = (uint32_t)(OWN * tid + u);
      at += h[u];
    }
  }
  lds_barrier();
  const uint32_t bin = __builtin_amdgcn_readfirstlane(sel[0]);
  const uint32_t bound = bin == kNoList ? kNoList : bins.lower_edge(bin);

  // ---- the list, in position order ----
  uint32_t cnt = 0u;
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
    for (int c = 0; c < 4; ++c) cnt += (uint32_t)__popcll(__ballot(key[jj][c] >= bound));
  if (lane == 0) scan[wave] = cnt;
  lds_barrier();
  uint32_t base = 0u, total = 0u;
#pragma unroll
  for (int w = 0; w < NWA; ++w) {
    base += w < wave ? scan[w] : 0u;
    total += scan[w];
  }
  base = __builtin_amdgcn_readfirstlane(base);
  total = __builtin_amdgcn_readfirstlane(total);
  const int cap = len / 2;  // keys, behind them half as many words of positions, at the end three words about the list
  const bool fits = bin != kNoList && total <= (uint32_t)cap && (len - cap - (cap + 1) / 2) >= 3;
  if (tid == 0) {
    out[len - 3] = fits ? total : kNoList;
    out[len - 2] = bound;
    out[len - 1] = bins.ref;
  }
  if (!fits || cnt == 0u) return;
  uint16_t* pos = reinterpret_cast<uint16_t*>(out + cap);
#pragma unroll
  for (int jj = 0; jj < NJ; ++jj) {
    unsigned long long b[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) b[c] = __ballot(key[jj][c] >= bound);
    if ((b[0] | b[1] | b[2] | b[3]) == 0ull) continue;
    uint32_t at = base + bits_below(b[0]) + bits_below(b[1]) + bits_below(b[2]) + bits_below(b[3]);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (key[jj][c] >= bound) {
        out[at] = key[jj][c];
        pos[at] = (uint16_t)(p0 + 256 * jj + c);
        ++at;
      }
    }
    base += (uint32_t)(__popcll(b[0]) + __popcll(b[1]) + __popcll(b[2]) + __popcll(b[3]));
  }
}

// The second step: the kk largest of the listed keys, their positions in ascending order in `keep` (LDS).  False, and nothing
// left behind, if a stretch has no list or more than kOpen keys share the bin of the kk-th largest.  The largest bound of
// any stretch is a bound for the unit: its own stretch holds kk keys that reach it.  Wave w takes the w-th of 16 parts of
// the lists; the keys are read again in every pass (they are few, and near).
__device__ __forceinline__ bool select_merge(const uint32_t* lists, const Stretches st, int npre, int kk, uint32_t* keep,
                                             uint32_t* tab, uint32_t* hist, uint32_t* scan, uint32_t* sel) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t cnt = 0u, bound = 0u, ref = 0u;
  if (lane < st.count) {
    const uint32_t* foot = lists + min((lane + 1) * st.len, npre) - 3;
    cnt = foot[0];
    bound = foot[1];
    ref = foot[2];
  }
  reinterpret_cast<uint2*>(hist)[tid] = make_uint2(0u, 0u);
  if (tid == 0) sel[3] = 0u;
  if (__ballot(cnt == kNoList) != 0ull) return false;  // (the same in every wave)
  bound = (uint32_t)__builtin_amdgcn_readlane((int)wave_max_lane63(bound), 63);
  const KeyBins<HIST> bins{(uint32_t)__builtin_amdgcn_readlane((int)wave_max_lane63(ref), 63)};
  const int psh = st.count <= 4 ? 2 : st.count <= 8 ? 1 : 0;  // parts per stretch
  const int pieces = st.count << psh;
  // fn(keys of a chunk, lane l those 64 u + l from its first entry on (0 behind the last), piece, first chunk of the piece,
  // first position of the stretch, positions of the chunk) for the wave's pieces; a wave whose one piece is one chunk reads it
  // once and for all
  constexpr int U = 8;
  struct Chunk {
    uint32_t x[U];
  };
  auto load = [&](const uint32_t* k, int left) {
    Chunk c;
#pragma unroll
    for (int u = 0; u < U; ++u) c.x[u] = 64 * u + lane < left ? k[64 * u + lane] : 0u;
    return c;
  };
  struct Piece {
    int t0, e0, e1, cap;
  };
  auto piece = [&](int p) -> Piece {
    const int s = p >> psh, part = p & ((1 << psh) - 1);
    const int t0 = s * st.len, c = __builtin_amdgcn_readlane((int)cnt, s);
    const int seg = (((c + (1 << psh) - 1) >> psh) + 63) & ~63;
    const int e0 = min(part * seg, c);
    return {t0, e0, min(e0 + seg, c), min(st.len, npre - t0) / 2};
  };
  const Piece first = piece(min(wave, pieces - 1));
  const bool one = pieces <= NW && first.e1 - first.e0 <= 64 * U;  // (uniform within the wave)
  const Chunk kept = load(lists + first.t0 + first.e0, one ? first.e1 - first.e0 : 0);
  auto for_chunks = [&](auto fn) {
    if (one) {
      if (wave < pieces)
        fn(kept, wave, true, first.t0, reinterpret_cast<const uint16_t*>(lists + first.t0 + first.cap) + first.e0);
    } else {
      for (int p = wave; p < pieces; p += NW) {
        const Piece q = piece(p);
        for (int i0 = q.e0; i0 < q.e1 || i0 == q.e0; i0 += 64 * U)
          fn(load(lists + q.t0 + i0, q.e1 - i0), p, i0 == q.e0, q.t0, reinterpret_cast<const uint16_t*>(lists + q.t0 + q.cap) + i0);
      }
    }
  };
  lds_barrier();
  for_chunks([&](const Chunk& c, int, bool, int, const uint16_t*) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c.x[u] >= bound) atomicAdd(&hist[bins.of(c.x[u])], 1u);
  });
  lds_barrier();
  (void)find_bin(hist, (uint32_t)kk, scan, sel);  // (there is such a bin: at least kk keys reach the bound)
  const uint32_t bin = __builtin_amdgcn_readfirstlane(sel[0]);
  const uint32_t need = (uint32_t)kk - __builtin_amdgcn_readfirstlane(sel[1]);
  const uint32_t n_open = __builtin_amdgcn_readfirstlane(sel[2]);
  const uint32_t lo = max(bins.lower_edge(bin), bound);
  uint32_t T = lo - 1u;  // the whole bin is kept
  if (need != n_open) {
    if (n_open > kOpen) return false;
    for_chunks([&](const Chunk& c, int, bool, int, const uint16_t*) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c.x[u] >= bound && bins.of(c.x[u]) == bin) hist[atomicAdd(&sel[3], 1u)] = c.x[u] - lo;
    });
    T = rank_open(hist, n_open, need, lo, sel);
  }
  uint32_t cgt = 0u, ceq = 0u;  // (T >= 1 wherever the equal ones matter: an entry that does not exist is none of them)
  for_chunks([&](const Chunk& c, int p, bool start, int, const uint16_t*) {
    if (start) cgt = ceq = 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      cgt += (uint32_t)__popcll(__ballot(c.x[u] > T));
      ceq += (uint32_t)__popcll(__ballot(c.x[u] == T));
    }
    if (lane == 0) {
      tab[p] = cgt;
      tab[kMaxStretches + p] = ceq;
    }
  });
  lds_barrier();
  const uint32_t ngt = lane < pieces ? tab[lane] : 0u, neq = lane < pieces ? tab[kMaxStretches + lane] : 0u;
  const uint32_t gt_incl = wave_inclusive_sum(ngt), eq_incl = wave_inclusive_sum(neq);
  const uint32_t need_eq = (uint32_t)kk - (uint32_t)__builtin_amdgcn_readlane((int)gt_incl, 63);
  uint32_t gt_before = 0u, eq_before = 0u;
  for_chunks([&](const Chunk& c, int p, bool start, int t0, const uint16_t* pos) {
    if (start) {
      gt_before = (uint32_t)__builtin_amdgcn_readlane((int)(gt_incl - ngt), p);
      eq_before = (uint32_t)__builtin_amdgcn_readlane((int)(eq_incl - neq), p);
    }
    uint32_t at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) at[u] = c.x[u] >= max(T, 1u) ? (uint32_t)t0 + pos[64 * u + lane] : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool gt = c.x[u] > T, eq = c.x[u] == T;
      const unsigned long long bgt = __ballot(gt), beq = __ballot(eq);
      const uint32_t gtb = gt_before + bits_below(bgt), eqb = eq_before + bits_below(beq);
      if (gt) keep[gtb + min(eqb, need_eq)] = at[u];
      if (eq && eqb < need_eq) keep[gtb + eqb] = at[u];
      gt_before += (uint32_t)__popcll(bgt);
      eq_before += (uint32_t)__popcll(beq);
    }
  });
  lds_barrier();
  return true;
}

// PMAX: positions per thread that the launch's longest prefix needs (4 .. 32), LONG: prefixes beyond 32768.
// fuse_gather: once the unit's kept positions are known, the same workgroup copies the unit's K and V rows (a7): for
// the few hundred rows of a small budget a launch of its own costs more than the copy.
template <int PMAX, bool LONG>
__global__ __launch_bounds__(NT, PMAX <= 16 ? 8 : 4) void pool_select_batch_kernel(const SelectBatchArgs a,
                                                                                   const GatherBatchArgs ga,
                                                                                   const int fuse_gather) {
  extern __shared__ uint32_t area[];  // select_area_words(PMAX) entries
  __shared__ __attribute__((aligned(16))) uint32_t hist[HIST];
  __shared__ uint32_t scan32[2 * NW];
  __shared__ uint32_t sel[4];
  uint16_t* keep = reinterpret_cast<uint16_t*>(area + PMAX * 768);  // behind the list's keys and positions

  const int tid = threadIdx.x;
  const int BH = a.B * a.Hkv;
  const int u = blockIdx.x;
  const int l = u / BH;
  const int bg = u - l * BH;
  const int b = bg / a.Hkv;
  const int g = bg - b * a.Hkv;
  const SelectLayer& ly = a.layer[l];
  const GatherLayer& gl = ga.layer[l];
  int n = a.N;
  if (a.seq_lens) {
    n = a.seq_lens[b];
    n = n < 0 ? 0 : (n > a.N ? a.N : n);
  }
  const int count = ly.k_l < n ? ly.k_l : n;
  // a scoring kernel that gave up a wait leaves meaningless scores: the caller learns it from the count
  if (g == 0 && tid == 0) ly.count_out[b] = (a.err && *a.err != 0) ? -1 : count;
  int32_t* idx = ly.idx_out + (size_t)bg * ly.k_cap;
  if (ly.k_l >= n) {  // keep everything
    for (int j = tid; j < ly.k_cap; j += NT) idx[j] = j < n ? j : -1;
    if (fuse_gather) gather_unit(ga, gl, b, g, [&](int j) { return j < n ? j : -1; });
    return;
  }
  if (a.flags && a.flags[(size_t)l * BH + bg] == 0) {  // the kept set is there
    if (fuse_gather) gather_unit(ga, gl, b, g, [&](int j) { return idx[j]; });
    return;
  }
  const int npre = n - a.alpha;
  const int kk = ly.k_l - a.alpha;  // prefix tokens to select; kk < npre
  const size_t rb_stride = (size_t)BH * a.N;
  const float* raw = a.raw + ((size_t)l * a.nrb * BH + bg) * a.N;
  float* pooled = ly.pooled + (size_t)bg * a.N;
  bool in_lds = false, merged = false;
  auto run = [&](auto P) {
    if constexpr (decltype(P)::value <= PMAX)
      in_lds = select_short<decltype(P)::value, PMAX>(a, raw, rb_stride, ly.write_pooled ? pooled : nullptr, idx, npre,
                                                       kk, area, hist, scan32, sel, keep);
  };
  if (PMAX <= 8 && npre <= 4 * NT) run(std::integral_constant<int, 4>{});
  else if (npre <= 8 * NT) run(std::integral_constant<int, 8>{});
  else if (npre <= 16 * NT) run(std::integral_constant<int, 16>{});
  else if (!LONG || npre <= kLdsKeys) run(std::integral_constant<int, 32>{});
  else if constexpr (LONG) {
    const Stretches st = stretches(npre, kk, a.listed != 0, ly.write_pooled != 0);
    if (st.count != 0)
      merged = select_merge(reinterpret_cast<const uint32_t*>(pooled), st, npre, kk, area, area + PMAX * 512, hist, scan32, sel);
    if (!merged)
      select_long(raw, a.nrb, rb_stride, a.inv_G, pooled, idx, npre, kk, a.alpha, a.pool, a.pool_w, area, hist, scan32, sel);
  }
  if (in_lds || merged) {
    auto pos = [&](int j) { return j >= kk ? npre + j - kk : merged ? (int)area[j] : (int)keep[j]; };
    for (int j = tid; j < ly.k_l; j += NT) idx[j] = pos(j);
    if (fuse_gather) gather_unit(ga, gl, b, g, pos);
  } else {
    for (int t = tid; t < a.alpha; t += NT) idx[kk + t] = npre + t;
    if (fuse_gather) {
      __syncthreads();  // the unit's kept positions are complete (all of them written by this workgroup)
      gather_unit(ga, gl, b, g, [&](int j) { return idx[j]; });
    }
  }
}

constexpr size_t select_area_words(int pmax) { return (size_t)pmax * NT + 2 * kPad; }

template <int PMAX, bool LONG>
hipError_t launch_select(const SelectBatchArgs& a, const GatherBatchArgs& ga, bool fuse_gather, int nlayers, hipStream_t s) {
  static bool attr_set[kMaxDevices];
  const size_t dyn = select_area_words(PMAX) * sizeof(uint32_t);
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {  // allow that much dynamic LDS, once per device (idempotent; no allocation)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(pool_select_batch_kernel<PMAX, LONG>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  hipLaunchKernelGGL((pool_select_batch_kernel<PMAX, LONG>), dim3(nlayers * a.B * a.Hkv), dim3(NT), dyn, s, a, ga,
                     fuse_gather ? 1 : 0);
  return hipGetLastError();
}

// Candidates of the prefixes beyond 32768 keys, a workgroup per stretch.
hipError_t launch_stretches(SelectBatchArgs& a, int nlayers, hipStream_t s) {
  const int most = stretch_count(a.N - a.alpha);
  const int64_t units = (int64_t)nlayers * a.B * a.Hkv;
  bool wanted = false;
  for (int l = 0; l < nlayers; ++l) wanted = wanted || (!a.layer[l].write_pooled && a.layer[l].k_l > a.alpha);
  // (65535: the second dimension of a grid)
  if (!wanted || most > kMaxStretches || units > 65535) return hipSuccess;  // select_long takes all
  a.listed = 1;
  static bool attr_set[kMaxDevices];
  const size_t dyn = kStretchWords * sizeof(uint32_t);
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(select_stretch_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  hipLaunchKernelGGL(select_stretch_kernel, dim3(most, (unsigned)units), dim3(kStretchThreads), dyn, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pool_select_batch(SelectBatchArgs& a, const GatherBatchArgs& ga, bool fuse_gather, int nlayers,
                                    hipStream_t s) {
  const int npre = a.N - a.alpha;  // of the longest sequence
  if (npre <= 8 * NT) return launch_select<8, false>(a, ga, fuse_gather, nlayers, s);
  if (npre <= 16 * NT) return launch_select<16, false>(a, ga, fuse_gather, nlayers, s);
  if (npre <= kLdsKeys) return launch_select<32, false>(a, ga, fuse_gather, nlayers, s);
  const hipError_t e = launch_stretches(a, nlayers, s);
  if (e != hipSuccess) return e;
  return launch_select<32, true>(a, ga, fuse_gather, nlayers, s);
}

// ---- attention recall rate (appendix, "Attention Recall Rate Experiment") ----
// The attention of a window query over all keys it sees sums to 1, so the share that falls on the kept keys is
// 1 - (mass on the dropped prefix keys); averaged over the G * alpha queries of a KV head that is
//   recall = 1 - (sum_{i < n-alpha} s_i - sum_{kept prefix i} s_i) / alpha
// with the un-pooled group-mean window scores s_i (the window keys are always kept).  One workgroup per
// (layer, sequence, KV head): one coalesced pass over the scores, one gather over the kept positions.
namespace {
__global__ __launch_bounds__(256) void recall_kernel(const RecallArgs a) {
  const RecallLayer& ly = a.layer[blockIdx.y];
  const int bg = blockIdx.x;
  const int b = bg / a.Hkv;
  const int BH = a.B * a.Hkv;
  int n = a.N;
  if (a.seq_lens) {
    n = a.seq_lens[b];
    n = n < 0 ? 0 : (n > a.N ? a.N : n);
  }
  __shared__ float red[2][256];
  float all = 0.f, kept = 0.f;
  if (ly.k_l < n) {
    const int npre = n - a.alpha, kk = ly.k_l - a.alpha;
    const bool sifted = a.flags && a.flags[(size_t)blockIdx.y * BH + bg] == 0;
    for (int p = 0; p < a.nrb; ++p) {
      const float* row = a.raw + (((size_t)blockIdx.y * a.nrb + p) * BH + bg) * a.N;
      if (sifted) all = threadIdx.x == 0 ? row[npre] : 0.f;
      else
        for (int i = threadIdx.x; i < npre; i += 256) all += row[i];
      for (int j = threadIdx.x; j < kk; j += 256) {
        const int i = ly.idx[(size_t)bg * ly.k_cap + j];
        if ((uint32_t)i < (uint32_t)npre) kept += row[i];
      }
    }
  }
  red[0][threadIdx.x] = all;
  red[1][threadIdx.x] = kept;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] += red[1][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0)
    ly.recall[bg] = (ly.k_l < n) ? 1.f - (red[0][0] - red[1][0]) * a.inv_G / (float)a.alpha : 1.f;
}
}  // namespace

hipError_t launch_recall(const RecallArgs& a, int nlayers, hipStream_t s) {
  hipLaunchKernelGGL(recall_kernel, dim3(a.B * a.Hkv, nlayers), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace pkv
