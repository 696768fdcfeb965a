// Pieces of the selection that more than one kernel of kSelectThreads threads uses: wave reductions, histogram bins over
// scores, pooling out of LDS.
#pragma once

#include <type_traits>

#include "pkv_internal.h"
#include "pkv_lds.h"

namespace pkv {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_u __attribute__((aligned(4)));   // four floats at any 4-byte boundary

constexpr int NT = kSelectThreads;
constexpr int NW = NT / 64;
constexpr int HIST = 2048;         // bins of the widest digit
constexpr int kPad = 32;           // neutral scores in LDS before the prefix and behind it (half a pooling window)

// Largest of a value over the 64 lanes of a wave, valid in lane 63.  Data-parallel-primitive row operations (no LDS
// traffic): running maximum within each row of 16 lanes by shifts of 1, 2, 4, 8 (lanes without a source take 0),
// then the last lane of row 0 / row 2 is handed to row 1 / row 3, and lane 31 to rows 2 and 3.
__device__ __forceinline__ uint32_t wave_max_lane63(uint32_t v) {
#define PKV_DPP_MAX(ctrl, rows) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, false))
  PKV_DPP_MAX(0x111, 0xF);  // row_shr:1
  PKV_DPP_MAX(0x112, 0xF);  // row_shr:2
  PKV_DPP_MAX(0x114, 0xF);  // row_shr:4
  PKV_DPP_MAX(0x118, 0xF);  // row_shr:8
  PKV_DPP_MAX(0x142, 0xA);  // row_bcast:15 into rows 1 and 3
  PKV_DPP_MAX(0x143, 0xC);  // row_bcast:31 into rows 2 and 3
#undef PKV_DPP_MAX
  return v;
}

// Largest of a value over each row of 16 lanes, valid in its last lane.
__device__ __forceinline__ uint32_t row_max_lane15(uint32_t v) {
#define PKV_DPP_MAX(ctrl) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xF, 0xF, false))
  PKV_DPP_MAX(0x111);  // row_shr:1
  PKV_DPP_MAX(0x112);  // row_shr:2
  PKV_DPP_MAX(0x114);  // row_shr:4
  PKV_DPP_MAX(0x118);  // row_shr:8
#undef PKV_DPP_MAX
  return v;
}

// Sum over the lanes up to and including each lane (the same row operations, additions).
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t v) {
#define PKV_DPP_ADD(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, false)
  PKV_DPP_ADD(0x111, 0xF);
  PKV_DPP_ADD(0x112, 0xF);
  PKV_DPP_ADD(0x114, 0xF);
  PKV_DPP_ADD(0x118, 0xF);
  PKV_DPP_ADD(0x142, 0xA);
  PKV_DPP_ADD(0x143, 0xC);
#undef PKV_DPP_ADD
  return v;
}

// The waves' 16 values in LDS, read one per lane: sum over the waves before `wave` (uniform), and over all of them.
__device__ __forceinline__ uint32_t sum_before(const uint32_t* per_wave, int wave, uint32_t& total) {
  uint32_t v = per_wave[threadIdx.x & 15];
#define PKV_DPP_ADD(ctrl) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xF, 0xF, false)
  PKV_DPP_ADD(0x111);
  PKV_DPP_ADD(0x112);
  PKV_DPP_ADD(0x114);
  PKV_DPP_ADD(0x118);
#undef PKV_DPP_ADD
  total = (uint32_t)__builtin_amdgcn_readlane((int)v, NW - 1);
  const uint32_t incl = (uint32_t)__builtin_amdgcn_readlane((int)v, wave > 0 ? wave - 1 : 0);
  return wave > 0 ? incl : 0u;
}

// The bin in which the count over ascending bins reaches kk: sel[0] = bin, sel[1] = count before it, sel[2] = count in it
// (untouched if there is none).  Returns the count over all bins.  Thread t owns bins 2t, 2t + 1 and leaves them cleared.
// Every thread returns after the answer is there.  (Bins 0 .. HIST - 1, `scan` holds NW entries.)
__device__ __forceinline__ uint32_t find_bin(uint32_t* hist, uint32_t kk, uint32_t* scan, uint32_t* sel) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint2 h = reinterpret_cast<uint2*>(hist)[tid];
  reinterpret_cast<uint2*>(hist)[tid] = make_uint2(0u, 0u);
  const uint32_t incl = wave_inclusive_sum(h.x + h.y);
  if (lane == 63) scan[wave] = incl;
  lds_barrier();
  uint32_t total;
  const uint32_t before = sum_before(scan, wave, total) + incl - h.x - h.y;
  const bool in0 = before < kk && before + h.x >= kk;
  const bool in1 = before + h.x < kk && before + h.x + h.y >= kk;
  if (in0 || in1) {
    sel[0] = (uint32_t)(2 * tid + (in1 ? 1 : 0));
    sel[1] = in1 ? before + h.x : before;
    sel[2] = in1 ? h.y : h.x;
  }
  lds_barrier();
  return total;
}

template <int NJ>
struct Scores {
  f32x4 v[NJ];
};

// Pooled scores of a thread's positions p0 + 256 * jj + c out of an LDS copy of the scores (half a window of them, or of
// neutral values, on both sides); v holds the scores on entry.  w0: first position of the wave, n: positions in all.
template <int NJ>
__device__ __forceinline__ Scores<NJ> pool_lds(const float* lsc, int p0, int w0, int n, int r, bool is_max, int pool_w,
                                               Scores<NJ> s) {
  f32x4* v = s.v;
  const float inv_w = 1.0f / (float)pool_w;
  // windows summed (or maximised) in ascending position order
  auto pool_fixed = [&](auto RR, auto MX) __attribute__((always_inline)) {
    constexpr int R = decltype(RR)::value;
    constexpr bool mx = decltype(MX)::value;
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      if (w0 + 256 * jj >= n) continue;
      const f32x4 lo = *reinterpret_cast<const f32x4*>(lsc + p0 + 256 * jj - 4);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(lsc + p0 + 256 * jj + 4);
      const f32x4 md = *reinterpret_cast<const f32x4*>(lsc + p0 + 256 * jj);
      const float x[12] = {lo[0], lo[1], lo[2], lo[3], md[0], md[1], md[2], md[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        float acc = x[4 + c - R];
#pragma unroll
        for (int u = -R + 1; u <= R; ++u) acc = mx ? fmaxf(acc, x[4 + c + u]) : acc + x[4 + c + u];
        v[jj][c] = mx ? acc : acc * inv_w;
      }
    }
  };
  using std::integral_constant;
  if (r <= 3) {
    if (is_max) {
      if (r == 1) pool_fixed(integral_constant<int, 1>{}, std::true_type{});
      else if (r == 2) pool_fixed(integral_constant<int, 2>{}, std::true_type{});
      else pool_fixed(integral_constant<int, 3>{}, std::true_type{});
    } else {
      if (r == 1) pool_fixed(integral_constant<int, 1>{}, std::false_type{});
      else if (r == 2) pool_fixed(integral_constant<int, 2>{}, std::false_type{});
      else pool_fixed(integral_constant<int, 3>{}, std::false_type{});
    }
  } else {
    // wider windows: one new score per step for the thread's four outputs
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      if (w0 + 256 * jj >= n) continue;
      const float* lp = lsc + p0 + 256 * jj - r;
      float x0 = lp[0], x1 = lp[1], x2 = lp[2];
      f32x4 acc = is_max ? f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY} : f32x4{0.f, 0.f, 0.f, 0.f};
      for (int u = 0; u <= 2 * r; ++u) {
        const float x3 = lp[u + 3];
        acc[0] = is_max ? fmaxf(acc[0], x0) : acc[0] + x0;
        acc[1] = is_max ? fmaxf(acc[1], x1) : acc[1] + x1;
        acc[2] = is_max ? fmaxf(acc[2], x2) : acc[2] + x2;
        acc[3] = is_max ? fmaxf(acc[3], x3) : acc[3] + x3;
        x0 = x1;
        x1 = x2;
        x2 = x3;
      }
      v[jj] = is_max ? acc : acc * inv_w;
    }
  }
  return s;
}

// Bins of the distance from a reference key, descending: the first half for keys from the reference up, 1/8 of a binade
// each (2^20 units of the bit pattern), the second half for those below it, 1/64 of a binade each (2^17 units; 16 binades in
// 1024 bins); the first and the last bin are open to the outside.
template <int BINS>
struct KeyBins {
  static constexpr int kUp = 20, kDown = 17;
  static constexpr uint32_t kMid = BINS / 2;
  uint32_t ref;
  __device__ __forceinline__ uint32_t of(uint32_t k) const {
    return k >= ref ? kMid - 1u - min((k - ref) >> kUp, kMid - 1u) : kMid + min((ref - 1u - k) >> kDown, kMid - 1u);
  }
  // smallest and largest key of a bin that holds one (never 0, the mark of a position that does not exist)
  __device__ __forceinline__ uint32_t lower_edge(uint32_t bin) const {
    if (bin < kMid) return max(ref + ((kMid - 1u - bin) << kUp), 1u);
    const uint32_t down = (bin - kMid + 1u) << kDown;
    return bin < BINS - 1u && down < ref ? ref - down : 1u;
  }
  __device__ __forceinline__ uint32_t upper_edge(uint32_t bin) const {
    if (bin >= kMid) return ref - 1u - ((bin - kMid) << kDown);
    const uint32_t up = ref + ((kMid - bin) << kUp) - 1u;
    return bin > 0u && up >= ref ? up : 0xFFFFFFFFu;
  }
};

}  // namespace
}  // namespace pkv
