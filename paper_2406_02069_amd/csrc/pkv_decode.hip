// The step after the compression path: one decoding query per sequence attends over the compacted cache of a
// layer (Sec. 3: after compression the model attends over K_s, V_s only).  The kept rows were copied bit for bit,
// so they carry the rotary phases of their original positions and nothing is re-rotated here (appendix on rotary
// embeddings); the cache is ragged (count_b rows per sequence) and may be paged with the layer's own block table
// (appendix "PyramidKV Implementation at vLLM").
//
// Work split: (sequence, KV head) x S key ranges, one workgroup of 4 .. 16 waves each; the G <= 8 query heads of a KV
// head share every key and value row.  The waves of a workgroup take the 16-key tiles (32-key at d = 64) of its range
// in turn, each on its own: K tile -> logits -> running softmax -> weighted V tile, the keys of the wave's next tile
// requested as soon as this tile's are multiplied and its values as soon as these are added, so that a wave always
// has loads in flight and no barrier separates the keys from the values.  One barrier at the end, when the waves'
// (maximum, sum, weighted values) meet in LDS.  With S > 1 the ranges leave un-normalised partial results in a
// workspace and a second small kernel merges them, with S = 1 the first kernel writes the result itself.  Few heads with S = 1 and a
// launch of their own: a workgroup per 32 output columns, each of which forms all logits (decode_columns_kernel).
//   logits  the G queries are rows 0 .. G-1 of the A operand of v_mfma_f32_16x16x32_bf16 (16-row tile, the other rows
//           zero; queries straight from memory into operand layout), 16 keys its columns, loaded straight into the
//           B-operand layout (16 rows x 64 bytes per load).  Lane (column l16, quad) ends with the logits of heads
//           4 quad .. 4 quad + 3 for key l16.
//   softmax a reference exponent per head and wave, moved to the exact maximum (and the sums rescaled) only when a
//           logit exceeds it by a factor 2^16: a wave-uniform branch, taken on the first tile and rarely afterwards.
//   values  a lane moves 16 bytes of a value row per load (a wave: 4 rows at d = 128), its weights come from a
//           wave-private LDS tile; every lane keeps GP x 8 partial outputs (GP = G rounded up to 1, 2, 4, 8).  From
//           GP = 4 on they are formed by v_mfma_f32_4x4x1_16b_f32 (fp32 products and sums): four neighbouring lanes
//           share a row, so one instruction adds weight x value for four heads (8 clk in the matrix pipe, against four
//           multiply-adds at 4 clk each in the vector pipe, which has the unpacking to do).
// HBM-bound: every kept K and V row is read once (2 x count x d x 2 bytes per head), the rest stays on chip.
#include <type_traits>

#include "pkv_internal.h"

namespace pkv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x8 as_frag(u32x4 u) { return __builtin_bit_cast(bf16x8, u); }

constexpr int kMaxSplits = 16;     // key ranges per (sequence, KV head), at most
// Waves of a workgroup, at most (always 4, 8 or 16): the outputs of eight heads need more than 128 registers.
constexpr int max_waves(int gp) { return gp > 4 ? 8 : 16; }
constexpr int kTabEntries = 1026;  // block-table entries of a key range kept in LDS (pages of 4 slots or more)

// LDS traffic of one wave to its own region needs ordering only inside the wave.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The value of the lane N places further round in the row of 16 lanes.
template <int N>
__device__ __forceinline__ float row_ror(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N, 0xF, 0xF, true));
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, row_ror<8>(x));
  x = fmaxf(x, row_ror<4>(x));
  x = fmaxf(x, row_ror<2>(x));
  return fmaxf(x, row_ror<1>(x));
}
__device__ __forceinline__ float row_sum(float x) {
  x += row_ror<8>(x);
  x += row_ror<4>(x);
  x += row_ror<2>(x);
  return x + row_ror<1>(x);
}
__device__ __forceinline__ float read_lane(float x, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}
// Sum of x over the wave's halves in the lower half, of y in the upper half (and the same over neighbouring rows of 16).
__device__ __forceinline__ float fold32(float x, float y) {
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float x, float y) {
  const u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false));
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Key range sp of (sequence b, KV head g) of one layer's cache; output columns part * DV .. part * DV + DV - 1 of D.
template <int D, int GP, bool PAGED, int DV = D>
__device__ __forceinline__ void decode_range(const DecodeArgs& a, int sp, int g, int b, float* dsm, int part = 0) {
  constexpr int KS = D / 32;             // matrix k-steps per dot product
  constexpr int NG = D == 128 ? 1 : 2;   // groups of 16 keys per tile (4 KB of keys and of values either way)
  constexpr int TK = 16 * NG;            // keys per tile
  constexpr int LPR = DV / 8;            // lanes per value row
  constexpr int RPL = 64 / LPR;          // value rows per load of a wave
  constexpr int NV = TK / RPL;           // value loads per tile
  constexpr int QH = GP > 4 ? 2 : 1;     // quads that hold logits of real heads
  static_assert(LPR >= 4 && DV >= TK, "lanes of a matrix block share a row; a wave's weights fit its outputs' place");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int l16 = lane & 15, quad = lane >> 4;
  const int sub = lane / LPR, col = lane - sub * LPR;
  // dsm: [nw][GP][DV] outputs of the waves (before that, each wave's region holds its tile's weights) | [nw][GP][2]
  // (max, sum) | [kTabEntries] block-table entries of this range
  float* s_o = dsm + (size_t)wave * GP * DV;
  float* s_mz = dsm + (size_t)nw * GP * DV;
  int* s_tab = reinterpret_cast<int*>(s_mz + nw * GP * 2);
  const int cnt_raw = a.count[b];
  const int j_lo = sp * a.chunk;
  const int nmax = min(a.k_cap - j_lo, a.chunk);  // rows the range can hold (<= 0: an empty last range)

  const uint16_t* Kb = a.K;
  const uint16_t* Vb = a.V;
  int q0 = 0;
  if constexpr (PAGED) {
    Kb += (size_t)g * a.page_size * D;
    Vb += (size_t)g * a.page_size * D;
    // this range's block-table entries once into LDS, so that a row's address costs one memory access
    if (a.page_size >= 4 && nmax > 0) {  // (at most chunk / 4 + 2 entries then)
      q0 = j_lo / a.page_size;
      const int n_ent = (j_lo + nmax - 1) / a.page_size - q0 + 1;
      for (int e = tid; e < n_ent; e += blockDim.x) s_tab[e] = a.table[(size_t)b * a.max_pages + q0 + e];
      __syncthreads();
    }
  } else {
    Kb += (size_t)b * a.c_sb + (size_t)g * a.c_sh + (size_t)j_lo * a.c_st;
    Vb += (size_t)b * a.c_sb + (size_t)g * a.c_sh + (size_t)j_lo * a.c_st;
  }
  Vb += part * DV;
  // Address of local row j (0 <= j < nmax) of Kb / Vb; paged: ok = its page number is in range (else the address is
  // that of some readable row)
  const uint64_t row_bytes = (uint64_t)a.c_st * 2u;
  auto row_ptr = [&](const uint16_t* base, int j, bool& ok) -> const char* {
    uint64_t off;
    if constexpr (PAGED) {
      j += j_lo;
      const int q = a.page_shift >= 0 ? j >> a.page_shift : (int)__umulhi((uint32_t)j, a.page_magic);
      const int slot = j - q * a.page_size;
      int pg = a.page_size >= 4 ? s_tab[q - q0] : a.table[(size_t)b * a.max_pages + q];
      ok = (uint32_t)pg < (uint32_t)a.num_pages;
      pg = ok ? pg : 0;
      off = (uint64_t)(uint32_t)pg * ((uint64_t)a.Hkv * a.page_size * (2 * D)) + (uint32_t)(slot * (2 * D));
    } else {
      ok = true;
      off = (uint32_t)j * row_bytes;
    }
    return reinterpret_cast<const char*>(base) + off;
  };
  bf16x8 kf[NG][KS];
  u32x4 vv[NV];
  bool kok[NG], vok[NV];
  // Keys / values of the wave's tile t; rows at or beyond lim are replaced by row lim - 1.  (The compiler may not move
  // loads across the empty statement behind each: it would sink them to their use in the next iteration, and nothing
  // would be in flight meanwhile.)
  auto load_k = [&](int t, int lim) {
#pragma unroll
    for (int gr = 0; gr < NG; ++gr) {
      const char* p = row_ptr(Kb, min(t * TK + 16 * gr + l16, lim - 1), kok[gr]) + 16 * quad;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[gr][ks] = as_frag(*reinterpret_cast<const u32x4*>(p + 64 * ks));
    }
    asm volatile("" ::: "memory");
  };
  auto load_v = [&](int t, int lim) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
      vv[i] = *reinterpret_cast<const u32x4*>(row_ptr(Vb, min(t * TK + RPL * i + sub, lim - 1), vok[i]) + 16 * col);
    asm volatile("" ::: "memory");
  };

  // m: reference exponent of each head (not necessarily the maximum so far, at most 2^kSlack below it; kNone, below every
  // finite logit and finite itself, so that logits of -inf have weight 0, before the first finite one), z: sum of this
  // lane's weights.  Outputs of column 8 col + c: oc[c] over four (eight) heads, or of[h][c].
  constexpr int NH = GP < 4 ? GP : 4;    // heads per quad
  constexpr bool MF = GP >= 4;           // values by matrix instructions
  constexpr float kSlack = 16.f, kNone = -3e38f;
  float m[NH], z[NH], of[MF ? 1 : GP][8];
  f32x4 oc[MF ? QH : 1][8];
#pragma unroll
  for (int v = 0; v < NH; ++v) {
    m[v] = kNone;
    z[v] = 0.f;
  }
#pragma unroll
  for (int c = 0; c < 8; ++c) {
#pragma unroll
    for (int q = 0; q < (MF ? QH : 1); ++q) oc[q][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int h = 0; h < (MF ? 1 : GP); ++h) of[h][c] = 0.f;
  }

  if (wave * TK < nmax) {
    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 w = u32x4{0u, 0u, 0u, 0u};
      if (l16 < a.G)
        w = *reinterpret_cast<const u32x4*>(a.q + ((size_t)b * a.Hq + (size_t)g * a.G + l16) * D + 32 * ks + 8 * quad);
      qf[ks] = as_frag(w);
    }
    // The first tile is requested before the count has arrived: every row below k_cap is readable, and what lies
    // beyond the count is masked below.
    load_k(wave, nmax);
    load_v(wave, nmax);
    const int cnt = min(max(cnt_raw, 0), a.k_cap);
    const int nloc = min(max(cnt - j_lo, 0), a.chunk);
    for (int t = wave; t * TK < nloc; t += nw) {
      const bool partial = PAGED || (t + 1) * TK > nloc;  // rows to mask (beyond the count, or of a bad page)
      f32x4 acc[NG];
      bool have[NG];
#pragma unroll
      for (int gr = 0; gr < NG; ++gr) {
        acc[gr] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc[gr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[ks], kf[gr][ks], acc[gr], 0, 0, 0);
        have[gr] = kok[gr] && t * TK + 16 * gr + l16 < nloc;
      }
      // (behind the wave's last tile this fetches one row once more: under a condition the waits below would have to
      // allow for either way in, and would wait for these keys as well)
      load_k(t + nw, nloc);
      // exponents relative to the heads' references; a reference is moved to the exact maximum only when some logit
      // exceeds it by more than 2^kSlack (always on the first tile): weights stay far inside fp32's range
      float y[NG][NH];
      auto exponents = [&]() {
        bool over = false;
#pragma unroll
        for (int gr = 0; gr < NG; ++gr)
#pragma unroll
          for (int v = 0; v < NH; ++v) {
            y[gr][v] = __builtin_fmaf(acc[gr][v], a.scale_log2, -m[v]);
            if (partial && !have[gr]) y[gr][v] = -INFINITY;
            over = over || y[gr][v] > kSlack;
          }
        return over;
      };
      if (__any(exponents() && quad < QH)) {
        float f[NH];
#pragma unroll
        for (int v = 0; v < NH; ++v) {
          float tm = -INFINITY;
#pragma unroll
          for (int gr = 0; gr < NG; ++gr) tm = fmaxf(tm, have[gr] ? acc[gr][v] * a.scale_log2 : -INFINITY);
          const float mn = fmaxf(m[v], row_max(tm));
          f[v] = __builtin_amdgcn_exp2f(m[v] - mn);
          z[v] *= f[v];
          m[v] = mn;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          if constexpr (MF) {
#pragma unroll
            for (int h = 0; h < GP; ++h) oc[h >> 2][c][h & 3] *= read_lane(f[h & 3], 16 * (h >> 2));
          } else {
#pragma unroll
            for (int h = 0; h < GP; ++h) of[h][c] *= read_lane(f[h], 0);
          }
        }
        (void)exponents();
      }
#pragma unroll
      for (int gr = 0; gr < NG; ++gr) {
        float p[NH];
#pragma unroll
        for (int v = 0; v < NH; ++v) {
          p[v] = __builtin_amdgcn_exp2f(y[gr][v]);
          z[v] += p[v];
        }
        if (quad < QH) {
          float* dst = s_o + (16 * gr + l16) * GP + 4 * quad;
          if constexpr (GP >= 4) *reinterpret_cast<f32x4*>(dst) = f32x4{p[0], p[1], p[2], p[3]};
          else if constexpr (GP == 2) *reinterpret_cast<f32x2*>(dst) = f32x2{p[0], p[1]};
          else *dst = p[0];
        }
      }
      wave_lds_fence();
      // rows beyond the count or of a bad page: their weights are zero, but what was read must not reach the sums
      if (partial) {
#pragma unroll
        for (int i = 0; i < NV; ++i)
          if (!(vok[i] && t * TK + RPL * i + sub < nloc)) vv[i] = u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const float* src = s_o + (RPL * i + sub) * GP;
        float pw[MF ? QH : GP];
        if constexpr (MF) {
          // one v_mfma_f32_4x4x1: four lanes of a row are a block, column block entry = the lane's value, row = head
#pragma unroll
          for (int q = 0; q < QH; ++q) pw[q] = src[4 * q + (lane & 3)];
        } else {
#pragma unroll
          for (int h = 0; h < GP; ++h) pw[h] = src[h];
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const uint32_t w = vv[i][c >> 1];
          const float x = __uint_as_float((c & 1) ? w & 0xFFFF0000u : w << 16);
          if constexpr (MF) {
#pragma unroll
            for (int q = 0; q < QH; ++q) oc[q][c] = __builtin_amdgcn_mfma_f32_4x4x1f32(pw[q], x, oc[q][c], 0, 0, 0);
          } else {
#pragma unroll
            for (int h = 0; h < GP; ++h) of[h][c] = __builtin_fmaf(pw[h], x, of[h][c]);
          }
        }
      }
      // (the sums are complete here: without this they move behind the requests below, whose registers then cannot be
      // the ones just read)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        if constexpr (MF) {
#pragma unroll
          for (int q = 0; q < QH; ++q) asm volatile("" : "+v"(oc[q][c]));
        } else {
#pragma unroll
          for (int h = 0; h < GP; ++h) asm volatile("" : "+v"(of[h][c]));
        }
      }
      wave_lds_fence();
      load_v(t + nw, nloc);
    }
  }
  auto o = [&](int h, int c) -> float {
    if constexpr (MF) return oc[h >> 2][c][h & 3];
    else return of[h][c];
  };

  // ---- the wave's result to LDS: outputs summed over the lanes that share columns (each lane keeps its share of the
  // heads as the sum proceeds), maxima and sums per head ----
#pragma unroll
  for (int v = 0; v < NH; ++v) {
    z[v] = row_sum(z[v]);
    if (l16 == 0 && quad < QH) {
      s_mz[(wave * GP + 4 * quad + v) * 2] = m[v];
      s_mz[(wave * GP + 4 * quad + v) * 2 + 1] = z[v];
    }
  }
  const int upper = lane >> 5, odd = (lane >> 4) & 1;
  constexpr int H1 = GP >= 2 ? GP / 2 : 1, H2 = GP >= 4 ? GP / 4 : 1;
  float r1[H1][8], r2[H2][8];
#pragma unroll
  for (int h = 0; h < H1; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) r1[h][c] = GP >= 2 ? fold32(o(h, c), o((h + H1) % GP, c)) : fold32(o(0, c), o(0, c));
#pragma unroll
  for (int h = 0; h < H2; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      r2[h][c] = GP >= 4 ? fold16(r1[h][c], r1[(h + H2) % H1][c]) : fold16(r1[0][c], r1[0][c]);
      if (LPR <= 8) r2[h][c] += row_ror<8>(r2[h][c]);
      if (LPR <= 4) r2[h][c] += row_ror<4>(r2[h][c]);
    }
  const int h0 = (GP >= 2 ? upper * H1 : 0) + (GP >= 4 ? odd * H2 : 0);
  const bool writes = (GP >= 2 || upper == 0) && (GP >= 4 || odd == 0) && (lane & (16 - LPR)) == 0;
  if (writes) {
#pragma unroll
    for (int h = 0; h < H2; ++h) {
      float* dst = s_o + (h0 + h) * DV + 8 * col;
      *reinterpret_cast<f32x4*>(dst) = f32x4{r2[h][0], r2[h][1], r2[h][2], r2[h][3]};
      *reinterpret_cast<f32x4*>(dst + 4) = f32x4{r2[h][4], r2[h][5], r2[h][6], r2[h][7]};
    }
  }
  __syncthreads();
  // ---- the waves' results meet, in wave order ----
  const size_t unit = (size_t)b * a.Hkv + g;
  for (int e = tid; e < a.G * DV; e += blockDim.x) {
    const int h = e / DV;
    float M = -INFINITY;
    for (int w0 = 0; w0 < nw; w0 += 4)  // (nw is a multiple of 4)
#pragma unroll
      for (int w = w0; w < w0 + 4; ++w) M = fmaxf(M, s_mz[(w * GP + h) * 2]);
    float zz = 0.f, xx = 0.f;
    for (int w0 = 0; w0 < nw; w0 += 4)
#pragma unroll
      for (int w = w0; w < w0 + 4; ++w) {
        const float f = __builtin_amdgcn_exp2f(s_mz[(w * GP + h) * 2] - M);  // (nothing here, M = kNone: zz and xx are 0)
        zz += f * s_mz[(w * GP + h) * 2 + 1];
        xx += f * dsm[(size_t)w * GP * DV + e];
      }
    const bool first = e == h * DV && part == 0;
    const int at = DV == D ? e : h * D + part * DV + (e - h * DV);
    if (a.S == 1) {
      a.out[((size_t)b * a.Hq + (size_t)g * a.G) * D + at] = zz > 0.f ? xx / zz : 0.f;
      if (first && a.lse)
        a.lse[(size_t)b * a.Hq + g * a.G + h] = zz > 0.f ? (M + __builtin_amdgcn_logf(zz)) * 0.69314718055994530942f : -INFINITY;
    } else {
      a.part_o[(unit * a.S + sp) * 8 * D + e] = xx;
      if (first) {
        a.part_mz[(unit * a.S + sp) * 16 + 2 * h] = M;
        a.part_mz[(unit * a.S + sp) * 16 + 2 * h + 1] = zz;
      }
    }
  }
}

template <int D, int GP, bool PAGED>
__global__ __launch_bounds__(64 * max_waves(GP)) void decode_partial_kernel(const DecodeArgs a) {
  extern __shared__ float dsm[];
  decode_range<D, GP, PAGED>(a, blockIdx.x, blockIdx.y, blockIdx.z, dsm);
}

// Few heads, one range each: a head's output columns over several workgroups.  Each forms all logits, so the keys are read D / 32
// times, but a compute unit has 5/8 (d = 64: 3/4) of the bytes to fetch, and nothing has to be merged.
constexpr int kColumns = 32;
template <int D, int GP, bool PAGED>
__global__ __launch_bounds__(64 * max_waves(GP)) void decode_columns_kernel(const DecodeArgs a) {
  extern __shared__ float dsm[];
  decode_range<D, GP, PAGED, kColumns>(a, 0, blockIdx.y, blockIdx.z, dsm, blockIdx.x);
}

// Merge of the S partial results of a (sequence, KV head): common reference exponent, sums, weighted values.
template <int D>
__device__ __forceinline__ void decode_merge(const DecodeArgs& a, int g, int b) {
  const size_t unit = (size_t)b * a.Hkv + g;
  const float* part_o = a.part_o + unit * a.S * 8 * D;
  const float* part_mz = a.part_mz + unit * a.S * 16;
  float* out = a.out + ((size_t)b * a.Hq + (size_t)g * a.G) * D;
  for (int e = threadIdx.x; e < a.G * D; e += 256) {
    const int h = e / D;
    // all loads first (S <= kMaxSplits, so the loops unroll): one memory round trip instead of one per range
    float pm[kMaxSplits], pz[kMaxSplits], px[kMaxSplits];
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {
      const bool have = s < a.S;
      pm[s] = have ? part_mz[s * 16 + 2 * h] : -INFINITY;
      pz[s] = have ? part_mz[s * 16 + 2 * h + 1] : 0.f;
      px[s] = have ? part_o[(size_t)s * 8 * D + e] : 0.f;
    }
    float M = -INFINITY;
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) M = fmaxf(M, pm[s]);
    float z = 0.f, x = 0.f;
#pragma unroll
    for (int s = 0; s < kMaxSplits; ++s) {
      const float f = __builtin_amdgcn_exp2f(pm[s] - M);
      z += pz[s] * f;
      x += px[s] * f;
    }
    out[e] = z > 0.f ? x / z : 0.f;
    if (a.lse && e == h * D)
      a.lse[(size_t)b * a.Hq + g * a.G + h] = z > 0.f ? (M + __builtin_amdgcn_logf(z)) * 0.69314718055994530942f : -INFINITY;
  }
}

template <int D>
__global__ __launch_bounds__(256) void decode_merge_kernel(const DecodeArgs a) {
  decode_merge<D>(a, blockIdx.x, blockIdx.y);
}

// ---- all layers of a decoding step in one launch ----
// The layers' caches are small at batch 1 (a few hundred rows each under a pyramidal budget), and a launch per layer
// costs more than the rows it reads; here workgroup w of the grid finds its layer from the table's running workgroup
// counts and works on one key range of one (sequence, KV head) of it, exactly as above.
__device__ __forceinline__ DecodeArgs layer_args(const DecodeBatchArgs& a, int l) {
  const DecodeLayer& ly = a.layer[l];
  DecodeArgs d;
  d.q = ly.q; d.K = ly.K; d.V = ly.V; d.table = ly.table; d.count = ly.count; d.out = ly.out; d.lse = ly.lse;
  d.part_o = a.part_o + (size_t)ly.part0 * 8 * a.d;
  d.part_mz = a.part_mz + (size_t)ly.part0 * 16;
  d.B = a.B; d.Hq = a.Hq; d.Hkv = a.Hkv; d.G = a.G; d.d = a.d; d.k_cap = ly.k_cap;
  d.page_size = a.page_size; d.num_pages = ly.num_pages; d.max_pages = ly.max_pages;
  d.page_shift = a.page_shift; d.page_magic = a.page_magic;
  d.S = ly.S; d.chunk = ly.chunk;
  d.c_sb = ly.c_sb; d.c_sh = ly.c_sh; d.c_st = ly.c_st;
  d.scale_log2 = a.scale_log2;
  return d;
}

template <int D, int GP, bool PAGED>
__global__ __launch_bounds__(64 * max_waves(GP)) void decode_partial_layers_kernel(const DecodeBatchArgs a) {
  extern __shared__ float dsm[];
  const int w = blockIdx.x;
  int l = 0;
  while (l + 1 < a.L && w >= a.layer[l + 1].wg0) ++l;  // (wave-uniform: scalar loads from the argument table)
  const DecodeArgs d = layer_args(a, l);
  const int rel = w - a.layer[l].wg0;          // [b][g][sp]
  const int sp = rel % d.S, bg = rel / d.S;
  const int g = bg % a.Hkv, b = bg / a.Hkv;
  decode_range<D, GP, PAGED>(d, sp, g, b, dsm);
}

template <int D>
__global__ __launch_bounds__(256) void decode_merge_layers_kernel(const DecodeBatchArgs a) {
  const int l = blockIdx.z;
  if (a.layer[l].S == 1) return;  // that layer's ranges wrote the result themselves
  const DecodeArgs d = layer_args(a, l);
  decode_merge<D>(d, blockIdx.x, blockIdx.y);
}

// Raises a kernel's dynamic LDS limit to what any launch of it can need, once per device (no allocation).
hipError_t grant_lds(const void* f, bool* granted, size_t lds_max) {
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (granted[dev]) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_max);
  if (e == hipSuccess) granted[dev] = true;
  return e;
}
constexpr size_t lds_bytes(int d, int gp, int nw, bool paged) {
  return (size_t)nw * gp * (d + 2) * sizeof(float) + (paged ? kTabEntries * sizeof(int) : 0);
}

template <int D, int GP, bool PAGED>
hipError_t launch_partial(const DecodeArgs& a, int nw, hipStream_t s) {
  static bool granted[kMaxDevices];
  const hipError_t e = grant_lds(reinterpret_cast<const void*>(decode_partial_kernel<D, GP, PAGED>), granted,
                                 lds_bytes(D, GP, max_waves(GP), PAGED));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((decode_partial_kernel<D, GP, PAGED>), dim3(a.S, a.Hkv, a.B), dim3(64 * nw),
                     lds_bytes(D, GP, nw, PAGED), s, a);
  return hipGetLastError();
}

template <int D, int GP, bool PAGED>
hipError_t launch_columns(const DecodeArgs& a, int nw, hipStream_t s) {
  static bool granted[kMaxDevices];
  const hipError_t e = grant_lds(reinterpret_cast<const void*>(decode_columns_kernel<D, GP, PAGED>), granted,
                                 lds_bytes(kColumns, GP, max_waves(GP), PAGED));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((decode_columns_kernel<D, GP, PAGED>), dim3(D / kColumns, a.Hkv, a.B), dim3(64 * nw),
                     lds_bytes(kColumns, GP, nw, PAGED), s, a);
  return hipGetLastError();
}

template <int D, int GP, bool PAGED>
hipError_t launch_partial_layers(const DecodeBatchArgs& a, int total_wgs, int nw, hipStream_t s) {
  static bool granted[kMaxDevices];
  const hipError_t e = grant_lds(reinterpret_cast<const void*>(decode_partial_layers_kernel<D, GP, PAGED>), granted,
                                 lds_bytes(D, GP, max_waves(GP), PAGED));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((decode_partial_layers_kernel<D, GP, PAGED>), dim3(total_wgs), dim3(64 * nw),
                     lds_bytes(D, GP, nw, PAGED), s, a);
  return hipGetLastError();
}

// Calls fn with (head dimension, padded group size, paged) as compile-time constants.
template <class Fn>
hipError_t with_variant(int d, int G, bool paged, Fn fn) {
  auto by_page = [&](auto D, auto GP) { return paged ? fn(D, GP, std::true_type{}) : fn(D, GP, std::false_type{}); };
  auto by_group = [&](auto D) {
    if (G == 1) return by_page(D, std::integral_constant<int, 1>{});
    if (G == 2) return by_page(D, std::integral_constant<int, 2>{});
    if (G <= 4) return by_page(D, std::integral_constant<int, 4>{});
    return by_page(D, std::integral_constant<int, 8>{});
  };
  if (d == 128) return by_group(std::integral_constant<int, 128>{});
  if (d == 64) return by_group(std::integral_constant<int, 64>{});
  return hipErrorInvalidValue;
}

}  // namespace

// Key ranges per (sequence, KV head) that the workspace has room for.
int decode_splits(int B, int Hkv, int k_cap) {
  int S = (512 + B * Hkv - 1) / (B * Hkv);
  if (S > kMaxSplits) S = kMaxSplits;
  const int by_len = k_cap / 128;
  if (S > by_len) S = by_len;
  return S < 1 ? 1 : S;
}

// Key ranges actually used.  One compute unit fetches 57 - 59 bytes per ns from beyond its L2 however much it has in
// flight, so the rows of a head are split over several when few heads leave the chip idle, but only where that saves
// more than the merge launch costs (about 4 us: 990 rows of 8 heads take 15.9 us in one range each, 6 + 4 in four).
int decode_splits_used(int B, int Hkv, int d, int k_cap) {
  const int most = decode_splits(B, Hkv, k_cap), units = B * Hkv;
  const int rows = d == 128 ? 256 : 512;  // per range
  if (k_cap <= 3 * rows || units > 128) return 1;
  int S = (k_cap + rows - 1) / rows;
  if (S > 512 / units) S = 512 / units;
  return S < most ? S : most;
}

// One range per head, but its output columns over several workgroups: up to 128 of them, where there is something to fetch.  Launches
// behind one another, us each, before -> with it: 8 heads of 4 queries, d = 128, 64 rows 4.1 -> 3.6, 256 rows 7.3 -> 6.6, 512 rows 9.6 ->
// 8.4, 768 rows 11.8 -> 10.0; of 8 queries, 512 rows 9.9 -> 8.0; 32 heads of one query, 64 rows 3.3 -> 3.8, 128 rows 4.3 -> 4.3, 512
// rows 8.6 -> 7.9; d = 64, 8 heads of 4 queries, 512 rows 6.9 -> 6.6.  256 workgroups: 64 heads of one query, 128 rows 4.4 -> 5.1, of
// 4 queries 5.4 -> 5.5, 512 rows 10.7 -> 10.7.
constexpr int kColumnsMaxWorkgroups = 128;
static bool decode_by_columns(const DecodeArgs& a) {
  return a.S == 1 && a.B * a.Hkv * (a.d / kColumns) <= kColumnsMaxWorkgroups && a.k_cap >= (a.G > 1 ? 64 : 128);
}

// Waves per workgroup: sixteen (one workgroup per compute unit) up to 256 workgroups, four beyond 1024.  In between
// eight, two workgroups per compute unit at a time, the next one starting where one is done (768 workgroups of 32 ..
// 1368 rows: 60 us, with four waves, all of them resident from the start, 75 us), but four where they are short (1024
// workgroups of 128 rows on average: 16 instead of 18 us).  Not many more than the longest range has tiles.
int decode_waves(int64_t workgroups, int64_t rows_total, int d, int G, int chunk) {
  int nw = workgroups <= 256 ? max_waves(G) : (workgroups <= 1024 && rows_total >= 256 * workgroups ? 8 : 4);
  const int tiles = (chunk + (d == 128 ? 15 : 31)) / (d == 128 ? 16 : 32);
  while (nw > 4 && nw / 2 >= tiles) nw /= 2;
  return nw;
}

// All layers in one launch: keys per range that the workspace has room for (about 512 ranges in all, 256 to 1024
// keys, at most 16 per head) ...
int decode_layers_chunk(int64_t rows_total) {
  int64_t c = (rows_total + 511) / 512;
  c = c < 256 ? 256 : (c > 1024 ? 1024 : c);
  return (int)((c + 31) / 32 * 32);
}
int decode_layers_splits(int k_cap, int chunk_target, int* chunk) {
  int S = (k_cap + chunk_target - 1) / chunk_target;
  S = S < 1 ? 1 : (S > kMaxSplits ? kMaxSplits : S);
  *chunk = ((k_cap + S - 1) / S + 31) / 32 * 32;
  return S;
}
// ... and those used, never shorter than that.  With a head for every compute unit: one range per head (no partial
// results, no merge launch: 768 heads of 32 .. 1368 rows 75 -> 60 us, 2048 heads of 133 .. 3963 rows 376 -> 355 us),
// except for few long heads, where the longest would outlast the rest (256 heads of 133 .. 3963 rows: 63 -> 60 us).
// With fewer heads: enough ranges for one per compute unit, of at least 256 keys.
int decode_layers_chunk_used(int64_t units, int64_t rows_total) {
  if (units >= 1024 || (units >= 256 && rows_total < 1536 * units)) return kDecodeMaxRows;
  if (units >= 256) return decode_layers_chunk(rows_total);
  int64_t c = (rows_total + 255) / 256;
  c = c < 256 ? 256 : (c > kDecodeMaxRows ? kDecodeMaxRows : c);
  return (int)((c + 31) / 32 * 32);
}

// q = j / page_size for 0 <= j < 4096: a shift, or the high half of a product with ceil(2^32 / page_size) (exact
// while j * page_size < 2^32; larger pages hold every row, so q = 0).
void decode_page_division(int page_size, int32_t* shift, uint32_t* magic) {
  *shift = -1;
  *magic = 0;
  if (page_size < 1) return;
  if ((page_size & (page_size - 1)) == 0) {
    *shift = __builtin_ctz((unsigned)page_size);
  } else if (page_size < kDecodeMaxRows) {
    *magic = (uint32_t)((((uint64_t)1 << 32) + page_size - 1) / page_size);
  }
}

hipError_t launch_decode_attention_layers(const DecodeBatchArgs& a, int total_wgs, int nw, bool any_split, hipStream_t s) {
  const hipError_t e = with_variant(a.d, a.G, a.page_size > 0, [&](auto D, auto GP, auto P) {
    return launch_partial_layers<decltype(D)::value, decltype(GP)::value, decltype(P)::value>(a, total_wgs, nw, s);
  });
  if (e != hipSuccess || !any_split) return e;
  if (a.d == 128) hipLaunchKernelGGL(decode_merge_layers_kernel<128>, dim3(a.Hkv, a.B, a.L), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(decode_merge_layers_kernel<64>, dim3(a.Hkv, a.B, a.L), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_decode_attention(const DecodeArgs& a, hipStream_t s) {
  if (decode_by_columns(a)) {
    const int nw = decode_waves((int64_t)a.B * a.Hkv * (a.d / kColumns), (int64_t)a.B * a.Hkv * a.k_cap, a.d, a.G, a.chunk);
    return with_variant(a.d, a.G, a.page_size > 0, [&](auto D, auto GP, auto P) {
      return launch_columns<decltype(D)::value, decltype(GP)::value, decltype(P)::value>(a, nw, s);
    });
  }
  const int nw = decode_waves((int64_t)a.S * a.B * a.Hkv, (int64_t)a.B * a.Hkv * a.k_cap, a.d, a.G, a.chunk);
  const hipError_t e = with_variant(a.d, a.G, a.page_size > 0, [&](auto D, auto GP, auto P) {
    return launch_partial<decltype(D)::value, decltype(GP)::value, decltype(P)::value>(a, nw, s);
  });
  if (e != hipSuccess || a.S == 1) return e;
  if (a.d == 128) hipLaunchKernelGGL(decode_merge_kernel<128>, dim3(a.Hkv, a.B), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(decode_merge_kernel<64>, dim3(a.Hkv, a.B), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace pkv
