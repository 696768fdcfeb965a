// Window scoring in two streaming launches over K for many query rows per KV head (G * alpha > 128; Sec. 4.2.2, Eq. Al
// and Eq. att_score) on MI355X; with supplied softmax denominators in one launch (G * alpha > 32, or few keys).
//
// With many query rows the scoring is bound by its products and exponentials and not by the bandwidth of K, so that
// reading K a second time is free, and what costs is everything that keeps the SIMDs from multiplying: waits for other
// workgroups and staging of Q.  Here there is neither: one launch forms the softmax statistics, the next one the scores,
// and no workgroup waits for another.  One workgroup of 512 threads per compute unit keeps ALL query rows of its unit
// (layer, sequence, KV head) in LDS (512 rows of 128 elements: 136 of 160 KB) and streams keys past them, two waves per
// SIMD that drift apart freely.
//
// Work split.  Units are cut into chunks of C keys (from one layer's shape, so that a call over many layers gives the
// results of one call per layer); workgroup j of W takes the chunks [j T / W, (j + 1) T / W), so that it changes units,
// and with them Q, a few times per launch.  In a chunk the workgroup takes 512 or 1024 keys per pass: each wave holds two 32-key
// tiles as matrix operands, multiplies them with all row tiles, and requests the next pass's keys meanwhile.
//
// Launch 1, per chunk and row: z = sum exp2(x - m) with the largest of the row's logits of 64 sampled keys, key 0 among
// them, as reference m: near the terms that count, so that x - m loses nothing to its rounding (with key 0's logit alone
// the scores were 1.0e-6 off those of 64 bits at 512 rows, the register-resident kernel's 0.6e-6), and the same for all
// keys.  The sampled keys alone contribute 1 to the unit's sum, so vanishing terms are as they should be; a sum beyond
// 2^100 makes the workgroup form its chunk again with the chunk's exact maxima (rare).
// Launch 2, when it takes up a unit, folds the statistics of its chunks into the normalisers c_r, rounded once (scores of 512
// rows 6.2e-7 -> 1.3e-7 off those of 64 bits, of 256 rows at d = 64 4.5e-7 -> 0.8e-7; the register-resident kernel 5.9e-7 and
// 4.2e-7), or takes the supplied denominators (then it is the only launch), and writes s_i = sum_r exp2(x_ri - c_r) / G.
//
// Inner loops as in the register-resident kernel: one product's matrix instructions are issued between the exponentials
// of the one before, in an order fixed in the source.
//
// What bounds it: the sweeps.  640 units of 32k keys, 512 rows: 3.04 + 2.62 ms (by the profiler, after 6.4 ms for the
// register-resident kernel's one launch) against 2.2 ms per sweep for a bare loop of these instructions at the clock the
// chip holds under them; 0.9 ms of that is what K takes to read.  The scores took 2.80 ms with eight waves; for the
// statistics sixteen do not help (3.04 -> 3.2 ms: their tables of sums do not fit beside 512 rows).
#include <type_traits>

#include "pkv_internal.h"
#include "pkv_tile.h"

namespace pkv {
namespace {

constexpr int kSums = 8;  // waves that form statistics

// End of a hand-ordered chunk of instructions: nothing is scheduled across it, and the running sums are pinned here.
#define PKV_CHUNK_END_SUMS(s0, s1)                 \
  do {                                             \
    asm volatile("" : "+v"(s0), "+v"(s1));         \
    __builtin_amdgcn_sched_barrier(0);             \
  } while (0)
// c as three bf16 summands (to 2^-24): the first three k-elements of a matrix operand.  -inf stays -inf.
__device__ __forceinline__ u64 split3(float c) {
  const __bf16 hi = (__bf16)c;
  float r = c - (float)hi;
  if (c == -INFINITY) r = 0.f;
  const __bf16 mid = (__bf16)r;
  r -= (float)mid;
  const __bf16 lo = (__bf16)r;
  const uint32_t w0 = (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, mid) << 16);
  return ((u64)__builtin_bit_cast(uint16_t, lo) << 32) | w0;
}

template <int D, bool SCORE>
constexpr size_t sweep_lds(int Rs) {
  // Q with a row pitch of D / 8 + 1 sixteen-byte slots (bank-free); a zero slot; normalisers, or references (in use,
  // original) and sums by wave, and the flag
  return (size_t)Rs * (D / 8 + 1) * 16 + 16 + (SCORE ? (size_t)Rs * 8 : (size_t)Rs * 4 * (2 + kSums) + 16);
}
static_assert(sweep_lds<128, false>(kResidentMaxRows) <= 160 * 1024, "one workgroup per compute unit");

// kW: waves per workgroup, 8, or 16 for the scores of launches with several passes per workgroup.
template <int D, bool SCORE, int kW>
__global__ __launch_bounds__(64 * kW, kW / 4) void score_sweep_kernel(const SweepArgs a) {
  static_assert(SCORE || kW == kSums, "a table of sums per wave");
  constexpr int kT = kW * 64, kPassKeys = 64 * kW;  // threads; keys of a pass
  constexpr int KS = D / 16, SEG = D / 8, PITCH = SEG + 1;
  constexpr int TPM = 16 / KS;  // logits per lane handled between two matrix instructions
  extern __shared__ u32x4 smem[];
  u32x4* s_q = smem;
  u32x4* s_zero = s_q + a.Rs * PITCH;
  u64* s_c = reinterpret_cast<u64*>(s_zero + 1);      // [Rs] -c_r / kappa, split (SCORE)
  float* s_m = reinterpret_cast<float*>(s_zero + 1);  // [Rs] references in use (else)
  float* s_m0 = s_m + a.Rs;                           // [Rs] references of the unit
  float* s_z = s_m0 + a.Rs;                           // [kW][Rs] sums by wave
  int* s_bad = reinterpret_cast<int*>(s_z + kW * a.Rs);  // [2] a chunk's reference does not fit; used in turn

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hf = lane >> 5;
  const int BH = a.B * a.Hkv, nrt = a.Rs / 32;
  const int C = SCORE ? a.score_C : a.C, nchunk = SCORE ? a.score_nchunk : a.nchunk;

  auto length = [&](int b) {
    int n = a.N;
    if (a.seq_lens) {
      n = a.seq_lens[b];
      n = n < 0 ? 0 : (n > a.N ? a.N : n);
    }
    return n;
  };

  // One pass of the workgroup (all fields wave-uniform): its keys from `key` on of chunk `chunk` of unit u.
  struct Pass {
    int u, n, chunk, key, left;  // left: chunks of this workgroup behind this one
    const uint16_t* Q;
    const uint16_t* K;
  };
  auto open_unit = [&](Pass& p) {  // pointers and length of unit p.u; false: the unit needs no scores
    const int l = p.u / BH, bg = p.u - l * BH;
    const int b = bg / a.Hkv, g = bg - b * a.Hkv;
    p.n = length(b);
    p.Q = a.layer[l].Q + (size_t)b * a.q_sb + (size_t)(g * a.G) * a.q_sh;
    p.K = a.layer[l].K + (size_t)b * a.kv_sb + (size_t)g * a.kv_sh;
    return a.layer[l].k_l < p.n;
  };
  Pass cur;
  {
    // first chunk and number of chunks of this workgroup
    int total, u0 = 0, c0 = 0;
    if (a.uniform) {
      total = a.L * BH * nchunk;
      const int lo = (int)((int64_t)blockIdx.x * total / gridDim.x), hi = (int)((int64_t)(blockIdx.x + 1) * total / gridDim.x);
      u0 = lo / nchunk;
      c0 = lo - u0 * nchunk;
      cur.left = hi - lo;
    } else {
      int* wsum = reinterpret_cast<int*>(smem);  // [kW] sums of the waves, [kW], [kW + 1] the first chunk's place
      const int E = a.L * a.B;
      int lo = 0, hi = 0;
      for (int round = 0; round < 2; ++round) {  // how many chunks there are; then who owns the first one
        int run = 0;
        for (int e0 = 0; e0 < E; e0 += kT) {
          const int e = e0 + tid;
          int c = 0, parts = 0;
          if (e < E) {
            const int l = e / a.B, n = length(e - l * a.B);
            parts = a.layer[l].k_l < n ? (n + C - 1) / C : 0;
            c = a.Hkv * parts;
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
          before += v - c;
          if (round == 1 && lo >= before && lo < before + c) {
            const int rem = lo - before, g = rem / parts;
            wsum[kW] = e * a.Hkv + g;
            wsum[kW + 1] = rem - g * parts;
          }
        }
        if (round == 0) {
          lo = (int)((int64_t)blockIdx.x * run / gridDim.x);
          hi = (int)((int64_t)(blockIdx.x + 1) * run / gridDim.x);
        }
      }
      __syncthreads();
      cur.left = hi - lo;
      if (cur.left > 0) {
        u0 = __builtin_amdgcn_readfirstlane(wsum[kW]);
        c0 = __builtin_amdgcn_readfirstlane(wsum[kW + 1]);
      }
      __syncthreads();
    }
    if (cur.left == 0) return;
    --cur.left;
    cur.u = u0;
    cur.chunk = c0;
    cur.key = c0 * C;
    (void)open_unit(cur);
  }
  // The pass after p; false if there is none (p is then a pass over the unit's first key alone).
  auto advance = [&](Pass& p) {
    p.key += kPassKeys;
    if (p.key < min((p.chunk + 1) * C, p.n)) return true;
    if (p.left == 0) {
      p.key = 0;
      p.n = 1;
      return false;
    }
    --p.left;
    ++p.chunk;
    if (p.chunk * C >= p.n) {
      p.chunk = 0;
      do ++p.u;
      while (!open_unit(p));  // (there is one: a chunk is left)
    }
    p.key = p.chunk * C;
    return true;
  };

  // Queries of a unit into LDS, and the normalisers (SCORE).  Barriers around it are the caller's.
  auto stage = [&](const Pass& p) {
    const int seg = tid & (SEG - 1);
    const char* src = reinterpret_cast<const char*>(p.Q) + 16 * seg;
    for (int row0 = tid / SEG; row0 < a.Rs; row0 += 4 * (kT / SEG)) {  // (uniform over a wave)
      u32x4 v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = row0 + j * (kT / SEG);
        v[j] = u32x4{0u, 0u, 0u, 0u};
        if (row < a.R) {
          const int hh = row / a.alpha, t = row - hh * a.alpha;
          v[j] = *reinterpret_cast<const u32x4*>(src + (uint32_t)((hh * a.q_sh + t * a.q_st) * 2));
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = row0 + j * (kT / SEG);
        if (row < a.Rs) s_q[row * PITCH + seg] = v[j];
      }
    }
    if (SCORE) {
      if (tid < a.Rs) {
        u64 w3 = split3(-INFINITY);  // -c / kappa; padding rows contribute exp2(-inf) = 0
        if (tid < a.R) {
          if (a.lse_mode) {
            const int l = p.u / BH, bg = p.u - l * BH, b = bg / a.Hkv, g = bg - b * a.Hkv;
            const float c = a.layer[l].lse[((size_t)b * a.Hq + (size_t)g * a.G) * a.alpha + tid] * 1.44269504088896340736f;
            w3 = split3(-c * a.inv_kappa);
          } else {
            const u64* st = a.stats + (size_t)p.u * a.nchunk * a.Rs + tid;
            const int parts = (p.n + a.C - 1) / a.C;
            float m = -INFINITY, z = 0.f;
            for (int q0 = 0; q0 < parts; q0 += 8) {
              u64 w[8];
#pragma unroll
              for (int k = 0; k < 8; ++k) w[k] = st[(size_t)min(q0 + k, parts - 1) * a.Rs];
              float M = m;
#pragma unroll
              for (int k = 0; k < 8; ++k) M = fmaxf(M, __uint_as_float((uint32_t)w[k]));
              const float Ms = (M == -INFINITY) ? 0.f : M;
              z *= fast_exp2(m - Ms);
#pragma unroll
              for (int k = 0; k < 8; ++k)
                if (q0 + k < parts)
                  z = __builtin_fmaf(__uint_as_float((uint32_t)(w[k] >> 32)), fast_exp2(__uint_as_float((uint32_t)w[k]) - Ms), z);
              m = M;
            }
            // c = m + log2 z, divided by kappa and rounded once: the logarithm of the mantissa alone (between 0 and 1, its
            // error is below 2^-24; that of log2 z, not centred on 0, showed in all scores of a row), the sum's rounding
            // error and the quotient's remainder are carried along
            const float e = (float)(__builtin_amdgcn_frexp_expf(z) - 1), lf = fast_log2(__builtin_amdgcn_frexp_mantf(z) * 2.f);
            const float t = m + e, t1 = t - m, err = (m - (t - t1)) + (e - t1);
            const float q = -t * a.inv_kappa, rem = __builtin_fmaf(q, a.kappa, t);
            w3 = split3(__builtin_fmaf(-(rem + (err + lf)), a.inv_kappa, q));
          }
        }
        s_c[tid] = w3;
      }
    }
  };

  // Keys of a wave's two tiles as matrix operands: lane (l32, hf) holds elements 16 ks + 8 hf of key 32 t + l32.  Keys
  // at or beyond n are replaced by the last one.
  bf16x8 kf[2][KS], kn[2][KS];
  auto issue_k = [&](const Pass& p, int t, int lo, int hi, bf16x8 (&f)[2][KS]) {
    const int ln = fresh(lane);
    const int key = min(p.key + 64 * wave + 32 * t + (ln & 31), p.n - 1);
    const char* rowp = reinterpret_cast<const char*>(p.K) + 16 * (ln >> 5) + (uint32_t)key * ((uint32_t)a.kv_st * 2u);
#pragma unroll
    for (int ks = lo; ks < hi; ++ks) f[t][ks] = as_frag(*reinterpret_cast<const u32x4*>(rowp + 32 * ks));
    __builtin_amdgcn_sched_barrier(0);
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const u32x4* q_lane = s_q + l32 * PITCH + hf;
  auto q_frag = [&](int rt, int ks) { return as_frag(q_lane[32 * rt * PITCH + 2 * ks]); };
  // References of a unit's rows: the largest logit over 64 keys spread evenly over the prefix, key 0 among them.  The keys
  // are requested before the queries are staged (into kf, free at that time); wave w takes the row tiles w, w + 8, ...
  auto sample_keys = [&](const Pass& p) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int ln = fresh(lane), key = (int)((int64_t)(32 * t + (ln & 31)) * (p.n - a.alpha) >> 6);
      const char* rowp = reinterpret_cast<const char*>(p.K) + 16 * (ln >> 5) + (uint32_t)key * ((uint32_t)a.kv_st * 2u);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[t][ks] = as_frag(*reinterpret_cast<const u32x4*>(rowp + 32 * ks));
    }
  };
  auto set_references = [&]() {
#pragma unroll 1
    for (int rt = wave; rt < nrt; rt += kW) {
      float m = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x16 y = zero16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) y = PKV_MFMA32(kf[t][ks], q_frag(rt, ks), y);
#pragma unroll
        for (int v = 0; v < 16; ++v) m = fmaxf(m, y[v]);
      }
      m = both_halves<true>(m) * a.kappa;
      if (hf == 0) s_m[32 * rt + l32] = s_m0[32 * rt + l32] = m;
    }
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using INONE = std::integral_constant<int, -1>;

  if (tid == 0) {
    *s_zero = u32x4{0u, 0u, 0u, 0u};
    if (!SCORE) s_bad[0] = s_bad[1] = 0;
  }
  if constexpr (SCORE) {
    stage(cur);
    issue_k(cur, 0, 0, KS, kf);
    issue_k(cur, 1, 0, KS, kf);
    lds_barrier();
  } else {
    sample_keys(cur);
    issue_k(cur, 0, 0, KS, kn);
    issue_k(cur, 1, 0, KS, kn);
    stage(cur);
    lds_barrier();
    set_references();
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) kf[t][ks] = kn[t][ks];
    lds_barrier();
  }

  bool first = true;  // first pass of a chunk
  int turn = 0;       // of the flags
  for (;;) {
    Pass nxt = cur;
    const bool has_next = advance(nxt);
    const int wkey = cur.key + 64 * wave;
    const int npre = cur.n - a.alpha;
    bf16x8 qf[KS];
    f32x16 fin, out;
    // half a tile of the next pass's keys is requested at a time, at fixed places of the first two row tiles
    auto refill = [&](auto RF, int half) {
      if constexpr (decltype(RF)::value >= 0) issue_k(nxt, decltype(RF)::value, half * (KS / 2), half * (KS / 2) + KS / 2, kn);
    };
    if constexpr (!SCORE) {
      // Product rows = keys (element v of a lane: key mrow0(v) + 4 hf of the tile), columns = query rows (l32).
      float* z_lane = s_z + wave * a.Rs + l32;
      const bool dirty = wkey + 64 > npre;  // a tile reaches into the causal window or beyond the end
      bool bad = false;
      auto pass = [&](auto MASKED) {
        constexpr bool masked = decltype(MASKED)::value;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = q_frag(0, ks);
        fin = zero16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fin = PKV_MFMA32(kf[0][ks], qf[ks], fin);
        // The product of tile TN goes into `nx` while `fi`, that of tile 1 - TN, turns into exponentials.
        auto step = [&](auto TN, auto RF, int rt_next, float nref, int lim, const f32x16& fi, f32x16& nx, float& s0, float& s1) {
          constexpr int tn = decltype(TN)::value, tc = 1 - tn;
          const float kap = a.kappa;
          nx = zero16;
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            nx = PKV_MFMA32(kf[tn][ks], qf[ks], nx);
            if (tn == 1) qf[ks] = q_frag(rt_next, ks);  // (last use of this row tile's fragment)
            float x[TPM];
#pragma unroll
            for (int j = 0; j < TPM; ++j) {
              x[j] = __builtin_fmaf(fi[TPM * ks + j], kap, nref);
              if (masked && 32 * tc + mrow0(TPM * ks + j) > lim) x[j] = -INFINITY;
            }
#pragma unroll
            for (int j = 0; j < TPM; ++j) x[j] = fast_exp2(x[j]);
#pragma unroll
            for (int j = 0; j < TPM; ++j) {
              if (j & 1) s1 += x[j]; else s0 += x[j];
            }
            PKV_CHUNK_END_SUMS(s0, s1);
            if (ks == KS / 2 - 1) refill(RF, tn == 1 ? 0 : 1);
          }
        };
        auto iter = [&](auto RF, int rt) {
          const int rt_next = rt + 1 < nrt ? rt + 1 : 0;  // (the last product of the pass is not used)
          const float nref = -s_m[32 * rt + l32];
          int lim = 0;
          if (masked) lim = npre + (32 * rt + l32) % a.alpha - wkey - 4 * hf;  // last key the lane's query sees
          float s0 = 0.f, s1 = 0.f;
          step(I1{}, RF, rt_next, nref, lim, fin, out, s0, s1);
          step(I0{}, RF, rt_next, nref, lim, out, fin, s0, s1);
          float z = both_halves<false>(s0 + s1);
          bad = bad || !(z <= 0x1p100f);
          if (!first) z += z_lane[32 * rt];
          if (hf == 0) z_lane[32 * rt] = z;
        };
        iter(I0{}, 0);
        if (nrt > 1) iter(I1{}, 1);
        else issue_k(nxt, 1, 0, KS, kn);
#pragma unroll 1
        for (int rt = 2; rt < nrt; ++rt) iter(INONE{}, rt);
      };
      if (dirty) pass(std::true_type{});
      else pass(std::false_type{});
      if (__any(bad) && lane == 0) s_bad[turn] = 1;

      const bool ends = !has_next || nxt.chunk != cur.chunk || nxt.u != cur.u;
      if (ends) {
        lds_barrier();
        if (tid == 0) s_bad[turn ^ 1] = 0;
        if (s_bad[turn] != 0) {
          // rare: a reference that does not fit; round 0 finds the chunk's maxima, round 1 forms the sums with them
          const int end = min((cur.chunk + 1) * C, cur.n);
          for (int round = 0; round < 2; ++round) {
            for (int r = lane; r < a.Rs; r += 64) s_z[wave * a.Rs + r] = round == 0 ? -INFINITY : 0.f;
            lds_barrier();
            Pass q = cur;
            for (q.key = cur.chunk * C; q.key < end; q.key += kPassKeys) {
              issue_k(q, 0, 0, KS, kf);
              issue_k(q, 1, 0, KS, kf);
#pragma unroll 1
              for (int rt = 0; rt < nrt; ++rt) {
                const float ref = s_m[32 * rt + l32];
                const int lim = npre + (32 * rt + l32) % a.alpha - q.key - 64 * wave - 4 * hf;
                float acc = round == 0 ? -INFINITY : 0.f;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                  f32x16 y = zero16;
#pragma unroll
                  for (int ks = 0; ks < KS; ++ks) y = PKV_MFMA32(kf[t][ks], q_frag(rt, ks), y);
#pragma unroll
                  for (int v = 0; v < 16; ++v) {
                    const bool hidden = 32 * t + mrow0(v) > lim;
                    if (round == 0) acc = fmaxf(acc, hidden ? -INFINITY : y[v] * a.kappa);
                    else acc += hidden ? 0.f : fast_exp2(__builtin_fmaf(y[v], a.kappa, -ref));
                  }
                }
                acc = round == 0 ? both_halves<true>(acc) : both_halves<false>(acc);
                const float old = z_lane[32 * rt];
                if (hf == 0) z_lane[32 * rt] = round == 0 ? fmaxf(old, acc) : old + acc;
              }
            }
            lds_barrier();
            if (round == 0) {
              if (tid < a.Rs) {
                float m = -INFINITY;
#pragma unroll
                for (int w = 0; w < kW; ++w) m = fmaxf(m, s_z[w * a.Rs + tid]);
                s_m[tid] = m == -INFINITY ? 0.f : m;
              }
              lds_barrier();
            }
          }
        }
        if (tid < a.Rs) {
          float z = 0.f;
#pragma unroll
          for (int w = 0; w < kW; ++w) z += s_z[w * a.Rs + tid];
          // (nothing to add up: no reference either, lest the stand-in for one of -inf outweighs the other chunks')
          const float m = z == 0.f ? -INFINITY : s_m[tid];
          a.stats[((size_t)cur.u * a.nchunk + cur.chunk) * a.Rs + tid] = ((u64)__float_as_uint(z) << 32) | __float_as_uint(m);
          s_m[tid] = s_m0[tid];
        }
        lds_barrier();
        turn ^= 1;
      }
      first = ends;
    } else {
      // Product rows = query rows (element v of a lane: row mrow0(v) + 4 hf), columns = keys (l32).  The normalisers
      // enter through one more matrix instruction: (hi, mid, lo) of the lane's row times ones, in the first wave half.
      const u32x4 ones_u = (hf == 0) ? u32x4{0x3F803F80u, 0x00003F80u, 0u, 0u} : u32x4{0u, 0u, 0u, 0u};
      const bf16x8 ones = as_frag(ones_u);
      const u64* c_lane = (hf == 0) ? s_c + l32 : reinterpret_cast<const u64*>(s_zero);
      const int c_step = (hf == 0) ? 32 : 0;
      bf16x8 bfr;
      auto load_bias = [&](int rt) {
        const u64 w = c_lane[c_step * rt];
        bfr = as_frag(u32x4{(uint32_t)w, (uint32_t)(w >> 32), 0u, 0u});
      };
      float e0 = 0.f, e1 = 0.f;
      if constexpr (kW == 16) {
        // Four waves per SIMD with half the registers each: a wave multiplies both tiles, then forms the exponentials,
        // and the others fill the gaps.  Its keys are requested again as soon as they have been multiplied.
        auto tile = [&](int rt, bool last) {
          load_bias(rt);
          f32x16 x0 = PKV_MFMA32(bfr, ones, zero16), x1 = PKV_MFMA32(bfr, ones, zero16);
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 q = q_frag(rt, ks);
            x0 = PKV_MFMA32(q, kf[0][ks], x0);
            x1 = PKV_MFMA32(q, kf[1][ks], x1);
          }
          if (last) {
            __builtin_amdgcn_sched_barrier(0);
            issue_k(nxt, 0, 0, KS, kf);
            issue_k(nxt, 1, 0, KS, kf);
          }
          // (the order of the sums is the eight waves': the scores do not depend on who writes them)
          float s0 = 0.f, s1 = 0.f, t0 = 0.f, t1 = 0.f;
#pragma unroll
          for (int v = 0; v < 16; v += 2) {
            s0 += fast_exp2(x0[v] * a.kappa);
            s1 += fast_exp2(x0[v + 1] * a.kappa);
            t0 += fast_exp2(x1[v] * a.kappa);
            t1 += fast_exp2(x1[v + 1] * a.kappa);
          }
          e0 += s0 + s1;
          e1 += t0 + t1;
        };
#pragma unroll 1
        for (int rt = 0; rt + 1 < nrt; ++rt) tile(rt, false);
        tile(nrt - 1, true);
      } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = q_frag(0, ks);
        load_bias(0);
        fin = PKV_MFMA32(bfr, ones, zero16);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fin = PKV_MFMA32(qf[ks], kf[0][ks], fin);
        auto step = [&](auto TN, auto RF, int rt_next, const f32x16& fi, f32x16& nx, float& e) {
          constexpr int tn = decltype(TN)::value;
          float s0 = 0.f, s1 = 0.f;
          float kap = a.kappa;
          asm volatile("" : "+s"(kap));
          nx = PKV_MFMA32(bfr, ones, zero16);
          if (tn == 1) load_bias(rt_next);
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) {
            nx = PKV_MFMA32(qf[ks], kf[tn][ks], nx);
            if (tn == 1) qf[ks] = q_frag(rt_next, ks);
            float x[TPM];
#pragma unroll
            for (int j = 0; j < TPM; ++j) x[j] = fi[TPM * ks + j] * kap;
#pragma unroll
            for (int j = 0; j < TPM; ++j) x[j] = fast_exp2(x[j]);
#pragma unroll
            for (int j = 0; j < TPM; ++j) {
              if (j & 1) s1 += x[j]; else s0 += x[j];
            }
            PKV_CHUNK_END_SUMS(s0, s1);
            if (ks == KS / 2 - 1) refill(RF, tn == 1 ? 0 : 1);
          }
          e += s0 + s1;
        };
        auto iter = [&](auto RF, int rt) {
          const int rt_next = rt + 1 < nrt ? rt + 1 : 0;
          step(I1{}, RF, rt_next, fin, out, e0);
          step(I0{}, RF, rt_next, out, fin, e1);
        };
        iter(I0{}, 0);
        if (nrt > 1) iter(I1{}, 1);
        else issue_k(nxt, 1, 0, KS, kn);
#pragma unroll 1
        for (int rt = 2; rt < nrt; ++rt) iter(INONE{}, rt);
      }
      const float s = both_halves<false>(e0), t = both_halves<false>(e1);
      const int key = wkey + lane;
      if (key < npre) a.raw[(size_t)cur.u * a.N + key] = (hf == 0 ? s : t) * a.inv_G;
    }
    if (!has_next) break;
    if (nxt.u != cur.u) {
      if (SCORE) lds_barrier();  // every wave is done with the unit's queries (else: the barrier behind the statistics)
      if constexpr (!SCORE) sample_keys(nxt);
      stage(nxt);
      lds_barrier();
      if constexpr (!SCORE) {
        set_references();
        lds_barrier();
      }
    }
    if constexpr (kW == 8) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kf[t][ks] = kn[t][ks];
    }
    cur = nxt;
  }
}

template <int D, bool SCORE, int kW>
hipError_t launch_sweep(const SweepArgs& a, hipStream_t s) {
  static bool attr_set[kMaxDevices];
  const int dev = current_device_slot();
  if (dev < 0) return hipErrorInvalidDevice;
  if (!attr_set[dev]) {  // raise the dynamic LDS limit once per device (idempotent; no allocation)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(score_sweep_kernel<D, SCORE, kW>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sweep_lds<D, SCORE>(kResidentMaxRows));
    if (e != hipSuccess) return e;
    attr_set[dev] = true;
  }
  const size_t lds = sweep_lds<D, SCORE>(a.Rs);
  hipLaunchKernelGGL((score_sweep_kernel<D, SCORE, kW>), dim3(a.grid), dim3(64 * kW), lds, s, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_sweep(const SweepArgs& a, hipStream_t s) {
  if (a.d != 64 && a.d != 128) return hipErrorInvalidValue;
  if (!a.lse_mode) {
    const hipError_t e = a.d == 128 ? launch_sweep<128, false, 8>(a, s) : launch_sweep<64, false, 8>(a, s);
    if (e != hipSuccess) return e;
  }
  if (a.score_waves == 16) return a.d == 128 ? launch_sweep<128, true, 16>(a, s) : launch_sweep<64, true, 16>(a, s);
  return a.d == 128 ? launch_sweep<128, true, 8>(a, s) : launch_sweep<64, true, 8>(a, s);
}

}  // namespace pkv
