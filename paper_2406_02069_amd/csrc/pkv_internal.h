// Internal declarations shared by the translation units of libpkv (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "pkv.h"
#include "pkv_measure.h"

namespace pkv {

// Upper bounds the kernels are written for; the host rejects anything beyond them.
constexpr int kMaxAlpha = 64;
constexpr int kMaxPoolW = 63;
constexpr int kKeysPerTile = 32;     // one MFMA tile of keys
constexpr int kWavesPerBlock = 4;    // score kernels
constexpr int kSelectThreads = 1024; // pool + select kernel

constexpr int kMaxLayers = 1024;     // layers per call

// How a call is split over the device; derived from the shape and the layer count only (never from
// k_l), so that one workspace size serves every budget.
struct Plan {
  int G;         // query heads per KV head
  int R;         // query rows sharing one KV head: G * alpha
  int BH;        // B * Hkv
  int L;
  // register-resident scoring
  bool resident_ok;
  int res_Rpad, res_nrb;  // rows padded to 128-row blocks
  int TPU;       // 512-key parts per unit
  int ngroups;   // independent workgroup groups (512 / group size)
  int UPG;       // units in flight per group
  // per-layer streaming scoring
  int RT;        // 32-row MFMA tiles per row block (1, 2 or 4)
  int RB;        // rows per row block: 32 * RT
  int nrb;       // row blocks: ceil(R / RB)
  int Rpad;      // nrb * RB
  int KC;        // keys per score workgroup (multiple of 128)
  int nchunk;    // ceil(N / KC)
  // workspace carve-up (byte offsets, each 256-aligned)
  size_t off_cnt, off_part, off_cfin, off_raw, off_pooled, total;
  size_t sync_bytes;  // error word + counters + tagged normalisers (zeroed before each resident launch)
};

Plan make_plan(const pkv_layer_desc& d, int L);

struct ScoreArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const int32_t* seq_lens;
  float2* part;  // [BH][Rpad][nchunk] per-chunk softmax statistics (max, sum) in the log2 domain
  float* cfin;   // [BH][Rpad] per-row log2 normaliser: max + log2(sum)
  float* raw;    // [nrb][BH][N] un-pooled scores, one partial per row block
  int32_t B, Hq, Hkv, G, alpha, N, k_l, R, Rpad, nrb, KC, nchunk, RT, d;
  int64_t q_sb, q_sh, q_st, kv_sb, kv_sh, kv_st;
  float kappa;   // log2(e) / sqrt(d)
  const float* lse;  // [B][Hq][alpha] supplied natural-log softmax denominators, or null
};


// ---- register-resident scoring over many layers (pkv_resident.hip) ----
constexpr int kResidentCUs = 256;       // compute units the persistent grid is sized for
constexpr int kResidentGrid = 512;      // persistent workgroups: two per compute unit, one wave per SIMD each
constexpr int kResidentKeys = 512;      // keys held in registers by one workgroup (4 waves x 4 tiles x 32)
constexpr int kResidentMaxRows = 512;   // G * alpha (padded to 128) the LDS normaliser table can hold
constexpr int kResidentMaxLayers = 96;  // per launch (kernel-argument table)

struct ResidentLayer {
  const uint16_t* Q;
  const uint16_t* K;
  const float* lse;  // [B][Hq][alpha] supplied natural-log softmax denominators, or null (two-sweep scoring)
  int32_t k_l;
  int32_t slot;  // (lagging kernel) the layer's place among the score arrays
};

struct ResidentArgs {
  ResidentLayer layer[kResidentMaxLayers];
  const int32_t* seq_lens;
  float* raw;     // [U][N] un-pooled scores
  float2* part;   // [nslots][TPU][Rpad] per-part softmax statistics (log2 domain), reused from unit to unit
  int32_t* cnt;   // [U] arrivals per unit
  int32_t* err;   // in front of cnt: set to 1 if a bounded wait gave up; cleared by the first launch of a call only
  int32_t* zero_base;  // start of the words to zero before the launch (err or cnt)
  unsigned long long* cbuf;  // [nslots][Rpad] (unit tag << 32 | normaliser bits), behind err, 8-byte aligned
  int32_t sync_words;  // 32-bit words to zero from zero_base: (error word,) counters, cbuf
  int32_t L, B, Hq, Hkv, G, alpha, N, R, Rpad, nrb, TPU, U, d;
  int32_t ngroups;  // independent groups of workgroups: 512 / group size
  int32_t UPG;      // units a group works on at the same time: group size / TPU
  int32_t tagged;   // 1: statistics words carry a phase bit, parts fold their own rows (no arrival counter)
  int32_t part_words;  // 32-bit words of the per-part statistics (zeroed before a tagged launch)
  int32_t set1_w;   // share (of 32) of a group pair's units that goes to the group of second workgroups
  int32_t stagger;  // start offset between consecutive groups, in 10 ns ticks
  int32_t lse_mode;    // 1: every layer carries lse; one sweep, no exchange between workgroups
  int32_t wait_ticks;  // wall-clock bound (10 ns ticks) of a wait for other workgroups; beyond it the workgroup
                       // raises the error word and carries on (0: give up at once)
  int64_t q_sb, q_sh, q_st, kv_sb, kv_sh, kv_st;
  float kappa, inv_kappa, inv_G;
};

// ---- one-pass scoring for few query rows, over many layers (pkv_stream.hip) ----
constexpr int kStreamGrid = 256;    // persistent workgroups, one per compute unit
constexpr int kStreamMaxRows = 64;  // G * alpha
constexpr int kStreamItems = 272;   // items of a workgroup per launch, at most (table in LDS)
constexpr int kStreamUnits = 2048;  // layers x sequences per launch, at most (prefix table in LDS)

struct StreamArgs {
  ResidentLayer layer[kResidentMaxLayers];
  const int32_t* seq_lens;
  float* raw;                 // [U][N] un-pooled scores
  unsigned long long* stats;  // [words][word_rows] statistics (log2 domain; the sign bit of the sum marks a word as there);
                              // cleared before the launch
  int32_t* err;
  int32_t L, B, Hq, Hkv, G, alpha, N, R, d;
  int32_t uniform;            // 1: every unit has N keys and none is kept whole
  int32_t grid, items;        // workgroups (kStreamGrid, fewer if there are fewer items); items, if every unit has N keys
  int32_t item_keys, words_per_item, word_rows;  // keys of an item; its statistics words; rows of a word's place
  int32_t wait_ticks;
  int64_t q_sb, q_sh, q_st, kv_sb, kv_sh, kv_st;
  float kappa, inv_G;
};
// clear_err: the first launch of a call also clears the error word
hipError_t launch_score_stream(const StreamArgs& a, bool clear_err, hipStream_t s);

// ---- one-pass scoring, probabilities waiting on the chip for two steps of 64 rows, over many layers (pkv_lag.hip) ----
constexpr int kLagItems = 255;      // items of a workgroup per launch, at most (table in LDS)
constexpr int kLagKeys = 512;       // keys of an item
// Whether a unit of that many items may lie in two rounds of the workgroups, 256 items each, without the workgroups waiting for
// each other in a ring: not where its ends, a round apart, wait for what lies between (measured beside the host's rule).
__host__ __device__ constexpr bool lag_unit_straddles(int64_t parts, int groups) {
  return parts <= 88 || (groups == 1 && (parts <= 102 || (parts > 125 && parts <= 176)));
}
constexpr int kLagGroupBytes = 2048;   // of the workspace, per unit and group of 64 query rows
constexpr int kLagGroupBytes4 = 512;   // ... and of the last words for large sums, where there is room

constexpr int kLagRefs = 24, kLagMax = 28;  // places of the references and of the maxima in a block of 32 words (8 rows)
__device__ __forceinline__ uint32_t lag_half_word(int which, int row) { return (uint32_t)(2 * which + (row >> 3) * 64 + (row & 7)); }

struct LagArgs {
  ResidentLayer layer[kResidentMaxLayers];
  const int32_t* seq_lens;
  int32_t* flags;             // [layer slot][B][Hkv] of the sifting kernels: only what they have not scored, or null: all
  float* raw;                 // [layer slot][B][Hkv][N] un-pooled scores
  unsigned long long* words;  // [units][groups][256] sums, references, maxima; cleared by the first of the two kernels
  unsigned long long* words4; // [units][groups][64] last words for large sums, or null; likewise
  int32_t* err;
  int32_t L, B, Hq, Hkv, G, alpha, N, R, d;
  int32_t uniform;            // 1: every unit has N keys and none is kept whole
  int32_t parts;              // uniform: items of a unit (those beyond its end are empty)
  int32_t grid;               // workgroups (kStreamGrid, fewer if there are fewer items)
  int32_t wait_ticks;
  int32_t groups;             // of 64 query rows
  uint32_t alpha_magic;       // ceil(2^16 / alpha): row / alpha = (row alpha_magic) >> 16 for rows below 512
  uint32_t bh_magic, hkv_magic;  // floor((2^32 - 1) / x) of B Hkv and Hkv: u / x = ((u + 1) magic) >> 32 while (u + 1) x <= 2^32
  int64_t q_sb, q_sh, q_st, kv_sb, kv_sh, kv_st;
  float kappa, inv_G;
};
// prepared: the references and words are there
hipError_t launch_score_lag(const LagArgs& a, bool clear_err, bool prepared, hipStream_t s);

// ---- estimated scores of all keys, exact ones of those that can be kept, over many layers (pkv_sift.hip) ----
constexpr int kSiftMaxKeys = 131072;  // of a prefix
constexpr int kSiftJob = 256;         // keys scored exactly by a workgroup
// ... of a unit, at most: an eighth of its keys
__host__ __device__ constexpr int sift_list(int N) { return N / 8 / kSiftJob * kSiftJob; }
constexpr int kSiftMinKeys = 4096;    // of a prefix
// Estimates are no use where the scores of 63 keys spread by less than kSiftSpread binades (standard deviation; with average pooling,
// whose lists are longer, kSiftSpreadAvg): about 0.18 without a common direction of the queries, 0.35 at a strength of 0.2 (the rest:
// 0.9), 0.48 at 0.3, 0.63 at 0.4, 0.8 at 0.5, 1.2 at 0.8, 1.8 at 1.2.  Whole calls of 8 heads x 32k keys, us, without estimates and with them from
// this spread on:
//   24 layers, 512 rows, max, 0.36, 0.42, 0.5 and 0.58: 0.25 1317, 1530, 1342, 1342, -; 0.3 1314, 1228, 1273, 1356, 1341; 0.35 1325, 1117, 1144,
//     1193, 1346; 0.4 1328, -, 1069, 1122, 1197.  Window 13: 0.25 1331, 1594, 1352, 1348; 0.3 1326, 1306, 1354, 1357; no pooling: 0.25 1311, 1154, 1345, 1341
//   32 layers, 128 rows, max, likewise: 0.25 675, 678, 693, 699, -; 0.3 680, 609, 632, 694, 692; 0.35 671, 588, 583, 611, 690
//   24 layers, 512 rows, average, 0.62, 0.7 and 0.78: 0.4 1311, 1360, 1359, 1354; 0.45 1311, 1485, 1358, 1358; 0.5 1318, 1285, 1319, 1359; 0.6 1325,
//     1140, 1151, 1187
//   32 layers, 128 rows, average: 0.4 672, 702, 695, 692; 0.45 683, 716, 696, 697; 0.5 680, 649, 661, 696; 0.6 677, 591, 596, 604
// The spread is seen before the sample is multiplied, so that heads without a common direction cost little more than their references.
// (A count of 256 sampled keys near the cut told the strengths apart worse, and later.)
constexpr float kSiftSpread = 0.42f, kSiftSpreadAvg = 0.7f;
// The guess of tau: the estimate that kSiftRank times the groups that the kept keys are thought to fill reach, times what the mean
// ratio of weight to estimate is below the largest, times kSiftSlack (0.95 and 1: one head in a hundred fails the check).
constexpr float kSiftSlack = 0.9f, kSiftRank = 1.2f;
// Less by kSiftApart binades per unit of the ratios' relative deviation from kSiftApartFrom on, where the rows' weights lie apart, as
// they do with key channels of unequal scales.  32 layers x 8 heads x 32k keys, 128 rows, average and max pooling, and 24 layers, 512
// rows, max, us, without estimates, without this (and a failing head handing on its sequence) and with it: scales LogNormal(0, 0.6) 675,
// 941, 583; 675, 1042, 588; 1323, 2297, 1117; LogNormal(0, 0.95) 697, 1205, 738; 699, 1203, 791; 1470, 2481, 1567; LogNormal(0, 1.1) 856, 1354,
// 1008; 857, 1349, 1100; 1563, 2547, 2061 (of the heads 3 %, 25 % and 55 % are handed on: that the rows' weights lie apart so far is seen
// only behind the pass.  3 from 0.12 on: 594, 589, 1140; 779, 832, 1600; 8 from 0.15 on: 598, 597, 1137; 737, 775, 1628).
constexpr float kSiftApart = 5.f, kSiftApartFrom = 0.15f;
constexpr int kSiftMaxPoolW = 17;

// (two where they fit the LDS beside the queries)
__host__ __device__ constexpr int sift_zbufs(int Rs) { return Rs <= 384 ? 2 : 1; }

struct SiftLayer {
  const uint16_t* Q;
  const uint16_t* K;
  int32_t* idx;   // [BH][k_l] kept positions
  int32_t k_l;
  int32_t slot;   // as ResidentLayer
};

struct SiftArgs {
  SiftLayer layer[kResidentMaxLayers];
  const int32_t* seq_lens;
  float* raw;                 // [layer slot][B][Hkv][N] scores
  float* omega;               // [units][Rs] estimated weights of the rows: 1 / (G z)
  unsigned long long* zsum;   // [units][Rs] their sums, as the other kernel's words hold them (bit 63: large ones in further words; 62: beyond those)
  unsigned long long* zlarge; // [units][3][Rs] the further words
  int32_t* flags;             // [layer slot][B][Hkv] 0: scored, or kept whole; else bits of kSiftLeft: left to the lagging kernel
  float* window;              // [units][Rs] sums of the rows over the window keys
  int32_t* done;              // [units] jobs done
  int32_t* total;             // [units] keys listed
  float* bound;               // [units] what the kept number of them has to reach
  uint32_t* list;             // [units][sift_list(N)] positions of keys that can be kept, ascending
  unsigned long long *words, *words4;  // of the kernel that takes the rest, prepared by the way
  int32_t* err;
  uint32_t scored[(kResidentMaxLayers + 31) / 32];  // layers whose scores are asked for: left to that kernel
  int32_t L, B, Hq, Hkv, G, alpha, N, R, Rs, d;     // Rs: rows padded to 64
  int32_t grid, groups;       // workgroups of the pass over K; groups of 64 rows
  int32_t zbufs;              // tables of sums by wave, used in turn
  int32_t pool, pool_w;
  int32_t sample_tiles;       // of 32 keys, per wave (8 waves): 2 or 4
  int32_t sample_shift;       // log2 of the sample's runs of eight keys
  int32_t min_share;          // keys of a prefix per key to keep, at least
  int32_t min_items;          // of a launch that are worth it
  float min_spread;           // of the scores of some keys
  uint32_t alpha_magic, bh_magic, hkv_magic;  // as LagArgs
  int64_t q_sb, q_sh, q_st, kv_sb, kv_sh, kv_st;
  float kappa, inv_G;
};
hipError_t launch_score_sift(const SiftArgs& a, bool clear_err, hipStream_t s);
// How many heads of a (layer, sequence) have none of the bits set, and the k-th of them; how many have one, and the k-th of those.
template <bool SET>
__device__ __forceinline__ int sift_heads(const int32_t* flags, int Hkv, int32_t bits) {
  int n = 0;
  for (int g0 = 0; g0 < Hkv; g0 += 8) {
    int f[8];
#pragma unroll
    for (int g = 0; g < 8; ++g) f[g] = flags[g0 + g < Hkv ? g0 + g : 0];
#pragma unroll
    for (int g = 0; g < 8; ++g) n += g0 + g < Hkv && ((f[g] & bits) != 0) == SET ? 1 : 0;
  }
  return n;
}
template <bool SET>
__device__ __forceinline__ int sift_head(const int32_t* flags, int Hkv, int32_t bits, int k) {
  int g = 0;
  for (; g < Hkv; ++g)
    if (((flags[g] & bits) != 0) == SET && k-- == 0) break;
  return g;
}
constexpr int32_t kSiftObjects = 1, kSiftFailed = 2, kSiftTooFew = 4, kSiftLeft = 7;

// ---- scoring in two streaming launches for many query rows, over many layers (pkv_sweep.hip) ----
constexpr int kSweepGrid = 256;     // workgroups, one per compute unit

struct SweepArgs {
  ResidentLayer layer[kResidentMaxLayers];
  const int32_t* seq_lens;
  float* raw;                 // [U][N] un-pooled scores
  unsigned long long* stats;  // [U][nchunk][Rs] (reference, sum) of a row over a chunk (log2 domain)
  int32_t L, B, Hq, Hkv, G, alpha, N, R, Rs, d;  // Rs: rows padded to 64
  int32_t C, nchunk;          // keys per chunk (a multiple of 512), chunks per unit
  int32_t score_C, score_nchunk;  // the split of the launch that writes the scores (a multiple of 64 keys per wave)
  int32_t score_waves;        // 8 or 16 per workgroup
  int32_t uniform;            // 1: every unit has N keys and none is kept whole
  int32_t grid;
  int32_t lse_mode;           // 1: every layer carries lse; no statistics
  int64_t q_sb, q_sh, q_st, kv_sb, kv_sh, kv_st;
  float kappa, inv_kappa, inv_G;
};
hipError_t launch_score_sweep(const SweepArgs& a, hipStream_t s);

// ---- pooling + selection and gather over many layers ----
constexpr int kBatchMaxLayers = 32;  // per launch (kernel-argument tables: selection + gather together < 4 KB)

struct SelectLayer {
  float* pooled;       // [BH][N]: scores_out of the layer, else workspace
  int32_t* idx_out;    // [BH][k_cap]
  int32_t* count_out;  // [B]
  int32_t k_l, k_cap;
  int32_t write_pooled;  // the caller asked for scores_out
  int32_t pad;
};

struct SelectBatchArgs {
  SelectLayer layer[kBatchMaxLayers];
  const float* raw;    // [L][nrb][BH][N], first layer of this launch
  const int32_t* seq_lens;
  int32_t B, Hkv, N, alpha, pool, pool_w;
  int32_t nrb;         // partial score arrays to add per layer
  float inv_G;         // factor applied to the sum of the partials
  const int32_t* err;  // error word of the scoring kernel (non-zero: a wait was given up), or null
  const int32_t* flags;  // [layer][B][Hkv] of the sifting kernels: where they scored a head, its kept positions are there; or null
  int32_t listed;      // a launch before this one has listed the candidates of long prefixes
};

struct GatherLayer {
  const uint16_t* K;
  const uint16_t* V;
  uint16_t* K_out;
  uint16_t* V_out;
  const int32_t* idx;
  const int32_t* table;  // paged output: [B][max_pages] page numbers of this layer, else null
  int32_t* count_out;    // paged output: [B], set to -2 where a page number is out of range
  int64_t o_sb, o_sh, o_st;
  int32_t k_cap, pad;
};

struct GatherBatchArgs {
  GatherLayer layer[kBatchMaxLayers];
  int32_t L, B, Hkv, d, k_cap_max;
  int32_t N;  // rows per head in K and V: positions outside [0, N) are never dereferenced
  int32_t page_size, num_pages, max_pages;  // page_size 0: compact output through the o_* strides
  int64_t kv_sb, kv_sh, kv_st;
};

// 16 bytes (segment seg) of kept row j of (sequence b, KV head g): from the cache into the compact cache or the
// layer's page pool.  An index outside [0, N) is never dereferenced: the compact slot is cleared, a pool slot is
// left alone.  d / 8 neighbouring lanes move one row.
__device__ __forceinline__ void gather_row_segment(const GatherBatchArgs& a, const GatherLayer& ly, int b, int g, int j,
                                                   int seg) {
  const int src = ly.idx[((size_t)b * a.Hkv + g) * ly.k_cap + j];
  if (a.page_size > 0) {
    if ((uint32_t)src >= (uint32_t)a.N) return;  // unused slot: the pool keeps its content
    const int q = j / a.page_size, slot = j - q * a.page_size;
    const int pg = q < a.max_pages ? ly.table[(size_t)b * a.max_pages + q] : -1;
    if ((uint32_t)pg >= (uint32_t)a.num_pages) {  // never written through a bad page number: reported instead
      ly.count_out[b] = -2;
      return;
    }
    const size_t off = (size_t)b * a.kv_sb + (size_t)g * a.kv_sh + (size_t)src * a.kv_st + seg * 8;
    const size_t o = (((size_t)pg * a.Hkv + g) * a.page_size + slot) * a.d + seg * 8;
    *reinterpret_cast<uint4*>(ly.K_out + o) = *reinterpret_cast<const uint4*>(ly.K + off);
    *reinterpret_cast<uint4*>(ly.V_out + o) = *reinterpret_cast<const uint4*>(ly.V + off);
    return;
  }
  uint4 kv = make_uint4(0, 0, 0, 0), vv = kv;
  if ((uint32_t)src < (uint32_t)a.N) {  // -1 marks an unused slot; anything else out of range is not dereferenced either
    const size_t off = (size_t)b * a.kv_sb + (size_t)g * a.kv_sh + (size_t)src * a.kv_st + seg * 8;
    kv = *reinterpret_cast<const uint4*>(ly.K + off);
    vv = *reinterpret_cast<const uint4*>(ly.V + off);
  }
  const size_t o = (size_t)b * ly.o_sb + (size_t)g * ly.o_sh + (size_t)j * ly.o_st + seg * 8;
  *reinterpret_cast<uint4*>(ly.K_out + o) = kv;
  *reinterpret_cast<uint4*>(ly.V_out + o) = vv;
}

// ---- attention recall of the kept set, from the un-pooled scores a compress call left in its workspace ----
struct RecallLayer {
  const int32_t* idx;  // [BH][k_cap] kept positions of the layer
  float* recall;       // [BH]
  int32_t k_l, k_cap;
};

struct RecallArgs {
  RecallLayer layer[kBatchMaxLayers];
  const float* raw;    // [L][nrb][BH][N], first layer of this launch
  const int32_t* seq_lens;
  int32_t B, Hkv, N, alpha, nrb;
  float inv_G;         // factor applied to the sum of the partials
  const int32_t* flags;  // [layer][B][Hkv] of the sifting kernels, first layer of this launch: where they scored a head,
                         // the sum over all keys lies behind its scores; or null
};

// ---- decoding attention over a compacted (possibly paged) cache ----
constexpr int kDecodeMaxRows = 4096;  // kept rows per sequence
struct DecodeArgs {
  const uint16_t* q;     // [B][Hq][d]
  const uint16_t* K;     // compact [B][Hkv][k_cap][d] (strides c_*) or pool [num_pages][Hkv][page_size][d]
  const uint16_t* V;
  const int32_t* table;  // [B][max_pages], paged only
  const int32_t* count;  // [B]
  float* out;            // [B][Hq][d]
  float* lse;            // [B][Hq] or null
  float* part_o;         // [B][Hkv][S][8][d] un-normalised partial outputs (S > 1)
  float* part_mz;        // [B][Hkv][S][8][2] reference exponent and sum of the partial result
  int32_t B, Hq, Hkv, G, d, k_cap, page_size, num_pages, max_pages;
  int32_t page_shift;    // log2(page_size), or -1: division by page_magic (decode_page_division)
  uint32_t page_magic;
  int32_t S, chunk;      // key ranges per (sequence, head); keys per range (multiple of 32)
  int64_t c_sb, c_sh, c_st;
  float scale_log2;      // log2(e) / sqrt(d)
};
int decode_splits(int B, int Hkv, int k_cap);
int decode_splits_used(int B, int Hkv, int d, int k_cap);
int decode_waves(int64_t workgroups, int64_t rows_total, int d, int G, int chunk);
void decode_page_division(int page_size, int32_t* shift, uint32_t* magic);
hipError_t launch_decode_attention(const DecodeArgs& a, hipStream_t s);

// The same over the caches of several layers in one launch (per-layer pointers and cache sizes; shape shared).
struct DecodeLayer {
  const uint16_t* q;
  const uint16_t* K;
  const uint16_t* V;
  const int32_t* table;
  const int32_t* count;
  float* out;
  float* lse;
  int64_t c_sb, c_sh, c_st;
  int32_t k_cap, num_pages, max_pages;
  int32_t S, chunk;  // key ranges of this layer; keys per range
  int32_t wg0;       // first workgroup of this layer in the launch: layers follow one another, [b][g][range] inside
  int32_t part0;     // first partial-result record of this layer in the workspace ([b][g][range] inside)
  int32_t pad;
};
constexpr int kDecodeMaxLayers = 32;  // per launch (kernel-argument table)
struct DecodeBatchArgs {
  DecodeLayer layer[kDecodeMaxLayers];
  float* part_o;   // [records][8][d]
  float* part_mz;  // [records][8][2]
  int32_t L, B, Hq, Hkv, G, d, page_size;
  int32_t page_shift;
  uint32_t page_magic;
  float scale_log2;
};
int decode_layers_chunk(int64_t rows_total);
int decode_layers_chunk_used(int64_t units, int64_t rows_total);
int decode_layers_splits(int k_cap, int chunk_target, int* chunk);
hipError_t launch_decode_attention_layers(const DecodeBatchArgs& a, int total_wgs, int nw, bool any_split, hipStream_t s);

// Index of the current device for per-device launch state (dynamic LDS limits are set per device), or -1.
constexpr int kMaxDevices = 64;
inline int current_device_slot() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
  return dev;
}

hipError_t launch_score_resident(const ResidentArgs& a, hipStream_t s);
hipError_t launch_recall(const RecallArgs& a, int nlayers, hipStream_t s);
// fuse_gather: the selection workgroup of a unit also copies the unit's kept rows (compact output only)
hipError_t launch_pool_select_batch(SelectBatchArgs& a, const GatherBatchArgs& ga, bool fuse_gather, int nlayers,
                                    hipStream_t s);
hipError_t launch_gather_batch(const GatherBatchArgs& a, hipStream_t s);
hipError_t launch_probe_read(const void* buf, size_t bytes, uint32_t* sink, hipStream_t s);

// Each returns hipSuccess or the launch error.
hipError_t launch_score_stats(const ScoreArgs& a, hipStream_t s);
hipError_t launch_score_finalize(const ScoreArgs& a, hipStream_t s);
hipError_t launch_score_accum(const ScoreArgs& a, hipStream_t s);

}  // namespace pkv
