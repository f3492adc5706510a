// Attention mass for MANY spans (one per document of a re-ranking prompt) on many query rows of
// a few heads: a probe-only pass that computes no attention output.  The attention call itself
// then runs with probing switched off.
//
// Workgroup of the single-kernel form = (sequence, probed head, block of 16 selected rows), 16 waves.
//   pass 1  the waves share the keys [0, pos_max] (32-key groups round-robin), each lane keeps a
//           running (max, sum) for its row over the keys it sees; merged across lanes and waves
//           into the exact softmax maximum and normaliser of each row;
//   pass 2  the spans are dealt to the waves; a wave walks the keys of its span, recomputes the
//           scores, sums exp2(s - max) per row and writes sum / normaliser.
// Every (row, span) value is produced by one wave in a fixed order: no atomics, reproducible,
// spans may overlap or be empty.  Scores are bf16 x bf16 products accumulated in fp32 on the
// matrix cores (16x16x32: 16 keys x 16 rows per instruction), exponentials and sums fp32.
#include "../../include/hook_api.h"
#include "fp8_device.h"
#include "hook_device.h"

#include <cmath>

namespace hook {
namespace {

constexpr int kSmWaves = 16;
constexpr int kSmRows = 16;     // query rows per workgroup
constexpr int kSmGroup = 2;     // 16-key tiles per pipeline stage

struct SpanParams {
  int num_seqs, total_q, Hq, Hkv, G, max_blocks, num_blocks;
  float scale_log2;
  const float* k_scale;   // 8-bit cache: one fp32 scale per kv head, folded into the softmax scale
  const void* q;
  const void* k_cache;
  const int* block_table;
  const int* seq_lens;
  const int* cu_q_lens;
  int P;
  const int* probe_heads;
  int NQ;
  const int* query_sel;
  int S;
  const int* key_spans;
  float* mass;
  float2* stats;    // split path: (max, sum) of every (sequence, probed head, row slot, key split)
  int nsplit;       // key splits of pass 1
  int sgroups;      // span groups of pass 2
  int span_turn;    // spans of a workgroup of pass 2 at a time (8, 4, 2 or 1)
  int nq_pad;       // NQ rounded up to whole 16-row blocks
};

template <int D>
struct Frag {
  static constexpr int KSTEPS = D / 32;
  uint4 k[KSTEPS];
};

// K rows of 16 keys as the A operand: lane (key slot l % 16, quarter l / 16) takes the 16-byte
// chunks 4 s + quarter of its key's row.  `key` is this lane's absolute key (already clamped
// into the sequence), looked up through the block table.
// With an 8-bit cache (KV8) the same eight dimensions are eight bytes, widened to bf16 after the load.
template <int D, bool KV8>
__device__ __forceinline__ void load_keys(const SpanParams& p, int blk, int g, int key, int quarter, Frag<D>& f) {
  blk = ((unsigned)blk < (unsigned)p.num_blocks) ? blk : 0;
  const size_t row_index = ((size_t)blk * p.Hkv + g) * kBlock + (key & 15);
  if constexpr (KV8) {
    const uint2* row = static_cast<const uint2*>(p.k_cache) + row_index * (D / 8);
#pragma unroll
    for (int s = 0; s < Frag<D>::KSTEPS; ++s) f.k[s] = e4m3x8_to_bf16x8(row[4 * s + quarter]);
  } else {
    const uint4* row = static_cast<const uint4*>(p.k_cache) + row_index * (D / 8);
#pragma unroll
    for (int s = 0; s < Frag<D>::KSTEPS; ++s) f.k[s] = row[4 * s + quarter];
  }
}

template <int D>
__device__ __forceinline__ f32x4 scores(const Frag<D>& f, const bf16x8 (&qf)[D / 32]);

// (k_span_mass.)  A stream of key groups (kSmGroup tiles of 16 keys; group n starts at key first + n * step) run
// as a three-stage pipeline per wave: block ids two groups ahead, K rows one group ahead,
// arithmetic on the current group - so neither load latency sits on the critical path.
// `use(tile_first_key, scores[NB])` is called for every tile whose first key is below `end`; NB blocks
// of 16 query rows share every K fetch.
template <int D, int NB, bool KV8, typename F>
__device__ __forceinline__ void stream_keys(const SpanParams& p, const int* bt, int g, int j, int quarter,
                                            const bf16x8 (&qf)[NB][D / 32], int first, int step, int end, int pos_max,
                                            F&& use) {
  auto lane_key = [&](int base, int u) { return min(base + 16 * u + j, pos_max); };
  auto ids = [&](int base, int (&id)[kSmGroup]) {
#pragma unroll
    for (int u = 0; u < kSmGroup; ++u) id[u] = bt[lane_key(base, u) >> 4];
  };
  auto rows = [&](int base, const int (&id)[kSmGroup], Frag<D> (&f)[kSmGroup]) {
#pragma unroll
    for (int u = 0; u < kSmGroup; ++u) load_keys<D, KV8>(p, id[u], g, lane_key(base, u), quarter, f[u]);
  };
  auto work = [&](int base, const Frag<D> (&f)[kSmGroup]) {
#pragma unroll
    for (int u = 0; u < kSmGroup; ++u)
      if (base + 16 * u < end) {   // uniform
        f32x4 sc[NB];              // one K fetch serves the NB blocks of 16 rows
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) sc[nb] = scores<D>(f[u], qf[nb]);
        use(base + 16 * u, sc);
      }
  };
  if (first >= end) return;
  // Every load below is issued unconditionally - keys are clamped into the sequence, so reading a
  // group past `end` is harmless - because the compiler can only keep loads in flight across a
  // wait when their number does not depend on the path taken.
  int idA[kSmGroup], idB[kSmGroup];
  Frag<D> fA[kSmGroup], fB[kSmGroup];
  ids(first, idA);
  rows(first, idA, fA);
  ids(first + step, idB);
  for (int base = first; base < end; base += 2 * step) {
    // fA holds (or awaits) the rows of `base`, idB the ids of base + step.  Loads return in issue
    // order, so ids are requested BEFORE the rows of the group in front of them: waiting for ids
    // then never drains rows issued after them.
    int idC[kSmGroup];
    ids(base + 2 * step, idC);
    rows(base + step, idB, fB);
    work(base, fA);
    ids(base + 3 * step, idB);
    rows(base + 2 * step, idC, fA);
    work(base + step, fB);
  }
}

template <int D>
__device__ __forceinline__ f32x4 scores(const Frag<D>& f, const bf16x8 (&qf)[D / 32]) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < D / 32; ++s) {
    bf16x8 a;
    __builtin_memcpy(&a, &f.k[s], 16);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[s], acc, 0, 0, 0);
  }
  return acc;
}

// The tiles [0, ntiles) behind tile `first` of a sequence whose last block is last_blk, kTileRing of them requested ahead and the
// scores of the next one computed beside `use` of the one before.  Block ids come 64 at a time, one per lane, so a tile costs
// one scalar address instead of one per lane.  Past the end all lanes fetch the same 16 bytes, so that the compiler knows how many
// loads are in flight.  4 prompts of 40-100 documents on 8 heads 38.1 us with stream_keys, 36.4 so (4 tiles ahead 37.1), on 32 heads 119.8 and
// 108.5; 16 prompts 117.5 and 110.
constexpr int kTileRing = 2;
template <int D, int NB, bool KV8, typename F>
__device__ __forceinline__ void stream_tiles(const SpanParams& p, const int* bt, int g, int lane, const bf16x8 (&qf)[NB][D / 32],
                                             int first, int ntiles, int last_blk, F&& use) {
  constexpr int KS = D / 32, ESZ = KV8 ? 1 : 2;
  struct Raw { uint4 k[KV8 ? (KS + 1) / 2 : KS]; };      // 8-bit: two k-steps to a register quad, widened before use
  if (ntiles <= 0) return;
  const char* const base = static_cast<const char*>(p.k_cache) + (size_t)g * kBlock * D * ESZ;
  const unsigned blk_bytes = (unsigned)p.Hkv * kBlock * D * ESZ, lane_off = (unsigned)(lane & 15) * D * ESZ + 8 * ESZ * (lane >> 4);
  auto load_ids = [&](int t) {
    const int blk = bt[min(first + t + lane, last_blk)];
    return (unsigned)blk < (unsigned)p.num_blocks ? blk : 0;
  };
  int ids = load_ids(0), ids_next = 0;
  if (ntiles > 64) ids_next = load_ids(64);
  auto request = [&](int t, Raw& f) {
    const global_bytes src = (global_bytes)(base + (unsigned long long)(unsigned)__builtin_amdgcn_readlane(ids, t & 63) * blk_bytes);
    unsigned off = t < ntiles ? lane_off : 0;
    asm("" : "+v"(off));
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if constexpr (KV8) {
        const u32x2 v = *(const __attribute__((address_space(1))) u32x2*)(src + off + 32 * s);
        if (s & 1) { f.k[s / 2].z = v.x; f.k[s / 2].w = v.y; } else { f.k[s / 2].x = v.x; f.k[s / 2].y = v.y; }
      } else {
        f.k[s] = load_global16(src + off + 64 * s);
      }
    }
  };
  auto tile_scores = [&](const Raw& d, f32x4 (&sc)[NB]) {
    Frag<D> f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if constexpr (KV8) f.k[s] = e4m3x8_to_bf16x8((s & 1) ? make_uint2(d.k[s / 2].z, d.k[s / 2].w) : make_uint2(d.k[s / 2].x, d.k[s / 2].y));
      else f.k[s] = d.k[s];
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) sc[nb] = scores<D>(f, qf[nb]);
  };
  Raw ring[kTileRing];
#pragma unroll
  for (int u = 0; u < kTileRing; ++u) request(u, ring[u]);
  f32x4 sc[NB], next[NB];
  tile_scores(ring[0], sc);
  for (int t = 0; t < ntiles; t += kTileRing) {
#pragma unroll
    for (int u = 0; u < kTileRing; ++u) {
      if (u == 0 && ((t + kTileRing) & 63) == 0) {
        ids = ids_next;
        ids_next = load_ids(t + kTileRing + 64);
      }
      request(t + u + kTileRing, ring[u]);
      __builtin_amdgcn_sched_barrier(0);
      tile_scores(ring[(u + 1) % kTileRing], next);      // (beside the exponentials of the tile before it)
      if (u == 0 || t + u < ntiles) use(16 * (first + t + u), sc);      // uniform
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) sc[nb] = next[nb];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

template <int D, bool KV8>
__global__ __launch_bounds__(kSmWaves * 64) void k_span_mass(const SpanParams p) {
  __shared__ float sh_m[kSmWaves][kSmRows];
  __shared__ float sh_l[kSmWaves][kSmRows];

  const int i = blockIdx.z, ps = blockIdx.y, rb = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: keeps the key loops scalar
  const int j = lane & 15, quarter = lane >> 4;

  const int Lraw = p.seq_lens[i];
  const int row0 = p.cu_q_lens[i];
  const int n = p.cu_q_lens[i + 1] - row0;
  const int L = min(Lraw, p.max_blocks * kBlock);
  if (Lraw < 0 || n <= 0 || n > L || row0 < 0 || row0 + n > p.total_q) return;   // uniform
  const int h = p.probe_heads[ps];
  if ((unsigned)h >= (unsigned)p.Hq) return;
  const int g = h / p.G;
  const int qb = p.query_sel[2 * i];
  const int qe = min(min(p.query_sel[2 * i + 1], n), qb + p.NQ);
  const int slot0 = kSmRows * rb;                 // first mass slot of this block
  const int t_lo = max(qb + slot0, 0), t_hi = min(qb + slot0 + kSmRows, qe);   // valid rows [t_lo, t_hi)
  if (t_hi <= t_lo) return;
  const int t_mine = qb + slot0 + j;
  const bool row_ok = t_mine >= t_lo && t_mine < t_hi;
  const int t = min(max(t_mine, t_lo), t_hi - 1);  // lanes without a row shadow a valid one
  const int pos = L - n + t;
  const int pos_max = L - n + t_hi - 1;

  const int* bt = p.block_table + (size_t)i * p.max_blocks;
  bf16x8 qf[1][D / 32];
  {
    const bf16x8* qp = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(p.q) +
                                                        ((size_t)(row0 + t) * p.Hq + h) * D);
#pragma unroll
    for (int s = 0; s < D / 32; ++s) qf[0][s] = qp[4 * s + quarter];
  }
  const float c = KV8 ? p.scale_log2 * p.k_scale[g] : p.scale_log2;

  // ---- pass 1: row maximum and normaliser
  float m = -INFINITY, l = 0.0f;
  const int ntile = pos_max / 16 + 1;
  stream_keys<D, 1, KV8>(p, bt, g, j, quarter, qf, 16 * kSmGroup * wave, 16 * kSmGroup * kSmWaves, 16 * ntile, pos_max,
                    [&](int key0, const f32x4 (&sc)[1]) {
    const f32x4 s4 = sc[0];
    float sv[4];
    float mt = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = key0 + 4 * quarter + r;
      sv[r] = key <= pos ? s4[r] * c : -INFINITY;
      mt = fmaxf(mt, sv[r]);
    }
    // branch-free update (a divergent branch between the loads would make the compiler wait for
    // every load in flight): with everything masked so far the reference is 0 and all terms vanish
    const float mn = fmaxf(m, mt);
    const float ref = (mn == -INFINITY) ? 0.0f : mn;
    l *= fast_exp2(m - ref);                        // m = -inf: l is 0 and stays 0
#pragma unroll
    for (int r = 0; r < 4; ++r) l += fast_exp2(sv[r] - ref);
    m = mn;
  });
  // merge the four quarters of a row, then the waves
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float mo = __shfl_xor(m, off), lo = __shfl_xor(l, off);
    const float mn = fmaxf(m, mo);
    if (mn != -INFINITY) l = l * fast_exp2(m - mn) + lo * fast_exp2(mo - mn);
    m = mn;
  }
  if (quarter == 0) { sh_m[wave][j] = m; sh_l[wave][j] = l; }
  __syncthreads();
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kSmWaves; ++w) M = fmaxf(M, sh_m[w][j]);
  float Lsum = 0.0f;
#pragma unroll
  for (int w = 0; w < kSmWaves; ++w) {
    const float mw = sh_m[w][j];
    if (mw != -INFINITY) Lsum += sh_l[w][j] * fast_exp2(mw - M);
  }
  const float inv = 1.0f / Lsum;   // every valid row sees at least key 0, so Lsum >= 1 term

  // ---- pass 2: spans
  float* mrow = p.mass + (((size_t)i * p.P + ps) * p.NQ + (slot0 + j)) * p.S;
  for (int r = wave; r < p.S; r += kSmWaves) {
    const int a = max(p.key_spans[((size_t)i * p.S + r) * 2], 0);
    const int e = min(p.key_spans[((size_t)i * p.S + r) * 2 + 1], pos_max + 1);
    if (e <= a) continue;                          // uniform; mass was zero-filled
    float acc = 0.0f;
    stream_keys<D, 1, KV8>(p, bt, g, j, quarter, qf, a, 16 * kSmGroup, e, pos_max, [&](int key0, const f32x4 (&sc)[1]) {
      const f32x4 s4 = sc[0];
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int key = key0 + 4 * quarter + rr;
        acc += (key < e && key <= pos) ? fast_exp2(s4[rr] * c - M) : 0.0f;
      }
    });
    acc += __shfl_xor(acc, 16);
    acc += __shfl_xor(acc, 32);
    if (quarter == 0 && row_ok) mrow[r] = acc * inv;
  }
}

// ---- the same as two kernels, for callers that provide scratch memory: a single workgroup per row block has to pull a
// long sequence's keys through one CU (about 100 us per 10 k keys and pass); here the keys are split over the chip, and
// most spans are summed in the pass that finds the statistics, against the reference of their split.

// Sum and maximum over the four lanes of a row (l, l ^ 16, l ^ 32, l ^ 48), in all of them, without a trip through LDS.
__device__ __forceinline__ float row_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float row_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// What both kernels need to know about their row block; false if there is nothing to do.
struct RowBlock {
  int g, h, row0, pos, pos_max, slot0;
  bool row_ok;
};

// What it rests on, requested in one go.
struct RowSource { int L, first, end, head, sel_b, sel_e; };

__device__ __forceinline__ RowSource row_source(const SpanParams& p, int i, int ps) {
  const RowSource q = {cload(p.seq_lens, i), cload(p.cu_q_lens, i), cload(p.cu_q_lens, i + 1), cload(p.probe_heads, ps),
                       cload(p.query_sel, 2 * i), cload(p.query_sel, 2 * i + 1)};
  asm volatile("" :: "s"(q.L), "s"(q.first), "s"(q.end), "s"(q.head), "s"(q.sel_b), "s"(q.sel_e));      // (not one behind the other's check)
  return q;
}

__device__ __forceinline__ bool row_block(const SpanParams& p, const RowSource& q, int rb, int j, RowBlock& r) {
  r.row0 = q.first;
  const int n = q.end - r.row0;
  const int L = min(q.L, p.max_blocks * kBlock);
  if (q.L < 0 || n <= 0 || n > L || r.row0 < 0 || r.row0 + n > p.total_q) return false;
  r.h = q.head;
  if ((unsigned)r.h >= (unsigned)p.Hq) return false;
  r.g = r.h / p.G;
  const int qb = q.sel_b;
  const int qe = min(min(q.sel_e, n), qb + p.NQ);
  r.slot0 = kSmRows * rb;
  const int t_lo = max(qb + r.slot0, 0), t_hi = min(qb + r.slot0 + kSmRows, qe);
  if (t_hi <= t_lo) return false;
  const int t_mine = qb + r.slot0 + j;
  r.row_ok = t_mine >= t_lo && t_mine < t_hi;
  const int t = min(max(t_mine, t_lo), t_hi - 1);
  r.pos = L - n + t;
  r.pos_max = L - n + t_hi - 1;
  r.row0 += t;      // global q row of this lane
  return true;
}

template <int D>
__device__ __forceinline__ void load_q(const SpanParams& p, const RowBlock& r, int quarter, bf16x8 (&qf)[D / 32]) {
  const bf16x8* qp = reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(p.q) + ((size_t)r.row0 * p.Hq + r.h) * D);
#pragma unroll
  for (int s = 0; s < D / 32; ++s) qf[s] = qp[4 * s + quarter];
}

// Both kernels are bound by latency, not by the bytes (4 prompts of 6-14 k tokens, 8 heads: 84 MB of keys): a wave spends
// most of its time in the chain lengths -> rows -> block ids -> keys.  So the work is cut fine and the workgroups are small,
// which lets the chip start them all at once and even out sequences of unequal length: pass 1 takes 1024 keys with 4
// waves (2048 keys: 4 waves 38 us, 16 waves 40; 1024 keys: 16 waves 40 us, 8 waves 29, 4 waves 27).
constexpr int kStatWaves = 4;     // waves per workgroup of pass 1
constexpr int kSumWaves = 8;      // waves per workgroup of the second kernel, and spans at a time
constexpr int kSumWgs = 144, kSumWgsLong = 256;      // workgroups that it has at least, or else fewer spans to each; where spans can be long
constexpr int kSplitBlocks = 2;   // blocks of 16 rows per workgroup: they share every K fetch
constexpr int kSplitRows = kSplitBlocks * kSmRows;
constexpr int kSplitKeys = 1024;  // keys of one workgroup of pass 1 (until kMaxSplits is reached)
constexpr int kMaxSplits = 16;    // key splits of pass 1
// A span is summed by the workgroup whose split it begins in, which reads on behind its split to the end of its last span.
// The spans of a split have to be disjoint and in order for that, and at most kListSpans; where they are not, the split's
// sum of exponentials carries a minus sign, and every span that begins in it gets its own walk over its keys in the
// second kernel.  So does a span that ends behind its split in a sequence with a span of more than kOverhang keys: one such walk takes as
// long as many, and reading on would come on top.
// The list holds as many spans as leave four workgroups to a compute unit their LDS: 4 keys each in 1024 keys, 16 each in the
// 4096 keys that a split of a 64 k context has.  (64 spans: 654 documents of 5-20 keys in each of 4 prompts of 8200 tokens 106.8
// us, 48.0 so; 1024 of 30-50 in 65536 76.7 and 57.3; all walked, without the list in the first kernel, 105.4 and 72.7.)
constexpr int kListSpans = 256;
constexpr int kOverhang = 512;

// The kSplitBlocks row blocks of workgroup column `bx`.  A block without rows shadows the other one
// (same loads and arithmetic, nothing written); false if no block has rows.
__device__ __forceinline__ bool row_blocks(const SpanParams& p, int i, int ps, int bx, int j,
                                           RowBlock (&r)[kSplitBlocks], bool (&has)[kSplitBlocks], int& pos_max) {
  static_assert(kSplitBlocks == 2, "each block has one other block to shadow");
  const RowSource q = row_source(p, i, ps);
#pragma unroll
  for (int nb = 0; nb < kSplitBlocks; ++nb) has[nb] = row_block(p, q, kSplitBlocks * bx + nb, j, r[nb]);
  if (!has[0] && !has[1]) return false;
#pragma unroll
  for (int nb = 0; nb < kSplitBlocks; ++nb) {
    if (!has[nb]) {   // (a computed index here would move the whole array into LDS)
      r[nb] = r[1 - nb];
      r[nb].slot0 = kSmRows * (kSplitBlocks * bx + nb);
      r[nb].row_ok = false;
    }
  }
  pos_max = max(r[0].pos_max, r[1].pos_max);
  return true;
}

// 16-key tiles per split of a row block whose last row sits at pos_max
__device__ __forceinline__ int split_tiles(int pos_max, int nsplit) { return (pos_max / 16 + nsplit) / nsplit; }

// Pass 1, a workgroup per (sequence, probed head, 32 rows, split): the split's statistics - a reference near the
// maximum and the sum of exponentials against it, per row - and, into `mass`, the sums of the spans that begin in it against
// the same reference.  The waves take runs of tiles one behind the other, so a wave meets the spans in order and
// keeps the sum of the one it is in, in registers; a finished span's sum goes to LDS, where the waves are merged.  Two waves
// have at most one span in common, so slot k + w is written by no other wave than w.
// 4 prompts of 7-16 k tokens, 8 heads, 32 rows, documents of 64-256 keys: 25 us and 4.8 for the second kernel (24 and 30 when the
// second one read all documents again); 7 documents of 20-40 keys 10 + 3.8.
template <int D, bool KV8>
__global__ __launch_bounds__(kStatWaves * 64) void k_span_stats(const SpanParams p) {
  __shared__ float sh_m[kStatWaves][kSplitRows];
  __shared__ float sh_l[kStatWaves][kSplitRows];
  __shared__ float sh_part[kListSpans + kStatWaves - 1][kSplitRows];     // wave w's sum of span k in slot k + w
  __shared__ int sh_a[kListSpans], sh_e[kListSpans], sh_s[kListSpans];   // begin, end and number of the split's spans
  const int i = blockIdx.z / p.nsplit, sp = blockIdx.z % p.nsplit, ps = blockIdx.y;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15, quarter = lane >> 4;
  const int2* const spans = reinterpret_cast<const int2*>(p.key_spans) + (size_t)i * p.S;
  constexpr int kSpanLoads = 8;                    // the first 512 spans are requested with the lengths
  int2 coming[kSpanLoads];
#pragma unroll
  for (int u = 0; u < kSpanLoads; ++u) coming[u] = spans[min(64 * u + lane, p.S - 1)];
  RowBlock r[kSplitBlocks];
  bool has[kSplitBlocks];
  int pos_max;
  if (!row_blocks(p, i, ps, blockIdx.x, j, r, has, pos_max)) return;   // uniform
  const int* bt = p.block_table + (size_t)i * p.max_blocks;
  bf16x8 qf[kSplitBlocks][D / 32];
#pragma unroll
  for (int nb = 0; nb < kSplitBlocks; ++nb) load_q<D>(p, r[nb], quarter, qf[nb]);
  const float c = KV8 ? p.scale_log2 * p.k_scale[r[0].g] : p.scale_log2;
  const int ntile = pos_max / 16 + 1, per = split_tiles(pos_max, p.nsplit);
  const int lo = 16 * per * sp, hi = min(16 * per * (sp + 1), 16 * ntile);

  // The spans that begin in this split: every wave counts them, the first one writes the list.
  int count = 0;
  bool any_long = false;
  for (int s0 = 0; s0 < p.S && count <= kListSpans; s0 += 64 * kSpanLoads) {
#pragma unroll
    for (int u = 0; u < kSpanLoads; ++u) {
      if (s0 + 64 * u >= p.S) break;
      const int s = s0 + 64 * u + lane;
      const int a = max(coming[u].x, 0), e = min(coming[u].y, pos_max + 1);
      const unsigned long long hit = __builtin_amdgcn_ballot_w64(s < p.S && e > a && a >= lo && a < hi);
      any_long = any_long || __builtin_amdgcn_ballot_w64(s < p.S && e - a > kOverhang) != 0;
      const int at = count + __builtin_amdgcn_mbcnt_hi((unsigned)(hit >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hit, 0));
      if (wave == 0 && ((hit >> lane) & 1) && at < kListSpans) {
        sh_a[at] = a;
        sh_e[at] = e;
        sh_s[at] = s;
      }
      count += __builtin_popcountll(hit);
    }
    if (s0 + 64 * kSpanLoads < p.S) {
#pragma unroll
      for (int u = 0; u < kSpanLoads; ++u) coming[u] = spans[min(s0 + 64 * (kSpanLoads + u) + lane, p.S - 1)];
    }
  }
  __syncthreads();
  // lane i holds span 64 * window + i; most lists fit one window
  int window = 0, span_a = sh_a[lane], span_e = sh_e[lane];
  bool listed = count <= kListSpans &&
                __builtin_amdgcn_ballot_w64(lane > 0 && lane < count && span_a < sh_e[max(lane - 1, 0)]) == 0;
  for (int k0 = 64; k0 < count && listed; k0 += 64)
    listed = __builtin_amdgcn_ballot_w64(k0 + lane < count && sh_a[k0 + lane] < sh_e[k0 + lane - 1]) == 0;
  int summed = listed ? count : 0, stop = hi;      // stop: end of the keys to read
  if (summed > 0) {
    const int last_e = __builtin_amdgcn_readfirstlane(sh_e[summed - 1]);
    if (any_long && last_e > hi) --summed;
    else stop = max(hi, last_e);
  }

  // this wave's run of tiles, and its first span
  const int run = ((stop - lo + 15) / 16 + kStatWaves - 1) / kStatWaves;
  const int w_lo = lo + 16 * run * wave, w_hi = min(w_lo + 16 * run, stop);
  int k = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < summed && span_e <= w_lo));
  for (int k0 = 64; k0 < summed; k0 += 64)
    k += __builtin_popcountll(__builtin_amdgcn_ballot_w64(k0 + lane < summed && sh_e[k0 + lane] <= w_lo));
  const int k_first = k;
  int sa, se;
  auto find_span = [&]() {                         // (what it finds behind the last span is not used)
    if (k >> 6 != window) {
      window = k >> 6;
      span_a = sh_a[min(64 * window + lane, kListSpans - 1)];
      span_e = sh_e[min(64 * window + lane, kListSpans - 1)];
    }
    sa = __builtin_amdgcn_readlane(span_a, k & 63);
    se = __builtin_amdgcn_readlane(span_e, k & 63);
  };
  find_span();

  float m[kSplitBlocks], l[kSplitBlocks], acc[kSplitBlocks];      // m: one reference for the four lanes of a row
#pragma unroll
  for (int nb = 0; nb < kSplitBlocks; ++nb) { m[nb] = -INFINITY; l[nb] = 0.0f; acc[nb] = 0.0f; }
  auto flush = [&]() {
#pragma unroll
    for (int nb = 0; nb < kSplitBlocks; ++nb) {
      const float v = row_sum(acc[nb]);
      if (quarter == 0) sh_part[k + wave][kSmRows * nb + j] = v;
      acc[nb] = 0.0f;
    }
  };
  stream_tiles<D, kSplitBlocks, KV8>(p, bt, r[0].g, lane, qf, w_lo / 16, (w_hi - w_lo + 15) / 16, pos_max / 16,
                                     [&](int key0, const f32x4 (&sc)[kSplitBlocks]) {
    float ex[kSplitBlocks][4], sum[kSplitBlocks];
#pragma unroll
    for (int nb = 0; nb < kSplitBlocks; ++nb) {
      float mt = -INFINITY;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        ex[nb][q] = key0 + 4 * quarter + q <= r[nb].pos ? sc[nb][q] * c : -INFINITY;
        mt = fmaxf(mt, ex[nb][q]);
      }
      // the reference is raised by what exceeds it by kLazyTau, with the sums that refer to it
      if (__builtin_amdgcn_ballot_w64(mt > m[nb] + kLazyTau) != 0) {
        mt = row_max(mt);
        const float mn = mt > m[nb] + kLazyTau ? mt : m[nb];
        const float alpha = mn > m[nb] ? fast_exp2(m[nb] - mn) : 1.0f;
        l[nb] *= alpha;
        acc[nb] *= alpha;
        if (quarter == 0)
          for (int kk = k_first; kk < k; ++kk) sh_part[kk + wave][kSmRows * nb + j] *= alpha;
        m[nb] = mn;
      }
      const float ref = m[nb] == -INFINITY ? 0.0f : m[nb];
      sum[nb] = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        ex[nb][q] = fast_exp2(ex[nb][q] - ref);
        sum[nb] += ex[nb][q];
      }
      if (key0 < hi) l[nb] += sum[nb];
    }
    while (k < summed && sa < key0 + 16) {         // (se > key0)
      if (sa <= key0 && se >= key0 + 16) {
#pragma unroll
        for (int nb = 0; nb < kSplitBlocks; ++nb) acc[nb] += sum[nb];
      } else {
#pragma unroll
        for (int nb = 0; nb < kSplitBlocks; ++nb)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int key = key0 + 4 * quarter + q;
            acc[nb] += key >= sa && key < se ? ex[nb][q] : 0.0f;
          }
      }
      if (se > key0 + 16) break;
      flush();
      ++k;
      find_span();
    }
  });
  if (k < summed && sa < w_hi) flush();            // the span that the next wave goes on with
#pragma unroll
  for (int nb = 0; nb < kSplitBlocks; ++nb) {
    l[nb] = row_sum(l[nb]);
    if (quarter == 0) { sh_m[wave][kSmRows * nb + j] = m[nb]; sh_l[wave][kSmRows * nb + j] = l[nb]; }
  }
  __syncthreads();
  // thread: row, and every eighth span
  constexpr int kSpanStep = kStatWaves * 64 / kSplitRows;
  const int row = threadIdx.x % kSplitRows, slot = kSplitRows * blockIdx.x + row;
  float M = -INFINITY, wgt[kStatWaves], Ls = 0.0f;
#pragma unroll
  for (int w = 0; w < kStatWaves; ++w) M = fmaxf(M, sh_m[w][row]);
#pragma unroll
  for (int w = 0; w < kStatWaves; ++w) {
    wgt[w] = sh_m[w][row] == -INFINITY ? 0.0f : fast_exp2(sh_m[w][row] - M);
    Ls += sh_l[w][row] * wgt[w];
  }
  if (threadIdx.x < kSplitRows && slot < p.nq_pad)
    p.stats[(((size_t)i * p.P + ps) * p.nq_pad + slot) * p.nsplit + sp] = make_float2(M, listed ? Ls : -Ls);
  if (slot >= p.NQ) return;
  float* const mass = p.mass + (((size_t)i * p.P + ps) * p.NQ + slot) * p.S;
  for (int kk = threadIdx.x / kSplitRows; kk < summed; kk += kSpanStep) {
    const int a = sh_a[kk], e = sh_e[kk];
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kStatWaves; ++w)           // the waves whose runs the span meets
      v += a < lo + 16 * run * (w + 1) && e > lo + 16 * run * w ? sh_part[kk + w][row] * wgt[w] : 0.0f;
    mass[sh_s[kk]] = v;
  }
}

// Maximum and sum over the 16 lanes of a DPP row, in all of them.
template <int N>
__device__ __forceinline__ float rotate16(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float max16(float v) {
  v = fmaxf(v, rotate16<8>(v));
  v = fmaxf(v, rotate16<4>(v));
  v = fmaxf(v, rotate16<2>(v));
  return fmaxf(v, rotate16<1>(v));
}
__device__ __forceinline__ float sum16(float v) {
  v += rotate16<8>(v);
  v += rotate16<4>(v);
  v += rotate16<2>(v);
  return v + rotate16<1>(v);
}

// The second kernel: from the splits' references to the row's, divided by its normaliser; zeros where there is no row or
// no key; and the walk over the keys of spans that the first kernel left out.  A workgroup takes p.span_turn spans of 32 rows: a
// thread per row and split finds what the split's sums are multiplied by, a thread per row and span multiplies, so that
// eight neighbouring lanes read and write 32 bytes of a row of `mass` (a wave to a span, four bytes of every row at a time, took 8.0 us for
// 4 x 40-100 documents on 8 heads and 32 rows; this takes 4.8).  The waves share out the walks: 16 spans of 600-1500 keys 47.7 us with
// the first kernel and a wave to a walk, 33.4 so.
template <int D, bool KV8>
__global__ __launch_bounds__(kSumWaves * 64, 4) void k_span_sums(const SpanParams p) {
  static_assert(kSumWaves * 64 == kSplitRows * kMaxSplits && kSmRows == 16, "");
  __shared__ float sh_f[kSplitRows][kMaxSplits + 1];     // factor of a row's sums over the spans that begin in a split
  __shared__ float sh_M[kSplitRows], sh_inv[kSplitRows];
  __shared__ float sh_part[kSumWaves][kSplitRows];
  __shared__ unsigned sh_bits;                           // splits without a list; kLong: some span is long
  constexpr unsigned kLong = 1u << kMaxSplits;
  const int i = blockIdx.z / p.sgroups, sg = blockIdx.z % p.sgroups, ps = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, quarter = lane >> 4;
  float* const mass = p.mass + ((size_t)i * p.P + ps) * p.NQ * p.S;
  const int2* const spans = reinterpret_cast<const int2*>(p.key_spans) + (size_t)i * p.S;
  const int slot0 = kSplitRows * blockIdx.x, turn = p.span_turn, turn_log2 = 31 - __builtin_clz(turn);
  const int row = tid >> turn_log2, slot = slot0 + row, k = tid & (turn - 1);      // this thread's row, and its span of a turn
  const bool mine = row < kSplitRows && slot < p.NQ;
  if (tid == 0) sh_bits = 0;
  RowBlock r[kSplitBlocks];
  bool has[kSplitBlocks];
  int pos_max;
  if (!row_blocks(p, i, ps, blockIdx.x, j, r, has, pos_max)) {   // uniform
    for (int s = sg * turn + k; s < p.S; s += p.sgroups * turn)
      if (mine) mass[(size_t)slot * p.S + s] = 0.0f;
    return;
  }
  const int per = split_tiles(pos_max, p.nsplit);
  int s0 = sg * turn;
  if (s0 >= p.S) return;
  const unsigned rows_ok = ((unsigned)__builtin_amdgcn_ballot_w64(r[0].row_ok) & 0xffffu) |
                           ((unsigned)__builtin_amdgcn_ballot_w64(r[1].row_ok) << 16);
  const bool ok = mine && ((rows_ok >> (row & (kSplitRows - 1))) & 1);
  int2 span = spans[min(s0 + k, p.S - 1)];
  float out = ok && s0 + k < p.S ? mass[(size_t)slot * p.S + s0 + k] : 0.0f;
  {
    const int sp = tid % kMaxSplits, rr = tid / kMaxSplits;
    // (a block without rows reads the other one's)
    const int from = slot0 + (has[0] && has[1] ? rr : has[0] ? rr % kSmRows : kSmRows + rr % kSmRows);
    const float2 v = sp < p.nsplit ? p.stats[(((size_t)i * p.P + ps) * p.nq_pad + from) * p.nsplit + sp] : make_float2(-INFINITY, 0.0f);
    bool any_long = false;
    for (int s = tid; s < p.S; s += kSumWaves * 64) {
      const int2 x = spans[s];
      any_long = any_long || min(x.y, pos_max + 1) - max(x.x, 0) > kOverhang;
    }
    const float M = max16(v.x);
    const float inv = 1.0f / sum16(fabsf(v.y) * fast_exp2(v.x - M));      // an empty split adds 0
    sh_f[rr][sp] = v.x == -INFINITY ? 0.0f : fast_exp2(v.x - M) * inv;    // -inf: the row sees no key of this split
    if (sp == 0) { sh_M[rr] = M; sh_inv[rr] = inv; }
    unsigned long long hit = __builtin_amdgcn_ballot_w64(__float_as_int(v.y) < 0);
    hit |= hit >> 32;
    hit |= hit >> 16;
    const unsigned bits = ((unsigned)hit & (kLong - 1)) | (__builtin_amdgcn_ballot_w64(any_long) != 0 ? kLong : 0u);
    __syncthreads();
    if (lane == 0 && bits) atomicOr(&sh_bits, bits);
    __syncthreads();
  }
  const unsigned bits = sh_bits;
  for (;;) {
    const int s = s0 + k, a = max(span.x, 0), e = min(span.y, pos_max + 1);
    const bool some = s < p.S && e > a;
    const int sp = some ? a / 16 / per : 0;
    // (what the first kernel did not sum: any span of a split without a list, and behind a split with long spans in the sequence)
    const bool left_out = some && (((bits >> sp) & 1) || ((bits & kLong) && e > 16 * per * (sp + 1)));
    const unsigned walk = (unsigned)__builtin_amdgcn_ballot_w64(left_out) & ((1u << turn) - 1);      // (lane k of each wave: span k)
    if (mine && s < p.S && !((walk >> k) & 1)) mass[(size_t)slot * p.S + s] = ok && some ? out * sh_f[row][sp] : 0.0f;
    if (walk) {                                      // (the same in all waves)
      const int parts = kSumWaves >> turn_log2, wk = wave / parts, part = wave % parts;
      if ((walk >> wk) & 1) {
        const int wa = __builtin_amdgcn_readlane(a, wk), we = __builtin_amdgcn_readlane(e, wk);
        const int* bt = p.block_table + (size_t)i * p.max_blocks;
        bf16x8 qf[kSplitBlocks][D / 32];
#pragma unroll
        for (int nb = 0; nb < kSplitBlocks; ++nb) load_q<D>(p, r[nb], quarter, qf[nb]);
        const float c = KV8 ? p.scale_log2 * p.k_scale[r[0].g] : p.scale_log2;
        float acc[kSplitBlocks], M[kSplitBlocks];
#pragma unroll
        for (int nb = 0; nb < kSplitBlocks; ++nb) { acc[nb] = 0.0f; M[nb] = sh_M[kSmRows * nb + j]; }
        const int tiles = (we + 15) / 16 - wa / 16, run = (tiles + parts - 1) / parts;
        stream_tiles<D, kSplitBlocks, KV8>(p, bt, r[0].g, lane, qf, wa / 16 + run * part, min(run, tiles - run * part), pos_max / 16,
                                           [&](int key0, const f32x4 (&sc)[kSplitBlocks]) {
#pragma unroll
          for (int nb = 0; nb < kSplitBlocks; ++nb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int key = key0 + 4 * quarter + q;
              acc[nb] += (key >= wa && key < we && key <= r[nb].pos) ? fast_exp2(sc[nb][q] * c - M[nb]) : 0.0f;
            }
        });
#pragma unroll
        for (int nb = 0; nb < kSplitBlocks; ++nb) {
          const float v = row_sum(acc[nb]);
          if (quarter == 0) sh_part[wave][kSmRows * nb + j] = v;
        }
      }
      __syncthreads();
      if (mine && ((walk >> k) & 1)) {
        float v = 0.0f;
        for (int w = 0; w < parts; ++w) v += sh_part[k * parts + w][row];
        mass[(size_t)slot * p.S + s] = ok ? v * sh_inv[row] : 0.0f;
      }
      __syncthreads();
    }
    s0 += p.sgroups * turn;
    if (s0 >= p.S) break;
    span = spans[min(s0 + k, p.S - 1)];
    out = ok && s0 + k < p.S ? mass[(size_t)slot * p.S + s0 + k] : 0.0f;
  }
}

// geometry of the split path from host scalars only
struct SplitGeom { int nsplit, least, sgroups, span_turn, nq_pad; size_t bytes; bool usable; };

// Scratch memory for fewer key splits than one per this many keys is not used (nor touched): pass 1 would run on a small
// part of the chip.
constexpr int kLeastSplitKeys = 2 * kSplitKeys;

inline SplitGeom split_geometry(const hook_attn_probe_args* a) {
  SplitGeom g{};
  const long long max_ctx = (long long)a->max_blocks_per_seq * kBlock;
  g.nsplit = (int)((max_ctx + kSplitKeys - 1) / kSplitKeys);
  if (g.nsplit < 1) g.nsplit = 1;
  if (g.nsplit > kMaxSplits) g.nsplit = kMaxSplits;
  g.least = (int)((max_ctx + kLeastSplitKeys - 1) / kLeastSplitKeys);
  if (g.least > kMaxSplits) g.least = kMaxSplits;
  // as many as the launch grid's third dimension (65535) holds
  if ((long long)a->num_seqs * g.nsplit > 65535) g.nsplit = 65535 / a->num_seqs;
  if (g.least > g.nsplit) g.least = g.nsplit;
  // Spans eight at a time, fewer where that leaves compute units without work, as long as that dimension holds the groups.  Spans
  // that are walked (long ones, overlapping ones) should be spread over the chip, the others ask for fewer workgroups.  Wave-to-a-span form, 128
  // and 256 workgroups, us: 4 prompts on 8 heads, 16 spans of 600-1500 keys 63.5, 73.9 and 58.0, 16 overlapping ones of 170-270 24.2, 27.3 and 24.4,
  // 30 of 820-860 43.7, 65.1 and 43.8; 16 apart of 20-60 18.7, 18.7 and 18.8.  But 3 x 60 of 20-60 on 8 heads 20.2 with 192 and 21.4 with 360, 1 x 100 of
  // 64-256 on 12 22.7 with 156 and 23.6 with 300, so spans that can only be short on average (by the width of the table) need 144.
  // (100 overlapping spans of 2000 keys in each of 4 prompts: 416 workgroups, two on some compute units, 243 against 190 in the former form.)
  const long long blocks = (long long)a->num_seqs * a->num_probe_heads * ((a->max_sel_q + kSplitRows - 1) / kSplitRows);
  const bool can_be_long = (long long)a->max_blocks_per_seq * kBlock > (long long)kOverhang * a->max_spans;
  const int least_wgs = can_be_long ? kSumWgsLong : kSumWgs;
  g.span_turn = kSumWaves;
  while (g.span_turn > 1 && blocks * ((a->max_spans + g.span_turn - 1) / g.span_turn) < least_wgs) g.span_turn /= 2;
  g.sgroups = (a->max_spans + g.span_turn - 1) / g.span_turn;
  if (g.sgroups < 1) g.sgroups = 1;
  if (a->num_seqs > 0 && g.sgroups > 65535 / a->num_seqs) g.sgroups = 65535 / a->num_seqs;
  g.nq_pad = (a->max_sel_q + kSmRows - 1) / kSmRows * kSmRows;
  g.bytes = (size_t)a->num_seqs * a->num_probe_heads * g.nq_pad * g.nsplit * sizeof(float2);
  g.usable = g.nsplit >= 1 && g.sgroups >= 1;
  return g;
}

__global__ __launch_bounds__(256) void k_zero_mass(float* ptr, size_t n) {
  for (size_t x = (size_t)blockIdx.x * 256 + threadIdx.x; x < n; x += (size_t)gridDim.x * 256) ptr[x] = 0.0f;
}

}  // namespace
}  // namespace hook

extern "C" hook_status hook_span_mass(const hook_attn_probe_args* a) {
  using namespace hook;
  if (!a) return HOOK_ERR_NULL;
  if (a->num_seqs < 0 || a->total_q < 0 || a->num_q_heads <= 0 || a->num_kv_heads <= 0 ||
      a->max_blocks_per_seq <= 0 || a->num_blocks <= 0 || a->head_dim <= 0)
    return HOOK_ERR_SHAPE;
  if (a->num_q_heads % a->num_kv_heads != 0) return HOOK_ERR_SHAPE;
  if (a->block_size != HOOK_BLOCK_SIZE || a->dtype != HOOK_BF16 || (a->head_dim != 64 && a->head_dim != 128))
    return HOOK_ERR_UNSUPPORTED;
  if (a->max_blocks_per_seq > (1 << 26)) return HOOK_ERR_UNSUPPORTED;
  const int P = a->num_probe_heads;
  if (P < 1 || P > a->num_q_heads || a->max_sel_q < 1 || a->max_spans < 1) return HOOK_ERR_SHAPE;
  if (a->max_sel_q > HOOK_MAX_SEL_Q || a->max_spans > HOOK_MAX_SPANS_WIDE) return HOOK_ERR_UNSUPPORTED;
  if (a->num_seqs > 65535 || P > 65535) return HOOK_ERR_UNSUPPORTED;
  if (!a->probe_heads || !a->query_sel || !a->key_spans || !a->mass) return HOOK_ERR_NULL;
  if (a->num_seqs == 0) return HOOK_OK;
  if (!a->q || !a->k_cache || !a->block_table || !a->seq_lens || !a->cu_q_lens) return HOOK_ERR_NULL;
  if (a->kv_dtype != HOOK_KV_SAME && a->kv_dtype != HOOK_KV_FP8_E4M3) return HOOK_ERR_SHAPE;
  const bool kv8 = a->kv_dtype == HOOK_KV_FP8_E4M3;
  if (kv8 && !a->k_scale) return HOOK_ERR_NULL;

  SpanParams p{};
  p.k_scale = a->k_scale;
  p.num_seqs = a->num_seqs; p.total_q = a->total_q; p.Hq = a->num_q_heads; p.Hkv = a->num_kv_heads;
  p.G = p.Hq / p.Hkv; p.max_blocks = a->max_blocks_per_seq; p.num_blocks = a->num_blocks;
  const float scale = a->scale > 0.0f ? a->scale : 1.0f / std::sqrt((float)a->head_dim);
  p.scale_log2 = scale * 1.44269504088896340736f;
  p.q = a->q; p.k_cache = a->k_cache; p.block_table = a->block_table; p.seq_lens = a->seq_lens;
  p.cu_q_lens = a->cu_q_lens; p.P = P; p.probe_heads = a->probe_heads; p.NQ = a->max_sel_q;
  p.query_sel = a->query_sel; p.S = a->max_spans; p.key_spans = a->key_spans; p.mass = a->mass;
  hipStream_t st = static_cast<hipStream_t>(a->stream);

  // with enough scratch memory: pass 1 split over the keys, pass 2 over the spans
  // (as many key splits as the scratch memory holds; below the least number it is left alone)
  SplitGeom geo = split_geometry(a);
  const size_t per_split = geo.bytes / (size_t)geo.nsplit;
  if (a->workspace_bytes < geo.bytes) geo.nsplit = (int)(a->workspace_bytes / per_split);
  if (geo.usable && a->workspace && geo.nsplit >= geo.least && (reinterpret_cast<uintptr_t>(a->workspace) % 8) == 0) {
    p.stats = static_cast<float2*>(a->workspace);
    p.nsplit = geo.nsplit; p.sgroups = geo.sgroups; p.span_turn = geo.span_turn; p.nq_pad = geo.nq_pad;
    const unsigned gx = (unsigned)((geo.nq_pad / kSmRows + kSplitBlocks - 1) / kSplitBlocks);
    const dim3 ga(gx, (unsigned)P, (unsigned)(p.num_seqs * geo.nsplit)), gb(gx, (unsigned)P, (unsigned)(p.num_seqs * geo.sgroups));
    const dim3 ta(kStatWaves * 64), tb(kSumWaves * 64);
    if (a->head_dim == 128 && !kv8) {
      hipLaunchKernelGGL((k_span_stats<128, false>), ga, ta, 0, st, p);
      hipLaunchKernelGGL((k_span_sums<128, false>), gb, tb, 0, st, p);
    } else if (a->head_dim == 128) {
      hipLaunchKernelGGL((k_span_stats<128, true>), ga, ta, 0, st, p);
      hipLaunchKernelGGL((k_span_sums<128, true>), gb, tb, 0, st, p);
    } else if (!kv8) {
      hipLaunchKernelGGL((k_span_stats<64, false>), ga, ta, 0, st, p);
      hipLaunchKernelGGL((k_span_sums<64, false>), gb, tb, 0, st, p);
    } else {
      hipLaunchKernelGGL((k_span_stats<64, true>), ga, ta, 0, st, p);
      hipLaunchKernelGGL((k_span_sums<64, true>), gb, tb, 0, st, p);
    }
    return hipGetLastError() == hipSuccess ? HOOK_OK : HOOK_ERR_LAUNCH;
  }

  const size_t nmass = (size_t)p.num_seqs * p.P * p.NQ * p.S;
  size_t zb = (nmass + 2047) / 2048;
  if (zb > 2048) zb = 2048;
  hipLaunchKernelGGL(k_zero_mass, dim3((unsigned)zb), dim3(256), 0, st, p.mass, nmass);
  if (hipGetLastError() != hipSuccess) return HOOK_ERR_LAUNCH;
  const dim3 grid((unsigned)((p.NQ + kSmRows - 1) / kSmRows), (unsigned)P, (unsigned)p.num_seqs);
  const dim3 tb(kSmWaves * 64);
  if (a->head_dim == 128 && !kv8) hipLaunchKernelGGL((k_span_mass<128, false>), grid, tb, 0, st, p);
  else if (a->head_dim == 128) hipLaunchKernelGGL((k_span_mass<128, true>), grid, tb, 0, st, p);
  else if (!kv8) hipLaunchKernelGGL((k_span_mass<64, false>), grid, tb, 0, st, p);
  else hipLaunchKernelGGL((k_span_mass<64, true>), grid, tb, 0, st, p);
  return hipGetLastError() == hipSuccess ? HOOK_OK : HOOK_ERR_LAUNCH;
}

extern "C" size_t hook_span_mass_workspace_bytes(const hook_attn_probe_args* a) {
  if (!a || a->num_seqs <= 0 || a->num_probe_heads <= 0 || a->max_sel_q <= 0 || a->max_spans <= 0 ||
      a->max_blocks_per_seq <= 0)
    return 0;
  const hook::SplitGeom g = hook::split_geometry(a);
  return g.usable ? g.bytes : 0;
}
