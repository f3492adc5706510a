// fp32 attention + probe.  Full-precision inputs cannot go through the bf16 matrix cores without
// changing the result; the fp32 matrix instruction (16x16x4: fp32 products and sums) keeps every bit of
// them, so this path uses the same structure as the bf16 one at fp32 throughout.
//
// Workgroup = NW waves = 16 query rows of one sequence x one q head; the waves share the keys (one
// 16-key cache block at a time, round-robin), each keeps an online softmax with its share of the output
// in registers, and the shares are merged in LDS.  The contraction may take its terms in any order, so
// both operands are laid out for 16-byte loads: k-step (i, e) of S^T = K Q^T takes dimensions
// 16 i + 4 (lane / 16) + e, and row m of O^T = V^T P^T stands for the dimensions 64 i + 4 m + c.  The
// scores of a lane (query lane % 16, keys 4 (lane / 16) + r) are then the B operand of the second product
// without moving between lanes.
//
// What bounds it: small batches are all this path sees, so latency - the length of one wave's chain of
// dependent loads and the number of launches.  256 rows x 8 heads, d 64: one row per wave on the vector ALUs
// behind a clearing launch took 2.8 + 34 us, this takes one launch of 8.7 us (kernel trace).
#include "hook_device.h"

namespace hook {

namespace {

constexpr int kF32Rows = 16;

// Item numbering without a planner: sequence i owns the items from cu_q_lens[i] / 16 + i on, which
// leaves room for ceil(n_i / 16) items whatever the lengths are (some items stay empty).
__device__ __forceinline__ int first_item(const int* cu, int i) { return cu[i] / kF32Rows + i; }

// Does slot `slot` of (sequence i, probe entry ps) hold a row that the attention workgroups write?
__device__ __forceinline__ bool slot_is_written(const AttnParams& p, int i, int ps, int slot) {
  const int first = p.cu_q_lens[i], n = p.cu_q_lens[i + 1] - first;
  const int L = min(p.seq_lens[i], p.max_blocks * kBlock);
  if (first < 0 || n <= 0 || n > L) return false;
  const int t = p.query_sel[2 * i] + slot;
  if (t < 0 || t >= n || t >= p.query_sel[2 * i + 1] || first + t >= p.total_q) return false;
  const int head = p.probe_heads[ps];
  return (unsigned)head < (unsigned)p.Hq && find_probe_slot(p.probe_heads, p.P, head) == ps;
}

template <int D, int NW>
__device__ __forceinline__ void f32_block(const AttnParams& p, int seq, int first, int n, int rows, int L, int r0,
                                          int head) {
  constexpr int KI = D / 16, VI = D / 64, ST = D + 4;
  __shared__ __attribute__((aligned(16))) float red_o[NW][kF32Rows][ST];
  __shared__ float red_s[NW][kF32Rows][2 + kMaxSpans];   // max, sum, span sums

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15, quarter = lane >> 4;
  const int t = min(r0 + j, rows - 1);          // lanes without a row repeat the last one
  const int pos = L - n + t, pos_min = L - n + r0;
  const int ntile = (L - n + min(r0 + kF32Rows, rows) - 1) / kBlock + 1;
  const int kvh = head / p.G;

  const float* const kc = static_cast<const float*>(p.k_cache) + (size_t)kvh * kBlock * D;
  const float* const vc = static_cast<const float*>(p.v_cache) + (size_t)kvh * kBlock * D;
  const int* const bt = p.block_table + (size_t)seq * p.max_blocks;
  const size_t blk_stride = (size_t)p.Hkv * kBlock * D;

  float4 kf[2][KI], vf[2][4][VI];
  auto load_tile = [&](int kt, float4 (&k)[KI], float4 (&v)[4][VI]) {
    int blk = bt[min(kt, ntile - 1)];
    blk = ((unsigned)blk < (unsigned)p.num_blocks) ? blk : 0;
    const float4* kr = reinterpret_cast<const float4*>(kc + blk * blk_stride + (size_t)j * D) + quarter;
#pragma unroll
    for (int i = 0; i < KI; ++i) k[i] = kr[4 * i];
    // a value row past the last token may hold anything (0 * NaN), so it is replaced by the last token's
    const int last = L - 1 - kBlock * min(kt, ntile - 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float4* vr = reinterpret_cast<const float4*>(vc + blk * blk_stride + (size_t)min(4 * quarter + e, last) * D) + j;
#pragma unroll
      for (int i = 0; i < VI; ++i) v[e][i] = vr[16 * i];
    }
  };
  load_tile(w, kf[0], vf[0]);

  float4 qf[KI];
  {
    const float4* qr = reinterpret_cast<const float4*>(static_cast<const float*>(p.q) + ((size_t)(first + t) * p.Hq + head) * D) + quarter;
#pragma unroll
    for (int i = 0; i < KI; ++i) qf[i] = qr[4 * i];
  }

  int pslot = -1, qsel_b = 0, qsel_e = 0;
  int sp_a[kMaxSpans], sp_b[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) { sp_a[s] = 0; sp_b[s] = 0; }
  if (p.P > 0) {
    qsel_b = p.query_sel[2 * seq];
    qsel_e = min(p.query_sel[2 * seq + 1], qsel_b + p.NQ);
    if (qsel_b < r0 + kF32Rows && qsel_e > r0) pslot = find_probe_slot(p.probe_heads, p.P, head);
    if (pslot >= 0) load_spans(p.key_spans, seq, p.S, sp_a, sp_b);
  }

  const float c = p.scale_log2;
  float m_run = -INFINITY, l_run = 0.0f;
  float am[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) am[s] = 0.0f;
  f32x4 o[VI][4];
#pragma unroll
  for (int i = 0; i < VI; ++i)
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) o[i][cc] = {0.0f, 0.0f, 0.0f, 0.0f};

  auto comp = [](const float4& v, int e) { return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w; };
  auto tile = [&](int kt, const float4 (&k)[KI], const float4 (&v)[4][VI]) {
    f32x4 acc[4];     // four independent chains, summed afterwards
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < KI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp(k[i], e), comp(qf[i], e), acc[e], 0, 0, 0);
    float s[4];
    float bm = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = ((acc[0][r] + acc[1][r]) + (acc[2][r] + acc[3][r])) * c;
      if (kBlock * kt + 4 * quarter + r > pos) s[r] = -INFINITY;
      bm = fmaxf(bm, s[r]);
    }
    bm = fmaxf(bm, __shfl_xor(bm, 16));
    bm = fmaxf(bm, __shfl_xor(bm, 32));
    const float mn = fmaxf(m_run, bm);
    const float ref = (mn == -INFINITY) ? 0.0f : mn;      // nothing visible yet: every term is 0
    const float alpha = fast_exp2(m_run - ref);
    m_run = mn;
    float pr[4], psum = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pr[r] = fast_exp2(s[r] - ref);
      psum += pr[r];
    }
    l_run = l_run * alpha + psum;
#pragma unroll
    for (int i = 0; i < VI; ++i)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[i][cc][r] *= alpha;
    // A key that only some of the rows see meets the others with a probability of 0, and 0 * Inf is not 0: where such a
    // tile holds a value that is not finite, the product takes 0 in its place and the rows that see it add it afterwards.
    float poison = 0.0f;
    if (kBlock * kt + kBlock - 1 > pos_min) {      // uniform
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < VI; ++i)
#pragma unroll
          for (int cc = 0; cc < 4; ++cc) poison = __builtin_fmaf(comp(v[e][i], cc), 0.0f, poison);
    }
    if (__builtin_amdgcn_ballot_w64(poison != poison) == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < VI; ++i)
#pragma unroll
          for (int cc = 0; cc < 4; ++cc)
            o[i][cc] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp(v[e][i], cc), pr[e], o[i][cc], 0, 0, 0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < VI; ++i)
#pragma unroll
          for (int cc = 0; cc < 4; ++cc) {
            const float x = comp(v[e][i], cc);
            o[i][cc] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_isfinite(x) ? x : 0.0f, pr[e], o[i][cc], 0, 0, 0);
          }
#pragma unroll 1
      for (int kq = 0; kq < 4; ++kq)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float pk = __shfl(pr[e], 16 * kq + j);
          const bool sees = kBlock * kt + 4 * kq + e <= pos;
#pragma unroll
          for (int i = 0; i < VI; ++i)
#pragma unroll
            for (int cc = 0; cc < 4; ++cc)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float x = __shfl(comp(v[e][i], cc), 16 * kq + 4 * quarter + r);
                if (sees && !__builtin_isfinite(x)) o[i][cc][r] = __builtin_fmaf(pk, x, o[i][cc][r]);
              }
        }
    }
    if (pslot >= 0) {
#pragma unroll
      for (int sp = 0; sp < kMaxSpans; ++sp)
        if (sp < p.S) {
          float add = 0.0f;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int key = kBlock * kt + 4 * quarter + r;
            add += (key >= sp_a[sp] && key < sp_b[sp]) ? pr[r] : 0.0f;
          }
          am[sp] = am[sp] * alpha + add;
        }
    }
  };
  for (int kt = w; kt < ntile; kt += 2 * NW) {     // the next block's loads are in flight during a block's products
    load_tile(kt + NW, kf[1], vf[1]);
    tile(kt, kf[0], vf[0]);
    if (kt + NW < ntile) {
      load_tile(kt + 2 * NW, kf[0], vf[0]);
      tile(kt + NW, kf[1], vf[1]);
    }
  }

  // merge: the lanes of a row, then the waves
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s)
    if (s < p.S) {
      am[s] += __shfl_xor(am[s], 16);
      am[s] += __shfl_xor(am[s], 32);
    }
#pragma unroll
  for (int i = 0; i < VI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      *reinterpret_cast<float4*>(&red_o[w][j][64 * i + 4 * (4 * quarter + r)]) =
          make_float4(o[i][0][r], o[i][1][r], o[i][2][r], o[i][3][r]);
  if (quarter == 0) {
    red_s[w][j][0] = m_run;
    red_s[w][j][1] = l_run;
#pragma unroll
    for (int s = 0; s < kMaxSpans; ++s)
      if (s < p.S) red_s[w][j][2 + s] = am[s];
  }
  __syncthreads();
  auto weights = [&](int row, float (&wt)[NW]) {   // of the waves' shares, normalised
    float m = -INFINITY, l = 0.0f;
#pragma unroll
    for (int k = 0; k < NW; ++k) m = fmaxf(m, red_s[k][row][0]);
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      wt[k] = fast_exp2(red_s[k][row][0] - m);     // a wave without keys: exp2(-inf) = 0
      l += wt[k] * red_s[k][row][1];
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int k = 0; k < NW; ++k) wt[k] *= inv;
  };
  for (int x = tid; x < kF32Rows * D / 4; x += NW * 64) {
    const int row = x / (D / 4), col = 4 * (x % (D / 4));
    if (r0 + row >= rows) break;                   // rows come in order
    float wt[NW];
    weights(row, wt);
    float4 sum = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const float4 v = *reinterpret_cast<const float4*>(&red_o[k][row][col]);
      sum.x = __builtin_fmaf(wt[k], v.x, sum.x); sum.y = __builtin_fmaf(wt[k], v.y, sum.y);
      sum.z = __builtin_fmaf(wt[k], v.z, sum.z); sum.w = __builtin_fmaf(wt[k], v.w, sum.w);
    }
    *reinterpret_cast<float4*>(static_cast<float*>(p.out) + ((size_t)(first + r0 + row) * p.Hq + head) * D + col) = sum;
  }
  if (pslot >= 0) {
    for (int x = tid; x < kF32Rows * p.S; x += NW * 64) {
      const int row = x / p.S, s = x - row * p.S, tr = r0 + row;
      if (tr < rows && tr >= qsel_b && tr < qsel_e) {
        float wt[NW];
        weights(row, wt);
        float a = 0.0f;
#pragma unroll
        for (int k = 0; k < NW; ++k) a += wt[k] * red_s[k][row][2 + s];
        p.mass[(((size_t)seq * p.P + pslot) * p.NQ + (tr - qsel_b)) * p.S + s] = a;
      }
    }
  }
}

template <int D, int NW>
__global__ __launch_bounds__(NW * 64) void k_attn_f32(const AttnParams p) {
  const int item = blockIdx.x, head = blockIdx.y;
  int lo = 0, hi = p.num_seqs;      // largest i whose items begin at or before this one
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (first_item(p.cu_q_lens, mid) <= item) lo = mid; else hi = mid;
  }
  const int first = p.cu_q_lens[lo], n = p.cu_q_lens[lo + 1] - first;
  const int L = min(p.seq_lens[lo], p.max_blocks * kBlock);
  const int r0 = kF32Rows * (item - (first / kF32Rows + lo));
  const int rows = min(n, p.total_q - first);
  if (first >= 0 && r0 >= 0 && r0 < rows && n <= L) f32_block<D, NW>(p, lo, first, n, rows, L, r0, head);

  // every entry of `mass` without a row is zero (these stores and those of the rows never meet)
  const size_t nmass = (size_t)p.num_seqs * p.P * p.NQ * p.S;
  const size_t wg = (size_t)blockIdx.y * gridDim.x + blockIdx.x, step = (size_t)gridDim.x * gridDim.y * (NW * 64);
  for (size_t e = wg * (NW * 64) + threadIdx.x; e < nmass; e += step) {
    const size_t at = e / p.S;
    const int slot = (int)(at % p.NQ), ps = (int)(at / p.NQ % p.P), i = (int)(at / p.NQ / p.P);
    if (!slot_is_written(p, i, ps, slot)) p.mass[e] = 0.0f;
  }
  if (wg == 0) {   // the status bits that the planner of the bf16 path records
    __shared__ int status;
    if (threadIdx.x == 0) status = 0;
    __syncthreads();
    int bits = 0;
    for (int i = threadIdx.x; i < p.num_seqs; i += NW * 64) {
      const int ni = p.cu_q_lens[i + 1] - p.cu_q_lens[i], Li = p.seq_lens[i];
      if (ni <= 0) continue;
      if (Li < 0) bits |= kStatNegative;
      else if (ni > min(Li, p.max_blocks * kBlock)) bits |= kStatQGtL;
      if (Li > p.max_blocks * kBlock) bits |= kStatLenClamped;
    }
    if (bits) atomicOr(&status, bits);
    __syncthreads();
    if (threadIdx.x == 0) { p.hdr->n_prefill = 0; p.hdr->n_decode = 0; p.hdr->chunk_keys = 0; p.hdr->status = status; }
  }
}

}  // namespace

hipError_t launch_attn_f32(const AttnParams& p, int D, hipStream_t st) {
  const long long items = (long long)p.total_q / kF32Rows + p.num_seqs;
  if (items > 0x7fffffffLL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)items, (unsigned)p.Hq);
  // eight waves, or four where the merge buffer of eight would not fit the 64 KB of static LDS
  if (D == 128) hipLaunchKernelGGL((k_attn_f32<128, 4>), grid, dim3(256), 0, st, p);
  else if (D == 64) hipLaunchKernelGGL((k_attn_f32<64, 8>), grid, dim3(512), 0, st, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace hook
