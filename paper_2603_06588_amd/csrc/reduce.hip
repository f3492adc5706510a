// Score reductions over the mass tensor: one workgroup per sequence (and per 16 spans), fp32 sums in a
// fixed order (strided partial sums per thread, a butterfly inside the wave, the waves in turn), so the
// result does not depend on anything but the inputs.
#include "../../include/hook_api.h"
#include "hook_device.h"

namespace hook {
namespace {

struct ReduceParams {
  int num_seqs, P, NQ, S, mode, span_a, span_b, accumulate;
  int lanes_log2;   // SPAN_MEAN: 2^lanes_log2 neighbouring threads take neighbouring spans of one row
  const float* mass;
  const int* query_sel;
  const int* cu_q_lens;
  const float* w;
  float* scores;
};

// What is read is a few KB to a few MB and every pair of (head, row) is independent, so the kernel is
// bound by how many loads are in flight: kInFlight rows per thread, and as many threads as the pairs need
// (256, or 1024 from kManyPairs pairs on, where 256 threads would take several trips to memory in turn).
constexpr int kInFlight = 8;
constexpr int kManyPairs = 128;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

struct SeqRows { int skip, nv; };   // slots skip .. skip + nv - 1 hold selected rows

__device__ __forceinline__ SeqRows selected_slots(const ReduceParams& p, int i) {
  SeqRows s = {0, p.NQ};
  if (p.query_sel) {
    const int qb = p.query_sel[2 * i];
    int qe = min(p.query_sel[2 * i + 1], qb + p.NQ);
    if (p.cu_q_lens) qe = min(qe, p.cu_q_lens[i + 1] - p.cu_q_lens[i]);
    s.nv = max(qe - max(qb, 0), 0);
    // slots of rows before the chunk (negative t) come first and hold zeros; they do not count
    s.skip = qb < 0 ? min(-qb, p.NQ) : 0;
  }
  return s;
}

// Scores per span.  A row's spans are neighbours in memory, so neighbouring threads take neighbouring
// spans of one row and the groups of threads share the (head, row) pairs: every load is coalesced.
// (One wave per sequence, eight spans per pass over the pairs, read 4 x 8 heads x 32 rows x 88 spans in 96 us.  With 64
// spans to a workgroup, two batches of loads per thread and a division for each load 4 x 8 x 32 x 100 took 6.3 us in a
// kernel trace; with one batch and the pair counted on from load to load it takes 4.6 at 32 spans and 3.9 at 16, where a
// row's share is 64 bytes still.)
constexpr int kReduceSpansLog2 = 4;
template <int NT>
__global__ __launch_bounds__(NT) void k_reduce_spans(const ReduceParams p) {
  __shared__ float red[NT / 64][1 << kReduceSpansLog2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = blockIdx.x;
  const int lanes = 1 << p.lanes_log2;
  const int r = (blockIdx.y << kReduceSpansLog2) + (tid & (lanes - 1));
  const int sub = tid >> p.lanes_log2, nsub = NT >> p.lanes_log2;
  const SeqRows rows = selected_slots(p, i);
  const float* m = p.mass + (size_t)i * p.P * p.NQ * p.S + r;
  const int npairs = p.P * rows.nv;
  float acc = 0.0f;
  if (r < p.S && npairs > 0) {
    int ph = sub / rows.nv, t = sub - ph * rows.nv;               // the next pair, and how far it is to the one after
    const int dph = nsub / rows.nv, dt = nsub - dph * rows.nv;
    for (int e0 = sub; e0 < npairs; e0 += kInFlight * nsub) {
      float v[kInFlight], wp[kInFlight];
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) {
        const int h = min(ph, p.P - 1);                           // past the end: some load with weight 0
        v[u] = m[((size_t)h * p.NQ + rows.skip + t) * p.S];
        wp[u] = p.w ? p.w[h] : 1.0f / (float)p.P;
        ph += dph;
        t += dt;
        if (t >= rows.nv) { t -= rows.nv; ++ph; }
      }
#pragma unroll
      for (int u = 0; u < kInFlight; ++u) acc += (e0 + u * nsub < npairs) ? wp[u] * v[u] : 0.0f;
    }
  }
  for (int off = lanes; off < 64; off <<= 1) acc += __shfl_xor(acc, off);
  if (lane < lanes) red[wave][lane] = acc;
  __syncthreads();
  if (tid < lanes && r < p.S) {
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) sum += red[w][tid];
    const float v = sum * (rows.nv > 0 ? 1.0f / (float)rows.nv : 0.0f);
    float* dst = p.scores + (size_t)i * p.S + r;
    *dst = p.accumulate ? *dst + v : v;
  }
}

// One ratio per sequence: threads over the (head, row) pairs.
template <int NT>
__global__ __launch_bounds__(NT) void k_reduce_ratio(const ReduceParams p) {
  __shared__ float red[2][NT / 64];
  const int tid = threadIdx.x, i = blockIdx.x;
  const SeqRows rows = selected_slots(p, i);
  const float* m = p.mass + (size_t)i * p.P * p.NQ * p.S;
  const int npairs = p.P * rows.nv;
  float sa = 0.0f, sb = 0.0f;   // RATIO_MEAN uses sa only
  for (int e = tid; e < npairs; e += NT) {
    const int ph = e / rows.nv, t = rows.skip + e - ph * rows.nv;
    const float wp = p.w ? p.w[ph] : 1.0f / (float)p.P;
    const float* row = m + ((size_t)ph * p.NQ + t) * p.S;
    const float a = row[p.span_a], b = row[p.span_b];
    if (p.mode == HOOK_REDUCE_RATIO_MEAN) {
      const float den = a + b;
      sa += den != 0.0f ? wp * (a / den) : 0.0f;
    } else {
      sa += wp * a;
      sb += wp * b;
    }
  }
  sa = wave_sum(sa);
  sb = wave_sum(sb);
  if ((tid & 63) == 0) { red[0][tid >> 6] = sa; red[1][tid >> 6] = sb; }
  __syncthreads();
  if (tid != 0) return;
  float A = 0.0f, B = 0.0f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) { A += red[0][w]; B += red[1][w]; }
  const float inv_nv = rows.nv > 0 ? 1.0f / (float)rows.nv : 0.0f;
  A *= inv_nv;
  B *= inv_nv;
  const float v = p.mode == HOOK_REDUCE_RATIO_MEAN ? A : ((A + B) != 0.0f ? A / (A + B) : 0.0f);
  p.scores[i] = p.accumulate ? p.scores[i] + v : v;
}

}  // namespace
}  // namespace hook

extern "C" hook_status hook_reduce_mass(const hook_reduce_args* a) {
  using namespace hook;
  if (!a) return HOOK_ERR_NULL;
  if (a->num_seqs < 0 || a->num_probe_heads < 1 || a->max_sel_q < 1 || a->max_sel_q > HOOK_MAX_SEL_Q ||
      a->max_spans < 1 || a->max_spans > HOOK_MAX_SPANS_WIDE)
    return HOOK_ERR_SHAPE;
  if (a->mode != HOOK_REDUCE_SPAN_MEAN && a->mode != HOOK_REDUCE_RATIO_MEAN && a->mode != HOOK_REDUCE_RATIO_OF_SUMS)
    return HOOK_ERR_UNSUPPORTED;
  if (a->mode != HOOK_REDUCE_SPAN_MEAN &&
      (a->span_a < 0 || a->span_a >= a->max_spans || a->span_b < 0 || a->span_b >= a->max_spans))
    return HOOK_ERR_SHAPE;
  if (a->num_seqs == 0) return HOOK_OK;
  if (!a->mass || !a->scores) return HOOK_ERR_NULL;
  ReduceParams p{};
  p.num_seqs = a->num_seqs; p.P = a->num_probe_heads; p.NQ = a->max_sel_q; p.S = a->max_spans;
  p.mode = a->mode; p.span_a = a->span_a; p.span_b = a->span_b; p.accumulate = a->accumulate;
  p.mass = a->mass; p.query_sel = a->query_sel; p.cu_q_lens = a->cu_q_lens; p.w = a->head_weights;
  p.scores = a->scores;
  hipStream_t st = static_cast<hipStream_t>(a->stream);
  const bool many = (long long)p.P * p.NQ >= kManyPairs;
  if (p.mode == HOOK_REDUCE_SPAN_MEAN) {
    while ((1 << p.lanes_log2) < p.S && p.lanes_log2 < kReduceSpansLog2) ++p.lanes_log2;
    const dim3 grid((unsigned)p.num_seqs, (unsigned)((p.S + (1 << kReduceSpansLog2) - 1) >> kReduceSpansLog2));
    if (many) hipLaunchKernelGGL(k_reduce_spans<1024>, grid, dim3(1024), 0, st, p);
    else hipLaunchKernelGGL(k_reduce_spans<256>, grid, dim3(256), 0, st, p);
  } else if (many) {
    hipLaunchKernelGGL(k_reduce_ratio<1024>, dim3((unsigned)p.num_seqs), dim3(1024), 0, st, p);
  } else {
    hipLaunchKernelGGL(k_reduce_ratio<256>, dim3((unsigned)p.num_seqs), dim3(256), 0, st, p);
  }
  return hipGetLastError() == hipSuccess ? HOOK_OK : HOOK_ERR_LAUNCH;
}
