// Split-key decode attention (one query row per sequence) and the kernel that merges the
// per-chunk partial results.
//
// The path is bound by HBM: every live K and V element of a kv head is read exactly once
// and shared by the HP query heads of its group.  A workgroup owns one (range of the contexts, or
// sequence and key chunk; kv head); each of its 4 waves streams a contiguous run of 16-key cache blocks straight
// from global memory into registers (16-byte loads, one block ahead):
//   - the K block is the A operand of S^T = K Q^T (16x16x32 bf16 MFMA, keys = M, heads = N),
//     whose accumulator gives lane (head j, key group kq) the scores of 4 keys;
//   - every (head, key group) lane runs its own online softmax over the keys it sees, so
//     the loop has no cross-lane reduction; exponentials are handed to the lanes that hold
//     the matching V rows with a DPP broadcast, and P V is plain fp32 FMAs on V in its
//     natural layout;
//   - the key-group streams of a wave, the waves of a workgroup and finally the chunks of a
//     sequence are merged with the usual (max, sum) weights; probe span sums ride along with
//     the normaliser in every merge.
#include "decode_device.h"

namespace hook {

namespace {

// The planner's items: one (sequence, chunk) per workgroup, longest first.  Four workgroups to a compute unit over an
// 8-bit cache and at head size 64, where a wave has half the bytes in flight (three for groups of 8 heads).
template <int D, int HP, bool KV8>
__global__ __launch_bounds__(256, (HP == 8 ? 2 : 3) + (KV8 || D == 64 ? 1 : 0)) void k_decode(const AttnParams p) {
  __shared__ float red[4][HP][DecodeCfg<D>::PSTR];
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bid = blockIdx.x;
  const int kvh = bid % p.Hkv;
  const int rest = bid / p.Hkv;
  const int hg = rest % p.dec_hgroups;
  const int turn = rest / p.dec_hgroups;
  // the grid covers the whole item capacity, so the turn's records can be fetched together with the
  // item count instead of after it
  const WorkItem it = p.dec_items[2 * turn];
  const int slot = p.dec_items[2 * turn + 1].x;
  if (turn >= p.hdr->n_decode) return;
  // the clamp only matters if the planner's capacity bound were ever violated
  const int item = min(max(slot, 0), p.dec_cap - 1);
  const int CH = p.hdr->chunk_keys;
  const int kstart = it.y * CH;
  decode_range<D, HP, KV8, lines_always<D, HP, KV8>(), 1>(p, red, tid, tid & 63, w, kvh, kvh * p.G + hg * HP, it.x, it.w, kstart, min(it.z, kstart + CH),
                           item, NewRows{-1, 0, false});
}

template <int D, int HP, bool KV8, bool WHOLE_LINES, int PER_LANE>
__global__ __launch_bounds__(256, HP == 8 ? 2 : 3) void k_decode_stream(const AttnParams p) {
  __shared__ float red[4][HP][DecodeCfg<D>::PSTR];
  stream_range<D, HP, KV8, WHOLE_LINES, PER_LANE, 1, false>(p, red, blockIdx.x);
}

// What a planner would have done besides, by one workgroup of the merge kernel: the header with the status word, zeros
// for elements of the head list that no head owns.
template <int NT>
__device__ __forceinline__ void settle_batch(const AttnParams& p) {
  __shared__ int sh_bits;
  if (threadIdx.x == 0) sh_bits = 0;
  __syncthreads();
  int bits = p.plan_fresh && bad_head_list<NT>(p) ? kBadHeadList : 0;
  for (int i = threadIdx.x; i < p.num_seqs; i += NT)
    bits |= decode_seq(p, p.seq_lens[i], p.cu_q_lens[i], p.cu_q_lens[i + 1]).bits;
  if (bits) atomicOr(&sh_bits, bits);
  __syncthreads();
  bits = sh_bits;
  if (threadIdx.x == 0) { p.hdr->n_prefill = 0; p.hdr->n_decode = 0; p.hdr->chunk_keys = 0; p.hdr->status = bits & ~kBadHeadList; }
  if (bits & kBadHeadList) zero_unowned_mass<NT>(p);
}

// Merges the partial records of a sequence: WPH waves per q head take its records in turn (a workgroup is
// max(4, WPH) waves), lane = output columns.  In a self-planned batch the wave that owns a probed head also
// zero-fills the `mass` slots without a row.  Every first touch of a record is a trip to memory (other
// workgroups wrote them under other L2s), and trips are all this kernel's time, so a wave requests several
// whole records before it waits for any: 8 where several waves share a head, and where one wave has a head to itself 4,
// or 16 for a sequence with more than that (one context of 32768 tokens, 64 records, among 199 of 300, by fours 12.0 us in
// a kernel trace and the call 89.0 us, 85.7 so; over an 8-bit cache 60.9 and 57.4; contexts of up to 200 tokens alike).
template <int D, int WPH>
__global__ __launch_bounds__(64 * (WPH > 4 ? WPH : 4)) void k_combine(const AttnParams p) {
  using C = DecodeCfg<D>;
  constexpr int E = D / 64, NWV = WPH > 4 ? WPH : 4;
  __shared__ float sh_o[WPH > 1 ? NWV : 1][D + kMaxSpans];
  __shared__ float sh_m[NWV], sh_l[NWV];
  const int seq = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = wave % WPH;
  const int head = blockIdx.y * (NWV / WPH) + wave / WPH;
  const bool stream = p.dec_ranges > 0;
  if (seq == p.num_seqs) {      // the column behind the sequences': nothing to wait for but its own trip
    if (blockIdx.y == 0) settle_batch<64 * NWV>(p);
    return;
  }
  int2 sd = p.seq_dec[seq];
  const int qrow = p.cu_q_lens[seq];
  // (the clamps only matter if the work lists were not this batch's: no record outside the workspace is read)
  sd.x = min(max(sd.x, 0), p.dec_cap - 1);
  int count = min(sd.y, p.dec_cap - sd.x);
  if (stream) {     // (a self-planned batch announces records only for sequences that have some)
    const int Lraw = p.seq_lens[seq], n = p.cu_q_lens[seq + 1] - qrow;
    const DecodeSeq ds = decode_seq(p, Lraw, qrow, qrow + n);
    if (ds.nblk == 0) count = 0;
    // a row block's `mass` belongs to the kernel that computes it
    if (p.batch_kind == 0 && n >= 2 && ds.bits != kStatNegative && !(ds.bits & (kStatQGtL | kStatNegative))) return;
  }
  if (count <= 0 && !stream) return;
  const bool live = head < p.Hq && count > 0;

  int pslot = -1, slot_row = -1;       // this head's place in the probe list; the selected row's slot, -1: none
  if (p.P > 0 && head < p.Hq) {
    // (find_probe_slot's answer without its chain of loads, as long as the list is in order)
    bool ordered = true;
    for (int i0 = 0; i0 < p.P; i0 += 64) {
      const int i = i0 + lane;
      const int ph = i < p.P ? p.probe_heads[i] : -1, before = i < p.P && i > 0 ? p.probe_heads[i - 1] : -2;
      const unsigned long long hit = __builtin_amdgcn_ballot_w64(ph == head);
      if (hit && pslot < 0) pslot = i0 + __builtin_ctzll(hit);
      ordered = ordered && __builtin_amdgcn_ballot_w64(i < p.P && i > 0 && ph <= before) == 0;
    }
    if (!ordered) pslot = find_probe_slot(p.probe_heads, p.P, head);
    // row t = 0 sits in slot t - begin, as on every other path
    const int qb = p.query_sel[2 * seq], qe = min(p.query_sel[2 * seq + 1], qb + p.NQ);
    if (qb <= 0 && qe > 0) slot_row = -qb;
  }

  float m = -INFINITY, l = 0.0f, a = 0.0f;   // a: lane s < S merges span s
  float o[E];
#pragma unroll
  for (int e = 0; e < E; ++e) o[e] = 0.0f;
  if (live) {
    const size_t rstride = (size_t)p.Hq * C::PSTR;
    const float* rec0 = p.partials + ((size_t)sd.x * p.Hq + head) * C::PSTR;
    auto merge = [&](auto in_flight) {
      constexpr int kInFlight = decltype(in_flight)::value;
      for (int c = part; c < count; c += kInFlight * WPH) {
        float v[kInFlight][E], sp[kInFlight], rm[kInFlight], rl[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
          const float* r = rec0 + (size_t)min(c + u * WPH, count - 1) * rstride;
#pragma unroll
          for (int e = 0; e < E; ++e) v[u][e] = r[E * lane + e];
          sp[u] = (lane < kMaxSpans) ? r[D + 2 + lane] : 0.0f;
          rm[u] = c + u * WPH < count ? r[D] : -INFINITY;
          rl[u] = r[D + 1];
        }
        float mn = m;
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) mn = fmaxf(mn, rm[u]);
        const float keep = fast_exp2(m - mn);        // mn is finite: record c exists
        m = mn;
        l *= keep;
        a *= keep;
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] *= keep;
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
          const float wg = fast_exp2(rm[u] - mn);
          l = __builtin_fmaf(wg, rl[u], l);
          a = __builtin_fmaf(wg, sp[u], a);
#pragma unroll
          for (int e = 0; e < E; ++e) o[e] = __builtin_fmaf(wg, v[u][e], o[e]);
        }
      }
    };
    if constexpr (WPH > 1) merge(std::integral_constant<int, 8>{});
    else if (count <= 4) merge(std::integral_constant<int, 4>{});
    else merge(std::integral_constant<int, 16>{});
  }
  if constexpr (WPH > 1) {
    if (lane == 0) { sh_m[wave] = m; sh_l[wave] = l; }
#pragma unroll
    for (int e = 0; e < E; ++e) sh_o[wave][E * lane + e] = o[e];
    if (lane < kMaxSpans) sh_o[wave][D + lane] = a;
    __syncthreads();
    if (part == 0 && live) {
      float mn = m;
#pragma unroll
      for (int k = 1; k < WPH; ++k) mn = fmaxf(mn, sh_m[wave + k]);
      const float keep = fast_exp2(m - mn);
      l *= keep;
      a *= keep;
#pragma unroll
      for (int e = 0; e < E; ++e) o[e] *= keep;
#pragma unroll
      for (int k = 1; k < WPH; ++k) {
        const float wg = fast_exp2(sh_m[wave + k] - mn);
        l = __builtin_fmaf(wg, sh_l[wave + k], l);
        if (lane < kMaxSpans) a = __builtin_fmaf(wg, sh_o[wave + k][D + lane], a);
#pragma unroll
        for (int e = 0; e < E; ++e) o[e] = __builtin_fmaf(wg, sh_o[wave + k][E * lane + e], o[e]);
      }
    }
  }
  if (part == 0) {
    const float inv = 1.0f / l;
    if (live) {
      __bf16* og = static_cast<__bf16*>(p.out) + ((size_t)qrow * p.Hq + head) * D;
      if constexpr (E == 2) reinterpret_cast<uint32_t*>(og)[lane] = pack_bf16(o[0] * inv, o[1] * inv);
      else og[lane] = (__bf16)(o[0] * inv);
    }
    if (pslot >= 0) {
      float* const mass = p.mass + ((size_t)seq * p.P + pslot) * p.NQ * p.S;
      const bool has = live && slot_row >= 0;
      if (has && lane < p.S) mass[slot_row * p.S + lane] = a * inv;
      if (stream && p.plan_fresh) {
        const int lo = has ? slot_row * p.S : 0, hi = has ? lo + p.S : 0;
        for (int e = lane; e < p.NQ * p.S; e += 64)
          if (e < lo || e >= hi) mass[e] = 0.0f;
      }
    }
  }
}

template <int D, int HP>
hipError_t launch_decode_dh(const AttnParams& p, hipStream_t st) {
  if (p.dec_ranges > 0) {
    const long long grid = (long long)p.dec_ranges * p.Hkv * p.dec_hgroups;
    if (!grid_fits(grid)) return hipErrorInvalidValue;
    constexpr int kFew = kStreamSeqs / 64, kMany = kScanMaxSeqs / 64;
    const dim3 g((unsigned)grid);
    if (p.num_seqs > kStreamSeqs) {
      if (p.kv8) hipLaunchKernelGGL((k_decode_stream<D, HP, true, true, kMany>), g, dim3(256), 0, st, p);
      else hipLaunchKernelGGL((k_decode_stream<D, HP, false, lines_always<D, HP, false>(), kMany>), g, dim3(256), 0, st, p);
    } else if (p.kv8) {
      hipLaunchKernelGGL((k_decode_stream<D, HP, true, true, kFew>), g, dim3(256), 0, st, p);
    } else if (lines_always<D, HP, false>() || p.num_seqs <= kLineSeqs) {
      hipLaunchKernelGGL((k_decode_stream<D, HP, false, true, kFew>), g, dim3(256), 0, st, p);
    } else {
      hipLaunchKernelGGL((k_decode_stream<D, HP, false, lines_always<D, HP, false>(), kFew>), g, dim3(256), 0, st, p);
    }
    return hipGetLastError();
  }
  const long long grid = (long long)p.dec_cap * p.Hkv * p.dec_hgroups;
  if (grid <= 0) return hipSuccess;
  if (!grid_fits(grid)) return hipErrorInvalidValue;
  if (p.kv8) hipLaunchKernelGGL((k_decode<D, HP, true>), dim3((unsigned)grid), dim3(256), 0, st, p);
  else hipLaunchKernelGGL((k_decode<D, HP, false>), dim3((unsigned)grid), dim3(256), 0, st, p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_decode_d(const AttnParams& p, hipStream_t st) {
  switch (p.dec_hp) {
    case 8: return launch_decode_dh<D, 8>(p, st);
    case 4: return launch_decode_dh<D, 4>(p, st);
    case 2: return launch_decode_dh<D, 2>(p, st);
    case 1: return launch_decode_dh<D, 1>(p, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_decode(const AttnParams& p, int D, hipStream_t st) {
  if (D == 128) return launch_decode_d<128>(p, st);
  if (D == 64) return launch_decode_d<64>(p, st);
  return hipErrorInvalidValue;
}

hipError_t launch_combine(const AttnParams& p, int D, hipStream_t st) {
  if (p.dec_cap <= 0 || p.num_seqs <= 0) return hipSuccess;
  // as many waves per head as let most sequences' records be fetched in one go: a planned batch has many sequences, and
  // the few that are much longer than the rest have no more waves for their many records; a self-planned sequence has
  // about ranges / num_seqs + 2
  const int per_seq = p.dec_ranges > 0 ? p.dec_ranges / p.num_seqs + 2 : 1;
  const int wph = per_seq > 32 ? 16 : per_seq > 4 ? 4 : 1;
  const int settles = p.dec_ranges > 0 && p.batch_kind == 2 ? 1 : 0;
  const dim3 grid((unsigned)(p.num_seqs + settles), (unsigned)(wph == 1 ? (p.Hq + 3) / 4 : p.Hq));
  if (D == 128 && wph == 16) hipLaunchKernelGGL((k_combine<128, 16>), grid, dim3(1024), 0, st, p);
  else if (D == 128 && wph == 4) hipLaunchKernelGGL((k_combine<128, 4>), grid, dim3(256), 0, st, p);
  else if (D == 128) hipLaunchKernelGGL((k_combine<128, 1>), grid, dim3(256), 0, st, p);
  else if (D == 64 && wph == 16) hipLaunchKernelGGL((k_combine<64, 16>), grid, dim3(1024), 0, st, p);
  else if (D == 64 && wph == 4) hipLaunchKernelGGL((k_combine<64, 4>), grid, dim3(256), 0, st, p);
  else if (D == 64) hipLaunchKernelGGL((k_combine<64, 1>), grid, dim3(256), 0, st, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace hook
