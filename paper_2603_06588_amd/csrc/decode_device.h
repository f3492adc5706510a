// Device code of the split-key decode path (see decode.hip for how it works), shared by the kernels of decode.hip and the
// launch that serves query chunks and single rows together (mixed.hip).
#pragma once

#include "fp8_device.h"
#include "kv_write_device.h"

namespace hook {

namespace {

template <int D>
struct DecodeCfg {
  static constexpr int KSTEPS = D / 32;        // MFMA k-steps
  static constexpr int CHV = D / 8;            // 16-byte chunks per V row
  static constexpr int VK = 64 / CHV;          // V key groups per block (lanes / chunks)
  static constexpr int KPL = kBlock / VK;      // keys per V lane per block (4 or 2)
  static constexpr int PSTR = D + kPartialPad; // floats per partial record
};

// A pointer read through it is not known to point to global memory unless this says so.
template <typename T>
__device__ __forceinline__ T* in_global(T* ptr) {
  return (T*)(__attribute__((address_space(1))) T*)ptr;
}

// Value of `x` in lane H of this lane's group of 16 (a DPP move: no trip through LDS)
template <int H>
__device__ __forceinline__ float row_bcast(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), 0x150 + H, 0xf, 0xf, false));
}

// KV8: the caches hold 8-bit E4M3 bytes ([num_blocks, Hkv, 16, D] bytes), one fp32 scale per kv head.
// The key scale is folded into the softmax scale and the value scale into the partial output, so
// the loop differs from the 16-bit one only in its loads and conversions.
// The keys [kstart, kend) of one sequence for one (kv head, head group): four waves split the cache
// blocks, merge in LDS and leave one partial record per head in slot `item`.
// NewRows: the call brings the new key/value rows of its sequences, and nothing has written them into the cache
// before.  Lane i holds where the row of sequence i goes, so a wave knows of every block it streams which rows
// of it are new - its own sequence's or another's that shares the block - and takes those from k_new / v_new.
// The workgroup of `store` writes its own sequence's row into the cache on the way.
struct NewRows {
  int blk;      // cache block, -1: none
  int at;       // 16 * row of k_new / v_new + place in the block
  bool store;
};
// WHOLE_LINES: how K rows of 128 bytes and more are fetched (below).  Batches that are better off without are
// large and of 256-byte rows for up to four heads: 8 rows 26.4 -> 24.9 us (on caches not seen before 27.8 -> 27.0), 24
// 49.6 -> 48.9, but 64 of 1000-8000 tokens 190 -> 192 and 200 of 1000-4000 (planned) 331 -> 337.  Large ones for groups of 8 go
// either way and keep whole lines: 150 x 100-1000 tokens 85 -> 80, x 500-3000 212 -> 213, x 1000-8000 488 -> 500.
constexpr int kLineSeqs = 32;
template <int D, int HP, bool KV8>
constexpr bool lines_always() { return HP == 8 || KV8 || D == 64; }
template <int D, int HP, bool KV8, bool WHOLE_LINES, int AHEAD>
__device__ __forceinline__ void decode_range(const AttnParams& p, float (&red)[4][HP][DecodeCfg<D>::PSTR], int tid, int lane,
                                             int w, int kvh, int head0, int seq, int qrow, int kstart, int kend,
                                             int item, const NewRows& fresh) {
  using C = DecodeCfg<D>;
  constexpr int NW = 4;
  constexpr int ESZ = KV8 ? 1 : 2;                      // bytes per cache element
  const int blk0 = kstart >> 4;                         // first block of the range inside the sequence
  const int nblk = (kend - kstart + kBlock - 1) / kBlock;
  const int bpw = (nblk + NW - 1) / NW;
  const int b0 = min(w * bpw, nblk), b1 = min(b0 + bpw, nblk);

  const int* const bt = in_global(p.block_table) + (size_t)seq * p.max_blocks + blk0;
  const char* const kbase = static_cast<const char*>(in_global(p.k_cache)) + (size_t)kvh * kBlock * D * ESZ;
  const char* const vbase = static_cast<const char*>(in_global(p.v_cache)) + (size_t)kvh * kBlock * D * ESZ;
  const unsigned blk_bytes = (unsigned)p.Hkv * kBlock * D * ESZ;

  // score-lane role: head j = lane % 16 (real if j < HP), key group kq = lane / 16
  const int j = lane & 15, kq = lane >> 4;
  // K rows of at least a memory line (128 bytes) are fetched a line of eight rows at a time, lane (row lane % 8, 16-byte
  // piece lane / 8).  As the A operand of the score MFMA such a load holds the even pieces of its rows in operand rows
  // 0 .. 7 and the odd ones in 8 .. 15, so Q comes as two sets of columns, 0 .. 7 against the even pieces of a line and
  // 8 .. 15 against the odd ones, and a score is the sum of two accumulator entries (compute_block).  Otherwise operand
  // rows are key rows, and a load takes 64 bytes, half a line, of each of 16 rows.  Whole lines are 2-6 % faster (8 x 2500-4096
  // tokens 26.4 -> 24.9 us, 8-bit 20.0 -> 19.3, 256 x 1000-8192 of 8-bit 431 -> 425, 128 x 1000-4000 at d 64 121 -> 119) but
  // for large streams of 256-byte rows and up to four heads (kLineSeqs), where 1 KB in one piece (4 rows, four classes of
  // pieces) is slower still (64 x 1000-8000 190 -> 194).
  constexpr int ROWB = D * ESZ;
  constexpr bool LINES = WHOLE_LINES && ROWB >= 128;
  const int krow = LINES ? lane & 7 : j, kpiece = LINES ? lane >> 3 : kq;
  const int qhead = LINES ? j & 7 : j;
  // value-lane role: key group vk, 16-byte chunk ch; its keys KPL*vk .. KPL*vk+KPL-1 all
  // belong to score key group (KPL*vk)/4 = lane / 16, so exponentials only move inside a group of 16 lanes
  const int vk = lane / C::CHV, ch = lane % C::CHV;

  // everything that does not depend on block ids is requested together with the first of them: block
  // ids (64 to a register, one per lane), query rows, probed heads
  auto load_ids = [&](int first) {
    const int blk = bt[min(first + lane, nblk - 1)];
    return ((unsigned)blk < (unsigned)p.num_blocks) ? blk : 0;
  };
  int ids = load_ids(b0), ids_next = 0;
  if (bpw > 64) ids_next = load_ids(b0 + 64);
  int qb = 0, qe = 0, ph0 = -1;
  if (p.P > 0) {
    qb = cload(p.query_sel, 2 * seq);
    qe = min(cload(p.query_sel, 2 * seq + 1), qb + p.NQ);
    if (lane < p.P) ph0 = in_global(p.probe_heads)[lane];
  }
  // the contraction may take the dimensions in any order as long as both operands agree: a 16-bit piece is one k-step of
  // eight dimensions, an 8-bit one (16 dimensions) two
  constexpr int NQF = LINES ? D / 64 : C::KSTEPS;
  bf16x8 qf[NQF];
#pragma unroll
  for (int s = 0; s < NQF; ++s) {
    uint4 v = make_uint4(0, 0, 0, 0);
    const int dim0 = KV8 ? 16 * (LINES ? 2 * kq + (j >> 3) : kq) + 8 * s
                         : LINES ? 64 * s + 16 * kq + 8 * (j >> 3) : 32 * s + 8 * kq;
    if (qhead < HP)
      v = *reinterpret_cast<const uint4*>(static_cast<const __bf16*>(in_global(p.q)) + ((size_t)qrow * p.Hq + head0 + qhead) * D + dim0);
    __builtin_memcpy(&qf[s], &v, 16);
  }

  // 16-byte pieces per lane and block: K rows for the score MFMA, V rows for P V (8-bit V: 8 bytes)
  constexpr int kKr = kBlock * ROWB / 1024;
  struct Block { uint4 k[kKr]; uint4 v[C::KPL]; int id; };
  const unsigned koff = (unsigned)krow * ROWB + 16 * kpiece;
  // load s: rows 8 (s / LPR) .., line s % LPR (the lines of a row one after the other); or 64 bytes of all rows
  constexpr int LPR = LINES ? ROWB / 128 : kKr;
  auto k_at = [](int s) { return (unsigned)(LINES ? 8 * (s / LPR) * ROWB + 128 * (s % LPR) : 64 * s); };
  const unsigned voff = (unsigned)(C::KPL * vk) * D * ESZ + 8 * ESZ * ch;
  // Rows past the last token lie in a block the sequence owns, and what they hold (anything, NaN included) is
  // replaced before use in the range's last block.  Loads are always issued, so that the compiler knows how
  // many are outstanding at a wait; past the wave's last block all lanes fetch the same 16 bytes.
  auto load_block = [&](int b, Block& d) {
    d.id = __builtin_amdgcn_readlane(ids, (b - b0) & 63);
    const unsigned long long off = (unsigned long long)(unsigned)d.id * blk_bytes;
    global_bytes kb = (global_bytes)(kbase + off), vb = (global_bytes)(vbase + off);
    unsigned ko = b < b1 ? koff : 0, vo = b < b1 ? voff : 0;     // (opaque, so that the loads take a scalar base and a 32-bit lane offset)
    asm("" : "+v"(ko), "+v"(vo));
#pragma unroll
    for (int s = 0; s < kKr; ++s) d.k[s] = load_stream16(kb + ko + k_at(s));
#pragma unroll
    for (int i = 0; i < C::KPL; ++i) {
      if constexpr (KV8) {
        const uint2 v = load_stream8(vb + vo + i * D);
        d.v[i] = make_uint4(v.x, v.y, 0, 0);
      } else {
        d.v[i] = load_stream16(vb + vo + i * D * 2);
      }
    }
  };
  constexpr int RING = AHEAD + 1;
  static_assert(64 % RING == 0, "a turn of the ring ends with a register of ids");
  Block ring[RING];
  if (b0 < b1) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) load_block(b0 + u, ring[u]);
  }

  // probe set-up: per score lane (its head), spans uniform.  The single row t = 0 is selected when
  // begin <= 0 < min(end, begin + NQ); its slot is -begin
  int sp_a[kMaxSpans], sp_b[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) { sp_a[s] = 0; sp_b[s] = 0; }
  bool lane_probe = false;
  const bool any_probe = p.P > 0 && qb <= 0 && qe > 0;
  if (any_probe) {
    load_spans_uniform(p.key_spans, seq, p.S, sp_a, sp_b);
    // is head0 + h probed?  The list is read 64 entries at a time, one per lane, and matched
    // with a ballot, so the answer costs one load instead of a search per head
    for (int i0 = 0; i0 < p.P; i0 += 64) {
      const int ph = i0 == 0 ? ph0 : (i0 + lane < p.P) ? in_global(p.probe_heads)[i0 + lane] : -1;
#pragma unroll
      for (int h = 0; h < HP; ++h) {
        const bool hit = __builtin_amdgcn_ballot_w64(ph == head0 + h) != 0;
        if (j == h) lane_probe = lane_probe || hit;
      }
    }
  }

  float m_run = -INFINITY, l_run = 0.0f;
  float am[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) am[s] = 0.0f;
  float acc[HP][8];
#pragma unroll
  for (int h = 0; h < HP; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[h][e] = 0.0f;
  const float c = KV8 ? p.scale_log2 * cloadf(p.k_scale, kvh) : p.scale_log2;

  auto compute_block = [&](int b, Block& d) {
    const int key0 = kstart + b * kBlock;
    const bool last = key0 + kBlock >= kend;     // uniform
    for (unsigned long long hit = __builtin_amdgcn_ballot_w64(fresh.blk == d.id); hit != 0; hit &= hit - 1) {
      const int owner = __builtin_ctzll(hit), at = __builtin_amdgcn_readlane(fresh.at, owner), r = at & 15;
      const bool store = fresh.store && owner == seq;
      const size_t row = ((size_t)(at >> 4) * p.Hkv + kvh) * D * 2, off = (size_t)(unsigned)d.id * blk_bytes;
      global_bytes kn = (global_bytes)(unsigned long long)(size_t)p.kvw.k_new + row;
      global_bytes vn = (global_bytes)(unsigned long long)(size_t)p.kvw.v_new + row;
      char* kdst = const_cast<char*>(kbase) + off;
      char* vdst = const_cast<char*>(vbase) + off;
      // 16-bit rows are requested straight into the block's registers and stored once all of them are there
#pragma unroll
      for (int s = 0; s < kKr; ++s) {
        if (krow + 8 * (s / LPR) == r) {
          if constexpr (KV8) {
            const uint4 a = load_global16(kn + 32 * kpiece), b = load_global16(kn + 32 * kpiece + 16);
            const float sc = cloadf(p.k_scale, kvh);
            const uint2 lo = quantize_chunk_e4m3(a, sc), hi = quantize_chunk_e4m3(b, sc);
            d.k[s] = make_uint4(lo.x, lo.y, hi.x, hi.y);
          } else {
            d.k[s] = load_global16(kn + (LINES ? 128 : 64) * (s % LPR) + 16 * kpiece);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < C::KPL; ++i) {
        if (C::KPL * vk + i == r) {
          d.v[i] = load_global16(vn + 16 * ch);
          if constexpr (KV8) {
            const uint2 v = quantize_chunk_e4m3(d.v[i], cloadf(p.v_scale, kvh));
            d.v[i] = make_uint4(v.x, v.y, 0, 0);
          }
        }
      }
      // (and the blocks without a new row wait for their own loads only)
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0)
      __builtin_amdgcn_sched_barrier(0);
      if (store) {
#pragma unroll
        for (int s = 0; s < kKr; ++s)
          if (krow + 8 * (s / LPR) == r) *reinterpret_cast<uint4*>(kdst + koff + k_at(s)) = d.k[s];
#pragma unroll
        for (int i = 0; i < C::KPL; ++i) {
          if (C::KPL * vk + i == r) {
            if constexpr (KV8) *reinterpret_cast<uint2*>(vdst + voff + i * D) = make_uint2(d.v[i].x, d.v[i].y);
            else *reinterpret_cast<uint4*>(vdst + voff + i * D * 2) = d.v[i];
          }
        }
      }
    }
    if (last) {
#pragma unroll
      for (int i = 0; i < C::KPL; ++i)           // 0 * NaN would poison the output
        if (key0 + C::KPL * vk + i >= kend) d.v[i] = make_uint4(0, 0, 0, 0);
    }
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 sacc[2] = {zero, zero};          // rows 0 .. 7 and 8 .. 15 (LINES)
#pragma unroll
    for (int s = 0; s < kKr * (KV8 ? 2 : 1); ++s) {
      const uint4& w = d.k[KV8 ? s >> 1 : s];
      bf16x8 a;
      if constexpr (KV8) {
        // bytes 8 (s % 2) .. 8 (s % 2) + 7 of piece s / 2
        const uint4 cv = e4m3x8_to_bf16x8((s & 1) ? make_uint2(w.z, w.w) : make_uint2(w.x, w.y));
        __builtin_memcpy(&a, &cv, 16);
      } else {
        __builtin_memcpy(&a, &w, 16);
      }
      const int half = !LINES ? 0 : KV8 ? s >> 1 : s / LPR;
      sacc[half] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[KV8 ? s & 1 : s % LPR], sacc[half], 0, 0, 0);
    }
    // lane (j, kq): tt[r] = score of head j with key key0 + 4 kq + r.  LINES: entry (row i, column n) of a half holds the
    // even pieces of row i where i < 8 and n < 8 and the odd ones of row i - 8 where both are 8 or more; one swap of lane
    // halves brings the rows of both halves into place, and the odd pieces come from eight columns on.  (Lanes j >= 8 are left with
    // products of unlike pieces, for which no head asks.  They keep references of their own; one that rises sends the
    // wave through the raise below, where lanes that do not rise multiply by 1.)
    float tt[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float score = sacc[0][r];
      if constexpr (LINES) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(sacc[0][r]), __float_as_uint(sacc[1][r]), false, false);
        score = __uint_as_float(x[0]) + __uint_as_float(__builtin_amdgcn_update_dpp(0u, x[1], 0x128, 0xf, 0xf, false));   // row_ror:8
      }
      tt[r] = score * c;
    }
    if (last) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (key0 + 4 * kq + r >= kend) tt[r] = -INFINITY;
    }
    const float bm = fmaxf(fmaxf(tt[0], tt[1]), fmaxf(tt[2], tt[3]));
    const bool upd = bm > m_run + kLazyTau;
    if (__builtin_amdgcn_ballot_w64(upd) != 0) {
      const float alpha = upd ? fast_exp2(m_run - bm) : 1.0f;
      m_run = upd ? bm : m_run;
      l_run *= alpha;
#pragma unroll
      for (int s = 0; s < kMaxSpans; ++s) am[s] *= alpha;
      static_for<HP>([&](auto h) {
        const float ah = row_bcast<decltype(h)::value>(alpha);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[decltype(h)::value][e] *= ah;
      });
    }
    const float m_safe = (m_run == -INFINITY) ? 0.0f : m_run;
    float pr[4];
    float psum = 0.0f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pr[r] = fast_exp2(tt[r] - m_safe);
      psum += pr[r];
    }
    l_run += psum;
    if (any_probe) {
#pragma unroll
      for (int s = 0; s < kMaxSpans; ++s) {
        if (s < p.S) {
          const int a = sp_a[s], bnd = sp_b[s];
          if (bnd > key0 && a < key0 + kBlock) {
            float add = 0.0f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int key = key0 + 4 * kq + r;
              add += (key >= a && key < bnd) ? pr[r] : 0.0f;
            }
            am[s] += lane_probe ? add : 0.0f;
          }
        }
      }
    }
    // P V on the value lanes
#pragma unroll
    for (int i = 0; i < C::KPL; ++i) {
      const uint4 v = d.v[i];
      float vf[8];
      if constexpr (KV8) {
        const f32x2 a0 = __builtin_amdgcn_cvt_pk_f32_fp8(v.x, false), a1 = __builtin_amdgcn_cvt_pk_f32_fp8(v.x, true);
        const f32x2 a2 = __builtin_amdgcn_cvt_pk_f32_fp8(v.y, false), a3 = __builtin_amdgcn_cvt_pk_f32_fp8(v.y, true);
        vf[0] = a0[0]; vf[1] = a0[1]; vf[2] = a1[0]; vf[3] = a1[1];
        vf[4] = a2[0]; vf[5] = a2[1]; vf[6] = a3[0]; vf[7] = a3[1];
      } else {
        vf[0] = bf16_lo(v.x); vf[1] = bf16_hi(v.x);
        vf[2] = bf16_lo(v.y); vf[3] = bf16_hi(v.y);
        vf[4] = bf16_lo(v.z); vf[5] = bf16_hi(v.z);
        vf[6] = bf16_lo(v.w); vf[7] = bf16_hi(v.w);
      }
      // the exponential of this lane's key i sits in register i (four keys per lane), or in register
      // 2 (vk % 2) + i (two keys per lane)
      static_for<HP>([&](auto h) {
        float phv;
        if constexpr (C::KPL == 4) {
          phv = row_bcast<decltype(h)::value>(pr[i]);
        } else {
          const float lo = row_bcast<decltype(h)::value>(pr[i]);
          const float hi = row_bcast<decltype(h)::value>(pr[(2 + i) & 3]);
          phv = (vk & 1) ? hi : lo;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[decltype(h)::value][e] = __builtin_fmaf(phv, vf[e], acc[decltype(h)::value][e]);
      });
      __builtin_amdgcn_sched_barrier(0);   // one key's widened values at a time
    }
  };

  // stream this wave's blocks with the next blocks' loads in flight during the arithmetic on this one
  for (int b = b0; b < b1; b += RING) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      if (u == 1) {
        if (((b + RING - b0) & 63) == 0) {      // the next 64 block ids
          ids = ids_next;
          ids_next = load_ids(b + RING + 64);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      load_block(b + u + AHEAD, ring[(u + AHEAD) % RING]);
      __builtin_amdgcn_sched_barrier(0);
      if (u == 0 || b + u < b1) compute_block(b + u, ring[u]);
      if (u != 0) __builtin_amdgcn_sched_barrier(0);
    }
  }

  // merge the key-group streams of this wave
  float m_w = fmaxf(m_run, __shfl_xor(m_run, 16));
  m_w = fmaxf(m_w, __shfl_xor(m_w, 32));
  const float wgt = (m_run == -INFINITY) ? 0.0f : fast_exp2(m_run - m_w);
  float l_w = l_run * wgt;
  l_w += __shfl_xor(l_w, 16);
  l_w += __shfl_xor(l_w, 32);
  float am_w[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) {
    float v = am[s] * wgt;
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    am_w[s] = v;
  }
  static_for<HP>([&](auto h) {
    const float wh = row_bcast<decltype(h)::value>(wgt);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float v = acc[decltype(h)::value][e] * wh;
      if constexpr (C::VK == 8) v += __shfl_xor(v, 8);
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      acc[decltype(h)::value][e] = v;
    }
  });
  // lanes with vk == 0 hold o[h][8 ch + e]; score lanes with kq == 0 hold (m, l, a) of head j
  if (vk == 0) {
#pragma unroll
    for (int h = 0; h < HP; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) red[w][h][8 * ch + e] = acc[h][e];
  }
  if (kq == 0 && j < HP) {
    red[w][j][D] = m_w;
    red[w][j][D + 1] = l_w;
#pragma unroll
    for (int s = 0; s < kMaxSpans; ++s) red[w][j][D + 2 + s] = am_w[s];
  }
  __syncthreads();

  // merge the 4 waves and write one partial record per head
  const float vscale = KV8 ? cloadf(p.v_scale, kvh) : 1.0f;
  for (int idx = tid; idx < HP * C::PSTR; idx += 256) {
    const int h = idx / C::PSTR, col = idx % C::PSTR;
    float mm = red[0][h][D];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) mm = fmaxf(mm, red[ww][h][D]);
    float out = 0.0f;
    if (col == D) {
      out = mm;
    } else if (col < D + 2 + kMaxSpans) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const float mw = red[ww][h][D];
        const float e = (mw == -INFINITY) ? 0.0f : fast_exp2(mw - mm);
        out += e * red[ww][h][col];
      }
      if (KV8 && col < D) out *= vscale;
    }
    in_global(p.partials)[((size_t)item * p.Hq + head0 + h) * C::PSTR + col] = out;
  }
}

// What a batch of single rows looks like to the kernel that plans itself: cache blocks of sequence i to
// stream, 0 where there is nothing to compute.
struct DecodeSeq { int L, qrow, nblk, bits; };

__device__ __forceinline__ DecodeSeq decode_seq(const AttnParams& p, int Lraw, int r0, int r1) {
  const int max_ctx = p.max_blocks * kBlock, n = r1 - r0;
  DecodeSeq s = {min(Lraw, max_ctx), r0, 0, 0};
  if (Lraw < 0 || n < 0) { s.bits = kStatNegative; return s; }
  if (Lraw > max_ctx) s.bits |= kStatLenClamped;
  if (n > s.L) s.bits |= kStatQGtL;
  else if (r0 < 0 || r0 + n > p.total_q) s.bits |= kStatNegative;
  else if (n > 1) s.bits |= p.batch_kind == 2 ? kStatHint : 0;   // a row block (in a batch promised to hold single rows)
  else if (n == 1) s.nblk = (s.L + kBlock - 1) / kBlock;
  return s;
}

// A batch of single rows that plans itself.  The cache blocks of all its sequences, laid end to end, are cut
// into p.dec_ranges equal ranges (one resident round of workgroups per kv head and head group), so every
// workgroup streams the same number of blocks however ragged the contexts are; a range may cover the end of
// one sequence and the beginning of the next.  A workgroup finds its range by a scan over the lengths (each
// wave on its own, lane l takes sequences l K .. l K + K - 1), which costs about a microsecond instead of a
// planning launch (8 us in a kernel trace).  Range g and sequence i share at most one piece and the path through the pairs is a
// staircase, so g + i numbers the partial records without gaps between the records of one sequence.
// A piece costs a workgroup its start-up (ids, query, first keys, merge), so where whole sequences can be dealt
// out to the ranges with hardly more blocks each, no range covers two: a sequence then takes its blocks divided by
// `bpr` ranges, rounded up, which fits while bpr is at least total / (ranges - sequences).  kPieceBlocks is about
// what a second piece costs in blocks.
// SHARED_LAUNCH: row blocks in the same launch may call for fewer ranges than there are workgroups (dec_few; the last of them find
// nothing to do).
// PER_LANE: sequences that a lane has room for (with room for kScanMaxSeqs in every batch 1 x 1237 tokens take 11.13 instead
// of 10.98 us).
constexpr int kPieceBlocks = 4;

template <int PER_LANE>
struct BlockScan {
  int K;                        // sequences per lane
  int nblk[PER_LANE];           // blocks of this lane's sequences
  int L[PER_LANE], qrow[PER_LANE];
  int excl;                     // blocks in front of this lane's first sequence
  int total;                    // blocks of the batch
  int bpr;                      // blocks per range
  bool whole;                   // ranges end with their sequence
  int bits;                     // status bits of this lane's sequences
};

template <int PER_LANE, bool SHARED_LAUNCH>
__device__ __forceinline__ BlockScan<PER_LANE> scan_blocks(const AttnParams& p, int lane) {
  BlockScan<PER_LANE> sc;
  sc.K = (p.num_seqs + 63) >> 6;
  sc.bits = 0;
  int sum = 0;
#pragma unroll
  for (int u = 0; u < PER_LANE; ++u) {
    sc.nblk[u] = sc.L[u] = sc.qrow[u] = 0;
    const int i = lane * sc.K + u;
    if (u < sc.K && i < p.num_seqs) {
      const DecodeSeq s = decode_seq(p, p.seq_lens[i], p.cu_q_lens[i], p.cu_q_lens[i + 1]);
      sc.nblk[u] = s.nblk;
      sc.L[u] = s.L;
      sc.qrow[u] = s.qrow;
      sc.bits |= s.bits;
    }
    sum += sc.nblk[u];
  }
  const int incl = wave_scan(sum);
  sc.excl = incl - sum;
  sc.total = __builtin_amdgcn_readlane(incl, 63);
  int ranges = p.dec_ranges;
  if (SHARED_LAUNCH && p.dec_few > 0 && (long long)kRowsWeigh * (p.total_q - p.num_seqs) >= sc.total) ranges = p.dec_few;
  sc.bpr = max((sc.total + ranges - 1) / ranges, kStreamMinBlocks);
  const int spare = ranges - p.num_seqs;
  const int bpr_whole = spare > 0 ? max((sc.total + spare - 1) / spare, kStreamMinBlocks) : 0;
  sc.whole = spare > 0 && bpr_whole <= sc.bpr + kPieceBlocks;
  if (sc.whole) sc.bpr = bpr_whole;
  return sc;
}

// The work of workgroup `bid`.  AHEAD: blocks requested ahead of the one being computed.
template <int D, int HP, bool KV8, bool WHOLE_LINES, int PER_LANE, int AHEAD, bool SHARED_LAUNCH>
__device__ __forceinline__ void stream_range(const AttnParams& p, float (&red)[4][HP][DecodeCfg<D>::PSTR], int bid) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kvh = bid % p.Hkv;
  const int rest = bid / p.Hkv;
  const int hg = rest % p.dec_hgroups;
  const int g = rest / p.dec_hgroups;

  const BlockScan<PER_LANE> sc = scan_blocks<PER_LANE, SHARED_LAUNCH>(p, lane);

  // where the new rows go (at most one sequence per lane: dec_write).  A length beyond the block table is clamped, so
  // its new row has no place in the cache.
  NewRows fresh = {-1, 0, hg == 0};
  if (p.dec_write) {
    if (sc.nblk[0] > 0 && !(sc.bits & kStatLenClamped)) {
      const int blk = p.block_table[(size_t)lane * p.max_blocks + ((sc.L[0] - 1) >> 4)];
      fresh.blk = (unsigned)blk < (unsigned)p.num_blocks ? blk : -1;
      fresh.at = 16 * sc.qrow[0] + ((sc.L[0] - 1) & 15);
    }
    // Rows of a sequence that contradicts the hint are nobody's to store on the way: every workgroup writes all rows
    // (the same bytes) before it reads.
    if (__builtin_amdgcn_ballot_w64((sc.bits & kStatHint) != 0) != 0) {
      for (int t = 0; t * kKvRowTile < p.total_q; ++t)
        kv_write_tile<256, 1>(p.kvw, t, tid, reinterpret_cast<long long*>(&red[0][0][0]), p.kvw.cu_q_lens);
      __threadfence();
      __syncthreads();
    }
  }

  // the sequence that the range begins in, and its place there: by blocks, or by ranges where those end with
  // their sequence
  int at = g * sc.bpr, excl = sc.excl, total = sc.total;
  int size[PER_LANE];
#pragma unroll
  for (int u = 0; u < PER_LANE; ++u) size[u] = sc.nblk[u];
  if (sc.whole) {
    int sum = 0;
#pragma unroll
    for (int u = 0; u < PER_LANE; ++u) {
      if (u < sc.K) size[u] = (sc.nblk[u] + sc.bpr - 1) / sc.bpr;      // (uniform: few sequences, few divisions)
      sum += size[u];
    }
    const int incl = wave_scan(sum);
    at = g;
    excl = incl - sum;
    total = __builtin_amdgcn_readlane(incl, 63);
  }
  if (at >= total) return;
  int seq, o, L, qrow;
  {
    int my_seq = 0, my_o = 0, my_L = 0, my_row = 0, start = excl;
#pragma unroll
    for (int u = 0; u < PER_LANE; ++u) {
      if (at >= start && at < start + size[u]) {
        my_seq = lane * sc.K + u;
        my_o = (at - start) * (sc.whole ? sc.bpr : 1);
        my_L = sc.L[u];
        my_row = sc.qrow[u];
      }
      start += size[u];
    }
    const int from = __builtin_ctzll(__builtin_amdgcn_ballot_w64(at >= excl && at < start));
    seq = __builtin_amdgcn_readlane(my_seq, from);
    o = __builtin_amdgcn_readlane(my_o, from);
    L = __builtin_amdgcn_readlane(my_L, from);
    qrow = __builtin_amdgcn_readlane(my_row, from);
  }
  // [x, x1): the range's blocks, counted from any origin
  int x = sc.whole ? o : at;
  const int x1 = sc.whole ? min((L + kBlock - 1) / kBlock, o + sc.bpr) : min(total, at + sc.bpr);
  const int head0 = kvh * p.G + hg * HP;
  for (;;) {
    const int take = min((L + kBlock - 1) / kBlock - o, x1 - x);
    const int kend = min(L, (o + take) * kBlock);
    // Arguments and lane number are made opaque per piece: otherwise everything derived from them is kept in
    // registers across the loop (60 vector registers spilled instead of a few instructions repeated).
    const AttnParams& pp = reread_arguments();
    int ln = lane;
    asm volatile("" : "+v"(ln));
    decode_range<D, HP, KV8, WHOLE_LINES, AHEAD>(pp, red, w * 64 + ln, ln, w, kvh, head0, seq, qrow, o * kBlock, kend, g + seq, fresh);
    // where the merge kernel finds the sequence's records
    if (o == 0 && kvh == 0 && hg == 0 && tid == 0)
      p.seq_dec[seq] = make_int2(g + seq, sc.whole ? ((L + kBlock - 1) / kBlock + sc.bpr - 1) / sc.bpr
                                                   : (x + (L + kBlock - 1) / kBlock - 1) / sc.bpr - g + 1);
    x += take;
    if (x >= x1) break;
    __syncthreads();      // `red` is written again
    DecodeSeq s;
    do {
      ++seq;
      s = decode_seq(p, cload(p.seq_lens, seq), cload(p.cu_q_lens, seq), cload(p.cu_q_lens, seq + 1));
    } while (s.nblk == 0 && seq + 1 < p.num_seqs);
    if (s.nblk == 0) break;     // (never: x < total says that there is one)
    o = 0;
    L = s.L;
    qrow = s.qrow;
  }
}

}  // namespace

}  // namespace hook
