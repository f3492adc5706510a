// Tiled causal attention for query chunks (n_i >= 2), bf16 MFMA, head_dim 64 and 128, 16-bit and 8-bit caches.
//
// Workgroup = 4 waves = (hpw q heads of one kv head) x (4 / hpw blocks of 32 query rows),
// all sharing the K/V tiles (64 keys = 4 cache blocks) of their kv head.  Data movement is built around two
// gfx950 features:
//   * K and V go from the paged cache straight into LDS with 16-byte direct-to-LDS loads, so staging
//     costs no vector registers and almost no vector ALU work.  Wave w fetches cache block w of every
//     tile: the block of a kv head is one contiguous run, so one block id, one 64-bit address and
//     16 D bytes / 1 KB load instructions with constant offsets do it.  16-byte chunks are XOR-swizzled inside
//     each LDS row so that the MFMA operand reads below are free of bank conflicts although rows are
//     unpadded;
//   * V stays in its natural [key][dim] layout and is read TRANSPOSED with
//     ds_read_b64_tr_b16, which hands each lane four consecutive keys of one output
//     dimension - the A operand of O^T = V^T P^T.
//
// Per wave the score tile is computed transposed, S^T = K Q^T (32x32x16 MFMA, keys = M,
// queries = N): lane l owns query l % 32 and 16 keys per 32-key block, so softmax row
// statistics are in-lane reductions plus one exchange between lane halves, and the
// exponentials, rounded to bf16, already form the B operand of the second MFMA.
//
// The loop is software pipelined inside each wave: while the vector ALUs run the softmax
// of tile t, the matrix cores compute the scores of tile t+1 (the two instruction streams
// are interleaved explicitly), then P V of tile t follows.  K tiles are fetched two tiles
// ahead and V tiles one tile ahead, which makes one workgroup barrier per tile sufficient
// with two LDS buffers each.
//
// 8-bit caches (KV8): the bytes go direct to LDS too, one tile earlier, into a staging area of each wave's own
// (2 x 16 D bytes); in the P V stage of the tile before they are needed the wave reads its block back, widens it
// to bf16 (exact: every E4M3 number is a bf16 number) and writes it to the same swizzled buffers as
// above, so the rest of the loop is the 16-bit one and every byte is widened once for the four heads
// that share it.  The key scale goes into the softmax scale, the value scale into the normalisation of `out`.
//
// Probe span sums are taken from the fp32 exponentials under the same running reference
// as the normaliser and divided by it at the end: the captured mass is the exact softmax
// mass of the row.  Waves that probe run a second instantiation of the same loop whose
// arithmetic for `out` is identical.
#include "fp8_device.h"
#include "hook_device.h"

namespace hook {

namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));

template <int D, bool KV8>
struct Cfg {
  static constexpr int RB = 2 * D;                          // bytes of one key row in the bf16 LDS buffers
  static constexpr int TILE = kTileKeys * RB;
  static constexpr int KSTEPS = D / 16;                     // MFMA k-steps of the scores
  static constexpr int MB = D / 32;                         // 32-dimension blocks of the output
  static constexpr int BLK = kBlock * D * (KV8 ? 1 : 2);    // bytes of one (cache block, kv head) run
  static constexpr int NI = BLK / 1024;                     // load instructions per run
  static constexpr int RPI = kBlock / NI;                   // rows per load instruction
  static constexpr int LPR = 64 / RPI;                      // lanes (16-byte pieces) per row
  static constexpr int STAGE = KV8 ? 2 * BLK : 0;           // staging bytes per wave: K run, V run
  static constexpr int LDS = 4 * TILE + 4 * STAGE;          // K[2], V[2], staging
  static constexpr int CH = D / 8;                          // 16-byte chunks per bf16 row
};

// Swizzle of the 16-byte chunks of LDS row r (what a chunk index is XORed with): the 16 rows a K read touches
// and the four rows a transposed V read touches then lie in different banks (64 banks of 4 bytes; a row is
// all of them at D = 128 and half of them at D = 64).
template <int D> __device__ __forceinline__ int k_swizzle(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D> __device__ __forceinline__ int v_swizzle(int r) { return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); }

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 16-byte direct-to-LDS load: lane i's data lands at lds + OFF + 16 * i, from base + OFF + its own offset.
// Written as assembly so that its completion is tracked only by the explicit vmcnt waits; the compiler would
// otherwise make every later LDS read wait for the load.
template <int OFF>
__device__ __forceinline__ void dma16(unsigned long long base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
               :: "s"(lds_addr), "v"(voff), "s"(base), "n"(OFF) : "memory", "m0");
}

struct WaveCtx {
  // loop-invariant per-lane / per-wave values
  unsigned k_read_addr;   // LDS byte offset of this lane's K row with its swizzle term folded in
  unsigned v_read_addr;   // same for the transposed V reads
  int hf, qi;
  int pos;                // causal horizon of this lane's query row
  float c;                // scale * log2(e)
  int S;                  // number of spans
  // direct-to-LDS fetches
  unsigned long long kbase, vbase;   // cache + kv-head offset
  unsigned lds_base;      // LDS address of the buffers
  unsigned blk_bytes;     // bytes per cache block (all kv heads)
  int num_blocks;
  unsigned k_off, v_off;  // this lane's source offset in a run (first load instruction)
  int L, last_blk, w, lane;
};

// lane l and lane l ^ 32 hold the two key halves of one query: maximum over both (one swap between
// the lane halves instead of a round trip through LDS)
__device__ __forceinline__ float half_max(float mx) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// mask (optional) and row maximum of a raw score tile; both lane halves end up with the same value
template <bool MASK>
__device__ __forceinline__ float tile_max(const WaveCtx& cx, int key0, f32x16 (&S)[2]) {
  if constexpr (MASK) {
#pragma unroll
    for (int kbk = 0; kbk < 2; ++kbk)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = key0 + 32 * kbk + 8 * (r >> 2) + 4 * cx.hf + (r & 3);
        if (key > cx.pos) S[kbk][r] = -INFINITY;
      }
  }
  float m0 = fmaxf(S[0][0], S[0][1]), m1 = fmaxf(S[1][0], S[1][1]);
#pragma unroll
  for (int r = 2; r < 16; r += 2) {
    m0 = fmaxf(m0, fmaxf(S[0][r], S[0][r + 1]));
    m1 = fmaxf(m1, fmaxf(S[1][r], S[1][r + 1]));
  }
  return half_max(fmaxf(m0, m1));
}

// Block ids of 64 consecutive blocks (16 tiles) live in one register per lane; two registers
// cover the group being consumed and the next one.  They are kept as they come (ids outside the cache are
// replaced by block 0 when one is used), so that nothing waits for them before that.
struct BlockIds {
  int grp;
  int cur, nxt;
};

__device__ __forceinline__ int load_ids(const int* bt, int first, int lane, int last_blk) {
  return bt[min(first + lane, last_blk)];
}

// byte offset of a block in the cache
__device__ __forceinline__ unsigned long long block_bytes(const WaveCtx& cx, int blk) {
  return (unsigned long long)((unsigned)blk < (unsigned)cx.num_blocks ? (unsigned)blk : 0u) * cx.blk_bytes;
}

// the same for this wave's block of a tile (past the last block: the last block again)
__device__ __forceinline__ unsigned long long block_offset(const WaveCtx& cx, int sel, int tile) {
  const int bidx = min(4 * tile + cx.w, cx.last_blk);      // same 64-block group as block 4 * tile
  return block_bytes(cx, __builtin_amdgcn_readlane(sel, bidx & 63));
}

// Load instruction J of this wave's K run.  A K row past the last token may hold anything: it only
// produces scores of keys beyond every row's horizon, which are overwritten with -inf before use, and
// it still lies inside a block the sequence owns.
template <int D, bool KV8, int J>
__device__ __forceinline__ void fetch_k(const WaveCtx& cx, unsigned long long boff, unsigned lds) {
  // (the swizzle of rows RPI J .. differs from that of the first rows by bit 2 of the chunk index times J)
  unsigned off = cx.k_off;
  if constexpr (!KV8 && J > 0) {
    asm("" : "+v"(off));      // computed here and not kept in a register of its own across the loop
    off ^= 64u * J;
  }
  dma16<1024 * J>(cx.kbase + boff, off, lds);
}

// Load instruction J of this wave's V run.  CLAMP: rows past the last token re-read the last valid row of the
// last block - P is 0 there, and 0 * NaN would poison the output - so a lane's source row may differ from the
// row its data is meant for.
template <int D, bool KV8, int J, bool CLAMP>
__device__ __forceinline__ void fetch_v(const WaveCtx& cx, unsigned long long boff, int tile, unsigned lds) {
  using C = Cfg<D, KV8>;
  if constexpr (CLAMP) {
    int ln = cx.lane;
    asm("" : "+v"(ln));       // likewise
    const int r = C::RPI * J + ln / C::LPR;
    const int rmax = cx.L - 1 - kBlock * min(4 * tile + cx.w, cx.last_blk);      // >= 0
    const unsigned row_bytes = C::BLK / kBlock;
    dma16<0>(cx.vbase + boff, cx.v_off + (unsigned)(min(r, rmax) - ln / C::LPR) * row_bytes, lds + 1024 * J);
  } else {
    dma16<1024 * J>(cx.vbase + boff, cx.v_off, lds);
  }
}

template <int D>
__device__ __forceinline__ bf16x8 read_k(const WaveCtx& cx, const unsigned char* kb, int s, int kbk) {
  const unsigned a = cx.k_read_addr ^ (32u * s);
  return *reinterpret_cast<const bf16x8*>(kb + a + kbk * 32 * 2 * D);
}

template <int D>
__device__ __forceinline__ bf16x8 read_vt(const WaveCtx& cx, const unsigned char* vb, int m, int mb) {
  const unsigned a = (cx.v_read_addr ^ (64u * mb)) + (16 * m) * 2 * D;
  union { v4i16 h[2]; bf16x8 v; } av;
  av.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(vb + a));
  av.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(vb + a + 8 * 2 * D));
  return av.v;
}

// 8-bit caches: half of a 16-byte piece of this wave's staged run - eight bytes of row `r`, chunk `ch` - widened into
// an LDS buffer row
template <int D>
__device__ __forceinline__ void widen_to(unsigned char* buf, int r, int ch, int swz, unsigned lo, unsigned hi) {
  *reinterpret_cast<uint4*>(buf + r * 2 * D + ((ch ^ swz) << 4)) = e4m3x8_to_bf16x8(make_uint2(lo, hi));
}

template <int D>
__device__ __forceinline__ void qk_tile(const WaveCtx& cx, const unsigned char* kb, const bf16x8 (&qf)[D / 16],
                                        f32x16 (&S)[2]) {
#pragma unroll
  for (int kbk = 0; kbk < 2; ++kbk)
#pragma unroll
    for (int r = 0; r < 16; ++r) S[kbk][r] = 0.0f;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    S[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k<D>(cx, kb, s, 0), qf[s], S[0], 0, 0, 0);
    S[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k<D>(cx, kb, s, 1), qf[s], S[1], 0, 0, 0);
  }
}

// ---- one pipelined iteration --------------------------------------------------------------
// On entry Scur holds the raw (already masked) scores of tile kt and mx_cur their row maximum.
//   stage B  raise the running reference if needed (rare);
//   stage C  exponentials of tile kt on the vector ALUs while the matrix cores compute the
//            scores of tile kt+1 into Snext (8 slices: D / 64 MFMAs + 4 exponentials each);
//   stage D  O += P V of tile kt on the matrix cores (one MFMA per slice) while the scalar/vector units
//            issue the fetches of V(kt+1) and K(kt+2) (8-bit caches: widen those two from the staging area and fetch
//            V(kt+2) and K(kt+3) into it) and reduce the row maximum of tile kt+1; V^T operands are
//            requested two MFMAs ahead of their use (the first two during stage C).
// The slices are fenced so the instruction streams stay interleaved as written.  Fetches are
// issued unconditionally with the tile index clamped to the last tile: the buffers they land
// in are free by then and are never read again.
// boff: cache offset of this wave's block of the tile whose V comes next (its K was the last one fetched).
// Returns the row maximum of tile kt+1.
template <int D, bool KV8, bool MASKNEXT, bool NEXT, bool PROBE>
__device__ __forceinline__ float tile_iter(const WaveCtx& cx, unsigned char* smem, int kt, int ntiles,
                                           BlockIds& ids, const int* bt, unsigned long long& boff,
                                           f32x16 (&Scur)[2], float mx_cur, f32x16 (&Snext)[2],
                                           const bf16x8 (&qf)[D / 16], f32x16 (&O)[D / 32], float& m_run, float& l_run,
                                           float (&am)[kMaxSpans], const int (&sp_a)[kMaxSpans],
                                           const int (&sp_b)[kMaxSpans]) {
  using C = Cfg<D, KV8>;
  const int key0 = kt * kTileKeys;
  unsigned char* const Kbuf = smem;
  unsigned char* const Vbuf = smem + 2 * C::TILE;
  const unsigned char* kb = Kbuf + ((kt + 1) & 1) * C::TILE;  // K of tile kt+1
  const unsigned char* vb = Vbuf + (kt & 1) * C::TILE;        // V of tile kt

  // what was fetched one iteration ago has landed (and, widened, is written); after the barrier every wave
  // has also finished reading the buffers that this iteration fills
  wait_vmem();
  __syncthreads();

  // -- stage B
  const float mt = mx_cur * cx.c;
  const bool upd = mt > m_run + kLazyTau;
  if (__builtin_amdgcn_ballot_w64(upd) != 0) {
    const float alpha = upd ? fast_exp2(m_run - mt) : 1.0f;
    m_run = upd ? mt : m_run;
    l_run *= alpha;
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) O[mb][r] *= alpha;
    if constexpr (PROBE) {
#pragma unroll
      for (int s = 0; s < kMaxSpans; ++s) am[s] *= alpha;
    }
  }
  const float m_safe = (m_run == -INFINITY) ? 0.0f : m_run;
  // block-id registers: the K fetch (two tiles ahead, three with staging) may enter a new group of 64 blocks
  const int tv = min(kt + (KV8 ? 2 : 1), ntiles - 1), tk = min(kt + (KV8 ? 3 : 2), ntiles - 1);
  if ((tk >> 4) > ids.grp + 1) {
    ids.grp += 1;
    ids.cur = ids.nxt;
    ids.nxt = load_ids(bt, 64 * (ids.grp + 1), cx.lane, cx.last_blk);
  }
  const int sel = ((tk >> 4) == ids.grp) ? ids.cur : ids.nxt;
  __builtin_amdgcn_sched_barrier(0);

  // -- stage C
  float tsum = 0.0f;
  union PB { uint32_t u[4]; bf16x8 v; } pb[4];
  bf16x8 va[3];   // ring of V^T operands: requested two matrix instructions ahead of their use
  {
    constexpr int PER = C::KSTEPS / 4 > 1 ? 2 : 1;      // MFMAs per slice: D = 128 both key halves of one k-step, D = 64 one
    bf16x8 ka[2][PER];
    auto request = [&](int s) {
      if constexpr (PER == 2) {
        ka[s & 1][0] = read_k<D>(cx, kb, s, 0);
        ka[s & 1][PER - 1] = read_k<D>(cx, kb, s, 1);
      } else {
        ka[s & 1][0] = read_k<D>(cx, kb, s >> 1, s & 1);
      }
    };
    if constexpr (NEXT) request(0);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if constexpr (NEXT) {
        if (s < 7) {
          request(s + 1);
          __builtin_amdgcn_sched_barrier(0);   // requested a whole slice before their use
        }
        const f32x16 z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        if constexpr (PER == 2) {
          Snext[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s & 1][0], qf[s % C::KSTEPS], s == 0 ? z : Snext[0], 0, 0, 0);
          Snext[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s & 1][PER - 1], qf[s % C::KSTEPS], s == 0 ? z : Snext[1], 0, 0, 0);
        } else {
          Snext[s & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[s & 1][0], qf[s >> 1], s < 2 ? z : Snext[s & 1], 0, 0, 0);
        }
      }
      // the first V^T operands of the P V stage are requested here, two slices before their use
      if (s == 6) va[0] = read_vt<D>(cx, vb, 0, 0);
      if (s == 7) va[1] = read_vt<D>(cx, vb, 0, 1);
      // exponentials of elements 4s .. 4s+3 of the current tile
      const int kbk = s >> 2, r0 = 4 * (s & 3);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float ex = fast_exp2(__builtin_fmaf(Scur[kbk][r0 + e], cx.c, -m_safe));
        Scur[kbk][r0 + e] = ex;
        tsum += ex;
      }
      const int m = 2 * kbk + ((s & 3) >> 1);
      pb[m].u[2 * (s & 1)] = pack_bf16(Scur[kbk][r0], Scur[kbk][r0 + 1]);
      pb[m].u[2 * (s & 1) + 1] = pack_bf16(Scur[kbk][r0 + 2], Scur[kbk][r0 + 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  l_run += tsum;

  if constexpr (PROBE) {
#pragma unroll
    for (int s = 0; s < kMaxSpans; ++s) {
      if (s < cx.S) {
        const int a = sp_a[s], b = sp_b[s];
        if (b > key0 && a < key0 + kTileKeys) {
          if (a <= key0 && b >= key0 + kTileKeys) {
            am[s] += tsum;  // whole tile inside the span; masked keys contributed 0
          } else {
            float acc = 0.0f;
#pragma unroll
            for (int kbk = 0; kbk < 2; ++kbk)
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                const int key = key0 + 32 * kbk + 8 * (r >> 2) + 4 * cx.hf + (r & 3);
                acc += (key >= a && key < b) ? Scur[kbk][r] : 0.0f;
              }
            am[s] += acc;
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // -- stage D
  float mx_acc = -INFINITY;   // running maximum of the next tile's scores
  if constexpr (NEXT && MASKNEXT) {
#pragma unroll
    for (int kbk = 0; kbk < 2; ++kbk)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = key0 + kTileKeys + 32 * kbk + 8 * (r >> 2) + 4 * cx.hf + (r & 3);
        if (key > cx.pos) Snext[kbk][r] = -INFINITY;
      }
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(2);   // the matrix-core-bound stage wins issue arbitration over the other wave
  constexpr int NS = 4 * C::MB;    // slices
  constexpr int NI = C::NI;
  unsigned char* const v_dst = Vbuf + ((kt + 1) & 1) * C::TILE + cx.w * kBlock * C::RB;   // this wave's rows of V(kt+1)
  unsigned char* const k_dst = Kbuf + (kt & 1) * C::TILE + cx.w * kBlock * C::RB;         // and of K(kt+2)
  const unsigned lds_v = cx.lds_base + (2 + ((kt + 1) & 1)) * C::TILE + cx.w * kBlock * C::RB;
  const unsigned lds_k = cx.lds_base + (kt & 1) * C::TILE + cx.w * kBlock * C::RB;
  unsigned char* const stage = smem + 4 * C::TILE + cx.w * C::STAGE;
  const unsigned lds_stage = cx.lds_base + 4 * C::TILE + cx.w * C::STAGE;
  uint4 st[2];                     // staged pieces on their way through the registers
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int m = i / C::MB, mb = i % C::MB;
    if (i + 2 < NS) va[(i + 2) % 3] = read_vt<D>(cx, vb, (i + 2) / C::MB, (i + 2) % C::MB);
    __builtin_amdgcn_sched_barrier(0);
    O[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[i % 3], pb[m].v, O[mb], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NEXT) {   // the last tile of an item has nothing left to fetch
      if constexpr (!KV8) {
        if (i < NI) {
          // (only a tile that needs the causal mask can reach past the last token)
          switch (i) {
            case 0: fetch_v<D, false, 0, MASKNEXT>(cx, boff, tv, lds_v); break;
            case 1: fetch_v<D, false, (NI > 1 ? 1 : 0), MASKNEXT>(cx, boff, tv, lds_v); break;
            case 2: fetch_v<D, false, (NI > 2 ? 2 : 0), MASKNEXT>(cx, boff, tv, lds_v); break;
            case 3: fetch_v<D, false, (NI > 2 ? 3 : 0), MASKNEXT>(cx, boff, tv, lds_v); break;
          }
        } else if (i < 2 * NI) {
          if (i == NI) boff = block_offset(cx, sel, tk);
          switch (i - NI) {
            case 0: fetch_k<D, false, 0>(cx, boff, lds_k); break;
            case 1: fetch_k<D, false, (NI > 1 ? 1 : 0)>(cx, boff, lds_k); break;
            case 2: fetch_k<D, false, (NI > 2 ? 2 : 0)>(cx, boff, lds_k); break;
            case 3: fetch_k<D, false, (NI > 2 ? 3 : 0)>(cx, boff, lds_k); break;
          }
        }
      } else {
        // piece p = 0 .. 2 NI - 1 (K run, then V run): read in slice 2p, its halves widened in slices 2p+2 and 2p+3
        if (i % 2 == 0 && i / 2 < 2 * NI) {
          const int p = i / 2;
          st[p & 1] = *reinterpret_cast<const uint4*>(stage + (p / NI) * C::BLK + (p % NI) * 1024 + 16 * cx.lane);
        }
        if (i >= 2 && (i - 2) / 2 < 2 * NI) {
          const int p = (i - 2) / 2, half = i % 2;
          const int r = C::RPI * (p % NI) + cx.lane / C::LPR, ch = 2 * (cx.lane % C::LPR) + half;
          const uint4& v = st[p & 1];
          widen_to<D>(p < NI ? k_dst : v_dst, r, ch, p < NI ? k_swizzle<D>(r) : v_swizzle<D>(r), half ? v.z : v.x, half ? v.w : v.y);
        }
        // the staging area is free once its last piece sits in registers
        constexpr int F = 4 * NI + 2 < NS - 2 * NI ? 4 * NI + 2 : NS - 2 * NI;
        if (i >= F && i < F + 2 * NI) {
          if (i == F) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          const int q = i - F;
          if (q == 0) fetch_v<D, true, 0, true>(cx, boff, tv, lds_stage + C::BLK);
          if (NI > 1 && q == 1) fetch_v<D, true, (NI > 1 ? 1 : 0), true>(cx, boff, tv, lds_stage + C::BLK);
          if (q == NI) { boff = block_offset(cx, sel, tk); fetch_k<D, true, 0>(cx, boff, lds_stage); }
          if (NI > 1 && q == NI + 1) fetch_k<D, true, (NI > 1 ? 1 : 0)>(cx, boff, lds_stage);
        }
      }
      // scores of the next tile, four at a time, spread over the last eight slices
      if (i >= NS - 8) {
        const int q = i - (NS - 8);
        const int kbk = q >> 2, r0 = 4 * (q & 3);
        // three-operand maxima written out (fmaxf() would first canonicalise every score with a v_max
        // of its own), both in one statement so that nothing is put between them
        asm volatile("v_max3_f32 %0, %0, %1, %2\n\tv_max3_f32 %0, %0, %3, %4"
                     : "+v"(mx_acc)
                     : "v"(Snext[kbk][r0]), "v"(Snext[kbk][r0 + 1]), "v"(Snext[kbk][r0 + 2]), "v"(Snext[kbk][r0 + 3]));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __builtin_amdgcn_s_setprio(0);
  float mx_next = 0.0f;
  if constexpr (NEXT) {
    mx_next = half_max(mx_acc);
  }
  return mx_next;
}

// The same iteration for a wave that has no key left: the tiles behind its rows' positions are for the other row blocks
// of the workgroup (groups of fewer than four heads), and it only fetches its cache blocks of them.  (Going through
// them with every score masked would let 0 * Inf from their values into its rows.)
template <int D, bool KV8>
__device__ __forceinline__ void fetch_iter(const WaveCtx& cx, unsigned char* smem, int kt, int ntiles, BlockIds& ids,
                                           const int* bt, unsigned long long& boff) {
  using C = Cfg<D, KV8>;
  constexpr int NI = C::NI;
  wait_vmem();
  __syncthreads();
  if (kt == ntiles - 1) return;
  const int tv = min(kt + (KV8 ? 2 : 1), ntiles - 1), tk = min(kt + (KV8 ? 3 : 2), ntiles - 1);
  if ((tk >> 4) > ids.grp + 1) {
    ids.grp += 1;
    ids.cur = ids.nxt;
    ids.nxt = load_ids(bt, 64 * (ids.grp + 1), cx.lane, cx.last_blk);
  }
  const int sel = ((tk >> 4) == ids.grp) ? ids.cur : ids.nxt;
  const unsigned rows = cx.w * kBlock * C::RB, vb = (2 + ((kt + 1) & 1)) * C::TILE + rows, kb = (kt & 1) * C::TILE + rows;
  unsigned lds_v = cx.lds_base + vb, lds_k = cx.lds_base + kb;
  if constexpr (KV8) {
    const unsigned staged = 4 * C::TILE + cx.w * C::STAGE;
#pragma unroll
    for (int q = 0; q < 2 * NI; ++q) {
      const uint4 st = *reinterpret_cast<const uint4*>(smem + staged + (q / NI) * C::BLK + (q % NI) * 1024 + 16 * cx.lane);
      const int r = C::RPI * (q % NI) + cx.lane / C::LPR, ch = 2 * (cx.lane % C::LPR);
      unsigned char* const dst = smem + (q < NI ? kb : vb);
      const int swz = q < NI ? k_swizzle<D>(r) : v_swizzle<D>(r);
      widen_to<D>(dst, r, ch, swz, st.x, st.y);
      widen_to<D>(dst, r, ch + 1, swz, st.z, st.w);
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the staging area is free
    lds_k = cx.lds_base + staged;
    lds_v = lds_k + C::BLK;
  }
  fetch_v<D, KV8, 0, true>(cx, boff, tv, lds_v);
  if constexpr (NI > 1) fetch_v<D, KV8, 1, true>(cx, boff, tv, lds_v);
  if constexpr (NI > 2) { fetch_v<D, KV8, 2, true>(cx, boff, tv, lds_v); fetch_v<D, KV8, 3, true>(cx, boff, tv, lds_v); }
  boff = block_offset(cx, sel, tk);
  fetch_k<D, KV8, 0>(cx, boff, lds_k);
  if constexpr (NI > 1) fetch_k<D, KV8, 1>(cx, boff, lds_k);
  if constexpr (NI > 2) { fetch_k<D, KV8, 2>(cx, boff, lds_k); fetch_k<D, KV8, 3>(cx, boff, lds_k); }
}

// mine: tiles up to the position of the wave's last row.  SHARED: that can be fewer than the workgroup's.
template <int D, bool KV8, bool SHARED, bool PROBE>
__device__ __forceinline__ void run_tiles(const WaveCtx& cx, unsigned char* smem, int ntiles, int mine, int n_nomask, BlockIds& ids,
                                          unsigned long long& boff, const bf16x8 (&qf)[D / 16], f32x16 (&O)[D / 32],
                                          float& m_run, float& l_run, float (&am)[kMaxSpans],
                                          const int (&sp_a)[kMaxSpans], const int (&sp_b)[kMaxSpans], const int* bt) {
  // The lane values are made opaque here: what is derived from them would otherwise be computed once for both
  // instantiations (probing or not) and spilled (57 registers, some of them in the loop) instead of recomputed.
  WaveCtx cy = cx;
  asm volatile("" : "+v"(cy.k_read_addr), "+v"(cy.v_read_addr), "+v"(cy.pos), "+v"(cy.k_off), "+v"(cy.v_off), "+v"(cy.hf), "+v"(cy.lane));
  f32x16 S0[2], S1[2];
  qk_tile<D>(cy, smem, qf, S0);
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) O[mb][rr] = 0.0f;
  m_run = -INFINITY;
  l_run = 0.0f;
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) am[s] = 0.0f;
  float mx = (n_nomask > 0) ? tile_max<false>(cy, 0, S0) : tile_max<true>(cy, 0, S0);

  // tile kt+1 needs no mask while kt+1 < n_nomask
  int kt = 0;
  const int end_nomask = min(n_nomask - 1, ntiles - 1);
  // two tiles per trip so the score registers ping-pong without copies
  while (kt + 2 <= end_nomask) {
    mx = tile_iter<D, KV8, false, true, PROBE>(cy, smem, kt, ntiles, ids, bt, boff, S0, mx, S1, qf, O, m_run,
                                               l_run, am, sp_a, sp_b);
    mx = tile_iter<D, KV8, false, true, PROBE>(cy, smem, kt + 1, ntiles, ids, bt, boff, S1, mx, S0, qf, O,
                                               m_run, l_run, am, sp_a, sp_b);
    kt += 2;
  }
  if (kt < end_nomask) {
    mx = tile_iter<D, KV8, false, true, PROBE>(cy, smem, kt, ntiles, ids, bt, boff, S0, mx, S1, qf, O, m_run,
                                               l_run, am, sp_a, sp_b);
    S0[0] = S1[0]; S0[1] = S1[1];
    kt += 1;
  }
  // tiles whose successor needs the causal mask
  const int fetching = SHARED ? min(mine, ntiles - 1) : ntiles - 1;
  while (kt < fetching) {
    mx = tile_iter<D, KV8, true, true, PROBE>(cy, smem, kt, ntiles, ids, bt, boff, S0, mx, S1, qf, O, m_run,
                                              l_run, am, sp_a, sp_b);
    S0[0] = S1[0]; S0[1] = S1[1];
    kt += 1;
  }
  if (SHARED && mine < ntiles) {
    for (; kt < ntiles; ++kt) fetch_iter<D, KV8>(cy, smem, kt, ntiles, ids, bt, boff);
    return;
  }
  // last tile
  (void)tile_iter<D, KV8, true, false, PROBE>(cy, smem, kt, ntiles, ids, bt, boff, S0, mx, S1, qf, O, m_run,
                                              l_run, am, sp_a, sp_b);
}

// The first tiles of an item into the LDS buffers.  16-bit: K(0) is requested here, V(0) and K(1) by the second
// function once the query rows have arrived.  8-bit caches: K(0), V(0) and K(1) here, and the bytes of V(1)
// and K(2) into the staging area.
template <int D, bool KV8>
__device__ __forceinline__ void first_tiles(const WaveCtx& cx, unsigned char* smem, int ntiles, unsigned long long boff0,
                                            unsigned long long boff1, unsigned long long boff2) {
  using C = Cfg<D, KV8>;
  constexpr int NI = C::NI;
  const unsigned lds_k = cx.lds_base + cx.w * kBlock * C::RB;                    // this wave's rows of K buffer 0
  if constexpr (!KV8) {
    fetch_k<D, false, 0>(cx, boff0, lds_k);
    if constexpr (NI > 1) fetch_k<D, false, 1>(cx, boff0, lds_k);
    if constexpr (NI > 2) { fetch_k<D, false, 2>(cx, boff0, lds_k); fetch_k<D, false, 3>(cx, boff0, lds_k); }
  } else {
    // through registers: nothing to overlap with yet
    const int t1 = min(1, ntiles - 1);
    const int rmax = cx.L - 1 - kBlock * min(cx.w, cx.last_blk);
    uint4 k0[NI], v0[NI], k1[NI];
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) {
      const int r = C::RPI * jj + cx.lane / C::LPR;
      const unsigned piece = 16 * (cx.lane % C::LPR);
      k0[jj] = load_global16((global_bytes)(cx.kbase + boff0 + r * D + piece));
      v0[jj] = load_global16((global_bytes)(cx.vbase + boff0 + min(r, rmax) * D + piece));
      k1[jj] = load_global16((global_bytes)(cx.kbase + boff1 + r * D + piece));
    }
    // V(1), then K(2): the order in which the loop fetches
    const unsigned lds_stage = cx.lds_base + 4 * C::TILE + cx.w * C::STAGE;
    fetch_v<D, true, 0, true>(cx, boff1, t1, lds_stage + C::BLK);
    if constexpr (NI > 1) fetch_v<D, true, 1, true>(cx, boff1, t1, lds_stage + C::BLK);
    fetch_k<D, true, 0>(cx, boff2, lds_stage);
    if constexpr (NI > 1) fetch_k<D, true, 1>(cx, boff2, lds_stage);
    unsigned char* const kd = smem + cx.w * kBlock * C::RB;
#pragma unroll
    for (int jj = 0; jj < NI; ++jj) {
      const int r = C::RPI * jj + cx.lane / C::LPR, ch = 2 * (cx.lane % C::LPR);
      widen_to<D>(kd, r, ch, k_swizzle<D>(r), k0[jj].x, k0[jj].y);
      widen_to<D>(kd, r, ch + 1, k_swizzle<D>(r), k0[jj].z, k0[jj].w);
      widen_to<D>(kd + 2 * C::TILE, r, ch, v_swizzle<D>(r), v0[jj].x, v0[jj].y);
      widen_to<D>(kd + 2 * C::TILE, r, ch + 1, v_swizzle<D>(r), v0[jj].z, v0[jj].w);
      widen_to<D>(kd + C::TILE, r, ch, k_swizzle<D>(r), k1[jj].x, k1[jj].y);
      widen_to<D>(kd + C::TILE, r, ch + 1, k_swizzle<D>(r), k1[jj].z, k1[jj].w);
    }
  }
}

template <int D, bool KV8>
__device__ __forceinline__ void rest_of_first_tiles(const WaveCtx& cx, unsigned long long boff0, unsigned long long boff1) {
  using C = Cfg<D, KV8>;
  if constexpr (!KV8) {
    constexpr int NI = C::NI;
    const unsigned lds_k = cx.lds_base + cx.w * kBlock * C::RB;
    const unsigned lds_v = lds_k + 2 * C::TILE;
    fetch_v<D, false, 0, true>(cx, boff0, 0, lds_v);
    if constexpr (NI > 1) fetch_v<D, false, 1, true>(cx, boff0, 0, lds_v);
    if constexpr (NI > 2) { fetch_v<D, false, 2, true>(cx, boff0, 0, lds_v); fetch_v<D, false, 3, true>(cx, boff0, 0, lds_v); }
    fetch_k<D, false, 0>(cx, boff1, lds_k + C::TILE);
    if constexpr (NI > 1) fetch_k<D, false, 1>(cx, boff1, lds_k + C::TILE);
    if constexpr (NI > 2) { fetch_k<D, false, 2>(cx, boff1, lds_k + C::TILE); fetch_k<D, false, 3>(cx, boff1, lds_k + C::TILE); }
  }
}

// One work item: rows [row0, row0 + rows_per_wg) of sequence `seq` (context L, n rows, first q row
// qbase) for the heads of (kvh, hg).  ZERO_REST (self-planned calls): the wave that owns a probed
// head in the item of row 0 also writes zeros to that head's `mass` slots that hold no row, so that
// every entry of `mass` is written exactly once without a planner's zero-fill.
template <int D, bool KV8, bool SHARED, bool ZERO_REST>
__device__ __forceinline__ void prefill_item(const AttnParams& p, unsigned char* smem, int kvh, int hg, int seq,
                                             int row0, int L, int n, int qbase) {
  using C = Cfg<D, KV8>;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = w % p.hpw, rb = w / p.hpw;
  const int head = kvh * p.G + hg * p.hpw + hh;
  const int wrow0 = row0 + rb * kWaveRows;
  const bool wave_active = wrow0 < n;
  const int qi = lane & 31, hf = lane >> 5;
  const int t = max(min(wrow0 + qi, n - 1), 0);
  const int wave_pos_min = L - n + min(wrow0, n - 1);
  const int wg_pos_max = L - n + min(row0 + p.rows_per_wg, n) - 1;
  const int ntiles = wg_pos_max / kTileKeys + 1;
  const int n_nomask = (wave_pos_min + 1) / kTileKeys;   // tiles whose last key is within every row's horizon
  const int mine = (L - n + min(wrow0 + kWaveRows, n) - 1) / kTileKeys + 1;     // tiles with a key within some row's

  const int* const bt = p.block_table + (size_t)seq * p.max_blocks;
  WaveCtx cx;
  cx.L = L;
  cx.last_blk = (L - 1) >> 4;
  cx.w = w;
  cx.lane = lane;
  cx.blk_bytes = (unsigned)p.Hkv * C::BLK;
  // this wave's blocks of the first tiles by scalar loads: the wait for them leaves vector loads alone
  cx.num_blocks = p.num_blocks;
  auto first_id = [&](int tile) { return cload(bt, min(4 * min(tile, ntiles - 1) + w, cx.last_blk)); };
  const int id0 = first_id(0), id1 = first_id(1), id2 = KV8 ? first_id(2) : 0;

  // Query rows.  The compiler does not count the tile fetches (assembly), so its wait for these rows is a wait for
  // the fetches issued before it as well: only K(0) is (first_tiles / rest_of_first_tiles).
  uint4 qraw[C::KSTEPS];
  {
    const __bf16* const qg = static_cast<const __bf16*>(p.q) + ((size_t)(qbase + t) * p.Hq + head) * D + 8 * hf;
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) qraw[s] = load_global16((global_bytes)(unsigned long long)(size_t)(qg + 16 * s));
  }

  cx.hf = hf;
  cx.qi = qi;
  cx.pos = L - n + t;
  cx.c = KV8 ? p.scale_log2 * p.k_scale[kvh] : p.scale_log2;
  cx.S = p.S;
  // K reads: lane (row qi [+32], half hf) reads logical chunk 2s + hf
  cx.k_read_addr = (unsigned)qi * C::RB | ((unsigned)(hf ^ k_swizzle<D>(qi)) << 4);
  {
    // transposed V reads: within a 16-lane group lane s supplies row (s >> 2) and 8-byte piece (s & 3)
    const int g = lane >> 4, s16 = lane & 15;
    const int hfv = g >> 1, ddhalf = g & 1;
    const unsigned rowc = (unsigned)(4 * hfv + (s16 >> 2)) * C::RB;
    const unsigned lowc = (unsigned)(2 * ddhalf + ((s16 & 3) >> 1)) * 16 + (unsigned)(s16 & 1) * 8;
    const unsigned xorc = (unsigned)v_swizzle<D>(s16 >> 2) * 16;
    cx.v_read_addr = rowc | (lowc ^ xorc);
  }
  cx.kbase = (unsigned long long)(size_t)p.k_cache + (size_t)kvh * C::BLK;
  cx.vbase = (unsigned long long)(size_t)p.v_cache + (size_t)kvh * C::BLK;
  // per-lane source offsets of the direct-to-LDS loads: LDS slot (row r, physical chunk pc)
  // receives logical chunk pc ^ swizzle(r); bytes are staged as they lie in the cache
  {
    const int r = lane / C::LPR, pc = lane % C::LPR;
    const unsigned row = (unsigned)r * (C::BLK / kBlock);
    cx.k_off = row + (unsigned)(KV8 ? pc : pc ^ k_swizzle<D>(r)) * 16;
    cx.v_off = row + (unsigned)(KV8 ? pc : pc ^ v_swizzle<D>(r)) * 16;
  }
  cx.lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) const void*)smem;

  BlockIds ids;
  ids.grp = 0;
  ids.cur = load_ids(bt, 0, lane, cx.last_blk);
  ids.nxt = load_ids(bt, 64, lane, cx.last_blk);

  const unsigned long long boff0 = block_bytes(cx, id0), boff1 = block_bytes(cx, id1), boff2 = block_bytes(cx, id2);
  first_tiles<D, KV8>(cx, smem, ntiles, boff0, boff1, boff2);
  unsigned long long boff = KV8 ? boff2 : boff1;      // of the last K run fetched

  int pslot = -1, qsel_b = 0, qsel_e = 0;
  int sp_a[kMaxSpans], sp_b[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) { sp_a[s] = 0; sp_b[s] = 0; }
  if (p.P > 0) {
    pslot = find_probe_slot_uniform(p.probe_heads, p.P, head);
    qsel_b = cload(p.query_sel, 2 * seq);
    qsel_e = min(cload(p.query_sel, 2 * seq + 1), qsel_b + p.NQ);
    load_spans_uniform(p.key_spans, seq, p.S, sp_a, sp_b);
  }
  const bool wave_probe = wave_active && pslot >= 0 && qsel_b < min(wrow0 + kWaveRows, n) && qsel_e > wrow0;

  f32x16 O[C::MB];
  float m_run, l_run;
  float am[kMaxSpans];

  // the first scores need Q and K(0); V(0) and K(1) (2 NI loads; with staging K(2) and V(1)) may stay in flight
  // until the top of the first iteration
  bf16x8 qf[C::KSTEPS];
#pragma unroll
  for (int s = 0; s < C::KSTEPS; ++s) __builtin_memcpy(&qf[s], &qraw[s], 16);
#pragma unroll
  for (int s = 0; s < C::KSTEPS; ++s) asm volatile("" : "+v"(qf[s]) :: "memory");     // Q has arrived here
  rest_of_first_tiles<D, KV8>(cx, boff0, boff1);
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * C::NI) : "memory");
  __syncthreads();

  if (wave_probe)
    run_tiles<D, KV8, SHARED, true>(cx, smem, ntiles, mine, n_nomask, ids, boff, qf, O, m_run, l_run, am, sp_a, sp_b, bt);
  else
    run_tiles<D, KV8, SHARED, false>(cx, smem, ntiles, mine, n_nomask, ids, boff, qf, O, m_run, l_run, am, sp_a, sp_b, bt);

  // epilogue: normalise, transpose through LDS (16-byte chunks swizzled by row), coalesced stores
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const float inv_l = 1.0f / l_tot;
  const float inv = KV8 ? inv_l * p.v_scale[kvh] : inv_l;     // `out` carries the value scale, `mass` does not
  wait_vmem();   // the clamped fetches of the last iterations must have landed before LDS is reused
  __syncthreads();
  unsigned char* const ot = smem + w * (kWaveRows * C::RB);
  if (wave_active) {
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        uint2 v;
        v.x = pack_bf16(O[mb][4 * g4] * inv, O[mb][4 * g4 + 1] * inv);
        v.y = pack_bf16(O[mb][4 * g4 + 2] * inv, O[mb][4 * g4 + 3] * inv);
        const int ch = 4 * mb + g4;
        *reinterpret_cast<uint2*>(ot + qi * C::RB + ((ch ^ k_swizzle<D>(qi)) << 4) + 8 * hf) = v;
      }
  }
  __syncthreads();
  if (wave_active) {
    __bf16* const og = static_cast<__bf16*>(p.out);
#pragma unroll
    for (int j = 0; j < C::CH / 2; ++j) {
      const int rr = lane / C::CH + (64 / C::CH) * j;
      const int ch = lane % C::CH;
      const int tr = wrow0 + rr;
      if (tr < n) {
        const uint4 v = *reinterpret_cast<const uint4*>(ot + rr * C::RB + ((ch ^ k_swizzle<D>(rr)) << 4));
        *reinterpret_cast<uint4*>(og + ((size_t)(qbase + tr) * p.Hq + head) * D + 8 * ch) = v;
      }
    }
    if (wave_probe) {
#pragma unroll
      for (int s = 0; s < kMaxSpans; ++s) {
        if (s < p.S) {
          const float a_tot = am[s] + __shfl_xor(am[s], 32);
          const int tr = wrow0 + qi;
          if (hf == 0 && tr < n && tr >= qsel_b && tr < qsel_e)
            p.mass[(((size_t)seq * p.P + pslot) * p.NQ + (tr - qsel_b)) * p.S + s] = a_tot * inv_l;
        }
      }
    }
  }
  if constexpr (ZERO_REST) {
    if (row0 == 0 && rb == 0 && pslot >= 0 && p.plan_fresh) {
      const int lo = max(qsel_b, 0), hi = min(qsel_e, n);     // slots lo - qsel_b .. hi - qsel_b - 1 hold rows
      for (int e = lane; e < p.NQ * p.S; e += 64) {
        const int tr = qsel_b + e / p.S;
        if (tr < lo || tr >= hi) p.mass[((size_t)seq * p.P + pslot) * p.NQ * p.S + e] = 0.0f;
      }
    }
  }
}

// ---- batches that plan themselves ----------------------------------------------------------
// Row blocks in processing order without a planner.  The deep row blocks (many key tiles) should start first, or
// the launch ends with a few of them alone; a full sort is not needed for that.  The range of depths is cut
// into kDepthParts equal parts and the order is: the deepest part of every sequence, the next part of every sequence, ...
// with descending blocks inside.  An item's block then follows from sums over the sequences, which every wave forms
// for itself (lane l takes sequences l K .. l K + K - 1): one trip to memory for the lengths instead of a planning
// launch (8 us in a kernel trace of 16 prompts) and two trips for its record.  It costs a workgroup about a thousand cycles, so launches of many
// rounds keep the planner (kSelfPlanMaxWgs).  (2 or 8 parts: 1-3 % slower on 16 ragged prompts; 16: 7 %, as
// neighbouring workgroups then share fewer tiles in L2.)
constexpr int kSeqsPerLane = kScanMaxSeqs / 64;

struct ChunkSeq { int L, n, qbase, bits; bool valid; };

// one sequence as the planner sees it; valid: it has row blocks to compute
__device__ __forceinline__ ChunkSeq chunk_seq(const AttnParams& p, int Lraw, int r0, int r1) {
  const int max_ctx = p.max_blocks * kBlock;
  ChunkSeq s = {min(Lraw, max_ctx), r1 - r0, r0, 0, false};
  if (Lraw < 0 || s.n < 0) { s.bits = kStatNegative; return s; }
  if (Lraw > max_ctx) s.bits |= kStatLenClamped;
  if (s.n > s.L) s.bits |= kStatQGtL;
  else if (r0 < 0 || r1 > p.total_q) s.bits |= kStatNegative;
  else if (s.n == 1 && p.batch_kind == 1) s.bits |= kStatHint;   // a single row in a call promised to hold chunks: dropped
  else s.valid = s.n >= 2;
  return s;
}

constexpr int kDepthParts = 4;

// row blocks of a sequence with at most `tiles` key tiles (they are its first ones)
__device__ __forceinline__ int blocks_up_to(int L, int n, int nblk, int tiles, int rows_log2) {
  if (L <= kTileKeys * tiles) return nblk;
  return min(max((kTileKeys * tiles - (L - n)) >> rows_log2, 0), nblk);
}

struct ChunkItem { int seq, block, L, n, qbase; };

// the item-th row block in processing order; false: there are not that many
__device__ __forceinline__ bool find_item(const AttnParams& p, int item, int lane, ChunkItem& it) {
  if (p.num_seqs == 1) {
    const ChunkSeq s = chunk_seq(p, cload(p.seq_lens, 0), cload(p.cu_q_lens, 0), cload(p.cu_q_lens, 1));
    const int nblk = s.valid ? (s.n + p.rows_per_wg - 1) / p.rows_per_wg : 0;
    it = {0, nblk - 1 - item, s.L, s.n, s.qbase};
    return item < nblk;
  }
  const int K = (p.num_seqs + 63) >> 6;
  const int rows_log2 = p.rows_per_wg == 32 ? 5 : p.rows_per_wg == 64 ? 6 : 7;
  int nblk[kSeqsPerLane], L[kSeqsPerLane], n[kSeqsPerLane], qbase[kSeqsPerLane];
  int deepest = 0;
#pragma unroll
  for (int u = 0; u < kSeqsPerLane; ++u) {
    nblk[u] = L[u] = n[u] = qbase[u] = 0;
    const int i = lane * K + u;
    if (u < K && i < p.num_seqs) {
      const ChunkSeq s = chunk_seq(p, p.seq_lens[i], p.cu_q_lens[i], p.cu_q_lens[i + 1]);
      if (s.valid) {
        L[u] = s.L; n[u] = s.n; qbase[u] = s.qbase;
        nblk[u] = (s.n + p.rows_per_wg - 1) >> rows_log2;
        deepest = max(deepest, s.L);
      }
    }
  }
  constexpr int N = kDepthParts;
  // part q (0: deepest) holds the blocks of more than bound[N - 1 - q] and at most bound[N - q] tiles
  const int max_tiles = (wave_max(deepest) + kTileKeys - 1) / kTileKeys;
  int bound[N + 1], total[N + 1];
  bound[0] = total[0] = 0;
#pragma unroll
  for (int k = 1; k <= N; ++k) {
    bound[k] = max_tiles * k / N;
    int sum = 0;
#pragma unroll
    for (int u = 0; u < kSeqsPerLane; ++u)
      if (u < K) sum += blocks_up_to(L[u], n[u], nblk[u], bound[k], rows_log2);
    total[k] = __builtin_amdgcn_readlane(wave_scan(sum), 63);
  }
  if (item >= total[N]) return false;
  int first = 0, lo = bound[N - 1], hi = bound[N];
#pragma unroll
  for (int k = 1; k < N; ++k)
    if (item >= total[N] - total[N - k]) { first = total[N] - total[N - k]; lo = bound[N - k - 1]; hi = bound[N - k]; }
  const int rel = item - first;
  int mine = 0;
#pragma unroll
  for (int u = 0; u < kSeqsPerLane; ++u)
    if (u < K) mine += blocks_up_to(L[u], n[u], nblk[u], hi, rows_log2) - (lo ? blocks_up_to(L[u], n[u], nblk[u], lo, rows_log2) : 0);
  const int incl = wave_scan(mine);
  int start = incl - mine;
  const int from = __builtin_ctzll(__builtin_amdgcn_ballot_w64(rel >= start && rel < incl));
  ChunkItem f = {0, 0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < kSeqsPerLane; ++u)
    if (u < K) {
      const int end = blocks_up_to(L[u], n[u], nblk[u], hi, rows_log2);
      const int size = end - (lo ? blocks_up_to(L[u], n[u], nblk[u], lo, rows_log2) : 0);
      if (rel >= start && rel < start + size) f = {lane * K + u, end - 1 - (rel - start), L[u], n[u], qbase[u]};
      start += size;
    }
  it.seq = __builtin_amdgcn_readlane(f.seq, from);
  it.block = __builtin_amdgcn_readlane(f.block, from);
  it.L = __builtin_amdgcn_readlane(f.L, from);
  it.n = __builtin_amdgcn_readlane(f.n, from);
  it.qbase = __builtin_amdgcn_readlane(f.qbase, from);
  return true;
}

// What the planner does besides, by a workgroup of its own: the header with the status word, and zeros in the `mass`
// entries of sequences without row blocks (in a mixed batch the merge kernel of the single rows has those) and of elements
// of the head list that no head owns.
__device__ __forceinline__ void settle_chunks(const AttnParams& p, int* sh) {
  int* const skip = sh + 2;     // [kScanMaxSeqs]
  const int tid = threadIdx.x;
  if (tid < 2) sh[tid] = 0;
  __syncthreads();
  int bits = p.plan_fresh && bad_head_list<256>(p) ? kBadHeadList : 0, blocks = 0;
  for (int i = tid; i < p.num_seqs; i += 256) {
    const ChunkSeq s = chunk_seq(p, p.seq_lens[i], p.cu_q_lens[i], p.cu_q_lens[i + 1]);
    bits |= s.bits;
    if (s.valid) blocks += (s.n + p.rows_per_wg - 1) / p.rows_per_wg;
    skip[i] = s.valid ? 0 : 1;
  }
  if (bits) atomicOr(&sh[0], bits);
  if (blocks) atomicAdd(&sh[1], blocks);
  __syncthreads();
  if (tid == 0) { p.hdr->n_prefill = sh[1]; p.hdr->n_decode = 0; p.hdr->chunk_keys = 0; p.hdr->status = sh[0] & ~kBadHeadList; }
  if (p.batch_kind == 1 && p.plan_fresh && p.P > 0)
    for (int i = 0; i < p.num_seqs; ++i)
      if (skip[i])
        for (int e = tid; e < p.P * p.NQ * p.S; e += 256) p.mass[(size_t)i * p.P * p.NQ * p.S + e] = 0.0f;
  if (sh[0] & kBadHeadList) zero_unowned_mass<256>(p);
}

// PLANNED: the work item comes from the planner's list.  Otherwise the kernel finds it (above), the last workgroup
// of the grid settles the rest, and `mass` is written entry by entry by the waves that own the entries.
// SHARED: several row blocks to a workgroup (groups of fewer than four heads).  An instantiation of its own, because the
// spills that the fetch-only iterations bring cost a prompt of 2048 tokens at 32 / 8 heads 1.5 of its 49.5 us.
template <int D, bool KV8, bool SHARED, bool PLANNED>
__global__ __launch_bounds__(256, 2) void k_prefill(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int bid = blockIdx.x;
  const int kvh = bid % p.Hkv;
  const int rest = bid / p.Hkv;
  const int hg = rest % p.hgroups;
  const int item = rest / p.hgroups;
  if constexpr (PLANNED) {
    // the grid covers the whole item capacity, so both records can be fetched together with
    // the item count instead of after it
    const WorkItem it = p.pf_items[2 * item];
    const int qbase = p.pf_items[2 * item + 1].x, nitems = p.hdr->n_prefill;
    // (named before the branch, or the compiler moves the loads behind it, one trip to memory after the other)
    asm volatile("" :: "s"(it.x), "s"(it.y), "s"(it.z), "s"(it.w), "s"(qbase), "s"(nitems), "s"(p.block_table), "s"(p.q),
                 "s"(p.k_cache), "s"(p.v_cache));
    if (item >= nitems) return;
    prefill_item<D, KV8, SHARED, false>(p, smem, kvh, hg, it.x, it.y, it.z, it.w, qbase);
  } else {
    if (bid == (int)gridDim.x - 1) {
      settle_chunks(reread_arguments(), reinterpret_cast<int*>(smem));   // (or its arguments take registers from the rest)
      return;
    }
    ChunkItem it;
    const bool some = find_item(p, item, threadIdx.x & 63, it);
    asm volatile("" :: "s"(p.block_table), "s"(p.q), "s"(p.k_cache), "s"(p.v_cache));
    if (!some) return;
    prefill_item<D, KV8, SHARED, true>(p, smem, kvh, hg, it.seq, it.block * p.rows_per_wg, it.L, it.n, it.qbase);
  }
}

template <int D, bool KV8, bool SHARED, bool PLANNED>
hipError_t launch_kernel(const AttnParams& p, long long grid, hipStream_t st) {
  static std::atomic<unsigned long long> configured{0};
  constexpr int lds = Cfg<D, KV8>::LDS;
  const hipError_t e = raise_lds_limit_once(reinterpret_cast<const void*>(&k_prefill<D, KV8, SHARED, PLANNED>), lds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_prefill<D, KV8, SHARED, PLANNED>), dim3((unsigned)grid), dim3(256), lds, st, p);
  return hipGetLastError();
}

template <int D, bool KV8>
hipError_t launch(const AttnParams& p, long long grid, hipStream_t st) {
  if (p.rows_per_wg == kWaveRows)
    return p.pf_self ? launch_kernel<D, KV8, false, false>(p, grid, st) : launch_kernel<D, KV8, false, true>(p, grid, st);
  return p.pf_self ? launch_kernel<D, KV8, true, false>(p, grid, st) : launch_kernel<D, KV8, true, true>(p, grid, st);
}

}  // namespace

hipError_t launch_prefill(const AttnParams& p, int D, hipStream_t st) {
  const long long grid = (long long)p.pf_cap * p.Hkv * p.hgroups + (p.pf_self ? 1 : 0);
  if (grid <= 0) return hipSuccess;
  if (!grid_fits(grid)) return hipErrorInvalidValue;
  if (D == 128) return !p.kv8 ? launch<128, false>(p, grid, st) : launch<128, true>(p, grid, st);
  if (D == 64) return !p.kv8 ? launch<64, false>(p, grid, st) : launch<64, true>(p, grid, st);
  return hipErrorInvalidValue;
}

}  // namespace hook
