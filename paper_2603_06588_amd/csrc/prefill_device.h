// Tiled causal attention for query chunks (n_i >= 2), bf16 MFMA, head_dim 64 and 128, 16-bit and 8-bit caches: device code
// of the kernels in prefill.hip and mixed.hip.
//
// Workgroup = 4 or 8 waves = (hpw q heads of one kv head) x (waves / hpw blocks of 32 query rows),
// all sharing the K/V tiles (64 keys = 4 cache blocks) of their kv head.  Data movement is built around two
// gfx950 features:
//   * K and V go from the paged cache straight into LDS with 16-byte direct-to-LDS loads, so staging
//     costs no vector registers and almost no vector ALU work.  Wave w of four fetches cache block w of every
//     tile (two of eight waves half a block each): the block of a kv head is one contiguous run, so one block id, one 64-bit address and
//     16 D bytes / 1 KB load instructions with constant offsets do it.  16-byte chunks are XOR-swizzled inside
//     each LDS row so that the MFMA operand reads below are free of bank conflicts although rows are
//     unpadded; K rows are kept as D / 64 parts of 128 bytes, so that four addresses reach every operand of a tile;
//   * V stays in its natural [key][dim] layout and is read TRANSPOSED with
//     ds_read_b64_tr_b16, which hands each lane four consecutive keys of one output
//     dimension - the A operand of O^T = V^T P^T.
//
// Per wave the score tile is computed transposed, S^T = K Q^T (32x32x16 MFMA, keys = M,
// queries = N): lane l owns query l % 32 and 16 keys per 32-key block, so row sums are in-lane, and the
// exponentials, rounded to bf16, already form the B operand of the second MFMA.
//
// The loop goes by half tiles of 32 keys: the exponentials of one run on the vector ALUs while the matrix cores
// alternate between the scores of the next and P V of the one before, a matrix instruction and its share of the
// exponentials at a time.  That even mix is what the two waves of a SIMD need to keep its matrix core busy (synthetic
// loops with all operand reads and fetches in place: 33 cycles per 32-cycle matrix instruction; this loop 31-34 while
// both waves are inside it, 39 on a 32 k prompt, where the chip is at its power limit and holds 1.5-1.6 GHz).  Phases, with
// the scores of a tile under its predecessor's exponentials and P V after them, took 44.
// A row's softmax reference is its maximum over the first tile: no maxima and no exchange between lanes inside the loop (a fifth
// of its vector instructions), and nothing waits for a whole tile's scores.  The sums are exact softmax sums under any
// reference while they are finite.  Where they grow large because scores have risen far above the reference, it is raised
// (raise_reference); rows whose sums left the range of fp32 before that are done over (rows_alone).
// 32768 tokens at 64 / 8 heads 14.9 -> 14.4 ms, one prompt of 2048 at 32 / 8 51.1 -> 44.6 us, 16 ragged prompts of 512-2048
// 253.8 -> 242.8 us, the same at head size 64 156.4 -> 148 us, 8 chunks over an 8-bit cache 251 -> 243 us.
//
// K tiles are fetched two tiles ahead and V tiles one tile ahead, which makes one workgroup barrier per tile sufficient
// with two LDS buffers each.  (Fetches issued right behind the barrier instead of in the first slots of the next
// iteration: 3-6 % slower, with branches or with lanes switched off where nothing is left to fetch.)
//
// Query rows come through LDS as well, requested in one go with the first tiles (a compiler that does not count the tile
// fetches waits for all of them when it waits for rows loaded to registers).
//
// Eight waves share a tile's fetch where row blocks are deep and many (kEightWaveMinWgs in api.hip): half the fetches per
// matrix instruction, which matters because the chip is at its power limit there (all fetches left out of a copy
// of the kernel: 12 % less time on the 32 k prompt, 19 % on ragged prompts); a compute unit then holds one workgroup, whose
// start-up nothing covers, so short contexts keep four.
// (One workgroup per compute unit that goes from row block to row block, the next one's rows and tiles requested
// during the last tile of the one before: 244 us against 242 on the ragged prompts; the cycles it saves come back as
// a lower clock.  Three waves to a SIMD at head size 64: 149.5 -> 157.8 us.)
//
// 8-bit caches (KV8): the bytes go direct to LDS too, one tile earlier, into a staging area of each wave's own
// (2 x 16 D bytes); in the tile before they are needed the wave reads its block back, widens it
// to bf16 (exact: every E4M3 number is a bf16 number) and writes it to the same swizzled buffers as
// above, so the rest of the loop is the 16-bit one and every byte is widened once for the four heads
// that share it.  The key scale goes into the softmax scale, the value scale into the normalisation of `out`.
//
// Probe span sums are taken from the fp32 exponentials under the same reference
// as the normaliser and divided by it at the end: the captured mass is the exact softmax
// mass of the row.  Waves that probe run a second instantiation of the same loop whose
// arithmetic for `out` is identical.
#pragma once

#include "fp8_device.h"
#include "hook_device.h"

namespace hook {

namespace {

typedef short v4i16 __attribute__((ext_vector_type(4)));

template <int D, bool KV8, int NW>
struct Cfg {
  static constexpr int RB = 2 * D;                          // bytes of one bf16 row
  static constexpr int TILE = kTileKeys * RB;
  static constexpr int KBLK = kBlock * RB;                  // a cache block in a K buffer: D / 64 parts of 64 dimensions, rows of 128 bytes
  static constexpr int KSTEPS = D / 16;                     // MFMA k-steps of the scores of a half tile
  static constexpr int MB = D / 32;                         // 32-dimension blocks of the output
  static constexpr int SLOTS = KSTEPS + 2 * MB;             // matrix instructions per half tile (scores and P V alternate)
  static constexpr int BLK = kBlock * D * (KV8 ? 1 : 2);    // bytes of one (cache block, kv head) run
  static constexpr int WPB = NW / 4;                        // waves that share the fetch of a run
  static constexpr int SHARE = BLK / WPB;                   // bytes of it for each
  static constexpr int ROWS = kBlock / WPB;                 // rows of V (and of bytes) for each
  static constexpr int NI = SHARE / 1024;                   // load instructions for each
  static_assert(NI >= 1, "");
  static constexpr int LPR = BLK / kBlock / 16;             // lanes (16-byte pieces) per row of a run fetched as it lies (V, bytes)
  static constexpr int RPI = 64 / LPR;                      // rows per load instruction of 1 KB
  static constexpr int STAGE = KV8 ? 2 * SHARE : 0;         // staging bytes per wave: of the K run, of the V run
  static constexpr int QHALF = kBlock * RB;                 // half of a wave's query rows on their way through LDS (16-bit caches)
  static constexpr int OUT = NW == 4 ? 0 : 4 * TILE + NW * STAGE;           // output rows: over the K buffers, or behind everything
  // K[2], V[2], staging, query rows on their way in (eight waves: output rows on their way out)
  static constexpr int LDS = 4 * TILE + NW * STAGE + (NW == 8 ? NW * 2 * QHALF : KV8 ? 0 : NW * QHALF);
  static constexpr int CH = D / 8;                          // 16-byte chunks per bf16 row
  static constexpr int RING = 4;                            // operands requested ahead, K and V^T each
};

// Swizzles of the 16-byte chunks (what a chunk index is XORed with).  K buffers have rows of 128 bytes, half of the
// 64 banks: 16 neighbouring rows read with one chunk index then touch every bank once.  V rows have 2 D bytes: the four
// rows a transposed read touches lie in different banks.  The output rows on their way through LDS use out_swizzle.
__device__ __forceinline__ int k_swizzle(int r) { return (r >> 1) & 7; }
template <int D> __device__ __forceinline__ int v_swizzle(int r) { return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2); }
template <int D> __device__ __forceinline__ int out_swizzle(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }

// A wave's own LDS accesses complete in order, so data that only passes through it from lane to lane needs no wait; but the
// compiler has to leave them in order too (what is written as one type is read as another).
__device__ __forceinline__ void in_order() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// 16-byte direct-to-LDS loads, N of them: lane i's data of load j lands at lds + OFF + 1024 j + 16 i, from base + OFF + 1024 j +
// its own offset voff[j].
// Written as assembly so that their completion is tracked only by the explicit vmcnt waits; the compiler would
// otherwise make every later LDS read wait for them.
template <int N, int OFF>
__device__ __forceinline__ void dma16(unsigned long long base, const unsigned* voff, unsigned lds_addr) {
  static_assert(N == 1 || N == 2, "");
  if constexpr (N == 1)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                 :: "s"(lds_addr), "v"(voff[0]), "s"(base), "n"(OFF) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3 offset:%4\n\tglobal_load_lds_dwordx4 %2, %3 offset:%5"
                 :: "s"(lds_addr), "v"(voff[0]), "v"(voff[1]), "s"(base), "n"(OFF), "n"(OFF + 1024) : "memory", "m0");
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 x) { return __builtin_bit_cast(bf16x8, x); }

struct WaveCtx {
  // loop-invariant per-lane / per-wave values
  int hf;
  int pos;                // causal horizon of this lane's query row
  int pos_min;            // of the wave's first row
  float c;                // scale * log2(e)
  // direct-to-LDS fetches
  unsigned long long kbase, vbase;   // cache + kv-head offset
  unsigned lds_base;      // LDS address of the buffers
  unsigned blk_bytes;     // bytes per cache block (all kv heads)
  int num_blocks;
  unsigned k_off[4], v_off[2];  // this lane's source offsets in a run, less 1024 per load instruction before
  int L, last_blk, w, lane;
  int wb, ws;             // the block of every tile that this wave fetches, which share of it
};

// lane l and lane l ^ 32 hold the two key halves of one query: maximum over both (one swap between
// the lane halves instead of a round trip through LDS)
__device__ __forceinline__ float half_max(float mx) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// scores of the keys behind this lane's row; `key0`: first key of the half tile
__device__ __forceinline__ void mask_half(const WaveCtx& cx, int key0, f32x16& S) {
  const int last = cx.pos - key0 - 4 * cx.hf;
#pragma unroll
  for (int r = 0; r < 16; ++r)
    S[r] = 8 * (r >> 2) + (r & 3) > last ? -INFINITY : S[r];
}

// byte offset of a block in the cache
__device__ __forceinline__ unsigned long long block_bytes(const WaveCtx& cx, int blk) {
  return (unsigned long long)((unsigned)blk < (unsigned)cx.num_blocks ? (unsigned)blk : 0u) * cx.blk_bytes;
}

// Id of this wave's block of a tile (past the workgroup's last block: that block again).  It is loaded an iteration before the
// fetch that needs it, into a vector register: a scalar load would have every operand read from LDS wait for it.
__device__ __forceinline__ int load_id(const WaveCtx& cx, const int* bt, int tile) {
  int i = min(4 * tile + cx.wb, cx.last_blk);
  asm("" : "+v"(i));
  return bt[i];
}

// Load instructions J and, where there are as many, J + 1 of this wave's K run.  16-bit: instruction J takes eight rows of one
// 64-dimension part, rows 8 (J & 1) .. + 7 of part J >> 1; bytes: 1 KB of the run as it lies.  A K row past the last
// token may hold anything: it only produces scores of keys beyond every row's horizon, which are overwritten with -inf
// before use, and it still lies inside a block the sequence owns.
template <int D, bool KV8, int NW, int J>
__device__ __forceinline__ void fetch_k(const WaveCtx& cx, unsigned long long boff, unsigned lds) {
  using C = Cfg<D, KV8, NW>;
  dma16<(C::NI > 1 ? 2 : 1), 1024 * J>(cx.kbase + boff, cx.k_off + (KV8 ? 0 : J), lds);
}

// The same of this wave's V run: 1 KB each as it lies.  Rows past the last token are cleared once they have landed
// (clear_past_end): P is 0 there, and 0 * NaN would poison the output.
template <int D, bool KV8, int NW, int J>
__device__ __forceinline__ void fetch_v(const WaveCtx& cx, unsigned long long boff, unsigned lds) {
  using C = Cfg<D, KV8, NW>;
  dma16<(C::NI > 1 ? 2 : 1), 1024 * J>(cx.vbase + boff, cx.v_off, lds);
}

// whole runs
template <int D, bool KV8, int NW>
__device__ __forceinline__ void fetch_v_tile(const WaveCtx& cx, unsigned long long boff, unsigned lds) {
  fetch_v<D, KV8, NW, 0>(cx, boff, lds);
  if constexpr (Cfg<D, KV8, NW>::NI > 2) fetch_v<D, KV8, NW, 2>(cx, boff, lds);
}
template <int D, bool KV8, int NW>
__device__ __forceinline__ void fetch_k_tile(const WaveCtx& cx, unsigned long long boff, unsigned lds) {
  fetch_k<D, KV8, NW, 0>(cx, boff, lds);
  if constexpr (Cfg<D, KV8, NW>::NI > 2) fetch_k<D, KV8, NW, 2>(cx, boff, lds);
}

// LDS positions, in bytes from the start of the buffers: this wave's share of K buffer `b` (8-bit caches: its block) and of V
// buffer `b`, its staging area, its 32 rows of output
template <int D, bool KV8, int NW> __device__ __forceinline__ unsigned k_rows(const WaveCtx& cx, int b) {
  using C = Cfg<D, KV8, NW>;
  return b * C::TILE + cx.wb * C::KBLK + (KV8 ? 0 : cx.ws * C::SHARE);
}
template <int D, bool KV8, int NW> __device__ __forceinline__ unsigned v_rows(const WaveCtx& cx, int b) {
  using C = Cfg<D, KV8, NW>;
  return (2 + b) * C::TILE + cx.wb * kBlock * C::RB + (KV8 ? 0 : cx.ws * C::SHARE);
}
template <int D, bool KV8, int NW> __device__ __forceinline__ unsigned staged(const WaveCtx& cx) {
  return 4 * Cfg<D, KV8, NW>::TILE + cx.w * Cfg<D, KV8, NW>::STAGE;
}
template <int D, bool KV8, int NW> __device__ __forceinline__ unsigned out_rows(const WaveCtx& cx) {
  return Cfg<D, KV8, NW>::OUT + cx.w * kWaveRows * Cfg<D, KV8, NW>::RB;
}

// operand of score k-step s, half tile `half`; `addr`: LDS addresses of this lane's row of the K buffer
template <int D, bool KV8, int NW>
__device__ __forceinline__ bf16x8 read_k(const unsigned (&addr)[4], int s, int half) {
  return *(const __attribute__((address_space(3))) bf16x8*)(size_t)(addr[s & 3] + (s >> 2) * (kBlock * 128) + half * 2 * Cfg<D, KV8, NW>::KBLK);
}

// operand of P V: keys 16 m .. 16 m + 15 of the V buffer, dimensions 32 mb .. 32 mb + 31
template <int D>
__device__ __forceinline__ bf16x8 read_vt(const unsigned (&addr)[4], int m, int mb) {
  union { v4i16 h[2]; bf16x8 v; } av;
  const unsigned a = addr[mb] + 16 * m * 2 * D;
  av.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(size_t)a);
  av.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4i16*)(size_t)(a + 8 * 2 * D));
  return av.v;
}

// 8-bit caches: row of the block that a lane's piece of load j belongs to
template <int D, int NW> __device__ __forceinline__ int piece_row(const WaveCtx& cx, int j) {
  using C = Cfg<D, true, NW>;
  return cx.ws * C::ROWS + C::RPI * j + cx.lane / C::LPR;
}
// eight bytes (row `r` of this wave's block, 16-byte chunk `ch` of the bf16 row) widened into the block's rows of a
// K or V buffer
template <int D>
__device__ __forceinline__ void widen_to_k(unsigned char* rows, int r, int ch, unsigned lo, unsigned hi) {
  *reinterpret_cast<uint4*>(rows + (ch >> 3) * (kBlock * 128) + r * 128 + (((ch & 7) ^ k_swizzle(r)) << 4)) =
      e4m3x8_to_bf16x8(make_uint2(lo, hi));
}
template <int D>
__device__ __forceinline__ void widen_to_v(unsigned char* rows, int r, int ch, unsigned lo, unsigned hi) {
  *reinterpret_cast<uint4*>(rows + r * 2 * D + ((ch ^ v_swizzle<D>(r)) << 4)) = e4m3x8_to_bf16x8(make_uint2(lo, hi));
}

// What a wave carries from half tile to half tile.
template <int D>
struct Pipe {
  f32x16 S[2];            // raw scores (and exponentials) of a tile's two halves
  u32x4 P[2][2];          // probabilities of a half tile, rounded: [half][16-key group]
  bf16x8 ka[4], va[4];    // operand rings
  unsigned k_addr[4];     // LDS positions of this lane's K row in the buffer being read, one per k-step of a 64-dimension part
  unsigned v_addr[4];     // the same for the transposed V reads, one per 32-dimension block of the output
  f32x16 O[D / 32];
  float l;                // normaliser
  float am[kMaxSpans];    // span sums
};

// Exponentials of half a tile, EPS elements to a slot and software pipelined: an element's multiply-add, its exponential,
// and its sum and rounding lie in three neighbouring slots, so that none waits for the one before it.
struct HalfExp { float x[4], sum; };

template <int EPS>
__device__ __forceinline__ void exp_begin(const WaveCtx& cx, const f32x16& S, float m, HalfExp& h) {
  h.sum = 0.0f;
#pragma unroll
  for (int e = 0; e < EPS; ++e) h.x[e] = __builtin_fmaf(S[e], cx.c, -m);
}
__device__ __forceinline__ void exp_done(const f32x16& S, HalfExp& h, u32x4 (&P)[2], int e) {   // element e of S is an exponential
  h.sum += S[e];
  if (e & 1) P[e >> 3][(e & 7) >> 1] = pack_bf16(S[e - 1], S[e]);
}
template <int EPS>
__device__ __forceinline__ void exp_slot(const WaveCtx& cx, f32x16& S, float m, HalfExp& h, u32x4 (&P)[2], int j) {
#pragma unroll
  for (int e = 0; e < EPS; ++e) {
    const int n = j * EPS + e;
    float ex = fast_exp2(h.x[e]);
    asm volatile("" : "+v"(ex));       // (in this slot, not where it is used)
    if (n + EPS < 16) h.x[e] = __builtin_fmaf(S[n + EPS], cx.c, -m);
    if (j > 0) exp_done(S, h, P, n - EPS);
    S[n] = ex;
  }
}
template <int EPS>
__device__ __forceinline__ float exp_end(const f32x16& S, HalfExp& h, u32x4 (&P)[2]) {
#pragma unroll
  for (int e = 16 - EPS; e < 16; ++e) exp_done(S, h, P, e);
  return h.sum;
}

// Spans of a sequence; no span that is not behind us begins before key `lo` or ends after key `hi`.
struct Spans { int a[kMaxSpans], b[kMaxSpans], lo, hi, n; };

template <int S = 0>
__device__ __forceinline__ void add_span(const WaveCtx& cx, const Spans& sp, int key0, const f32x16& ex, float sum,
                                         float (&am)[kMaxSpans], int& next) {
  if constexpr (S < kMaxSpans) {
    if (S >= sp.n) return;
    const int a = sp.a[S], b = sp.b[S];
    if (b > key0 && a < key0 + 32) {
      if (a <= key0 && b >= key0 + 32) {
        am[S] += sum;
      } else {
        float acc = 0.0f;
        const unsigned lo = a - key0 - 4 * cx.hf, len = b - a;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc += 8 * (r >> 2) + (r & 3) - lo < len ? ex[r] : 0.0f;
        am[S] += acc;
      }
    }
    if (b > key0 + 32) next = min(next, a);
    add_span<S + 1>(cx, sp, key0, ex, sum, am, next);
  }
}

// Span sums of the half tile at key0 from its exponentials (masked keys are 0).
template <int D>
__device__ __forceinline__ void add_spans(const WaveCtx& cx, Spans& sp, int key0, const f32x16& ex, float sum,
                                          float (&am)[kMaxSpans]) {
  if (__builtin_expect(sp.hi > key0 && sp.lo < key0 + 32, 0)) {
    int next = sp.hi;
    add_span(cx, sp, key0, ex, sum, am, next);
    sp.lo = next;
  }
}

// the barrier after which the tiles fetched during an iteration may be read and the ones read in it overwritten
template <bool KV8>
__device__ __forceinline__ void tile_barrier() {
  if constexpr (!KV8) wait_vmem();     // (bytes only go to the wave's own staging area)
  __syncthreads();
}

// Every kRaiseTiles tiles, where some lane's normaliser has reached kRaiseSum: the reference of such a row is raised by the whole
// powers of two in it, and everything that counts from it comes down by them: output, sums, the probabilities that wait in
// P[0].  A row whose output has overflowed already is marked by its normaliser.  Scores of unit spread never get here
// (normalisers of 2^15 at 128 k tokens).
// What a wave pays for it is a comparison that its branch waits for, up to 0.6 % (32 k prompt 13.47 -> 13.53 ms, 16 ragged prompts 242 -> 243 us, at head
// size 64 143.5 -> 144.5; every tile 1 % more; at the end of a tile's code 80 vector registers are spilled, as the compiler
// then keeps the output twice, and in its middle head size 64 takes 10 % more).  Eight tiles instead of four: 0.2 % less, but rounding of up to 8 %
// more in span masses under scores of 16 units' spread.
// Before, rows that had risen by 2^64 were done over.  Keys from 96 on with scores of 12 natural units' spread, 32 / 8 heads, done
// over, now, and under a running maximum raised by 2^8 at a time: 2048 tokens 250, 44.7 and 51.7 us, 8192 2513, 472 and 501, 16 ragged prompts
// 954, 252 and 272, at head size 64 531, 146 and 163.
constexpr float kRaiseSum = 0x1p24f, kSumLimit = 0x1p120f;
constexpr int kRaiseTiles = 4;
template <int D, bool PROBE>
__device__ __forceinline__ void raise_reference(Pipe<D>& t, float& m) {
  const float l = half_max(t.l);
  const int k = l >= kRaiseSum && l < kSumLimit ? __builtin_amdgcn_frexp_expf(l) - 1 : 0;
  // what the reference really rises by: rounded where it has a fraction, and to less or nothing at all where it is far beyond 2^24
  const float raised = m + (float)k, by = raised - m;
  const float f = fast_exp2(-by), f16 = __builtin_ldexpf(1.0f, -(int)__builtin_rintf(by));      // (16-bit values keep their bits)
  m = raised;
  float z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      z[r & 3] = __builtin_fmaf(t.O[mb][r], 0.0f, z[r & 3]);
      t.O[mb][r] *= f;
    }
  t.l = t.l * f + (k > 0 ? (z[0] + z[1]) + (z[2] + z[3]) : 0.0f);
  if constexpr (PROBE) {
#pragma unroll
    for (int i = 0; i < kMaxSpans; ++i) t.am[i] *= f;
  }
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int i = 0; i < 4; ++i) t.P[0][g][i] = pack_bf16(bf16_lo(t.P[0][g][i]) * f16, bf16_hi(t.P[0][g][i]) * f16);
}

// ---- one pipelined iteration --------------------------------------------------------------
// On entry P[0] holds the probabilities of the first half of tile kt, S[1] the raw scores of its second half, and the
// rings the first operands of K(kt+1) and V(kt).  Half a tile at a time,
//   the matrix cores compute the scores of a half tile of kt+1 and P V of a half tile of kt, alternating,
//   the vector ALUs the exponentials of the half tile between the two,
// one matrix instruction and 16 / SLOTS exponentials to a slot; the slots are fenced so that the streams stay interleaved.
// Fetches of V(kt+1) and K(kt+2) (8-bit caches: the bytes of V(kt+2) and K(kt+3), once those of V(kt+1) and K(kt+2) are
// widened) are issued first; the barrier that closes the iteration stands as many slots before its end as operands are
// in flight, so nothing waits for the first operands of the next one.  A fetch behind the last tile takes the last tile's last block again:
// the buffers are free by then and are never read again.
// boff: cache offset of this wave's block of the tile whose V comes next (its K was the last one requested); id: its block
// of the tile after that.
template <int D, bool KV8, int NW, bool PROBE>
__device__ __forceinline__ void tile_iter(const WaveCtx& cx, unsigned char* smem, int kt, int& id,
                                          const int* bt, unsigned long long& boff, Pipe<D>& t, float m,
                                          const bf16x8 (&qf)[D / 16], Spans& sp) {
  using C = Cfg<D, KV8, NW>;
  constexpr int NS = C::SLOTS, EPS = 16 / NS, R = C::RING, NQ = C::KSTEPS, NP = 2 * C::MB, NI = C::NI;
  static_assert(NQ == NP && 2 * NQ % R == 0, "scores and P V alternate; the rings turn whole rounds");
  constexpr int BAR = 2 * NS - 2 * R + 2;              // slot in front of which the barrier stands
  const unsigned v_dst = v_rows<D, KV8, NW>(cx, (kt + 1) & 1), k_dst = k_rows<D, KV8, NW>(cx, kt & 1);
  const unsigned stage = staged<D, KV8, NW>(cx);
  uint4 st[2];                     // staged pieces on their way through the registers
  unsigned long long next_boff = 0;
  float sum[2];
  HalfExp h;
  // operand `n` of the scores / of P V, counted through the iteration; beyond it, the next iteration's
  auto request_k = [&](auto n) { t.ka[n % R] = read_k<D, KV8, NW>(t.k_addr, n % NQ, n % (2 * NQ) / NQ); };
  auto request_v = [&](auto n) { t.va[n % R] = read_vt<D>(t.v_addr, n % (2 * NP) / C::MB, n % C::MB); };
  static_for<2 * NS>([&](auto slot) {
    constexpr int i = slot, half = i / NS, j = i % NS, u = j / 2;
    // half 0: exponentials of the second half of kt, half 1: of the first half of kt + 1
    f32x16& Sx = t.S[half ^ 1];
    const int key0 = kTileKeys * kt + 32 * (half + 1);
    if (j == 0) {
      if (key0 + 31 > cx.pos_min) mask_half(cx, key0, Sx);
      __builtin_amdgcn_sched_barrier(0);
      exp_begin<EPS>(cx, Sx, m, h);
    }
    if (i == BAR) {
      __builtin_amdgcn_sched_barrier(0);
      tile_barrier<KV8>();
#pragma unroll
      for (int b = 0; b < 4; ++b) {       // on to the other buffers
        t.k_addr[b] += (kt & 1) ? C::TILE : -C::TILE;
        if (b < C::MB) t.v_addr[b] += (kt & 1) ? -C::TILE : C::TILE;
      }
      // what could not be requested before
      static_for<BAR / 2 + R - 2 * NQ>([&](auto k) {
        request_k(std::integral_constant<int, 2 * NQ + k>{});
        request_v(std::integral_constant<int, 2 * NP + k>{});
      });
      __builtin_amdgcn_sched_barrier(0);
    }
    if (j % 2 == 0) {
      const f32x16 z = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
      constexpr int n = half * NQ + u;
      t.S[half] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.ka[n % R], qf[u], u == 0 ? z : t.S[half], 0, 0, 0);
      if constexpr (n + R < 2 * NQ || i >= BAR) request_k(std::integral_constant<int, n + R>{});
    } else {
      constexpr int n = half * NP + u;
      t.O[n % C::MB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.va[n % R], as_bf16x8(t.P[half][(n / C::MB) % 2]), t.O[n % C::MB], 0, 0, 0);
      if constexpr (n + R < 2 * NP || i >= BAR) request_v(std::integral_constant<int, n + R>{});
    }
    if constexpr (!KV8) {
      if constexpr (i == 0) {
        next_boff = block_bytes(cx, __builtin_amdgcn_readfirstlane(id));
        id = load_id(cx, bt, kt + 3);
      }
      if constexpr (i == 1) fetch_v<D, false, NW, 0>(cx, boff, cx.lds_base + v_dst);
      if constexpr (i == 3 && NI > 2) fetch_v<D, false, NW, 2>(cx, boff, cx.lds_base + v_dst);
      if constexpr (i == 5) boff = next_boff;
      if constexpr (i == 5) fetch_k<D, false, NW, 0>(cx, boff, cx.lds_base + k_dst);
      if constexpr (i == 7 && NI > 2) fetch_k<D, false, NW, 2>(cx, boff, cx.lds_base + k_dst);
    } else {
      // piece p = 0 .. 2 NI - 1 (K run, then V run): read in slice 2p, its halves widened in slices 2p+2 and 2p+3
      if (i == 0) wait_vmem();
      if (i % 2 == 0 && i / 2 < 2 * NI) {
        const int p = i / 2;
        st[p & 1] = *reinterpret_cast<const uint4*>(smem + stage + (p / NI) * C::SHARE + (p % NI) * 1024 + 16 * cx.lane);
      }
      if (i >= 2 && (i - 2) / 2 < 2 * NI) {
        const int p = (i - 2) / 2, hh = i % 2;
        const int r = piece_row<D, NW>(cx, p % NI), ch = 2 * (cx.lane % C::LPR) + hh;
        const uint4& v = st[p & 1];
        if (p < NI) widen_to_k<D>(smem + k_dst, r, ch, hh ? v.z : v.x, hh ? v.w : v.y);
        else widen_to_v<D>(smem + v_dst, r, ch, hh ? v.z : v.x, hh ? v.w : v.y);
      }
      // the staging area is free once its last piece sits in registers
      constexpr int F = 4 * NI + 2;
      static_assert(F + 2 < 2 * NS, "");
      if constexpr (i == F) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      if constexpr (i == F - 1) next_boff = block_bytes(cx, __builtin_amdgcn_readfirstlane(id));
      if constexpr (i == F - 1) id = load_id(cx, bt, kt + 4);
      if constexpr (i == F) fetch_v<D, true, NW, 0>(cx, boff, cx.lds_base + stage + C::SHARE);
      if constexpr (i == F + 2) boff = next_boff;
      if constexpr (i == F + 2) fetch_k<D, true, NW, 0>(cx, boff, cx.lds_base + stage);
    }
    exp_slot<EPS>(cx, Sx, m, h, t.P[half ^ 1], j);
    __builtin_amdgcn_sched_barrier(0);
    if (j == NS - 1) {
      sum[half] = exp_end<EPS>(Sx, h, t.P[half ^ 1]);
      asm volatile("" : "+v"(t.P[half ^ 1][0]), "+v"(t.P[half ^ 1][1]), "+v"(sum[half]));      // (likewise)
      if constexpr (PROBE) {
        add_spans<D>(cx, sp, key0, Sx, sum[half], t.am);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  });
  t.l += sum[0] + sum[1];
}

// The same iteration for a wave that has no key left: the tiles behind its rows' positions are for the other row blocks
// of the workgroup (groups of fewer than four heads), and it only fetches its cache blocks of them.  (Going through
// them with every score masked would let 0 * Inf from their values into its rows.)
template <int D, bool KV8, int NW>
__device__ __forceinline__ void fetch_iter(const WaveCtx& cx, unsigned char* smem, int kt, int& id,
                                           const int* bt, unsigned long long& boff) {
  using C = Cfg<D, KV8, NW>;
  constexpr int NI = C::NI;
  if constexpr (KV8) {
    const unsigned v_dst = v_rows<D, KV8, NW>(cx, (kt + 1) & 1), k_dst = k_rows<D, KV8, NW>(cx, kt & 1), stage = staged<D, KV8, NW>(cx);
    wait_vmem();
#pragma unroll
    for (int q = 0; q < 2 * NI; ++q) {
      const uint4 st = *reinterpret_cast<const uint4*>(smem + stage + (q / NI) * C::SHARE + (q % NI) * 1024 + 16 * cx.lane);
      const int r = piece_row<D, NW>(cx, q % NI), ch = 2 * (cx.lane % C::LPR);
      if (q < NI) {
        widen_to_k<D>(smem + k_dst, r, ch, st.x, st.y);
        widen_to_k<D>(smem + k_dst, r, ch + 1, st.z, st.w);
      } else {
        widen_to_v<D>(smem + v_dst, r, ch, st.x, st.y);
        widen_to_v<D>(smem + v_dst, r, ch + 1, st.z, st.w);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const unsigned long long next = block_bytes(cx, __builtin_amdgcn_readfirstlane(id));
    id = load_id(cx, bt, kt + 4);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the staging area is free
    fetch_v_tile<D, true, NW>(cx, boff, cx.lds_base + stage + C::SHARE);
    boff = next;
    fetch_k_tile<D, true, NW>(cx, boff, cx.lds_base + stage);
    tile_barrier<true>();
  } else {
    const unsigned long long next = block_bytes(cx, __builtin_amdgcn_readfirstlane(id));
    id = load_id(cx, bt, kt + 3);
    fetch_v_tile<D, false, NW>(cx, boff, cx.lds_base + v_rows<D, KV8, NW>(cx, (kt + 1) & 1));
    boff = next;
    fetch_k_tile<D, false, NW>(cx, boff, cx.lds_base + k_rows<D, KV8, NW>(cx, kt & 1));
    tile_barrier<false>();
  }
}

// This wave's rows past the last token of the V buffer that holds the last tile.
template <int D, bool KV8, int NW>
__device__ __forceinline__ void clear_past_end(const WaveCtx& cx, unsigned char* smem, int kt) {
  using C = Cfg<D, KV8, NW>;
  const int first = cx.L - (kTileKeys * kt + kBlock * cx.wb + C::ROWS * cx.ws);      // first row of this wave's share past the end
  unsigned char* const rows = smem + v_rows<D, KV8, NW>(cx, kt & 1) + (KV8 ? cx.ws * C::ROWS * C::RB : 0);
#pragma unroll
  for (int j = 0; j < C::ROWS * C::CH / 64; ++j) {
    const int r = (64 / C::CH) * j + cx.lane / C::CH;
    if (r >= first) *reinterpret_cast<uint4*>(rows + r * C::RB + 16 * (cx.lane % C::CH)) = make_uint4(0, 0, 0, 0);
  }
}

// What is left once all K and V tiles lie in LDS: the last tile's second half and P V of both.
template <int D, bool KV8, int NW, bool PROBE>
__device__ __forceinline__ void last_tile(const WaveCtx& cx, int kt, Pipe<D>& t, float m, int pos_max, Spans& sp) {
  using C = Cfg<D, KV8, NW>;
  constexpr int R = C::RING, NP = 2 * C::MB, EPS = 16 / NP;
  const int key0 = kTileKeys * kt + 32;
  const bool second = key0 <= pos_max;            // some row sees keys of the second half
  HalfExp h;
  if (second) {
    mask_half(cx, key0, t.S[1]);
    exp_begin<EPS>(cx, t.S[1], m, h);
  }
  __builtin_amdgcn_sched_barrier(0);
  static_for<NP>([&](auto slot) {
    constexpr int n = slot;
    t.O[n % C::MB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.va[n % R], as_bf16x8(t.P[0][n / C::MB]), t.O[n % C::MB], 0, 0, 0);
    t.va[n % R] = read_vt<D>(t.v_addr, (n + R) / C::MB, (n + R) % C::MB);
    if (second) exp_slot<EPS>(cx, t.S[1], m, h, t.P[1], n);
    __builtin_amdgcn_sched_barrier(0);
  });
  if (!second) return;
  const float sum = exp_end<EPS>(t.S[1], h, t.P[1]);
  t.l += sum;
  if constexpr (PROBE) add_spans<D>(cx, sp, key0, t.S[1], sum, t.am);
  __builtin_amdgcn_sched_barrier(0);
  static_for<NP>([&](auto slot) {
    constexpr int n = NP + slot;
    t.O[n % C::MB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t.va[n % R], as_bf16x8(t.P[1][(n - NP) / C::MB]), t.O[n % C::MB], 0, 0, 0);
    if (n + R < 2 * NP) t.va[n % R] = read_vt<D>(t.v_addr, (n + R) / C::MB, (n + R) % C::MB);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// The first tile's scores, on which the softmax reference of each row rests (`m`: the row's maximum in them), and the
// probabilities of its first half.
// On entry K(0) lies in LDS; V(0) and K(1) are on their way, and there on return.
template <int D, bool KV8, int NW>
__device__ __forceinline__ void first_half(const WaveCtx& cx, const bf16x8 (&qf)[D / 16], Pipe<D>& t, float& m) {
  using C = Cfg<D, KV8, NW>;
  constexpr int EPS = 16 / C::SLOTS;
  // K reads: lane (row qi [+32], half hf) reads chunk 2s + hf of a 64-dimension part
  const int qi = cx.lane & 31;
#pragma unroll
  for (int s = 0; s < 4; ++s) t.k_addr[s] = cx.lds_base + (unsigned)(qi >> 4) * C::KBLK + (unsigned)(qi & 15) * 128 + ((unsigned)((2 * s + cx.hf) ^ k_swizzle(qi)) << 4);
  {
    // transposed V reads: within a 16-lane group lane s supplies row (s >> 2) and 8-byte piece (s & 3)
    const int g = cx.lane >> 4, s16 = cx.lane & 15;
    const int hfv = g >> 1, ddhalf = g & 1;
    const unsigned rowc = (unsigned)(4 * hfv + (s16 >> 2)) * C::RB;
    const unsigned lowc = (unsigned)(2 * ddhalf + ((s16 & 3) >> 1)) * 16 + (unsigned)(s16 & 1) * 8;
    const unsigned xorc = (unsigned)v_swizzle<D>(s16 >> 2) * 16;
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) t.v_addr[mb] = cx.lds_base + 2 * C::TILE + ((rowc | (lowc ^ xorc)) ^ (64u * mb));
  }
#pragma unroll
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int r = 0; r < 16; ++r) t.S[half][r] = 0.0f;
  }
#pragma unroll
  for (int s = 0; s < C::KSTEPS; ++s)
#pragma unroll
    for (int half = 0; half < 2; ++half)
      t.S[half] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k<D, KV8, NW>(t.k_addr, s, half), qf[s], t.S[half], 0, 0, 0);
  if (31 > cx.pos_min) mask_half(cx, 0, t.S[0]);
  if (63 > cx.pos_min) mask_half(cx, 32, t.S[1]);
  float mx = fmaxf(t.S[0][0], t.S[1][0]);
#pragma unroll
  for (int r = 1; r < 16; ++r) mx = fmaxf(mx, fmaxf(t.S[0][r], t.S[1][r]));
  mx = half_max(mx) * cx.c;
  m = mx == -INFINITY ? 0.0f : mx;
  HalfExp h;
  exp_begin<EPS>(cx, t.S[0], m, h);
#pragma unroll
  for (int j = 0; j < C::SLOTS; ++j) exp_slot<EPS>(cx, t.S[0], m, h, t.P[0], j);
  t.l = exp_end<EPS>(t.S[0], h, t.P[0]);
  // V(0) and K(1) (8-bit caches: they were there before, but every wave has to be done with K(0))
  if constexpr (!KV8) wait_vmem();
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    t.k_addr[s] += C::TILE;
    asm volatile("" : "+v"(t.k_addr[s]));       // (in registers of their own)
    if (s < C::MB) asm volatile("" : "+v"(t.v_addr[s]));
  }
#pragma unroll
  for (int n = 0; n < C::RING; ++n) {
    t.ka[n] = read_k<D, KV8, NW>(t.k_addr, n, 0);
    t.va[n] = read_vt<D>(t.v_addr, n / C::MB, n % C::MB);
  }
}

// All that follows.  mine: tiles up to the position of the wave's last row, pos_max.  SHARED: that can be fewer than the
// workgroup's.
template <int D, bool KV8, int NW, bool SHARED, bool PROBE>
__device__ __forceinline__ void run_tiles(const WaveCtx& cx, unsigned char* smem, int ntiles, int mine, int pos_max, int id,
                                          unsigned long long& boff, const bf16x8 (&qf)[D / 16], Pipe<D>& t, float& m,
                                          Spans& sp, const int* bt) {
  using C = Cfg<D, KV8, NW>;
  // The lane values are made opaque here: what is derived from them would otherwise be computed once for both
  // instantiations (probing or not) and spilled instead of recomputed.
  WaveCtx cy = cx;
  asm volatile("" : "+v"(cy.pos), "+v"(cy.k_off[0]), "+v"(cy.v_off[0]), "+v"(cy.hf), "+v"(cy.lane));
  cy.v_off[1] = cy.v_off[0];
  if constexpr (KV8) cy.k_off[1] = cy.k_off[0];
  else if constexpr (C::NI > 1) asm volatile("" : "+v"(cy.k_off[1]));
  if constexpr (C::NI > 2) asm volatile("" : "+v"(cy.k_off[2]), "+v"(cy.k_off[3]));
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) t.O[mb][r] = 0.0f;
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) t.am[s] = 0.0f;
  first_half<D, KV8, NW>(cy, qf, t, m);
  if constexpr (PROBE) add_spans<D>(cy, sp, 0, t.S[0], t.l, t.am);
  __builtin_amdgcn_sched_barrier(0);
  const int full = SHARED ? min(mine, ntiles - 1) : ntiles - 1;
  int kt = 0;
  while (kt < full) {
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(t.l >= kRaiseSum) != 0, 0)) raise_reference<D, PROBE>(t, m);
    const int stop = min(full, kt + kRaiseTiles);
    for (; kt < stop; ++kt) tile_iter<D, KV8, NW, PROBE>(cy, smem, kt, id, bt, boff, t, m, qf, sp);
  }
  if (SHARED)
    for (; kt < ntiles - 1; ++kt) fetch_iter<D, KV8, NW>(cy, smem, kt, id, bt, boff);
  if (kTileKeys * ntiles > cy.L) {        // (the same for all waves)
    clear_past_end<D, KV8, NW>(cy, smem, ntiles - 1);
    __syncthreads();
#pragma unroll
    for (int n = 0; n < C::RING; ++n) t.va[n] = read_vt<D>(t.v_addr, n / C::MB, n % C::MB);
  }
  if (!SHARED || mine == ntiles) last_tile<D, KV8, NW, PROBE>(cy, kt, t, m, pos_max, sp);
}

// 16-bit caches: where the two halves of this wave's query rows pass through LDS on their way to registers.  Four waves: the first
// lies in its rows of V buffer 1, which it fetches itself after that.  D = 128: a half is one 64-dimension part of all rows, D = 64: 16 rows.
template <int D, int NW>
__device__ __forceinline__ unsigned q_half(const WaveCtx& cx, int i) {
  using C = Cfg<D, false, NW>;
  if (NW == 8) return out_rows<D, false, NW>(cx) + i * C::QHALF;
  return i == 0 ? v_rows<D, false, NW>(cx, 1) : 4 * C::TILE + cx.w * C::QHALF;
}

// Requests the query rows, K(0), V(0) and K(1) of an item, in this order.  rows: the wave's first query row, of `n_rows`, which
// are `stride` bytes apart (rows past the last repeat it).
template <int D, int NW>
__device__ __forceinline__ void first_tiles(const WaveCtx& cx, unsigned long long rows, int n_rows, unsigned stride,
                                            unsigned long long boff0, unsigned long long boff1) {
  using C = Cfg<D, false, NW>;
#pragma unroll
  for (int j = 0; j < 4; j += 2) {      // 16 rows of 64 dimensions: two instructions of eight
    unsigned voff[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 8 * (j + i) + cx.lane / 8;
      voff[i] = (unsigned)min(r, n_rows - 1) * stride + (unsigned)((cx.lane % 8) ^ k_swizzle(r)) * 16 + 1024 * (1 - i);
    }
#pragma unroll
    for (int part = 0; part < D / 64; ++part)
      dma16<2, 0>(rows - 1024 + 128 * part, voff, cx.lds_base + (D == 128 ? q_half<D, NW>(cx, part) + 1024 * j : q_half<D, NW>(cx, j / 2)));
  }
  fetch_k_tile<D, false, NW>(cx, boff0, cx.lds_base + k_rows<D, false, NW>(cx, 0));
  fetch_v_tile<D, false, NW>(cx, boff0, cx.lds_base + v_rows<D, false, NW>(cx, 0));
  fetch_k_tile<D, false, NW>(cx, boff1, cx.lds_base + k_rows<D, false, NW>(cx, 1));
}

template <int D, int NW>
__device__ __forceinline__ void read_queries(const WaveCtx& cx, const unsigned char* smem, bf16x8 (&qf)[D / 16]) {
  const int qi = cx.lane & 31;
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    const unsigned a = D == 128 ? q_half<D, NW>(cx, s >> 2) + qi * 128 : q_half<D, NW>(cx, qi >> 4) + (qi & 15) * 128;
    qf[s] = *reinterpret_cast<const bf16x8*>(smem + a + (((2 * (s & 3) + cx.hf) ^ k_swizzle(qi)) << 4));
  }
}

// 8-bit caches: K(0), V(0) and K(1) through registers (there is nothing to overlap with yet), the bytes of V(1) and K(2)
// into the staging area.
template <int D, int NW>
__device__ __forceinline__ void first_tiles_kv8(const WaveCtx& cx, unsigned char* smem, unsigned long long boff0,
                                                unsigned long long boff1, unsigned long long boff2) {
  using C = Cfg<D, true, NW>;
  constexpr int NI = C::NI;
  uint4 k0[NI], v0[NI], k1[NI];
#pragma unroll
  for (int jj = 0; jj < NI; ++jj) {
    const int r = piece_row<D, NW>(cx, jj);
    const unsigned piece = 16 * (cx.lane % C::LPR);
    k0[jj] = load_global16((global_bytes)(cx.kbase + boff0 + r * D + piece));
    v0[jj] = load_global16((global_bytes)(cx.vbase + boff0 + r * D + piece));
    k1[jj] = load_global16((global_bytes)(cx.kbase + boff1 + r * D + piece));
  }
  // V(1), then K(2): the order in which the loop fetches
  const unsigned lds_stage = cx.lds_base + staged<D, true, NW>(cx);
  fetch_v_tile<D, true, NW>(cx, boff1, lds_stage + C::SHARE);
  fetch_k_tile<D, true, NW>(cx, boff2, lds_stage);
  unsigned char* const kd = smem + k_rows<D, true, NW>(cx, 0);
  unsigned char* const vd = smem + v_rows<D, true, NW>(cx, 0);
#pragma unroll
  for (int jj = 0; jj < NI; ++jj) {
    const int r = piece_row<D, NW>(cx, jj), ch = 2 * (cx.lane % C::LPR);
    widen_to_k<D>(kd, r, ch, k0[jj].x, k0[jj].y);
    widen_to_k<D>(kd, r, ch + 1, k0[jj].z, k0[jj].w);
    widen_to_v<D>(vd, r, ch, v0[jj].x, v0[jj].y);
    widen_to_v<D>(vd, r, ch + 1, v0[jj].z, v0[jj].w);
    widen_to_k<D>(kd + C::TILE, r, ch, k1[jj].x, k1[jj].y);
    widen_to_k<D>(kd + C::TILE, r, ch + 1, k1[jj].z, k1[jj].w);
  }
}

// One work item: rows [row0, row0 + rows_per_wg) of sequence `seq` (context L, n rows, first q row
// qbase) for the heads of (kvh, hg).
struct Item { int kvh, hg, seq, row0, L, n, qbase; };

// What a wave knows about its part of an item beyond WaveCtx.
struct WaveItem {
  int ntiles, mine, pos_max, head, wrow0;
  bool active;
  int pslot, qsel_b, qsel_e;      // probed head's place in the list (-1: not probed), selected rows
};

// Normalise, transpose through LDS (16-byte chunks swizzled by row; each wave in rows of its own of the K buffers, which
// are free), coalesced stores; the span sums.  rows: bit per row of the wave that is to be written.
template <int D, bool KV8, int NW, bool PROBE>
__device__ __forceinline__ void finish(const AttnParams& p, unsigned char* smem, const Item& it, const WaveItem& wi, const WaveCtx& cx,
                                       const Spans& sp, const Pipe<D>& t, float l_tot, unsigned rows) {
  using C = Cfg<D, KV8, NW>;
  const float inv_l = 1.0f / l_tot;
  const float inv = KV8 ? inv_l * p.v_scale[it.kvh] : inv_l;     // `out` carries the value scale, `mass` does not
  unsigned char* const ot = smem + out_rows<D, KV8, NW>(cx);
  const int qi = cx.lane & 31;
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      uint2 v;
      v.x = pack_bf16(t.O[mb][4 * g4] * inv, t.O[mb][4 * g4 + 1] * inv);
      v.y = pack_bf16(t.O[mb][4 * g4 + 2] * inv, t.O[mb][4 * g4 + 3] * inv);
      const int ch = 4 * mb + g4;
      *reinterpret_cast<uint2*>(ot + qi * C::RB + ((ch ^ out_swizzle<D>(qi)) << 4) + 8 * cx.hf) = v;
    }
  in_order();
  __bf16* const og = static_cast<__bf16*>(p.out);
#pragma unroll
  for (int j = 0; j < C::CH / 2; ++j) {
    const int rr = cx.lane / C::CH + (64 / C::CH) * j;
    const int ch = cx.lane % C::CH;
    const int tr = wi.wrow0 + rr;
    if (rows >> rr & 1) {
      const uint4 v = *reinterpret_cast<const uint4*>(ot + rr * C::RB + ((ch ^ out_swizzle<D>(rr)) << 4));
      *reinterpret_cast<uint4*>(og + ((size_t)(it.qbase + tr) * p.Hq + wi.head) * D + 8 * ch) = v;
    }
  }
  if constexpr (PROBE) {
#pragma unroll
    for (int s = 0; s < kMaxSpans; ++s) {
      if (s < sp.n) {
        const float a_tot = t.am[s] + __shfl_xor(t.am[s], 32);
        const int tr = wi.wrow0 + qi;
        if (cx.hf == 0 && (rows >> qi & 1) && tr >= wi.qsel_b && tr < wi.qsel_e)
          p.mass[(((size_t)it.seq * p.P + wi.pslot) * p.NQ + (tr - wi.qsel_b)) * p.S + s] = a_tot * inv_l;
      }
    }
  }
}

// A row's sums are exact under any reference that keeps them within range.  It is done over, under a running maximum, if scores
// rose beyond that between two looks at it (a sum of kSumLimit), if all scores of its first tile are -inf (there is no maximum to
// refer to then; every other row's sum holds the 1 of its first tile's maximum or what raised the reference from there), or if
// its output is not finite although large values alone are no reason for that (with sums below 2^8 they are).
template <int D>
__device__ __forceinline__ bool out_of_range(const Pipe<D>& t, float l_tot) {
  bool again = !(l_tot >= 0.5f && l_tot < kSumLimit);
  if (__builtin_amdgcn_ballot_w64(l_tot >= 0x1p8f) != 0) {
    float zs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) zs[r & 3] = __builtin_fmaf(t.O[mb][r], 0.0f, zs[r & 3]);
    float z = (zs[0] + zs[1]) + (zs[2] + zs[3]);
    z += __shfl_xor(z, 32);
    again = again || (l_tot >= 0x1p8f && !(z == 0.0f));
  }
  return again;
}

// The wave's rows under a running maximum, without the other waves: keys straight from the cache, values through the rows of LDS
// that its output passed through, both requested half a tile ahead.  Rows that need it are rare, so this is short rather than fast.
// All rows done over (keys from 96 on with 40 natural units' spread), 32 / 8 heads, in two passes without requests ahead, now, and by the
// former loop, which knew no such rows: 2048 tokens 250, 148 and 51 us, 8192 2493, 1575 and 474, 16 ragged prompts 1072, 710 and 245, at head
// size 64 576, 364 and 151.
template <int D, bool KV8, int NW>
__device__ __forceinline__ void rows_alone(const AttnParams& p, unsigned char* smem, const Item& it, const WaveItem& wi,
                                           const WaveCtx& cx, Spans& sp, const int* bt, unsigned rows) {
  using C = Cfg<D, KV8, NW>;
  constexpr int E = KV8 ? 1 : 2, LPR = D / 8, RPL = 64 / LPR, NV = 32 / RPL;      // lanes per row, rows per load (eight values to a lane), loads
  bf16x8 qf[C::KSTEPS];
  {
    const int t = wi.wrow0 + min(cx.lane & 31, it.n - 1 - wi.wrow0);
    const __bf16* const qg = static_cast<const __bf16*>(p.q) + ((size_t)(it.qbase + t) * p.Hq + wi.head) * D + 8 * cx.hf;
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) {
      const uint4 v = load_global16((global_bytes)(unsigned long long)(size_t)(qg + 16 * s));
      __builtin_memcpy(&qf[s], &v, 16);
    }
  }
  // eight values each: of this lane's key, one piece per k-step; of rows RPL j + lane / LPR
  std::conditional_t<KV8, u32x2, uint4> kp[C::KSTEPS], vp[NV];
  auto request = [&](int first) {      // the half tile that begins with block `first`
    const unsigned long long b0 = block_bytes(cx, cload(bt, min(first, cx.last_blk)));
    const unsigned long long b1 = block_bytes(cx, cload(bt, min(first + 1, cx.last_blk)));
    const unsigned long long ka = cx.kbase + (KV8 ? 0 : 2048) + (cx.lane & 16 ? b1 : b0) + (cx.lane & 15) * (D * E) + 8 * E * cx.hf;
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) {
      if constexpr (KV8) kp[s] = *(const __attribute__((address_space(1))) u32x2*)(global_bytes)(ka + 16 * s);
      else kp[s] = load_global16((global_bytes)(ka + 32 * s));
    }
    unsigned vo = (cx.lane / LPR) * (D * E) + 8 * E * (cx.lane % LPR);
    asm("" : "+v"(vo));       // (so that the loads take a scalar base and a 32-bit lane offset)
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const global_bytes va = (global_bytes)(cx.vbase + (j < NV / 2 ? b0 : b1)) + vo + RPL * (j % (NV / 2)) * (D * E);
      if constexpr (KV8) vp[j] = *(const __attribute__((address_space(1))) u32x2*)va;
      else vp[j] = load_global16(va);
    }
  };
  auto widened = [](const auto& x) {
    if constexpr (KV8) return e4m3x8_to_bf16x8(make_uint2(x.x, x.y));
    else return x;
  };
  request(0);
  float m = -INFINITY;
  sp.lo = 0;
  Pipe<D> t;
  t.l = 0.0f;
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) t.am[s] = 0.0f;
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) t.O[mb][r] = 0.0f;
  unsigned char* const vrows = smem + out_rows<D, KV8, NW>(cx);
  unsigned v_addr[4];
  {
    const int g = cx.lane >> 4, s16 = cx.lane & 15;
    const unsigned a = (4 * (g >> 1) + (s16 >> 2)) * C::RB + (((2 * (g & 1) + ((s16 & 3) >> 1)) ^ v_swizzle<D>(s16 >> 2)) << 4) + 8 * (s16 & 1);
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb) v_addr[mb] = cx.lds_base + out_rows<D, KV8, NW>(cx) + (a ^ (64u * mb));
  }
  for (int key0 = 0; key0 <= wi.pos_max; key0 += 32) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int r = RPL * j + cx.lane / LPR, ch = cx.lane % LPR;
      uint4 v = widened(vp[j]);
      if (key0 + r >= cx.L) v = make_uint4(0, 0, 0, 0);      // 0 * NaN would poison the output
      *reinterpret_cast<uint4*>(vrows + r * C::RB + ((ch ^ v_swizzle<D>(r)) << 4)) = v;
    }
    in_order();
    f32x16 S;
#pragma unroll
    for (int r = 0; r < 16; ++r) S[r] = 0.0f;
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) {
      const uint4 a = widened(kp[s]);
      bf16x8 av;
      __builtin_memcpy(&av, &a, 16);
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, qf[s], S, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    request(key0 / kBlock + 2);
    __builtin_amdgcn_sched_barrier(0);
    mask_half(cx, key0, S);
    float mx = S[0] * cx.c;
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, S[r] * cx.c);
    mx = half_max(mx);
    const bool up = mx > m + kLazyTau;
    if (__builtin_amdgcn_ballot_w64(up) != 0) {
      const float f = up ? fast_exp2(m - mx) : 1.0f;
      m = up ? mx : m;
      t.l *= f;
#pragma unroll
      for (int i = 0; i < kMaxSpans; ++i) t.am[i] *= f;
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) t.O[mb][r] *= f;
    }
    u32x4 P[2];
    HalfExp h;
    exp_begin<1>(cx, S, m == -INFINITY ? 0.0f : m, h);
#pragma unroll
    for (int j = 0; j < 16; ++j) exp_slot<1>(cx, S, m == -INFINITY ? 0.0f : m, h, P, j);
    const float sum = exp_end<1>(S, h, P);
    t.l += sum;
    add_spans<D>(cx, sp, key0, S, sum, t.am);
#pragma unroll
    for (int n = 0; n < 2 * C::MB; ++n)
      t.O[n % C::MB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_vt<D>(v_addr, n / C::MB, n % C::MB), as_bf16x8(P[n / C::MB]),
                                                              t.O[n % C::MB], 0, 0, 0);
    in_order();
  }
  finish<D, KV8, NW, true>(p, smem, it, wi, cx, sp, t, t.l + __shfl_xor(t.l, 32), rows);
}

template <int D, bool KV8, int NW, bool SHARED, bool PROBE>
__device__ __forceinline__ unsigned tiles_and_output(const AttnParams& p, unsigned char* smem, const Item& it, const WaveItem& wi,
                                                     const WaveCtx& cx, int id, unsigned long long boff,
                                                     const bf16x8 (&qf)[D / 16], Spans& sp, const int* bt) {
  Pipe<D> t;
  float m;
  run_tiles<D, KV8, NW, SHARED, PROBE>(cx, smem, wi.ntiles, wi.mine, wi.pos_max, id, boff, qf, t, m, sp, bt);
  if constexpr (KV8) wait_vmem();   // (bytes that nobody waits for any more: no fetch may outlive its buffers)
  const float l_tot = t.l + __shfl_xor(t.l, 32);
  const unsigned rows = wi.active ? (unsigned)((1ull << min(kWaveRows, it.n - wi.wrow0)) - 1) : 0u;
  if (wi.active) finish<D, KV8, NW, PROBE>(p, smem, it, wi, cx, sp, t, l_tot, rows);
  return rows & (unsigned)__builtin_amdgcn_ballot_w64(out_of_range<D>(t, l_tot));
}

// ZERO_REST (self-planned calls): the wave that owns a probed
// head in the item of row 0 also writes zeros to that head's `mass` slots that hold no row, so that
// every entry of `mass` is written exactly once without a planner's zero-fill.
template <int D, bool KV8, int NW, bool SHARED, bool ZERO_REST>
__device__ __forceinline__ void prefill_item(const AttnParams& p, unsigned char* smem, const Item& it) {
  using C = Cfg<D, KV8, NW>;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = it.L, n = it.n;
  const int hh = w % p.hpw, rb = w / p.hpw;
  const int head = it.kvh * p.G + it.hg * p.hpw + hh;
  const int wrow0 = it.row0 + rb * kWaveRows;
  const int qi = lane & 31, hf = lane >> 5;
  const int t = max(min(wrow0 + qi, n - 1), 0);
  const int wg_pos_max = L - n + min(it.row0 + p.rows_per_wg, n) - 1;
  const int ntiles = wg_pos_max / kTileKeys + 1;
  WaveItem wi;
  wi.ntiles = ntiles;
  wi.pos_max = L - n + min(wrow0 + kWaveRows, n) - 1;
  wi.mine = wi.pos_max / kTileKeys + 1;     // tiles with a key within some row's horizon
  wi.head = head;
  wi.wrow0 = wrow0;
  wi.active = wrow0 < n;

  const int* const bt = p.block_table + (size_t)it.seq * p.max_blocks;
  WaveCtx cx;
  cx.L = L;
  cx.last_blk = min((L - 1) >> 4, 4 * ntiles - 1);
  cx.w = w;
  cx.wb = w / C::WPB;
  cx.ws = w % C::WPB;
  cx.lane = lane;
  cx.blk_bytes = (unsigned)p.Hkv * C::BLK;
  // this wave's blocks of the first tiles by scalar loads: the wait for them leaves vector loads alone
  cx.num_blocks = p.num_blocks;
  auto first_id = [&](int tile) { return cload(bt, min(4 * min(tile, ntiles - 1) + cx.wb, cx.last_blk)); };
  const int id0 = first_id(0), id1 = first_id(1), id2 = first_id(2);

  int probe_list = p.P > 0 ? p.probe_heads[min(lane, p.P - 1)] : 0;
  bf16x8 qf[C::KSTEPS];
  uint4 qraw[KV8 ? C::KSTEPS : 1];
  if constexpr (KV8) {
    const __bf16* const qg = static_cast<const __bf16*>(p.q) + ((size_t)(it.qbase + t) * p.Hq + head) * D + 8 * hf;
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) qraw[s] = load_global16((global_bytes)(unsigned long long)(size_t)(qg + 16 * s));
  }

  cx.hf = hf;
  cx.pos = L - n + t;
  cx.pos_min = __builtin_amdgcn_readfirstlane(L - n + min(wrow0, n - 1));
  cx.c = KV8 ? p.scale_log2 * p.k_scale[it.kvh] : p.scale_log2;
  cx.kbase = (unsigned long long)(size_t)p.k_cache + (size_t)it.kvh * C::BLK;
  cx.vbase = (unsigned long long)(size_t)p.v_cache + (size_t)it.kvh * C::BLK;
  // per-lane source offsets of the direct-to-LDS loads: LDS slot (row r, physical chunk pc)
  // receives logical chunk pc ^ swizzle(r); bytes are staged as they lie in the cache
  {
    const int r = lane / C::LPR, pc = lane % C::LPR;
    if (KV8) {
      cx.v_off[0] = cx.v_off[1] = cx.k_off[0] = cx.k_off[1] = cx.ws * C::SHARE + 16 * lane;
    } else {
      cx.v_off[0] = cx.v_off[1] = cx.ws * C::SHARE + (unsigned)r * C::RB + (unsigned)(pc ^ v_swizzle<D>(r)) * 16;
      // (2048 more, which kbase is short of, so that none is negative)
#pragma unroll
      for (int i = 0; i < C::NI; ++i) {
        const int j = cx.ws * C::NI + i, rk = 8 * (j & 1) + lane / 8;
        cx.k_off[i] = (unsigned)rk * C::RB + (j >> 1) * 128 + (unsigned)((lane % 8) ^ k_swizzle(rk)) * 16 + 2048 - 1024 * i;
      }
      cx.kbase -= 2048;
    }
  }
  cx.lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) const void*)smem;

  int id = KV8 ? first_id(3) : id2;
  asm("" : "+v"(id));
  const unsigned long long boff0 = block_bytes(cx, id0), boff1 = block_bytes(cx, id1), boff2 = block_bytes(cx, id2);
  if constexpr (KV8) {
    first_tiles_kv8<D, NW>(cx, smem, boff0, boff1, boff2);
  } else {
    // (The compiler does not count these loads: what it counts has to have arrived before them, or waiting for that
    // would be waiting for all of them.)
    asm volatile("" : "+v"(probe_list));
    const int row = min(wrow0, n - 1);
    first_tiles<D, NW>(cx, (unsigned long long)(size_t)p.q + ((size_t)(it.qbase + row) * p.Hq + head) * C::RB, n - row, p.Hq * C::RB,
                   boff0, boff1);
  }

  Spans sp;
  sp.n = 0;
  wi.pslot = -1;
  wi.qsel_b = wi.qsel_e = 0;
  if (p.P > 0) {
    wi.pslot = p.P <= 64 ? find_probe_slot_lanes(probe_list, p.P, head) : find_probe_slot_uniform(p.probe_heads, p.P, head);
    wi.qsel_b = cload(p.query_sel, 2 * it.seq);
    wi.qsel_e = min(cload(p.query_sel, 2 * it.seq + 1), wi.qsel_b + p.NQ);
    sp.n = p.S;
    load_spans_uniform(p.key_spans, it.seq, p.S, sp.a, sp.b);
  }
  const bool wave_probe = wi.active && wi.pslot >= 0 && wi.qsel_b < min(wrow0 + kWaveRows, n) && wi.qsel_e > wrow0;
  if (!wave_probe) sp.n = 0;
  sp.lo = 0;
  sp.hi = 0;
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s)
    if (s < sp.n) {
      sp.b[s] = max(sp.b[s], sp.a[s]);      // (an empty one stays empty)
      sp.hi = max(sp.hi, sp.b[s]);
    }

  // the first scores need the query rows and K(0); V(0) and K(1) (2 NI loads; with staging K(2) and V(1)) may stay in flight
  if constexpr (KV8) {
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) __builtin_memcpy(&qf[s], &qraw[s], 16);
#pragma unroll
    for (int s = 0; s < C::KSTEPS; ++s) asm volatile("" : "+v"(qf[s]) :: "memory");     // (they have arrived here)
  }
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * C::NI) : "memory");
  if constexpr (!KV8) read_queries<D, NW>(cx, smem, qf);
  __syncthreads();
  const unsigned long long boff = KV8 ? boff2 : boff1;      // of the last K run fetched
  const unsigned again = wave_probe ? tiles_and_output<D, KV8, NW, SHARED, true>(p, smem, it, wi, cx, id, boff, qf, sp, bt)
                                    : tiles_and_output<D, KV8, NW, SHARED, false>(p, smem, it, wi, cx, id, boff, qf, sp, bt);
  // (with its arguments read again, or they take registers from the rest: 2 prompts of 200-300 tokens 11.9 instead of 12.1 us)
  if (__builtin_expect(again != 0, 0)) rows_alone<D, KV8, NW>(reread_arguments(), smem, it, wi, cx, sp, bt, again);
  if constexpr (ZERO_REST) {
    if (it.row0 == 0 && rb == 0 && wi.pslot >= 0 && p.plan_fresh) {
      const int lo = max(wi.qsel_b, 0), hi = min(wi.qsel_e, n);     // slots lo - qsel_b .. hi - qsel_b - 1 hold rows
      for (int e = lane; e < p.NQ * p.S; e += 64) {
        const int tr = wi.qsel_b + e / p.S;
        if (tr < lo || tr >= hi) p.mass[((size_t)it.seq * p.P + wi.pslot) * p.NQ * p.S + e] = 0.0f;
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
template <int NT>
__device__ __forceinline__ void settle_chunks(const AttnParams& p, int* sh) {
  int* const skip = sh + 2;     // [kScanMaxSeqs]
  const int tid = threadIdx.x;
  if (tid < 2) sh[tid] = 0;
  __syncthreads();
  int bits = p.plan_fresh && bad_head_list<NT>(p) ? kBadHeadList : 0, blocks = 0;
  for (int i = tid; i < p.num_seqs; i += NT) {
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
        for (int e = tid; e < p.P * p.NQ * p.S; e += NT) p.mass[(size_t)i * p.P * p.NQ * p.S + e] = 0.0f;
  if (sh[0] & kBadHeadList) zero_unowned_mass<NT>(p);
}

// PLANNED: the work item comes from the planner's list.  Otherwise the kernel finds it (above), the last workgroup
// of the grid settles the rest, and `mass` is written entry by entry by the waves that own the entries.
// SHARED: several row blocks to a workgroup.  An instantiation of its own, because the fetch-only iterations cost the others up to
// 2 % (one prompt of 700 tokens at head size 64 12.8 -> 13.1 us, 32 chunks of 64-200 rows 173.3 -> 174.7, long prompts nothing).
template <int D, bool KV8, int NW, bool SHARED, bool PLANNED>
__device__ __forceinline__ void row_block(const AttnParams& p, unsigned char* smem, int bid, int last) {
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
    prefill_item<D, KV8, NW, SHARED, false>(p, smem, {kvh, hg, it.x, it.y, it.z, it.w, qbase});
  } else {
    if (bid == last) {
      settle_chunks<64 * NW>(reread_arguments(), reinterpret_cast<int*>(smem));   // (or its arguments take registers from the rest)
      return;
    }
    ChunkItem it;
    const bool some = find_item(p, item, threadIdx.x & 63, it);
    asm volatile("" :: "s"(p.block_table), "s"(p.q), "s"(p.k_cache), "s"(p.v_cache));
    if (!some) return;
    prefill_item<D, KV8, NW, SHARED, true>(p, smem, {kvh, hg, it.seq, it.block * p.rows_per_wg, it.L, it.n, it.qbase});
  }
}

}  // namespace

}  // namespace hook
