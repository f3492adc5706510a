// Internal declarations shared by the HIP translation units of libhook (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

namespace hook {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kBlock = 16;          // tokens per KV block
constexpr int kMaxSpans = 8;        // compile-time bound on S
constexpr int kTileKeys = 64;       // keys per prefill tile
constexpr int kWaveRows = 32;       // query rows per prefill wave
constexpr int kPartialPad = 16;     // floats after the D output values of a decode partial: m, l, a[8], pad
constexpr int kPlanBuckets = 2048;  // counting-sort buckets (tile counts) of the prefill work list
// Decode chunking rule shared by the planner (which applies it) and the host (which bounds the
// number of items it can produce): the largest chunk of 512 << k keys, up to kMaxChunkKeys, that
// still yields kDecodeFillWgs decode workgroups; 256 keys when none does.  The planner halves it while it is longer than a
// workgroup's share of the batch and the items still fit the host's bound (plan.hip).
constexpr int kChunkSizes = 5;
constexpr int kMaxChunkKeys = 512 << (kChunkSizes - 1);
constexpr int kDecodeFillWgs = 2048;
// Batches of single rows with at most kStreamSeqs sequences, or more where there are few heads (stream_seqs in api.hip),
// plan themselves (decode.hip); ranges are cut no shorter than
// one block per wave of a workgroup (the last one of a batch, or of a sequence, may hold fewer).  More rows than that
// are worth the planning launch: the hardware deals its items out one by one, longest first, whereas equal ranges that
// start together do not end together (256 x 1000-8192 tokens: the first after 370, the last after 770 us).  At 32 / 8
// heads streamed and planned: 128 x 1000-8192 tokens 408 and 407 us, 200 x 300-1000 with new rows 109 and 106, 256 x
// 300-1000 130 and 124, 500 x 200-2000 414 and 391; 256 x 1000-8192 for groups of 8 heads 796 and 782, over an 8-bit
// cache 546 and 480.  Over 16-bit caches the line could lie higher for some batches, which lose the planning launch: 200 x
// 1000-4000 334 and 338, one of 32768 tokens among 199 of 300 82 and 86; but 256 x 20-200 takes 49 and 42.
constexpr int kStreamSeqs = 192;
constexpr int kScanMaxSeqs = 512;   // the most whose lengths a workgroup scans to plan itself, here and in prefill_device.h
constexpr int kStreamMinBlocks = 4;
// Cache blocks of single rows that a row of the row blocks in the same launch weighs: with fewer to each of them the single rows'
// workgroups leave a place on every compute unit free (dec_few).  Two of them to a compute unit and one, over an 8-bit cache,
// us: 28 x 16384 tokens and a chunk of 1000 rows (29 blocks to a row) 164 and 195, 20 x 4096 and 200 (26) 42.4 and 46.6, 16 x 3000-6000 and 2 x
// 1000 (2.3) 61.0 and 54.7, 28 x 4096 and 4 x 1024 (1.8) 90.9 and 88.8.
constexpr int kRowsWeigh = 5;
// A running maximum is only raised when a tile's maximum exceeds it by more than this many
// powers of two; exponentials then stay below 2^kLazyTau, far inside fp32 range, and the
// normaliser carries the same reference, so the result is the exact softmax.
constexpr float kLazyTau = 8.0f;

// Device-side status bits written by the plan kernel.
enum : int { kStatQGtL = 1, kStatLenClamped = 2, kStatNegative = 4, kStatHint = 8 };
constexpr int kBadHeadList = 1 << 16;   // beside them inside a kernel, never reported

struct PlanHeader {
  int n_prefill;   // prefill work items (row blocks)
  int n_decode;    // decode work items (key chunks)
  int chunk_keys;  // keys per decode work item
  int status;      // kStat* bits of the last attention call
  int problems;    // HOOK_BAD_* bits of the last hook_attn_probe_validate call (a word of its own)
  int pad[11];
};

// Work-list records.  prefill: two consecutive records per item,
// {seq, first chunk-local row, L, n} and {global row of the sequence's first query, 0, 0, 0};
// decode: one record {seq, chunk index, L, global q row}.
typedef int4 WorkItem;

// Cache write of the new tokens' rows (kv_write_device.h)
struct KvWriteParams {
  int num_seqs, total_q, Hkv, max_blocks, num_blocks;
  int row_chunks;   // 16-byte chunks per (token, kv head) row of k_new / v_new
  int kv8;          // the cache holds 8-bit E4M3 bytes: rows (bf16) are quantised on the way
  const uint4* k_new;
  const uint4* v_new;
  const int* block_table;
  const int* seq_lens;
  const int* cu_q_lens;
  void* k_cache;
  void* v_cache;
  const float* k_scale;   // [Hkv], kv8 only
  const float* v_scale;
};

struct AttnParams {
  int num_seqs, total_q, Hq, Hkv, G, max_blocks, num_blocks;
  float scale_log2;                 // softmax scale * log2(e)
  const void* q;
  const void* k_cache;
  const void* v_cache;
  const int* block_table;
  const int* seq_lens;
  const int* cu_q_lens;
  int P;
  const int* probe_heads;
  int NQ;
  const int* query_sel;
  int S;
  const int* key_spans;
  void* out;
  float* mass;
  // new tokens' key/value rows to be written into the cache before anything reads it (kvw.k_new != null)
  KvWriteParams kvw;
  // 8-bit (E4M3) key/value cache: bytes instead of `dtype` elements, one fp32 scale per kv head
  int kv8;
  const float* k_scale;
  const float* v_scale;
  // workspace carve-up
  PlanHeader* hdr;
  WorkItem* pf_items;
  int pf_cap;
  WorkItem* dec_items;              // two records per turn, longest chunks first: {seq, chunk, L, q row}, {partial slot, -, -, -}
  int dec_cap;
  int2* seq_dec;                    // per sequence {first partial record, number of records}
  float* partials;                  // [dec_cap, Hq, D + kPartialPad]
  int dec_ranges;                   // > 0: no planner; the blocks of all single rows are cut into this many ranges
  int dec_write;                    // the streaming kernel stores the new rows (k_new / v_new) itself
  int plan_fresh;                   // the call promises a fully written `mass` (not a reused plan)
  int one_launch;                   // row blocks and single rows share a launch (mixed.hip)
  int pf_self;                      // the chunk kernel finds its row blocks itself, no planner
  // geometry chosen on the host from G
  int batch_kind;                   // 0 mixed, 1 no single-row sequences, 2 only single-row sequences
  int pf_waves;                     // waves of a prefill workgroup (4 or 8)
  int hpw;                          // q heads per prefill workgroup (8, 4, 2 or 1)
  int rows_per_wg;                  // 32 * (pf_waves / hpw)
  int hgroups;                      // G / hpw
  int dec_hp;                       // q heads per decode workgroup (8, 4, 2 or 1)
  int dec_hgroups;                  // G / dec_hp
  int dec_few;                      // > 0: ranges instead of dec_ranges where row blocks of the same launch weigh more (kRowsWeigh)
};

// The kernel's argument block, through a pointer whose origin the compiler cannot see.
__device__ __forceinline__ const AttnParams& reread_arguments() {
  auto a = (const __attribute__((address_space(4))) void*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return *(const AttnParams*)(const __attribute__((address_space(4))) AttnParams*)a;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2 v = {lo, hi};
  bf16x2 b = __builtin_convertvector(v, bf16x2);  // v_cvt_pk_bf16_f32, round-to-nearest-even
  uint32_t u;
  __builtin_memcpy(&u, &b, 4);
  return u;
}

// 16-byte load of data that is read once and not again (K/V rows on the decode path): the
// non-temporal hint keeps the stream from displacing useful lines and measurably raises the
// sustained read rate on this chip.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  const u32x4 v = __builtin_nontemporal_load(static_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}

typedef const __attribute__((address_space(1))) char* global_bytes;   // a pointer that is known to be global memory
__device__ __forceinline__ uint4 load_stream16(global_bytes p) {
  const u32x4 v = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 load_global16(global_bytes p) {
  const u32x4 v = *(const __attribute__((address_space(1))) u32x4*)p;
  return make_uint4(v.x, v.y, v.z, v.w);
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 load_stream8(global_bytes p) {
  const u32x2 v = __builtin_nontemporal_load((const __attribute__((address_space(1))) u32x2*)p);
  return make_uint2(v.x, v.y);
}

// Element of an array that no kernel of the launch writes, at a uniform index: always a scalar load.  (Through
// an ordinary pointer the compiler may only use one while no store can have come before it.)
__device__ __forceinline__ int cload(const int* p, int i) {
  return ((const __attribute__((address_space(4))) int*)p)[i];
}

__device__ __forceinline__ float cloadf(const float* p, int i) {
  return ((const __attribute__((address_space(4))) float*)p)[i];
}

// 16-byte store of data that this kernel does not read again.
__device__ __forceinline__ void store_stream16(void* p, const uint4 v) {
  u32x4 x;
  x.x = v.x; x.y = v.y; x.z = v.z; x.w = v.w;
  __builtin_nontemporal_store(x, static_cast<u32x4*>(p));
}

// Inclusive prefix sum over the wave with DPP moves: inside the rows of 16 lanes, then across them.
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Maximum over the wave of a value that is not negative, in every lane.
__device__ __forceinline__ int wave_max(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));   // the moves of wave_scan
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

// Index of `head` in the strictly increasing list probe_heads[0..P), or -1: a binary search, so
// the chain of dependent loads is log2(P) long (a list that is not increasing just fails to
// find some heads).
__device__ __forceinline__ int find_probe_slot(const int* probe_heads, int P, int head) {
  int lo = 0, hi = P;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (probe_heads[mid] < head) lo = mid + 1; else hi = mid;
  }
  return (lo < P && probe_heads[lo] == head) ? lo : -1;
}

// The same for a uniform `head` on a path that has stored something before.
__device__ __forceinline__ int find_probe_slot_uniform(const int* probe_heads, int P, int head) {
  int lo = 0, hi = P;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (cload(probe_heads, mid) < head) lo = mid + 1; else hi = mid;
  }
  return (lo < P && cload(probe_heads, lo) == head) ? lo : -1;
}

// The same search in a list of at most 64 that the lanes hold (lane i: element min(i, P - 1)): one trip to memory instead of
// log2(P).
__device__ __forceinline__ int find_probe_slot_lanes(int list, int P, int head) {
  int lo = 0, hi = P;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (__builtin_amdgcn_readlane(list, mid) < head) lo = mid + 1; else hi = mid;
  }
  return (lo < P && __builtin_amdgcn_readlane(list, lo) == head) ? lo : -1;
}

// Calls without a planner: every entry of `mass` is written by the wave that owns its head, so elements of the head list
// that no head owns (find_probe_slot does not lead to them: repeated, out of range, out of order) are cleared by one
// workgroup of NT threads.  Whether there can be any: this thread's share of the list, to be fetched with whatever else
// that workgroup waits for.
template <int NT>
__device__ __forceinline__ bool bad_head_list(const AttnParams& p) {
  bool bad = false;
  for (int i = threadIdx.x; i < p.P; i += NT) {
    const int h = p.probe_heads[i];
    if ((unsigned)h >= (unsigned)p.Hq || (i > 0 && h <= p.probe_heads[i - 1])) bad = true;
  }
  return bad;
}

template <int NT>
__device__ __forceinline__ void zero_unowned_mass(const AttnParams& p) {
  const int per = p.NQ * p.S;
  for (int ps = 0; ps < p.P; ++ps) {
    const int h = p.probe_heads[ps];
    if ((unsigned)h < (unsigned)p.Hq && find_probe_slot(p.probe_heads, p.P, h) == ps) continue;
    for (int i = 0; i < p.num_seqs; ++i)
      for (int e = threadIdx.x; e < per; e += NT) p.mass[((size_t)i * p.P + ps) * per + e] = 0.0f;
  }
}

// Spans of one sequence, all fetched before any is waited for (entries past S repeat the last
// span and are never used).
__device__ __forceinline__ void load_spans(const int* key_spans, int seq, int S, int (&sp_a)[kMaxSpans],
                                           int (&sp_b)[kMaxSpans]) {
  const int2* sp = reinterpret_cast<const int2*>(key_spans) + (size_t)seq * S;
  int2 v[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) v[s] = sp[min(s, S - 1)];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) {
    sp_a[s] = s < S ? max(v[s].x, 0) : 0;
    sp_b[s] = s < S ? v[s].y : 0;
  }
}

// The same for a uniform `seq` on a path that has stored something before.
__device__ __forceinline__ void load_spans_uniform(const int* key_spans, int seq, int S, int (&sp_a)[kMaxSpans],
                                                   int (&sp_b)[kMaxSpans]) {
  const int* sp = key_spans + (size_t)seq * S * 2;
  int a[kMaxSpans], b[kMaxSpans];
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) { a[s] = cload(sp, 2 * min(s, S - 1)); b[s] = cload(sp, 2 * min(s, S - 1) + 1); }
#pragma unroll
  for (int s = 0; s < kMaxSpans; ++s) {
    sp_a[s] = s < S ? max(a[s], 0) : 0;
    sp_b[s] = s < S ? b[s] : 0;
  }
}

// f(0), f(1), ... f(N - 1) with the number as a constant
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// launchers (defined next to their kernels); all return hipGetLastError() after the launch
// The dynamic-LDS limit of a kernel is an attribute per device: it is raised on the first launch
// on each device (bit per device id in `done`), from whichever host thread gets there first.
inline hipError_t raise_lds_limit_once(const void* kernel, int bytes, std::atomic<unsigned long long>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const bool tracked = dev >= 0 && dev < 64;
  if (tracked && ((done.load(std::memory_order_acquire) >> dev) & 1ull)) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e != hipSuccess) return e;
  if (tracked) done.fetch_or(1ull << dev, std::memory_order_release);
  return hipSuccess;
}

// Launch grids are one-dimensional and must fit the 31-bit limit.
inline bool grid_fits(long long workgroups) { return workgroups >= 0 && workgroups <= 0x7fffffffLL; }

hipError_t launch_plan(const AttnParams& p, hipStream_t st);
hipError_t launch_kv_write(const KvWriteParams& p, hipStream_t st);
hipError_t launch_prefill(const AttnParams& p, int D, hipStream_t st);
hipError_t launch_mixed(const AttnParams& p, int D, hipStream_t st);
hipError_t launch_decode(const AttnParams& p, int D, hipStream_t st);
hipError_t launch_combine(const AttnParams& p, int D, hipStream_t st);
hipError_t launch_attn_f32(const AttnParams& p, int D, hipStream_t st);
hipError_t launch_steer(void* hidden, const void* vec, float alpha, const uint8_t* mask, int T, int D,
                        int dtype, hipStream_t st);

}  // namespace hook
