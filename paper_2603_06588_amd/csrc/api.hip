// Host side of the C ABI declared in include/hook_api.h: argument checks, workspace
// carve-up and the fixed launch sequence.  No device memory is allocated here and the
// stream is never synchronised (except in the explicit debug status call).
#include "../../include/hook_api.h"
#include "hook_device.h"

#include <algorithm>
#include <cmath>

namespace {

using namespace hook;

constexpr size_t kAlign = 256;
// Row blocks find their work themselves up to this many workgroups (two resident rounds).  Finding it costs every
// workgroup about a thousand cycles; the planning launch (8 us in a kernel trace of 16 prompts) costs a small call less
// than that and sorts better: 2 prompts of 200 tokens 16.2 us planned, 11.6 by themselves; 8 of 200-600 (800
// workgroups) 31.6 and 29.3; 3 of 1500-2048 (1350 workgroups) 81.1 and 82.7.
constexpr long long kSelfPlanMaxWgs = 1024;
// Row blocks go to workgroups of eight waves (twice the rows, or all eight heads of a group, to each fetched tile) from this
// many of those and so many rows to a sequence: two rounds of the compute units, and contexts deep enough to
// pay for a start-up that no second workgroup covers.  Four waves and eight, 32 / 8 heads, us: 1 x 2048 43.1 and 48.5, 3000 75.9
// and 78.8, 4096 131.8 and 124.6, 8192 474 and 459, 2 x 2048 75.8 and 75.9, 4 x 2048 143.0 and 139.6, 16 x 512-2048 243.7 and 241.2,
// 4 x 1000-1500 behind 3000 tokens 304 and 286, but 16 x 200-600 47.5 and 52.3, 8 x 300-1000 46.8 and 47.0; 64 / 8 heads: 1 x 2048
// 71.0 and 66.8, 8192 940 and 905, 8 x 300-1000 86.5 and 96.3.  (32 chunks of 64-200 rows behind 2000 tokens would
// gain, 188.8 and 179.3, but the host sees rows and not depths.)
constexpr long long kEightWaveMinWgs = 512;
constexpr long long kEightWaveMinRows = 768;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Layout {
  size_t off_hdr, off_pf, off_dec, off_seq, off_part;
  size_t needed, reported;      // smallest workspace that is accepted; size to ask for
  int pf_cap, dec_cap, ranges, pf_waves, hpw, rows_per_wg, hgroups, dec_hp, dec_hgroups;
};

bool shapes_supported(const hook_attn_probe_args* a) {
  if (a->num_seqs < 0 || a->total_q < 0 || a->num_q_heads <= 0 || a->num_kv_heads <= 0) return false;
  if (a->max_blocks_per_seq <= 0 || a->num_blocks <= 0) return false;
  if (a->num_q_heads % a->num_kv_heads != 0) return false;
  if (a->block_size != HOOK_BLOCK_SIZE) return false;
  if (a->dtype != HOOK_BF16 && a->dtype != HOOK_F32) return false;
  if (a->head_dim != 64 && a->head_dim != 128) return false;
  if (a->max_blocks_per_seq > (1 << 26)) return false;
  return true;
}

// Upper bound on the number of decode items the planner can produce, from host scalars only.
// The planner takes the largest chunk size c in {512, 1024, ..., kMaxChunkKeys} whose item count
// still gives kDecodeFillWgs workgroups, else 256 keys.  Halving a chunk at most doubles a
// sequence's item count, so whenever the next larger size was refused (fewer than kDecodeFillWgs
// workgroups, i.e. at most (kDecodeFillWgs - 1) / wg_per_item items) the chosen size yields at most
// twice that; and the largest size yields at most one item per kMaxChunkKeys keys of the longest
// context the block table allows.  (The 256-key tiling of every context is a bound as well.)  Where the planner halves
// its choice further, for a few long contexts among short ones, it stops at this bound, which it is given as dec_cap.
int decode_item_bound(long long num_decode_seqs, long long max_context, int wg_per_item) {
  const long long refused = 2 * ((kDecodeFillWgs - 1) / wg_per_item);
  const long long largest = num_decode_seqs * ((max_context + kMaxChunkKeys - 1) / kMaxChunkKeys);
  const long long finest = num_decode_seqs * ((max_context + 255) / 256);
  long long cap = refused > largest ? refused : largest;
  if (cap > finest) cap = finest;
  if (cap > (1ll << 30)) cap = 1ll << 30;
  return (int)cap;
}

// Ranges per kv head and head group that give every one of the 256 compute units `each` workgroups.
int ranges_of_one_round(const Layout& l, const hook_attn_probe_args* a, int each) {
  const long long wgs = (long long)a->num_kv_heads * l.dec_hgroups;
  return (int)((256 * each + wgs - 1) / wgs);
}

// Ranges of a self-planned batch of single rows (decode.hip): one resident
// round of workgroups - a second, partial round costs more than its finer balance gains - but no range shorter than
// kStreamMinBlocks.  A round is taken as 3 workgroups for each of 256 compute units, 2 for groups of 8 heads: what the
// kernel's launch bounds promise and head size 128 over a 16-bit cache holds.  (Instantiations with fewer registers,
// at head size 64 or over an 8-bit cache, hold 4 in some cases; a finer cut for them has not been measured.)
int stream_ranges(const hook_attn_probe_args* a, const Layout& l, int num_seqs) {
  // (and one range per sequence more, for ranges that end with their sequence)
  const long long finest = ((long long)num_seqs * a->max_blocks_per_seq + kStreamMinBlocks - 1) / kStreamMinBlocks + num_seqs;
  const long long ranges = ranges_of_one_round(l, a, l.dec_hp == 8 ? 2 : 3);
  return (int)(ranges < finest ? ranges : finest);
}

// Row blocks and single rows of a mixed batch share a launch (mixed.hip) where the single rows plan themselves and are few: no
// more sequences than ranges at one workgroup per compute unit, so that hardly a range pays for more than two start-ups, which
// nothing covers there.  Apart and together, 32 / 8 heads, us: 8 x 1000 tokens and a chunk of 512 rows 32.1 and 23.5, with new rows 37.8
// and 28.3, 4 x 6000 and 130 34.6 and 28.6, 16 x 3000-6000 and 2 x 1000 90.0 and 70.5, 28 x 4096 and 4 x 2048 230 and 205, 28 x 16384 and 130 over an
// 8-bit cache 172 and 161; 20 x 4096 and 200 at 64 / 8 heads over an 8-bit cache 66.5 and 55.0; 28 x 4096 and 4 x 2048 at 8 / 1 78.2 and 57.6.  (How
// many workgroups the single rows take there: share_compute_units.)  With more sequences, at one workgroup, either way: 60 x 4096 and 4 x 2048 312
// and 291, with new rows 326 and 332, 60 x 500-5000 and 200 over an 8-bit cache 88 and 99, 180 x 500-2000 and 2 x 300 184 and 193.  Groups of
// four heads and more; four waves to a row block (eight leave no room on their compute unit).
bool shares_launch(const hook_attn_probe_args* a, const Layout& l) {
  return a->dtype == HOOK_BF16 && a->batch_kind == HOOK_BATCH_MIXED && l.ranges > 0 && l.pf_waves == 4 && l.hpw == 4 &&
         a->num_seqs <= kStreamSeqs && a->num_seqs <= ranges_of_one_round(l, a, 1);
}

// Ranges of the single rows in such a launch.  One workgroup to a compute unit leaves a place for a row block, and streams as fast as
// memory where its waves' requests are large (16-bit rows of 256 bytes for four heads, three blocks ahead).  Elsewhere it takes two:
// with one, an 8-bit cache lost to two launches where contexts are deep and row blocks few (28 x 16384 tokens and a chunk of 130 rows at 64 / 8 heads
// 211 us in two launches, 266 with one workgroup, 202 with two; at 32 / 8 172, 192 and 161; 8 x 32768 and 64 at 64 / 8 124, 154 and 119), and so did groups of
// eight heads over 16-bit caches (8 x 32768 and 64 183, 189 and 177).  But row blocks that weigh more than the single rows
// want that place (kRowsWeigh; decided by the kernel, which knows the contexts, or here where no context can be long enough), and cutting
// each sequence into more than 16 ranges costs the merge more than it gains (8 x 16384 and 130 at 8 / 1 heads 25.0 with one, 28.8 with two).
// Without a row to spare there is no row block to leave a place for (a batch of single rows without a hint: 8 x 1000 tokens at 32 / 8
// heads 18.3 in two launches, 20.2 with one workgroup, 16.5 with two; 28 x 16384 of 8 bits at 64 / 8 204, 267 and 203); one sequence alone
// has enough ranges with one (1 x 32768 at 32 / 8 heads 32.6, 32.1 and 33.8).
void share_compute_units(const hook_attn_probe_args* a, const Layout& l, hook::AttnParams& p) {
  const int one = std::min(l.ranges, ranges_of_one_round(l, a, 1)), two = std::min(l.ranges, ranges_of_one_round(l, a, 2));
  const bool large = a->kv_dtype != HOOK_KV_FP8_E4M3 && a->head_dim == 128 && l.dec_hp == 4;
  const long long rows = (long long)a->total_q - a->num_seqs, most_blocks = (long long)a->num_seqs * a->max_blocks_per_seq;
  p.dec_few = 0;
  if (rows <= 0) {
    p.dec_ranges = large && a->num_seqs == 1 ? one : two;
  } else if (large || two > 16 * a->num_seqs || hook::kRowsWeigh * rows >= most_blocks) {
    p.dec_ranges = one;
  } else {
    p.dec_ranges = two;
    p.dec_few = one;
  }
}

// Sequences up to which single rows plan themselves; up to kStreamSeqs of them do in any case (why there: hook_device.h).
// Where an item is few workgroups the planner cuts contexts down to 256 keys to fill the chip, so more sequences are
// better off in equal ranges.  Streamed and planned, contexts of 100-1000, 500-4000 and 2000-8000 tokens: 4 / 1 heads, 200
// rows 23 / 51 / 91 and 27 / 60 / 103 us, 500 rows 43 / 102 / 202 and 40 / 111 / 218; 8 / 2 heads, 300 rows 43 / 121 / 252 and
// 45 / 134 / 272, 500 rows 67 / 192 / 409 and 65 / 201 / 422; 16 / 4 heads, 200 rows 52 / 163 / 341 and 56 / 172 / 354.
// Contexts shorter than a range are the planner's (8 / 2 heads, 500 rows of 20-200 tokens 34 and 30).
// Groups of 8 heads have fewer ranges and pass earlier: 8 / 1 heads, 300 rows 37 / 75 / 140 and 37 / 90 / 159, 500 rows 54 / 113 /
// 222 and 49 / 123 / 232; 16 / 2, 300 rows 53 / 137 / 270 and 55 / 147 / 289; 32 / 4, 200 rows 63 / 181 / 360 and 68 / 185 / 361, but 44
// and 33 of 20-200 tokens.  So do key rows of half the bytes, where more planned workgroups are resident: 8 / 2 heads over an 8-bit
// cache, 300 rows 33 / 73 / 145 and 33 / 78 / 145; 16 / 4 heads at head size 64, 200 rows 32 / 62 / 115 and 34 / 58 / 103.
int stream_seqs(const hook_attn_probe_args* a, const Layout& l) {
  const int wgs = a->num_kv_heads * l.dec_hgroups;
  int n = wgs == 1 ? kScanMaxSeqs : wgs == 2 ? 384 : wgs <= 4 ? 288 : kStreamSeqs;
  if (l.dec_hp == 8) n = wgs <= 2 ? 5 * n / 6 : kStreamSeqs;
  if (a->head_dim == 64 || a->kv_dtype == HOOK_KV_FP8_E4M3) n = 2 * n / 3;
  return n > kStreamSeqs ? n : kStreamSeqs;
}

// Carves the workspace up for the layout's capacities; returns its size.
size_t place(const hook_attn_probe_args* a, Layout& l) {
  size_t off = 0;
  l.off_hdr = off;  off = align_up(off + sizeof(PlanHeader));
  l.off_pf = off;   off = align_up(off + 2 * sizeof(WorkItem) * (size_t)l.pf_cap);
  l.off_dec = off;  off = align_up(off + 2 * sizeof(WorkItem) * (size_t)l.dec_cap);
  l.off_seq = off;  off = align_up(off + sizeof(int2) * (size_t)(a->num_seqs > 0 ? a->num_seqs : 1));
  l.off_part = off;
  off = align_up(off + sizeof(float) * (size_t)l.dec_cap * a->num_q_heads * (a->head_dim + kPartialPad));
  return off;
}

// The layout for a workspace of `bytes`.  Single rows of up to stream_seqs() sequences, whose lengths every
// workgroup can afford to scan, plan themselves where their records fit; those are numbered by range + sequence, which
// can take more slots than the planner's items.  A smaller workspace keeps the planner, so every size that holds the
// planner's items is accepted.
// The size reported is no smaller for a larger batch (one buffer, asked for once, serves every batch up to that one with
// the kernels that its own size would have got it): beyond stream_seqs() it still holds the records of that many, and
// up to the static scratch's size it asks for no more than that.
Layout make_layout(const hook_attn_probe_args* a, size_t bytes) {
  Layout l{};
  const int G = a->num_q_heads / a->num_kv_heads;
  l.pf_waves = 4;
  l.hpw = (G % 4 == 0) ? 4 : (G % 2 == 0) ? 2 : 1;
  const int rows = kWaveRows * (4 / l.hpw);      // of a workgroup of four waves
  if (a->head_dim == 128 && G % 4 == 0 && (long long)(a->total_q / (2 * rows)) * a->num_kv_heads * (G / 4) >= kEightWaveMinWgs &&
      a->total_q >= kEightWaveMinRows * a->num_seqs) {
    l.pf_waves = 8;
    if (G % 8 == 0) l.hpw = 8;
  }
  l.rows_per_wg = kWaveRows * (l.pf_waves / l.hpw);
  l.hgroups = G / l.hpw;
  l.dec_hp = (G % 8 == 0) ? 8 : (G % 4 == 0) ? 4 : (G % 2 == 0) ? 2 : 1;
  l.dec_hgroups = G / l.dec_hp;
  if (a->dtype == HOOK_BF16) {
    l.pf_cap = a->total_q / rows + a->num_seqs;
    l.dec_cap = decode_item_bound(a->num_seqs < a->total_q ? a->num_seqs : a->total_q,
                                  (long long)a->max_blocks_per_seq * kBlock, a->num_kv_heads * l.dec_hgroups);
    l.needed = l.reported = place(a, l);
    if (a->num_seqs > 0) {
      const int planned_cap = l.dec_cap, most = stream_seqs(a, l), n = a->num_seqs < most ? a->num_seqs : most;
      const int ranges = stream_ranges(a, l, n);
      if (l.dec_cap < ranges + n) l.dec_cap = ranges + n;
      const size_t streaming = place(a, l), fixed = (size_t)HOOK_STATIC_SCRATCH_BYTES;
      l.reported = l.needed > fixed || streaming < fixed ? streaming : fixed;
      if (n == a->num_seqs && bytes >= streaming) { l.ranges = ranges; return l; }
      l.dec_cap = planned_cap;
    }
  }
  const size_t total = place(a, l);
  if (a->dtype != HOOK_BF16) l.needed = l.reported = total;
  return l;
}

}  // namespace

extern "C" {

size_t hook_attn_probe_workspace_bytes(const hook_attn_probe_args* a) {
  if (!a || !shapes_supported(a)) return 0;
  return make_layout(a, 0).reported;
}

}  // extern "C"

namespace hook {
// Validates, carves the workspace and launches.  With `ev` (5 events) the launches are
// bracketed by event records so a profiling caller can read per-kernel durations (used by the
// separate measurement library, which links these objects; not part of the exported ABI).
// Everything about a call that the host can check without its workspace.  HOOK_OK with *nothing_to_do
// set means a valid call that has no work (no sequences or no rows).
__attribute__((visibility("hidden"))) hook_status check_attn_probe_args(const hook_attn_probe_args* a, bool* nothing_to_do) {
  *nothing_to_do = false;
  if (!a) return HOOK_ERR_NULL;
  if (a->num_seqs < 0 || a->total_q < 0 || a->num_q_heads <= 0 || a->num_kv_heads <= 0 ||
      a->max_blocks_per_seq <= 0 || a->num_blocks <= 0 || a->head_dim <= 0)
    return HOOK_ERR_SHAPE;
  if (a->num_q_heads % a->num_kv_heads != 0) return HOOK_ERR_SHAPE;
  if (!shapes_supported(a)) return HOOK_ERR_UNSUPPORTED;
  if (a->batch_kind < HOOK_BATCH_MIXED || a->batch_kind > HOOK_BATCH_DECODE_ONLY) return HOOK_ERR_SHAPE;
  if (a->plan_mode != HOOK_PLAN_FRESH && a->plan_mode != HOOK_PLAN_REUSE) return HOOK_ERR_SHAPE;
  const int P = a->num_probe_heads;
  if (P < 0 || P > a->num_q_heads) return HOOK_ERR_SHAPE;
  if (P > 0) {
    if (a->max_sel_q < 1 || a->max_spans < 1) return HOOK_ERR_SHAPE;
    if (a->max_sel_q > HOOK_MAX_SEL_Q || a->max_spans > HOOK_MAX_SPANS) return HOOK_ERR_UNSUPPORTED;
    if (!a->probe_heads || !a->query_sel || !a->key_spans || !a->mass) return HOOK_ERR_NULL;
  }
  if (a->kv_dtype != HOOK_KV_SAME && a->kv_dtype != HOOK_KV_FP8_E4M3) return HOOK_ERR_SHAPE;
  const bool kv8 = a->kv_dtype == HOOK_KV_FP8_E4M3;
  // the 8-bit cache goes with bf16 queries
  if (kv8 && a->dtype != HOOK_BF16) return HOOK_ERR_UNSUPPORTED;
  if (a->num_seqs == 0 || a->total_q == 0) { *nothing_to_do = true; return HOOK_OK; }
  if (!a->q || !a->k_cache || !a->v_cache || !a->block_table || !a->seq_lens || !a->cu_q_lens || !a->out)
    return HOOK_ERR_NULL;
  if (kv8 && (!a->k_scale || !a->v_scale)) return HOOK_ERR_NULL;
  if ((a->k_new == nullptr) != (a->v_new == nullptr)) return HOOK_ERR_NULL;
  return HOOK_OK;
}

// (for a caller that times the launches)
__attribute__((visibility("hidden"))) bool attn_probe_shares_launch(const hook_attn_probe_args* a) {
  return shares_launch(a, make_layout(a, a->workspace_bytes));
}

__attribute__((visibility("hidden"))) hook_status run_attn_probe(const hook_attn_probe_args* a, hipEvent_t* ev,
                                                                 void* workspace, size_t workspace_bytes) {
  bool nothing_to_do = false;
  const hook_status checked = check_attn_probe_args(a, &nothing_to_do);
  if (checked != HOOK_OK || nothing_to_do) return checked;
  const int P = a->num_probe_heads;
  const bool kv8 = a->kv_dtype == HOOK_KV_FP8_E4M3;
  const Layout l = make_layout(a, workspace_bytes);
  // one-dimensional launch grids over the item capacities
  if (a->dtype == HOOK_BF16 &&
      (!grid_fits((long long)l.pf_cap * a->num_kv_heads * l.hgroups) ||
       !grid_fits((long long)l.dec_cap * a->num_kv_heads * l.dec_hgroups)))
    return HOOK_ERR_UNSUPPORTED;
  if (!workspace || workspace_bytes < l.needed || (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
    return HOOK_ERR_WORKSPACE;

  AttnParams p{};
  p.num_seqs = a->num_seqs;
  p.total_q = a->total_q;
  p.Hq = a->num_q_heads;
  p.Hkv = a->num_kv_heads;
  p.G = p.Hq / p.Hkv;
  p.max_blocks = a->max_blocks_per_seq;
  p.num_blocks = a->num_blocks;
  const float scale = a->scale > 0.0f ? a->scale : 1.0f / std::sqrt((float)a->head_dim);
  p.scale_log2 = scale * 1.44269504088896340736f;
  p.q = a->q; p.k_cache = a->k_cache; p.v_cache = a->v_cache;
  p.block_table = a->block_table; p.seq_lens = a->seq_lens; p.cu_q_lens = a->cu_q_lens;
  p.P = P;
  p.probe_heads = a->probe_heads;
  p.NQ = P > 0 ? a->max_sel_q : 0;
  p.query_sel = a->query_sel;
  p.S = P > 0 ? a->max_spans : 0;
  p.key_spans = a->key_spans;
  p.out = a->out;
  p.mass = a->mass;
  p.kv8 = kv8 ? 1 : 0;
  p.k_scale = a->k_scale;
  p.v_scale = a->v_scale;
  const bool writes_kv = a->k_new != nullptr;
  if (writes_kv) {
    const int esize = a->dtype == HOOK_BF16 ? 2 : 4;
    KvWriteParams& w = p.kvw;
    w.num_seqs = a->num_seqs; w.total_q = a->total_q; w.Hkv = a->num_kv_heads; w.max_blocks = a->max_blocks_per_seq;
    w.num_blocks = a->num_blocks; w.row_chunks = a->head_dim * esize / 16; w.kv8 = p.kv8;
    w.k_new = static_cast<const uint4*>(a->k_new); w.v_new = static_cast<const uint4*>(a->v_new);
    w.block_table = a->block_table; w.seq_lens = a->seq_lens; w.cu_q_lens = a->cu_q_lens;
    w.k_cache = const_cast<void*>(a->k_cache); w.v_cache = const_cast<void*>(a->v_cache);
    w.k_scale = a->k_scale; w.v_scale = a->v_scale;
  }
  char* ws = static_cast<char*>(workspace);
  p.hdr = reinterpret_cast<PlanHeader*>(ws + l.off_hdr);
  p.pf_items = reinterpret_cast<WorkItem*>(ws + l.off_pf);
  p.pf_cap = l.pf_cap;
  p.dec_items = reinterpret_cast<WorkItem*>(ws + l.off_dec);
  p.dec_cap = l.dec_cap;
  p.seq_dec = reinterpret_cast<int2*>(ws + l.off_seq);
  p.partials = reinterpret_cast<float*>(ws + l.off_part);
  p.pf_waves = l.pf_waves; p.hpw = l.hpw; p.rows_per_wg = l.rows_per_wg; p.hgroups = l.hgroups;
  p.dec_hp = l.dec_hp; p.dec_hgroups = l.dec_hgroups;
  p.batch_kind = a->batch_kind;
  // single rows of few sequences find their work themselves (make_layout), and so do row blocks while there are
  // few of them (or the planner would have nothing to sort)
  const bool streams = a->dtype == HOOK_BF16 && l.ranges > 0 && a->batch_kind != HOOK_BATCH_PREFILL_ONLY;
  p.dec_ranges = streams ? l.ranges : 0;
  p.pf_self = a->dtype == HOOK_BF16 && a->num_seqs <= kScanMaxSeqs && a->batch_kind != HOOK_BATCH_DECODE_ONLY &&
              (streams || a->batch_kind == HOOK_BATCH_PREFILL_ONLY) &&
              (a->num_seqs == 1 || (long long)(a->total_q / l.rows_per_wg) * a->num_kv_heads * l.hgroups * (l.pf_waves / 4) <= kSelfPlanMaxWgs);
  p.one_launch = shares_launch(a, l) ? 1 : 0;
  if (p.one_launch) share_compute_units(a, l, p);
  // The streaming kernel can do without a write ahead of it while a wave can hold every new row's place, one per lane.
  // (A launch ahead costs a call 4 us: 1 x 1237 tokens 16.6 us against 11.7, 8 x 4096 30.2 against 26.3, 64 x 2048 77.2
  // against 72.8.  Where to look would take more registers for more sequences, and the loop has none to spare.)
  p.dec_write = writes_kv && streams && a->batch_kind == HOOK_BATCH_DECODE_ONLY && a->num_seqs <= 64 && a->total_q <= a->num_seqs;
  p.plan_fresh = a->plan_mode == HOOK_PLAN_FRESH;

  hipStream_t st = static_cast<hipStream_t>(a->stream);
  auto mark = [&](int i) { return !ev || hipEventRecord(ev[i], st) == hipSuccess; };
  if (!mark(0)) return HOOK_ERR_LAUNCH;
  // a small batch of single rows writes its rows while streaming, the planning launch carries the cache write where
  // there is one, else it gets a launch of its own
  const bool plans = a->dtype == HOOK_BF16 && a->plan_mode == HOOK_PLAN_FRESH &&
                     !(a->batch_kind == HOOK_BATCH_DECODE_ONLY ? streams : p.pf_self != 0);
  if (writes_kv && !p.dec_write && !plans && launch_kv_write(p.kvw, st) != hipSuccess)
    return HOOK_ERR_LAUNCH;
  if (a->dtype == HOOK_F32) {
    if (launch_attn_f32(p, a->head_dim, st) != hipSuccess) return HOOK_ERR_LAUNCH;
    for (int i = 1; i < 5; ++i)
      if (!mark(i)) return HOOK_ERR_LAUNCH;
    return HOOK_OK;
  }
  // (a reusing call finds the work lists of the same batch in the workspace)
  if ((plans && launch_plan(p, st) != hipSuccess) || !mark(1)) return HOOK_ERR_LAUNCH;
  const bool chunks = a->batch_kind != HOOK_BATCH_DECODE_ONLY, singles = a->batch_kind != HOOK_BATCH_PREFILL_ONLY;
  if ((p.one_launch ? launch_mixed(p, a->head_dim, st) : chunks ? launch_prefill(p, a->head_dim, st) : hipSuccess) != hipSuccess || !mark(2))
    return HOOK_ERR_LAUNCH;
  if ((singles && !p.one_launch && launch_decode(p, a->head_dim, st) != hipSuccess) || !mark(3)) return HOOK_ERR_LAUNCH;
  if ((singles && launch_combine(p, a->head_dim, st) != hipSuccess) || !mark(4)) return HOOK_ERR_LAUNCH;
  return HOOK_OK;
}
}  // namespace hook

using hook::run_attn_probe;

extern "C" {

hook_status hook_attn_probe(const hook_attn_probe_args* a) {
  return a ? run_attn_probe(a, nullptr, a->workspace, a->workspace_bytes) : HOOK_ERR_NULL;
}

// ---- the same call on the library's own scratch memory ---------------------------------------
// Work lists and decode partials live in a fixed array in device memory instead of a caller
// workspace, so the call needs nothing allocated by anybody.  Every GPU holds its own copy of the
// array at its own address; the host learns that address once per device.
static __device__ __attribute__((used)) __align__(256) unsigned char scratch[HOOK_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];   // zero-initialised: address of `scratch` on each device

// Device address of `scratch` on the current device (null on failure).  The array's name is a
// host-side handle, not an address: only the pointer returned here may be given to kernels.
void* scratch_on_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr) return ptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
  g_scratch_ptr[dev].store(ptr, std::memory_order_release);   // racing threads store the same value
  return ptr;
}
}  // namespace

size_t hook_attn_probe_static_capacity(void) { return (size_t)HOOK_STATIC_SCRATCH_BYTES; }

hook_status hook_attn_probe_static(const hook_attn_probe_args* a) {
  // the argument and size checks come first, so that a call that is refused never touches the device
  bool nothing_to_do = false;
  const hook_status checked = hook::check_attn_probe_args(a, &nothing_to_do);
  if (checked != HOOK_OK || nothing_to_do) return checked;
  if (make_layout(a, 0).needed > (size_t)HOOK_STATIC_SCRATCH_BYTES) return HOOK_ERR_WORKSPACE;
  void* ws = scratch_on_current_device();
  if (!ws) return HOOK_ERR_LAUNCH;
  return run_attn_probe(a, nullptr, ws, (size_t)HOOK_STATIC_SCRATCH_BYTES);
}


hook_status hook_attn_probe_device_status(const void* workspace, void* stream, int32_t* status_bits) {
  if (!workspace || !status_bits) return HOOK_ERR_NULL;
  PlanHeader h{};
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(&h, workspace, sizeof h, hipMemcpyDeviceToHost, st) != hipSuccess) return HOOK_ERR_LAUNCH;
  if (hipStreamSynchronize(st) != hipSuccess) return HOOK_ERR_LAUNCH;
  *status_bits = h.status;
  return HOOK_OK;
}

hook_status hook_steer(void* hidden, const void* vec, float alpha, const uint8_t* token_mask,
                       int32_t num_tokens, int32_t hidden_dim, int32_t dtype, void* stream) {
  if (num_tokens < 0 || hidden_dim < 0) return HOOK_ERR_SHAPE;
  if (dtype != HOOK_BF16 && dtype != HOOK_F32) return HOOK_ERR_UNSUPPORTED;
  if (hidden_dim % (dtype == HOOK_BF16 ? 8 : 4) != 0) return HOOK_ERR_UNSUPPORTED;
  if (num_tokens == 0 || hidden_dim == 0) return HOOK_OK;
  if (!hidden || !vec || !token_mask) return HOOK_ERR_NULL;
  if ((reinterpret_cast<uintptr_t>(hidden) | reinterpret_cast<uintptr_t>(vec)) % 16 != 0) return HOOK_ERR_UNSUPPORTED;
  if (alpha == 0.0f) return HOOK_OK;
  return launch_steer(hidden, vec, alpha, token_mask, num_tokens, hidden_dim, dtype,
                      static_cast<hipStream_t>(stream)) == hipSuccess ? HOOK_OK : HOOK_ERR_LAUNCH;
}

hook_status hook_parse_layer_heads(const char* text, int32_t* layers, int32_t* heads, int32_t capacity,
                                   int32_t* count) {
  if (!text || !count || capacity < 0 || (capacity > 0 && (!layers || !heads))) return HOOK_ERR_NULL;
  *count = 0;
  const char* c = text;
  auto skip_blank = [&]() { while (*c == ' ' || *c == '\t' || *c == '\n' || *c == '\r') ++c; };
  auto number = [&](int32_t* out) -> bool {   // blanks, digits, blanks
    skip_blank();
    if (*c < '0' || *c > '9') return false;
    long long v = 0;
    while (*c >= '0' && *c <= '9') {
      v = v * 10 + (*c - '0');
      if (v > (1ll << 30)) return false;
      ++c;
    }
    skip_blank();
    *out = (int32_t)v;
    return true;
  };
  int32_t n = 0;
  for (;;) {
    skip_blank();
    if (*c == '\0') break;
    if (*c == ';') { ++c; continue; }          // empty part
    int32_t layer = 0;
    if (!number(&layer) || *c != ':') return HOOK_ERR_SHAPE;
    ++c;
    int32_t in_part = 0;
    for (;;) {
      int32_t head = 0;
      if (!number(&head)) return HOOK_ERR_SHAPE;
      if (n < capacity) { layers[n] = layer; heads[n] = head; }
      ++n;
      ++in_part;
      if (*c == ',') { ++c; continue; }
      break;
    }
    if (in_part == 0) return HOOK_ERR_SHAPE;
    if (*c == ';') { ++c; continue; }
    if (*c == '\0') break;
    return HOOK_ERR_SHAPE;
  }
  *count = n;
  return n > capacity ? HOOK_ERR_WORKSPACE : HOOK_OK;
}

const char* hook_status_string(hook_status s) {
  switch (s) {
    case HOOK_OK: return "ok";
    case HOOK_ERR_NULL: return "null pointer";
    case HOOK_ERR_SHAPE: return "inconsistent shape";
    case HOOK_ERR_UNSUPPORTED: return "unsupported configuration";
    case HOOK_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case HOOK_ERR_LAUNCH: return "kernel launch failed";
  }
  return "unknown status";
}

int hook_version(void) { return 2; }

}  // extern "C"
