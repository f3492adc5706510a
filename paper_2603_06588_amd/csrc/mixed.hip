// Query chunks and single rows of one batch in one launch: a chunk kernel that is bound by the matrix cores and a stream that
// is bound by memory.  What that saves is mostly a launch with its start-up and drain, which is why it is for batches of few
// sequences (shares_launch in api.hip); the two overlap less than one would think.  A workgroup of each on every compute unit
// (where they land has been checked): 64 contexts of 4096 tokens stream in 225 instead of 172 us, but the chunks run at a quarter of
// their speed, since their tile fetches wait their turn behind the stream's in the compute unit's memory path (with the stream's
// blocks in L2 both take 207 us, with the chunks' tiles in L2 284, as it is 320, one after the other 312).  On compute units of their own
// the chunks run at full speed, but eight waves stream 30-40 GB/s (their arithmetic), and workgroups that draw their work by
// compute unit leave a tail of 60 us: 336.
#include "decode_device.h"
#include "prefill_device.h"

namespace hook {

namespace {

// The first workgroups take ranges of the single rows' contexts, one or two workgroups to a compute unit (dec_ranges), the rest row blocks.
// Three blocks are requested ahead: the registers are there, and a wave has its SIMD's single rows to itself or shares them with one other.
// (Groups of eight heads over a 16-bit cache at head size 128 would spill eight registers, and have two workgroups to a
// compute unit instead: one workgroup and three blocks, two and three, two and one, 28 x 16384 tokens and a chunk of 130 rows 320, 335 and
// 305 us, 28 x 4096 and 100 92, 101 and 87.)
// K rows by half lines at head size 128 for groups of four, as in the launch of their own beyond kLineSeqs: whole lines, 32 / 8 heads, 16 x 3000-6000
// tokens and 2 x 1000 rows 69.9 -> 65.9, 28 x 4096 and 4 x 2048 199 -> 191, but 8 x 32768 and 64 168 -> 172, 28 x 8192 and 130 150 -> 152,
// and no line between the two has been looked for.
template <int D, bool KV8, int HP, bool PLANNED>
__global__ __launch_bounds__(256, 2) void k_mixed(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  typedef float Red[4][HP][DecodeCfg<D>::PSTR];
  static_assert(sizeof(Red) <= Cfg<D, KV8, 4>::LDS, "");
  constexpr int AHEAD = HP == 8 && D == 128 && !KV8 ? 1 : 3;
  const int rows = p.dec_ranges * p.Hkv * p.dec_hgroups, first = (rows + 7) & ~7;      // (row blocks keep their chiplets)
  const int bid = blockIdx.x;
  if (bid < first) {
    if (bid < rows)
      stream_range<D, HP, KV8, lines_always<D, HP, KV8>(), kStreamSeqs / 64, AHEAD, true>(p, *reinterpret_cast<Red*>(smem), bid);
    return;
  }
  row_block<D, KV8, 4, false, PLANNED>(p, smem, bid - first, gridDim.x - first - 1);
}

template <int D, bool KV8, int HP, bool PLANNED>
hipError_t launch_kernel(const AttnParams& p, long long grid, hipStream_t st) {
  static std::atomic<unsigned long long> configured{0};
  constexpr int lds = Cfg<D, KV8, 4>::LDS;
  const hipError_t e = raise_lds_limit_once(reinterpret_cast<const void*>(&k_mixed<D, KV8, HP, PLANNED>), lds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_mixed<D, KV8, HP, PLANNED>), dim3((unsigned)grid), dim3(256), lds, st, p);
  return hipGetLastError();
}

template <int D, bool KV8>
hipError_t launch(const AttnParams& p, long long grid, hipStream_t st) {
  if (p.dec_hp == 8) return p.pf_self ? launch_kernel<D, KV8, 8, false>(p, grid, st) : launch_kernel<D, KV8, 8, true>(p, grid, st);
  return p.pf_self ? launch_kernel<D, KV8, 4, false>(p, grid, st) : launch_kernel<D, KV8, 4, true>(p, grid, st);
}

}  // namespace

hipError_t launch_mixed(const AttnParams& p, int D, hipStream_t st) {
  const long long rows = ((long long)p.dec_ranges * p.Hkv * p.dec_hgroups + 7) & ~7ll;
  const long long grid = rows + (long long)(p.total_q / p.rows_per_wg + p.num_seqs) * p.Hkv * p.hgroups + (p.pf_self ? 1 : 0);
  if (!grid_fits(grid)) return hipErrorInvalidValue;
  if (D == 128) return !p.kv8 ? launch<128, false>(p, grid, st) : launch<128, true>(p, grid, st);
  if (D == 64) return !p.kv8 ? launch<64, false>(p, grid, st) : launch<64, true>(p, grid, st);
  return hipErrorInvalidValue;
}

}  // namespace hook
