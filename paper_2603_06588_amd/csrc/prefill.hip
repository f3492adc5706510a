// Launches of query chunks (prefill_device.h says how the kernel works).
#include "prefill_device.h"

namespace hook {

namespace {

template <int D, bool KV8, int NW, bool SHARED, bool PLANNED>
__global__ __launch_bounds__(64 * NW, 2) void k_prefill(const AttnParams p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  row_block<D, KV8, NW, SHARED, PLANNED>(p, smem, blockIdx.x, gridDim.x - 1);
}

template <int D, bool KV8, int NW, bool SHARED, bool PLANNED>
hipError_t launch_kernel(const AttnParams& p, long long grid, hipStream_t st) {
  static std::atomic<unsigned long long> configured{0};
  constexpr int lds = Cfg<D, KV8, NW>::LDS;
  const hipError_t e = raise_lds_limit_once(reinterpret_cast<const void*>(&k_prefill<D, KV8, NW, SHARED, PLANNED>), lds, configured);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_prefill<D, KV8, NW, SHARED, PLANNED>), dim3((unsigned)grid), dim3(64 * NW), lds, st, p);
  return hipGetLastError();
}

template <int D, bool KV8, int NW>
hipError_t launch(const AttnParams& p, long long grid, hipStream_t st) {
  if (p.rows_per_wg == kWaveRows)
    return p.pf_self ? launch_kernel<D, KV8, NW, false, false>(p, grid, st) : launch_kernel<D, KV8, NW, false, true>(p, grid, st);
  return p.pf_self ? launch_kernel<D, KV8, NW, true, false>(p, grid, st) : launch_kernel<D, KV8, NW, true, true>(p, grid, st);
}

template <int D, bool KV8>
hipError_t launch(const AttnParams& p, long long grid, hipStream_t st) {
  if constexpr (D == 128)
    if (p.pf_waves == 8) return launch<D, KV8, 8>(p, grid, st);
  return launch<D, KV8, 4>(p, grid, st);
}

}  // namespace

hipError_t launch_prefill(const AttnParams& p, int D, hipStream_t st) {
  const long long grid = (long long)(p.total_q / p.rows_per_wg + p.num_seqs) * p.Hkv * p.hgroups + (p.pf_self ? 1 : 0);
  if (grid <= 0) return hipSuccess;
  if (!grid_fits(grid)) return hipErrorInvalidValue;
  if (D == 128) return !p.kv8 ? launch<128, false>(p, grid, st) : launch<128, true>(p, grid, st);
  if (D == 64) return !p.kv8 ? launch<64, false>(p, grid, st) : launch<64, true>(p, grid, st);
  return hipErrorInvalidValue;
}

}  // namespace hook
