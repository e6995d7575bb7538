// kernels_mixed.hip -- kernels that take series of both dtypes in one launch
// (the wave branches on the dtype of each chunk's series), and their
// launchers.
#include "codec_kernels.hpp"

namespace falcon_dev {

template <bool DIRECT>
__global__ __launch_bounds__(64 * kWavesD) __attribute__((amdgpu_waves_per_eu(4))) void k_decompress_mixed(
    DecompressArgs a) {
  __shared__ BlockLdsT<kWavesD> sm;
  __shared__ uint64_t tiles[DIRECT ? 1 : 64];
  const uint64_t t_start = now_ticks();
  const int lane = lane_id();
  load_tables(sm.tab);
  if (!DIRECT) load_tiles(a, tiles, lane);
  empty_series_checks(a);
  __syncthreads();
  const int wid = (int)uniform(threadIdx.x >> 6);  // wave-uniform: keeps the chunk loop scalar
  uint8_t* buf = wave_bytes(sm, wid);
  decompress_loop<DIRECT, true>(a, tiles, buf, kWaveLds, lane, wid, t_start,
                  [&](const DecompressSeries& sd, uint64_t c, uint32_t S, uint32_t pad, uint32_t total, bool bad) {
                    if (uniform(sd.dtype) == 2)
                      decompress_chunk<TF64>(sm.tab, buf, sd, c, S, pad, total, bad, a.epoch, lane, a.ctl);
                    else
                      decompress_chunk<TF32>(sm.tab, buf, sd, c, S, pad, total, bad, a.epoch, lane, a.ctl);
                  });
}

hipError_t launch_decompress_mixed(const DecompressArgs& a, bool direct, int grid, hipStream_t s) {
  if (direct) hipLaunchKernelGGL((k_decompress_mixed<true>), dim3(grid), dim3(64 * kWavesD), 0, s, a);
  else hipLaunchKernelGGL((k_decompress_mixed<false>), dim3(grid), dim3(64 * kWavesD), 0, s, a);
  return hipGetLastError();
}

const void* decompress_kernel_mixed() { return reinterpret_cast<const void*>(&k_decompress_mixed<false>); }

hipError_t launch_compress_queue_mixed(const CompressArgs& a, int nw, int grid, hipStream_t s) {
  if (nw == 8) hipLaunchKernelGGL((k_compress_queue_mixed<8>), dim3(grid), dim3(64 * 8), 0, s, a);
  else hipLaunchKernelGGL((k_compress_queue_mixed<4>), dim3(grid), dim3(64 * 4), 0, s, a);
  return hipGetLastError();
}

const void* compress_queue_kernel_mixed(int nw) {
  return nw == 8 ? reinterpret_cast<const void*>(&k_compress_queue_mixed<8>)
                 : reinterpret_cast<const void*>(&k_compress_queue_mixed<4>);
}

}  // namespace falcon_dev
