// kernels_f32.hip -- the f32 instantiations of the compression and
// decompression kernels (codec_kernels.hpp) and their launchers.
#include "codec_kernels.hpp"

namespace falcon_dev {

constexpr int kPassWaves = pass_waves(1);

hipError_t launch_compress_f32(const CompressArgs& a, int pass, int grid, hipStream_t s) {
  if (pass == 1) hipLaunchKernelGGL((k_compress_pass<TF32, kPassWaves, 1>), dim3(grid), dim3(64 * kPassWaves), 0, s, a);
  else hipLaunchKernelGGL((k_compress_pass<TF32, kPassWaves, 2>), dim3(grid), dim3(64 * kPassWaves), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_decompress_f32(const DecompressArgs& a, bool direct, int grid, hipStream_t s) {
  const dim3 g(grid), b(64 * kWavesD);
  if (a.many) {
    if (direct) hipLaunchKernelGGL((k_decompress<TF32, true, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_decompress<TF32, false, true>), g, b, 0, s, a);
  } else {
    if (direct) hipLaunchKernelGGL((k_decompress<TF32, true, false>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_decompress<TF32, false, false>), g, b, 0, s, a);
  }
  return hipGetLastError();
}

const void* compress_kernel_f32(int pass) {
  if (pass == 1) return reinterpret_cast<const void*>(&k_compress_pass<TF32, kPassWaves, 1>);
  return reinterpret_cast<const void*>(&k_compress_pass<TF32, kPassWaves, 2>);
}

template <int V>
static const void* size_pass_variant_f32() {
  return reinterpret_cast<const void*>(&k_compress_pass<TF32, kVariantWaves, 1, V, kVarWaveBlocks>);
}

// The write pass follows the flags the size pass stored, so one write
// kernel serves every variant.
const void* compress_variant_kernel_f32(int variant, int pass) {
  if (pass == 2)
    return reinterpret_cast<const void*>(&k_compress_pass<TF32, kVariantWaves, 2, kVarFalcon, kVarWaveBlocks>);
  if (variant == kVarElf) return size_pass_variant_f32<kVarElf>();
  if (variant == kVarSparse) return size_pass_variant_f32<kVarSparse>();
  if (variant == kVarDense) return size_pass_variant_f32<kVarDense>();
  return nullptr;
}

// For the occupancy.  A launch of one series would fit 7 waves a SIMD instead
// of 6, and is slower for it (1 GiB in fixed shares: 354 against 343 us).
const void* decompress_kernel_f32() { return reinterpret_cast<const void*>(&k_decompress<TF32, false, true>); }

template <int NW>
static void launch_queue(const CompressArgs& a, int grid, hipStream_t s) {
  if (a.many) hipLaunchKernelGGL((k_compress_queue<TF32, NW, true>), dim3(grid), dim3(64 * NW), 0, s, a);
  else hipLaunchKernelGGL((k_compress_queue<TF32, NW, false>), dim3(grid), dim3(64 * NW), 0, s, a);
}

hipError_t launch_compress_queue_f32(const CompressArgs& a, int nw, int grid, hipStream_t s) {
  if (nw == queue_large(1)) launch_queue<queue_large(1)>(a, grid, s);
  else launch_queue<4>(a, grid, s);
  return hipGetLastError();
}

// for the occupancy; launches of one series hold as many workgroups per CU
const void* compress_queue_kernel_f32(int nw) {
  return nw == queue_large(1) ? reinterpret_cast<const void*>(&k_compress_queue<TF32, queue_large(1), true>)
                              : reinterpret_cast<const void*>(&k_compress_queue<TF32, 4, true>);
}

}  // namespace falcon_dev
