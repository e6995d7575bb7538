// kernels_common.hip -- prefix scans of chunk sizes (two-pass compression,
// decompression), fill, and the dispatch of launches to the per-form translation units.
#include "codec_kernels.hpp"

namespace falcon_dev {

// ---------------------------------------------------------------------------
// Prefix sum of a chunk size array into chunk offsets (two-pass compression).
// Three small kernels over tiles of kScanTile sizes: tile sums, a scan of the
// tile sums, and the per-tile scan.
// ---------------------------------------------------------------------------
static_assert(kScanTile == 256 * 16, "256 threads x 16 sizes");

__device__ __forceinline__ uint64_t block_excl_scan256(uint64_t v, uint64_t* tmp, uint64_t& total) {
  // tmp: 4 words of LDS (one per wave)
  const int lane = lane_id(), wid = threadIdx.x >> 6;
  const uint64_t incl = wave_incl_scan64(v, lane);
  if (lane == 63) tmp[wid] = incl;
  __syncthreads();
  uint64_t before = 0;
  for (int i = 0; i < wid; ++i) before += tmp[i];
  total = tmp[0] + tmp[1] + tmp[2] + tmp[3];
  __syncthreads();
  return before + incl - v;
}

__global__ __launch_bounds__(256) void k_scan_tiles(const uint32_t* sizes, uint64_t n, uint64_t* tile_sum) {
  __shared__ uint64_t tmp[4];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + threadIdx.x * 16;
  uint64_t sum = 0;
  for (int k = 0; k < 16; ++k)
    if (base + k < n) sum += sizes[base + k];
  uint64_t total;
  block_excl_scan256(sum, tmp, total);
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_scan_tile_sums(uint64_t* tile_sum, uint64_t ntiles) {
  __shared__ uint64_t tmp[4];
  uint64_t carry = 0;
  for (uint64_t b0 = 0; b0 < ntiles; b0 += 256) {
    const uint64_t i = b0 + threadIdx.x;
    const uint64_t v = i < ntiles ? tile_sum[i] : 0;
    uint64_t total;
    const uint64_t ex = block_excl_scan256(v, tmp, total);
    if (i < ntiles) tile_sum[i] = carry + ex;  // becomes the tile's offset
    carry += total;
  }
}

__global__ __launch_bounds__(256) void k_scan_apply(const uint32_t* sizes, uint64_t n, const uint64_t* tile_off,
                                                    uint64_t* offsets) {
  __shared__ uint64_t tmp[4];
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + threadIdx.x * 16;
  uint32_t v[16];
  uint64_t sum = 0;
  for (int k = 0; k < 16; ++k) {
    v[k] = base + k < n ? sizes[base + k] : 0u;
    sum += v[k];
  }
  uint64_t total;
  uint64_t run = tile_off[blockIdx.x] + block_excl_scan256(sum, tmp, total);
  for (int k = 0; k < 16; ++k) {
    if (base + k < n) offsets[base + k] = run;
    run += v[k];
  }
}

__global__ void k_fill_u64(uint64_t* p, size_t n, uint64_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// ---------------------------------------------------------------------------
// Decompression's scan (Sec. 4: the size array is scanned into the offset
// array), as far as one launch gets without waiting: offsets inside each tile
// and the tile sums.  The decoder's waves add the tile sums themselves, which
// saves two launches: 43 -> 14 us before the decoder on 261,889 chunks.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_scan_local(DecompressSeries one, const DecompressSeries* many, uint32_t ns,
                                                    uint64_t n, uint32_t* local, uint64_t* tile_sum,
                                                    uint64_t* times) {
  __shared__ uint64_t tmp[4];
  if (times && blockIdx.x == 0 && threadIdx.x == 0) times[0] = times[1] = now_ticks();
  const uint64_t base = (uint64_t)blockIdx.x * kScanTile + threadIdx.x * 16;
  uint32_t v[16];
  uint64_t sum = 0;
  if (base < n) {
    // a thread's chunks lie in one series, or in a few in a row
    uint32_t i = many ? find_index(many, ns, base) : 0;
    DecompressSeries sd = one;
    uint64_t end = n;
    auto enter = [&]() {
      sd = many[i];
      end = i + 1 < ns ? many[i + 1].chunk0 : n;
    };
    if (many) enter();
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const uint64_t t = base + k;
      v[k] = 0;
      if (t < n) {
        while (t >= end) {
          ++i;
          enter();
        }
        v[k] = scan_size(reinterpret_cast<const uint32_t*>(sd.in + kHdrBytes)[t - sd.chunk0]);
        sum += v[k];
      }
    }
  }
  uint64_t total;
  uint32_t run = (uint32_t)block_excl_scan256(sum, tmp, total);
  if (base < n) {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (base + k < n) local[base + k] = run;
      run += v[k];
    }
  }
  if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

hipError_t launch_scan_local(DecompressArgs* a, uint64_t total_chunks, uint32_t* local, uint64_t* tiles,
                             hipStream_t s) {
  const uint64_t ntiles = scan_tiles(total_chunks);
  a->local = local;
  a->tiles = tiles;
  a->ntiles = (uint32_t)ntiles;
  a->tiles_scanned = ntiles > 64;  // up to 64 (262,144 chunks) the decoder's waves add them
  hipLaunchKernelGGL(k_scan_local, dim3((unsigned)ntiles), dim3(256), 0, s, a->one, a->many, a->nseries, total_chunks,
                     local, tiles, a->times);
  if (a->tiles_scanned) hipLaunchKernelGGL(k_scan_tile_sums, dim3(1), dim3(256), 0, s, tiles, ntiles);
  return hipGetLastError();
}

hipError_t launch_compress(const CompressArgs& a, int form, int pass, int grid, hipStream_t s) {
  return form == 2 ? launch_compress_f64(a, pass, grid, s) : launch_compress_f32(a, pass, grid, s);
}

hipError_t launch_compress_queue(const CompressArgs& a, int form, int nw, int grid, hipStream_t s) {
  if (form == 2) return launch_compress_queue_f64(a, nw, grid, s);
  if (form == 1) return launch_compress_queue_f32(a, nw, grid, s);
  return launch_compress_queue_mixed(a, nw, grid, s);
}

hipError_t launch_compress_variant(const CompressArgs& a, int form, int variant, int pass, int grid, hipStream_t s) {
  const void* fn = form == 2 ? compress_variant_kernel_f64(variant, pass)
                             : form == 1 ? compress_variant_kernel_f32(variant, pass) : nullptr;
  if (!fn) return hipErrorInvalidValue;
  CompressArgs copy = a;
  void* args[] = {&copy};
  return hipLaunchKernel(fn, dim3(grid), dim3(64 * kVariantWaves), args, 0, s);
}

hipError_t launch_decompress(const DecompressArgs& a, int form, bool direct, int grid, hipStream_t s) {
  if (form == 2) return launch_decompress_f64(a, direct, grid, s);
  if (form == 1) return launch_decompress_f32(a, direct, grid, s);
  return launch_decompress_mixed(a, direct, grid, s);
}

hipError_t launch_scan_sizes(const uint32_t* sizes, uint64_t n, uint64_t* tile_tmp, uint64_t* offsets,
                             hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint64_t ntiles = (n + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)ntiles), dim3(256), 0, s, sizes, n, tile_tmp);
  hipLaunchKernelGGL(k_scan_tile_sums, dim3(1), dim3(256), 0, s, tile_tmp, ntiles);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)ntiles), dim3(256), 0, s, sizes, n, tile_tmp, offsets);
  return hipGetLastError();
}
uint64_t scan_tiles(uint64_t n) { return (n + kScanTile - 1) / kScanTile; }

hipError_t launch_fill_u64(uint64_t* p, size_t n, uint64_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

static int max_grid_of(const void* fn, int device, int block) {
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, device) != hipSuccess) return 256;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, block, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  return per_cu * prop.multiProcessorCount;
}

int max_grid_compress(int device, int form, int pass) {
  return max_grid_of(form == 2 ? compress_kernel_f64(pass) : compress_kernel_f32(pass), device, 64 * pass_waves(form));
}

int max_grid_compress_queue(int device, int form, int nw) {
  const void* fn = form == 2 ? compress_queue_kernel_f64(nw)
                             : form == 1 ? compress_queue_kernel_f32(nw) : compress_queue_kernel_mixed(nw);
  return max_grid_of(fn, device, 64 * nw);
}

int max_grid_compress_variant(int device, int form, int variant, int pass) {
  const void* fn = form == 2 ? compress_variant_kernel_f64(variant, pass)
                             : form == 1 ? compress_variant_kernel_f32(variant, pass) : nullptr;
  return fn ? max_grid_of(fn, device, 64 * kVariantWaves) : 0;
}

int max_grid_decompress(int device, int form) {
  const void* fn = form == 2 ? decompress_kernel_f64() : form == 1 ? decompress_kernel_f32()
                                                                    : decompress_kernel_mixed();
  return max_grid_of(fn, device, 64 * kWavesD);
}

}  // namespace falcon_dev
