// internal.hpp -- launch interface between the C ABI (api.cpp) and the
// kernels (kernels_*.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "offsets.hpp"

namespace falcon_dev {

// Control block of a launch queue, in pinned host memory so that the host
// reads it without a copy: the decompression error word (receives the launch
// epoch when a chunk fails a check) and the compression error word (set when
// a wait for an offset gives up, which a correct run never does).
struct Ctl {
  uint32_t error;
  uint32_t qerror;
  uint64_t pad;
};

// Compression takes chunks from ticket counters, each in a 128-byte line of
// its own (a counter is one word every kQueueStride): a launch in workgroups
// of NW waves uses the first NW of kQueueGroups counters.  The lines after
// them elect the scanning workgroup.
constexpr int kQueueGroups = 12;
constexpr int kRoleLines = 16;
constexpr int kQueueStride = 16;
// and those of decompression's draws, kDrawGroups lines from kDrawLine on,
// used by launches of more than kDrawFrom chunks a wave: shorter ones gain
// nothing.  Walks, fixed against drawn, us a call: float64 3 chunks a wave 46.8
// / 46.8, 4 56.6 / 56.5, 5 66.3 / 63.0, 6 76.4 / 73.4, 8 95.5 / 91.5; float32 3
// 35.8 / 37.6, 4 42.2 / 40.4, 5 47.8 / 48.0, 6 55.0 / 52.5, 8 68.5 / 65.1.
constexpr int kDrawLine = kQueueGroups + 1 + kRoleLines;
constexpr int kDrawGroups = 64;
constexpr uint64_t kDrawFrom = 4;
constexpr int kQueueWords = kQueueStride * (kDrawLine + kDrawGroups);
constexpr int kQueueSlack = 8192;  // size and offset words past the chunks (the scan reads ahead)

// Time stamps of a timed launch, in ticks of the device's constant-rate
// clock: words 0-2 the launch's start and, for compression, when the last
// size and the last offset were known; then kTimeEnds lines of kTimeStride
// words whose maximum is the launch's end.
constexpr int kTimeStride = 16;
constexpr int kTimeEnds = 16;
constexpr int kTimeWords = kTimeStride * (1 + kTimeEnds);

// One array to compress.  chunk0 is the global index of its first chunk in
// the launch (prefix of the chunk counts of the series before it).
struct CompressSeries {
  const void* in;
  uint8_t* out;
  uint64_t n;
  uint64_t chunk0;
  uint32_t dtype;    // 1 = f32, 2 = f64
  uint32_t idx;      // position of the series in the caller's list (lens[idx])
};

struct DecompressSeries {
  const uint8_t* in;
  uint8_t* out;
  uint64_t n;
  uint64_t chunk0;
  uint64_t payload_bytes;  // ~0: read from the stream header on the device
  uint64_t in_len;         // stream bytes
  uint32_t dtype;
  uint32_t idx;
};

// What the size pass of compression learns about a chunk and the write pass
// reuses: the row scheme flags (bit p set = plane p is written dense), the
// chunk's byte count, and its header bytes alpha_max, beta_hat_max, w.
struct ChunkMeta {
  uint64_t flags;
  uint32_t S;
  uint8_t A, B, w, pad;
};

// A batch's descriptors are followed by an index into them: the series of
// every 64th launch chunk, up to the last chunk's block and one more.  A chunk's
// series is then one of a few (find_series), where a search over all
// descriptors is eleven dependent loads for 2,000 of them: decompressing those
// 259 -> 237 us, compressing 342 -> 324; of 200, 54 -> 51 and 73 -> 73.
constexpr int kIndexShift = 6;

struct CompressArgs {
  CompressSeries one;            // the series of a one-series launch (many == null)
  const CompressSeries* many;    // device array, sorted by chunk0, for batch launches
  const uint32_t* index;  // batch launches: index[k] is the series of launch chunk 64k (see kIndexShift)
  uint32_t nseries;
  uint32_t total_waves;
  uint64_t total_chunks;  // chunks of this launch: launch chunks t0 .. t0 + total_chunks - 1
  uint64_t t0;
  uint64_t* lens;      // batch launches: stream length of each series (device), else null
  ChunkMeta* meta;     // one per launch chunk, written by the size pass
  uint32_t* gsizes;    // chunk sizes by launch chunk (scan input), written by the size pass
  const uint64_t* offsets;  // exclusive prefix of gsizes, read by the write pass
  // one launch (work queue and scanning workgroup): kQueueWords counters, and one
  // size word and one offset word per chunk of the launch, all 0 at the
  // launch's start and again at its end
  uint64_t* qctr;
  uint32_t* qsize;
  uint64_t* qoff;
  Ctl* ctl;
  uint64_t* times;     // kTimeWords, or null
};

struct DecompressArgs {
  DecompressSeries one;
  const DecompressSeries* many;
  const uint32_t* index;  // batch launches: index[k] is the series of launch chunk 64k (see kIndexShift)
  uint32_t nseries;
  uint32_t total_waves;
  uint64_t total_chunks;
  uint64_t t0;
  // offsets of the chunks, unless the launch adds them up itself (direct):
  // each launch chunk's inside its tile, and the tiles' sums (tiles_scanned:
  // the sums of the tiles before)
  const uint32_t* local;
  const uint64_t* tiles;
  uint32_t tiles_scanned;
  uint32_t ntiles;
  uint32_t epoch;
  uint32_t pad;
  uint64_t* qctr;      // kQueueWords counters as in CompressArgs, where total_chunks > kDrawFrom * total_waves
  Ctl* ctl;
  uint64_t* times;     // kTimeWords, or null
};

// A decompression launch adds up its chunks' offsets itself (direct) when no
// series is longer than this many chunks; else k_scan_local runs before it.
// One series, direct against scanned, us a call: float64 1 chunk 9.9 / 13.3,
// 1,024 11.7 / 17.1, 4,093 17.8 / 22.3, 6,000 26.5 / 26.7, 8,000 36.2 / 37.5, 12,000
// 52 / 47; float32 6.6 / 9.9, 8.5 / 13.8, 14.2 / 17.7, 18.9 / 20.8, 22.3 / 21.7,
// 35.5 / 27.0.  So one series gains up to some 6,000 chunks; the line is lower
// for what a batch of many long series loses, whose adding up is hidden by
// nothing.  Plans: 200 series of 1-360 chunks 57 / 67 us, 2,000 309 / 323;
// float64 1,024 series of 256 chunks 887 / 895, 128 of 2,048 915 / 860, 64 of 4,096
// 953 / 862, float32 500 / 503, 489 / 460, 544 / 466.
constexpr uint64_t kDirectChunks = 4096;

// Wavefronts per workgroup of the two compression passes.  The float32
// passes run 6 waves per SIMD (their LDS buffer is half the float64 one and
// their registers are held to 80), which workgroups of 8 waves fill (3 per
// CU); 16-wave workgroups would fit only one.
constexpr int pass_waves(int dtype) { return dtype == 1 ? 8 : 16; }
constexpr int kDecompressWaves = 4;   // wavefronts per decompression workgroup

// Wavefronts per workgroup of a compression launch, which sets its ticket
// counters and its scanning waves too: 4 up to 1,024 chunks (queue_waves),
// beyond that 8, and 12 in float32 (two workgroups hold a CU's 24 waves).
// float32 chunks are half as large, and one scanning workgroup of 8 waves
// kept up with 490 of them a microsecond: 512 MiB of mixed float32, 8 against
// 12 waves, 271 / 250 us, 256 MiB of decimals 143 / 124, 32 MiB 36.2 / 33.2;
// 16 waves leave 4 a SIMD (286 / 141 / 33.3).  float64 in 16-wave
// workgroups: 2 GiB of readings 781 / 827.
constexpr int queue_large(int form) { return form == 1 ? 12 : 8; }
constexpr int queue_nw(int form, int nw) { return nw == 4 ? 4 : queue_large(form); }

// Kernel forms: one instantiation per dtype (1 = f32, 2 = f64) and a mixed
// one (3) that takes either dtype per series.
constexpr int kFormMixed = 3;
// The two-pass compression of falcon_compress_noalloc, one dtype per launch
// (form 1 or 2), pass_waves(form) wavefronts per workgroup.  pass 1: the
// size pass (meta, gsizes and the stream's size array); pass 2: the write
// pass, after a scan of gsizes into offsets.
hipError_t launch_compress(const CompressArgs& a, int form, int pass, int grid, hipStream_t s);
// direct: no series of the launch has more than kDirectChunks chunks, and
// a.local and a.tiles are not used.
hipError_t launch_decompress(const DecompressArgs& a, int form, bool direct, int grid, hipStream_t s);
// One-launch compression (work queue over chunks, a scanning workgroup for the
// offsets, so at least two workgroups), nw = 4 or queue_large(form) wavefronts
// per workgroup: a.qctr, a.qsize, a.qoff, a.ctl set.
hipError_t launch_compress_queue(const CompressArgs& a, int form, int nw, int grid, hipStream_t s);
hipError_t launch_compress_queue_f64(const CompressArgs& a, int nw, int grid, hipStream_t s);
hipError_t launch_compress_queue_f32(const CompressArgs& a, int nw, int grid, hipStream_t s);
hipError_t launch_compress_queue_mixed(const CompressArgs& a, int nw, int grid, hipStream_t s);
const void* compress_queue_kernel_f64(int nw);
const void* compress_queue_kernel_f32(int nw);
const void* compress_queue_kernel_mixed(int nw);
int max_grid_compress_queue(int device, int form, int nw);
// per-form entry points (one translation unit each)
hipError_t launch_compress_f64(const CompressArgs& a, int pass, int grid, hipStream_t s);
hipError_t launch_compress_f32(const CompressArgs& a, int pass, int grid, hipStream_t s);
hipError_t launch_decompress_f64(const DecompressArgs& a, bool direct, int grid, hipStream_t s);
hipError_t launch_decompress_f32(const DecompressArgs& a, bool direct, int grid, hipStream_t s);
hipError_t launch_decompress_mixed(const DecompressArgs& a, bool direct, int grid, hipStream_t s);
const void* compress_kernel_f64(int pass);
const void* compress_kernel_f32(int pass);
const void* decompress_kernel_f64();
const void* decompress_kernel_f32();
const void* decompress_kernel_mixed();
hipError_t launch_fill_u64(uint64_t* p, size_t n, uint64_t v, hipStream_t s);
// Exclusive prefix of n chunk sizes into offsets; tile_tmp holds
// scan_tiles(n) words.
hipError_t launch_scan_sizes(const uint32_t* sizes, uint64_t n, uint64_t* tile_tmp, uint64_t* offsets, hipStream_t s);
uint64_t scan_tiles(uint64_t n);
// Decompression, before launches that are not direct: every launch chunk's
// offset inside its tile into a->local (total_chunks words) and the tile sums
// into a->tiles (scan_tiles(total_chunks) words), from the sizes at the
// streams of a->one or a->many; sets a->ntiles and a->tiles_scanned.
hipError_t launch_scan_local(DecompressArgs* a, uint64_t total_chunks, uint32_t* local, uint64_t* tiles, hipStream_t s);
// Compression under an ablation variant of Sec. 5.4.2 (variant 1: Elf's
// decimal places, 2: every row sparse, 3: every row dense), one dtype per
// launch (form 1 or 2), kVariantWaves wavefronts per workgroup.
constexpr int kVariantWaves = 8;
hipError_t launch_compress_variant(const CompressArgs& a, int form, int variant, int pass, int grid, hipStream_t s);
const void* compress_variant_kernel_f64(int variant, int pass);
const void* compress_variant_kernel_f32(int variant, int pass);
// Largest number of co-resident workgroups of each kernel on the device.
int max_grid_compress(int device, int form, int pass);
int max_grid_compress_variant(int device, int form, int variant, int pass);
int max_grid_decompress(int device, int form);

}  // namespace falcon_dev
