// offsets.hpp -- the arithmetic of decompression's chunk offsets.  The sizes
// come from the stream and may hold anything, so every step here has to stay
// right, or at least inside the stream, for any of them.  constexpr: used by
// the kernels, and by a host program that checks it.
#pragma once

#include <stdint.h>

namespace falcon_dev {

// A chunk's size as a scan counts it.  No chunk is larger than an all-dense
// float64 one; a larger size fails its own chunk whatever it counts for, and
// counted in full it would run the 32-bit offsets inside a tile over, from
// which the series behind it in the tile would get offsets before their
// payload.
constexpr uint32_t kSizeCap = 3 + 8 + 8 + 64 * 128;
constexpr int kScanTile = 4096;  // chunk sizes per workgroup of the scans
static_assert((uint64_t)kScanTile * kSizeCap < 1ull << 32, "offsets inside a tile fit 32 bits");
constexpr uint32_t scan_size(uint32_t size) { return size < kSizeCap ? size : kSizeCap; }

// Whether a payload of S bytes at offset off lies inside the payload_bytes of
// its stream, and the last one ends with them.  No sum that could wrap.
constexpr bool payload_inside(uint64_t off, uint32_t S, uint64_t payload_bytes, bool last) {
  return off <= payload_bytes && (last ? S == payload_bytes - off : S <= payload_bytes - off);
}

}  // namespace falcon_dev
