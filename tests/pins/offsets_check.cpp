// Chunk offsets of a batch as decompression's scan finds them (offsets.hpp),
// over series whose size words are damaged.  Checked for every chunk: one that
// is accepted lies inside its series' payload (in 128 bits, where nothing
// wraps); a series without damage gets its exact offsets, all accepted, wherever
// in a tile it lies; one with damage has a chunk refused.  "wrapping" runs the
// same with sums that wrap (sizes counted in full, off + S compared).
// Prints: chunks N accepted-outside N wrong-neighbours N missed N
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <random>
#include <vector>

#include "../../paper_2511_04140_amd/csrc/offsets.hpp"

using namespace falcon_dev;
typedef unsigned __int128 u128;

struct Series {
  std::vector<uint32_t> sizes;
  uint64_t payload = 0;
  bool damaged = false;
  uint64_t chunk0 = 0;
};

static uint64_t n_chunks, n_outside, n_neighbours, n_missed;

static void check(std::vector<Series>& ss, bool wrapping) {
  std::vector<uint32_t> local;
  std::vector<uint64_t> tile;  // sums, then their exclusive prefix
  uint64_t t = 0, run = 0;
  for (auto& s : ss) {
    s.chunk0 = t;
    for (uint32_t w : s.sizes) {
      if (t++ % kScanTile == 0) {
        if (t > 1) tile.push_back(run);
        run = 0;
      }
      local.push_back((uint32_t)run);
      run += wrapping ? w : scan_size(w);
    }
  }
  tile.push_back(run);
  uint64_t sum = 0;
  for (auto& v : tile) {
    const uint64_t own = v;
    v = sum;
    sum += own;
  }
  auto before = [&](uint64_t x) { return tile[x / kScanTile] + local[x]; };
  for (const auto& s : ss) {
    const uint64_t nc = s.sizes.size();
    uint64_t exact = 0;
    bool refused = false;
    for (uint64_t c = 0; c < nc; ++c) {
      const uint64_t x = s.chunk0 + c, off = before(x) - (c == x ? 0 : before(x - c));
      const uint32_t S = s.sizes[c];
      const bool last = c == nc - 1;
      const bool inside = wrapping ? !(off + S > s.payload || (last && off + S != s.payload))
                                   : payload_inside(off, S, s.payload, last);
      const bool ok = S >= 7 && S <= kSizeCap && inside;
      ++n_chunks;
      if (ok && (u128)off + S > s.payload) ++n_outside;
      if (!s.damaged && (!ok || off != exact)) ++n_neighbours;
      refused |= !ok;
      exact += S;
    }
    if (s.damaged && !refused) ++n_missed;
  }
}

int main(int argc, char** argv) {
  const bool wrapping = argc > 1 && !strcmp(argv[1], "wrapping");
  std::mt19937_64 rng(20251105);
  auto pick = [&](uint64_t lo, uint64_t hi) { return lo + rng() % (hi - lo + 1); };
  // short damaged series whose second chunk would start before the payload
  {
    std::vector<Series> ss(3);
    for (int i = 0; i < 5; ++i) ss[0].sizes.push_back(8000), ss[0].payload += 8000;
    ss[1].sizes = {0u - 6000u, 7000, 5000};
    ss[1].payload = 20000;
    ss[1].damaged = true;
    for (int i = 0; i < 5000; ++i) ss[2].sizes.push_back(11 + i), ss[2].payload += 11 + i;
    check(ss, wrapping);
    ss[1].sizes = {0u - 100u, 5000, 4000};
    check(ss, wrapping);
    ss[1].sizes = {0u - 8000u, 8100, 4000};
    check(ss, wrapping);
  }
  for (int rep = 0; rep < 400; ++rep) {
    std::vector<Series> ss(pick(1, 60));
    for (auto& s : ss) {
      const uint64_t nc = rep % 4 == 0 ? pick(1, 3000) : pick(1, 12);
      for (uint64_t c = 0; c < nc; ++c) s.sizes.push_back((uint32_t)pick(7, kSizeCap)), s.payload += s.sizes.back();
      if (pick(0, 2) == 0) {
        s.damaged = true;
        for (uint64_t k = pick(1, 3); k; --k) {
          uint32_t& w = s.sizes[pick(0, nc - 1)];
          switch (pick(0, 4)) {
            case 0: w = 0u - (uint32_t)pick(1, 9000); break;
            case 1: w = (uint32_t)rng(); break;
            case 2: w = kSizeCap + (uint32_t)pick(1, 3); break;
            case 3: w = 0; break;
            default: w ^= 1u << pick(0, 31); break;
          }
        }
        uint64_t sum = 0;
        bool all = true;
        for (uint32_t w : s.sizes) sum += w, all &= w >= 7 && w <= kSizeCap;
        s.damaged = !(all && sum == s.payload);  // flips that cancel out
      }
    }
    check(ss, wrapping);
  }
  printf("chunks %llu accepted-outside %llu wrong-neighbours %llu missed %llu\n", (unsigned long long)n_chunks,
         (unsigned long long)n_outside, (unsigned long long)n_neighbours, (unsigned long long)n_missed);
  return 0;
}
