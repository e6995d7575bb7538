// queue_wait.hpp -- when the scanning workgroup of a compression launch gives
// up waiting for a chunk's size.  constexpr: used by the kernel, and by a host
// program that checks it.
#pragma once

#include <stdint.h>

namespace falcon_dev {

// Whether launch chunk t, whose size is the first still missing, has a
// resident workgroup to come from.  fits: the workgroups number themselves and
// workgroup 1 + k takes the chunks k NW to k NW + NW - 1; word counts those
// that came (the scanning one first), and is 0 again when all have.  Else the
// chunks are drawn, and a workgroup that has come stays until the last is:
// word counts the draws from the first counter, which chunk 0 comes from.
constexpr bool chunk_taken(bool fits, uint32_t word, uint64_t t, uint32_t nw) {
  return fits ? word == 0 || (uint64_t)(word - 1) * nw > t : t != 0 || word != 0;
}

// The scanning workgroup polls.  A chunk that is taken has its size within
// microseconds, whatever else the device runs: its wave is resident and waits
// for nothing before.  One that is not waits for the device to start the
// workgroup, for as long as other launches hold the chip; that is no failure,
// and its limit only ends a launch whose words were not clear.  A round takes
// about a microsecond.
struct ScanWait {
  static constexpr uint32_t kLookEvery = 256;     // quiet rounds from one look at the queue to the next
  static constexpr uint32_t kLimit = 1u << 22;    // looks without a workgroup: a quarter of an hour and more
  static constexpr uint32_t kTakenWeight = 256;   // a taken chunk's count for as many: seconds
  uint32_t quiet = 0, looks = 0;

  // A new size has come.
  constexpr void progress() { quiet = looks = 0; }
  // Once a round: whether to look at the queue now.
  constexpr bool look() { return (++quiet & (kLookEvery - 1)) == 0; }
  // What the look found; true: give up.
  constexpr bool give_up(bool another_gave_up, bool taken) {
    looks += taken ? kTakenWeight : 1;
    return another_gave_up || looks > kLimit;
  }
};

}  // namespace falcon_dev
