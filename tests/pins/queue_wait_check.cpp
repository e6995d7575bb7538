// The scanning workgroup's waits (queue_wait.hpp) on the host.  Prints one line
// per check; the last is the count of wrong answers.
#include <stdint.h>
#include <stdio.h>

#include <random>
#include <vector>

#include "../../paper_2511_04140_amd/csrc/queue_wait.hpp"

using namespace falcon_dev;

// Rounds until a wait gives up, at most max (0: it did not).
template <class Taken, class Failed>
static uint64_t rounds(uint64_t max, Taken taken, Failed failed) {
  ScanWait w;
  for (uint64_t r = 1; r <= max; ++r)
    if (w.look() && w.give_up(failed(r), taken(r))) return r;
  return 0;
}

int main() {
  uint64_t wrong = 0;
  auto never = [](uint64_t) { return false; };
  auto always = [](uint64_t) { return true; };
  auto say = [&](const char* what, uint64_t got, bool ok) {
    printf("%s %llu\n", what, (unsigned long long)got);
    wrong += !ok;
  };
  // a minute in which no working workgroup finds a place on the chip
  uint64_t r = rounds(60000000, never, never);
  say("absent-minute", r, r == 0);
  // it comes after that minute: its chunk still has seconds
  r = rounds(70000000, [](uint64_t i) { return i > 60000000; }, never);
  say("late-comer", r, r > 63000000);
  // a taken chunk whose size never comes, and one that never gets a taker
  r = rounds(1ull << 31, always, never);
  say("taken", r, r > 1000000 && r < 10000000);
  r = rounds(1ull << 31, never, never);
  say("absent", r, r > 600000000);
  // another wave gave up
  r = rounds(10000, never, [](uint64_t i) { return i > 1000; });
  say("another", r, r > 1000 && r <= 1000 + 2 * ScanWait::kLookEvery);
  // progress starts the limits anew
  ScanWait w;
  for (int i = 0; i < 4000000; ++i) wrong += w.look() && w.give_up(false, true);
  w.progress();
  for (int i = 0; i < 4000000; ++i) wrong += w.look() && w.give_up(false, true);

  // workgroups that number themselves: chunk t is taken once 2 + t / NW have come
  for (uint32_t nw : {4u, 8u, 12u})
    for (uint64_t total : {1ull, 3ull, 8ull, 100ull, 515ull}) {
      const uint64_t grid = 1 + (total + nw - 1) / nw;
      for (uint64_t come = 1; come <= grid; ++come)
        for (uint64_t t = 0; t < total; ++t)
          wrong += chunk_taken(true, come == grid ? 0 : come, t, nw) != (2 + t / nw <= come);
    }
  // tickets, drawn in any order by grid - 1 waves a counter, each past the end once
  std::mt19937_64 rng(7);
  uint64_t looked = 0;
  for (int rep = 0; rep < 300; ++rep) {
    const uint32_t nw = rep % 3 == 0 ? 4 : rep % 3 == 1 ? 8 : 12;
    const uint64_t grid = 2 + rng() % 6, total = (grid - 1) * nw + 1 + rng() % 200;
    std::vector<uint64_t> ctr(nw, 0), left(nw, grid - 1);
    std::vector<char> drawn(total, 0), cleared(nw, 0);
    for (bool any = true; any;) {
      any = false;
      const uint32_t g = rng() % nw;
      if (left[g]) {
        const uint64_t k = ctr[g]++, t = k * nw + g;
        if (t < total) drawn[t] = 1;
        else {
          --left[g];
          const uint64_t valid = (total + nw - 1 - g) / nw;
          if (k == valid + grid - 2) ctr[g] = 0, cleared[g] = 1;
        }
      }
      for (uint64_t l : left) any |= l != 0;
      wrong += chunk_taken(false, ctr[0], 0, nw) != (drawn[0] && !cleared[0]);  // cleared: its wave is at work
      for (uint64_t t = 1; t < total; ++t) wrong += drawn[t - 1] && !chunk_taken(false, ctr[0], t, nw);
      ++looked;
    }
    for (uint64_t c : ctr) wrong += c != 0;
    for (char d : drawn) wrong += !d;
  }
  say("looked", looked, looked > 10000);
  printf("wrong %llu\n", (unsigned long long)wrong);
  return 0;
}
