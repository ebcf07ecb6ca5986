// A grid's workgroups meeting at the grid barrier, one memory operation at a time
// in an order drawn at random, with some of them held up for long stretches.
// Prints how many times a workgroup left a barrier with other list lengths than
// the grid had appended since the barrier before it, for the library's protocol
// and for one that keeps a single word per group.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "iwpp_barrier.hpp"

using namespace iwpp;

struct TwoWords {  // the library's
  static uint32_t slot(uint32_t gen) { return barrier::slot(gen); }
  static bool arrived(unsigned long long v, uint32_t gen) { return barrier::arrived(v, gen); }
};
struct OneWord {
  static uint32_t slot(uint32_t) { return 0u; }
  static bool arrived(unsigned long long v, uint32_t gen) { return (uint32_t)v != gen; }
};

constexpr uint32_t kBarriers = 12;

struct Wg {
  uint32_t gen = 0, phase = 0, appended = 0, lane = 0;
  uint32_t seen[8] = {}, held = 0;
  unsigned long long total = 0, v[8] = {};
};

template <class Protocol>
long run(uint32_t nwg, uint64_t seed) {
  std::mt19937_64 rng(seed);
  GridBarrier b{};
  const uint32_t groups = nwg < 8u ? nwg : 8u;
  // Every third barrier carries no lengths (the pairs around a full round).
  auto silent = [](uint32_t gen) { return gen % 3u == 2u; };
  std::vector<std::vector<uint32_t>> truth(kBarriers, std::vector<uint32_t>(8, 0u));
  std::vector<Wg> wg(nwg);
  long wrong = 0;
  uint32_t running = nwg;
  for (long steps = 0; running > 0; ++steps) {
    if (steps > 20000000) return -1;  // a workgroup waits for ever
    const uint32_t i = (uint32_t)(rng() % nwg), g = i & 7u, in_group = (nwg - g + 7u) >> 3;
    Wg& w = wg[i];
    if (w.gen == kBarriers) continue;
    if (w.held > 0) {
      --w.held;
      continue;
    }
    if (rng() % 64 == 0) w.held = (uint32_t)(rng() % 400);
    unsigned long long* words = b.word[Protocol::slot(w.gen)];
    switch (w.phase) {
      case 0:  // the round's work: a few workgroups append
        if (!silent(w.gen) && rng() % 3 == 0) {
          const uint32_t n = (uint32_t)(rng() % 5);
          w.appended += n;
          truth[w.gen][g] += n;
        }
        w.phase = rng() % 2 ? 1 : 0;
        break;
      case 1: {
        const unsigned long long one = barrier::arrival(silent(w.gen) ? 0u : w.appended);
        b.group[g][0] += one;
        w.total = b.group[g][0];
        if (!silent(w.gen)) w.appended = 0;
        w.phase = barrier::last(w.total, w.gen, in_group) ? 2 : 3;
        break;
      }
      case 2:
        words[g] = barrier::word(w.total, w.gen);
        w.phase = 3;
        break;
      case 3:  // a poll's loads return one by one, in any order
        {
          const uint32_t x = (w.lane * 5u + i) % 8u;
          w.v[x] = words[x];
        }
        if (++w.lane < 8) break;
        w.lane = 0;
        {
          bool all = true;
          for (uint32_t x = 0; x < groups; ++x) all = all && Protocol::arrived(w.v[x], w.gen);
          if (!all) break;
        }
        if (!silent(w.gen))
          for (uint32_t x = 0; x < groups; ++x) {
            const uint32_t n = barrier::items(w.v[x]) - w.seen[x];
            wrong += n != truth[w.gen][x];
            w.seen[x] = barrier::items(w.v[x]);
          }
        w.phase = 0;
        if (++w.gen == kBarriers) --running;
        break;
    }
  }
  return wrong;
}

template <class Protocol>
long sweep() {
  long wrong = 0;
  for (uint32_t nwg : {1u, 3u, 8u, 9u, 17u, 40u})
    for (uint64_t seed = 0; seed < 300; ++seed) {
      const long w = run<Protocol>(nwg, seed * 64 + nwg);
      if (w < 0) {
        std::printf("stuck: %u workgroups, seed %llu\n", nwg, (unsigned long long)seed);
        return -1;
      }
      wrong += w;
    }
  return wrong;
}

int main() {
  std::printf("library %ld\n", sweep<TwoWords>());
  std::printf("one_word %ld\n", sweep<OneWord>());
  return 0;
}
