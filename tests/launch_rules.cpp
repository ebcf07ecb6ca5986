// Waves per workgroup for "wg_waves persistent_blocks tiles compute_units" given as
// arguments: reconstruction, distance transform.  Host code only.
#include <cstdio>
#include <cstdlib>

#include "iwpp_internal.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i + 3 < argc; i += 4) {
    const int waves = std::atoi(argv[i]), blocks = std::atoi(argv[i + 1]);
    std::printf("%u %u\n", iwpp::recon_waves(waves, blocks),
                iwpp::edt_waves(waves, blocks, std::strtoull(argv[i + 2], nullptr, 10), std::atoi(argv[i + 3])));
  }
  return 0;
}
