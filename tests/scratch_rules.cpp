// Scratch of one distance transform: what admission to a server counts and what a
// launch lays out, for the sizes given as arguments "h w h w ...".  Host code only.
#include <cstdio>
#include <cstdlib>

#include "iwpp_runtime.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) {
    const int h = std::atoi(argv[i]), w = std::atoi(argv[i + 1]);
    // Addresses that are only compared with each other, 2^34 apart.
    const iwpp_job j{IWPP_OP_EDT, 8, h, w, reinterpret_cast<const uint8_t*>(1ull << 34), nullptr,
                     reinterpret_cast<void*>(2ull << 34), reinterpret_cast<int32_t*>(3ull << 34)};
    iwpp_ctx ctx;
    iwpp::rt::Plan plan;
    if (iwpp::rt::build_plan(&ctx, &j, 1, "scratch", plan) != IWPP_OK) return 1;
    std::printf("%d %d %zu %zu\n", h, w, iwpp::rt::job_scratch_bytes(IWPP_OP_EDT, h, w),
                iwpp::rt::align256(plan.scratch_bytes) + plan.table_bytes);
  }
  return 0;
}
