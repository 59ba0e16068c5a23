// CPU check of the step's cache policy (lbm_internal.hpp, keep_sixteenths):
// prints the share of blocks that keep, for states of so many MB in all.
//
// Usage: cache_policy_check value_bytes MB...
#include <cstdio>
#include <cstdlib>

#include "../paper_1710_04751_amd/csrc/lbm_internal.hpp"

int main(int argc, char** argv) {
    for (int i = 2; i < argc; ++i)
        std::printf("%u\n", lbm::keep_sixteenths((uint64_t)std::atoll(argv[i]) << 20, std::atoi(argv[1])));
    return 0;
}
