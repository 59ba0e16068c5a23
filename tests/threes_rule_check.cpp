// CPU check of which boxes go three steps a launch (lbm_internal.hpp).
//
// Usage: threes_rule_check units precision q general stochastic specular nx ny nz
#include <cstdio>
#include <cstdlib>

#include "../paper_1710_04751_amd/csrc/lbm_internal.hpp"

int main(int argc, char** argv) {
    if (argc != 10) return 2;
    int v[10];
    for (int i = 1; i < 10; ++i) v[i] = std::atoi(argv[i]);
    lbm::Geom g = {};
    g.nx = v[7], g.ny = v[8], g.nz = v[9];
    std::printf("%d\n", (int)lbm::steps_in_threes((lbm::Prec)v[2], v[3], v[4] != 0, v[5] != 0, v[6] != 0, g,
                                                 v[1]));
    return 0;
}
