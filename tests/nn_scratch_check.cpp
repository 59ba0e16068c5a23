// CPU check of the weight gradient's scratch (nn_plan.hpp): what a network
// made for `batch` samples sets aside must hold the partial sums of every
// layer for every smaller call, whatever number of blocks the device runs at
// once.
//
// Usage: nn_scratch_check grid blocks_one blocks_two
#include <cstdio>
#include <cstdlib>

#include "../paper_1710_04751_amd/csrc/nn_plan.hpp"

using namespace lbmnn;

int main(int argc, char** argv) {
    if (argc != 4) return 2;
    const WgradBlocks resident = {std::atoll(argv[2]), std::atoll(argv[3])};
    int lg0 = 0;
    while ((1 << lg0) < std::atoi(argv[1])) ++lg0;
    auto geom = [&](int l, int n) {
        const LayerDef& d = kDefs[l];
        return make_geom(n, lg0 - d.level, d.taps, d.c1, d.c2, d.cout);
    };
    int rising = 0;
    for (int batch = 1; batch <= 64; ++batch) {
        int64_t given = 0;
        for (int l = 0; l < kLayers - 1; ++l)
            given = std::max(given, wgrad_scratch_floats(geom(l, batch), resident));
        for (int l = 0; l < kLayers - 1; ++l)
            for (int n = 1; n <= batch; ++n) {
                const WgradPlan p = wgrad_plan(geom(l, n), 0, resident);
                // the last bias partial and the last slice sum lie inside
                const int64_t slices = p.slices ? (p.rows + kRowSlice - 1) / kRowSlice : 0;
                const int64_t end = std::max(p.bias_off + p.rows * p.bwidth,
                                             p.part_floats + slices * (p.wwidth + p.bwidth));
                if (p.bias_off < p.rows * p.wwidth || end > p.scratch_floats ||
                    p.scratch_floats > given) {
                    std::printf("FAIL batch %d: %s with %d samples needs %lld floats of %lld\n", batch,
                                kDefs[l].name, n, (long long)p.scratch_floats, (long long)given);
                    return 1;
                }
                rising += p.scratch_floats > wgrad_plan(geom(l, batch), 0, resident).scratch_floats;
            }
    }
    std::printf("ok %d\n", rising);
    return 0;
}
