// CPU check of the blocks of consecutive cells (lbm_index.hpp, flat_start and
// flat_cell): every lane of every block of a box must get the cell its number
// names, lanes past the last cell z >= nz, and every offset of the cell must
// lie inside the window that starts at the block's first row and address what
// the same cell addresses from a window of its own row.
//
// Usage: flat_index_check nx ny nz qt value_bytes threads
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "../paper_1710_04751_amd/csrc/lbm_index.hpp"

using namespace lbm::idx;

int main(int argc, char** argv) {
    if (argc != 7) return 2;
    const int nx = std::atoi(argv[1]), ny = std::atoi(argv[2]), nz = std::atoi(argv[3]);
    const int qt = std::atoi(argv[4]), vb = std::atoi(argv[5]), threads = std::atoi(argv[6]);
    const int gs = rows_log2(nx, ny, nz, vb), rq = 15 + qt;
    const uint32_t mx = small_magic((uint32_t)nx), my = small_magic((uint32_t)ny);
    const int64_t ncell = (int64_t)nx * ny * nz;
    for (int64_t c0 = 0; c0 < ncell; c0 += threads) {
        const FlatStart f = flat_start((uint32_t)c0, nx, ny);
        const Window w = window_of((int)f.z0, (int)f.y0, nx, ny, nz, gs, rq, vb);
        for (int t = 0; t < threads; ++t) {
            const int64_t c = c0 + t;
            int x, y, z;
            flat_cell(f, (uint32_t)t, nx, ny, mx, my, &x, &y, &z);
            if (c >= ncell ? z < nz
                           : x != c % nx || y != (c / nx) % ny || z != c / ((int64_t)nx * ny)) {
                std::printf("FAIL cell %lld: (%d, %d, %d)\n", (long long)c, x, y, z);
                return 1;
            }
            if (c >= ncell) continue;
            const CellAt a = cell_at(w, x, y, z, nx, ny, nz);
            const Window wo = window_of(z, y, nx, ny, nz, gs, rq, vb);
            const CellAt b = cell_at(wo, x, y, z, nx, ny, nz);
            auto check = [&](uint32_t got, uint32_t own) {
                if ((int64_t)w.g0 * w.glen + got != (int64_t)wo.g0 * wo.glen + own ||
                    (uint64_t)got * vb + vb > (uint64_t)w.bytes) {
                    std::printf("FAIL offset of cell (%d, %d, %d)\n", x, y, z);
                    std::exit(1);
                }
            };
            for (int k = 0; k < 15; ++k) check(flow_load(w, a, k), flow_load(wo, b, k));
            for (int k = 0; k < qt; ++k) {
                if (qt == 7)
                    check(scalar_load<7, false>(w, a, k).off, scalar_load<7, false>(wo, b, k).off);
                else
                    check(scalar_load<15, true>(w, a, k).off, scalar_load<15, true>(wo, b, k).off);
            }
            for (int k = 0; k < rq; ++k) check(store_at(w, a, k), store_at(wo, b, k));
        }
    }
    std::printf("ok\n");
    return 0;
}
