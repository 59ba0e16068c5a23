// Host arithmetic of the warm-start network's layers: their shapes and the
// launch plans of the weight gradient with the scratch these need.  No GPU
// code and no GPU calls, so every grid and batch can be enumerated on the CPU.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace lbmnn {

inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
inline int round_up(int a, int b) { return (a + b - 1) / b * b; }

// One convolution over n samples on a cubic grid of edge 2^lg.  The input
// is the channel concatenation of x1 (c1s stored channels on this grid, of
// which c1 are real; the rest hold zeros) and, when c2 > 0, x2 (c2 channels
// on the grid of edge 2^(lg-1), read through nearest-neighbour upsampling).
struct ConvGeom {
    int32_t n, lg;
    int32_t taps;       // 27 (3x3x3) or 1 (1x1x1)
    int32_t c1, c1s, c2;
    int32_t cin;        // c1s + c2: stored input channels, K per tap
    int32_t K, kpad;    // taps * cin, rounded up to 32
    int32_t cout;       // real output channels
    int32_t coutp;      // rows of the packed weight: cout rounded up to 16
    int32_t ys;         // stored channels of the output and its gradient: cout rounded up to 8
    int32_t kpad_t;     // columns of the transposed weight: taps * ys rounded up to 32
    int32_t cinp;       // rows of the transposed weight: cin rounded up to 16
};

inline ConvGeom make_geom(int n, int lg, int taps, int c1, int c2, int cout) {
    ConvGeom g;
    g.n = n;
    g.lg = lg;
    g.taps = taps;
    g.c1 = c1;
    g.c1s = round_up(c1, 8);
    g.c2 = c2;
    g.cin = g.c1s + c2;
    g.K = taps * g.cin;
    g.kpad = round_up(g.K, 32);
    g.cout = cout;
    g.coutp = round_up(cout, 16);
    g.ys = round_up(cout, 8);
    g.kpad_t = round_up(taps * g.ys, 32);
    g.cinp = round_up(g.cin, 16);
    return g;
}

// Layer table: input x1 (c1 channels on the layer's level), optional x2
// (c2 channels one level coarser, upsampled), output channels, kernel taps,
// level (0 = G, 1 = G/2, ...).
struct LayerDef {
    const char* name;
    int c1, c2, cout, taps, level, relu;
};
constexpr int kLayers = 16;
constexpr LayerDef kDefs[kLayers] = {
    {"enc1a", 4, 0, 16, 27, 0, 1},    {"enc1b", 16, 0, 16, 27, 0, 1},
    {"enc2a", 16, 0, 32, 27, 1, 1},   {"enc2b", 32, 0, 32, 27, 1, 1},
    {"enc3a", 32, 0, 64, 27, 2, 1},   {"enc3b", 64, 0, 64, 27, 2, 1},
    {"bota", 64, 0, 128, 27, 3, 1},   {"botb", 128, 0, 128, 27, 3, 1},
    {"botc", 128, 0, 128, 27, 3, 1},  {"dec3a", 64, 128, 64, 27, 2, 1},
    {"dec3b", 64, 0, 64, 27, 2, 1},   {"dec2a", 32, 64, 32, 27, 1, 1},
    {"dec2b", 32, 0, 32, 27, 1, 1},   {"dec1a", 16, 32, 16, 27, 0, 1},
    {"dec1b", 16, 0, 16, 27, 0, 1},   {"head", 16, 0, 4, 1, 0, 0},
};

// Rows a thread adds up in the first reduction pass (k_sum_row_slices).
constexpr int kRowSlice = 16;

// Blocks of the brick weight gradient that the device runs at once, for one
// and for two output groups of 16 channels a block.
struct WgradBlocks {
    int64_t one, two;
};

// Launch plan of the weight gradient: a brick kernel (grids of at least 16
// cells, 27 taps, 16/32 output channels with >= 8 input channels, 64 with
// >= 16) or the tiled kernel, its grid, and the floats of partial sums it
// writes.
struct WgradPlan {
    bool small;          // 8-cell grids: k_wgrad_small, one block per (group, sample, 32 channels)
    bool brick;
    int rs, cs;
    int chunks, groups;  // brick: channel groups x brick ranges
    int64_t per;         // brick: bricks per range
    int kt, ct, nz;      // tiled: column tiles, row tiles, voxel chunks
    int64_t vchunk;
    int64_t part_floats, bias_off;  // partial sums of every block
    int64_t rows, wwidth, bwidth;   // rows of partials, weight / bias floats per row
    int64_t scratch_floats;         // partials + the first reduction pass
    bool slices;                    // whether the first reduction pass runs
};

// Scratch of the first reduction pass, after the partials: the weight rows
// and the bias rows summed over slices of kRowSlice rows.
inline void finish_plan(WgradPlan* p) {
    p->slices = p->rows > 2 * kRowSlice;
    const int64_t sl = p->slices ? (p->rows + kRowSlice - 1) / kRowSlice : 0;
    p->scratch_floats = p->part_floats + sl * (p->wwidth + p->bwidth);
}

// Partial sums kept to about 32 MB and 1024 blocks: enough blocks to fill
// the chip, and a second pass that reads far less than the layer's inputs.
constexpr int64_t kPartFloats = 8 << 20;
constexpr int64_t kPartBlocks = 1024;

// (The brick kernel reads the output gradient unmasked: relu != 0 takes the
// tiled kernel.)
inline WgradPlan wgrad_plan(const ConvGeom& g, int relu, const WgradBlocks& resident) {
    WgradPlan p = {};
    const int64_t M = (int64_t)g.n << (3 * g.lg);
    // (8 input channels, the network's first layer, takes a channel group
    // of 16 whose upper half loads zeros; only k_wgrad_tr is checked for
    // that, so 64 output channels need 16.)
    p.small = !relu && g.lg == 3 && g.taps == 27 && g.c2 == 0 && g.cin % 16 == 0 &&
              g.coutp % 32 == 0;
    if (p.small) {
        p.rs = g.coutp / 16;
        p.chunks = g.cin / 16;
        p.groups = g.n;  // partial rows: one per sample
        const int64_t blk_floats = (int64_t)27 * g.coutp * 16;
        p.bias_off = (int64_t)g.n * p.chunks * blk_floats;
        p.part_floats = p.bias_off + (int64_t)g.n * g.coutp;
        p.rows = g.n;
        p.wwidth = (int64_t)p.chunks * blk_floats;
        p.bwidth = g.coutp;
        p.slices = false;
        p.scratch_floats = p.part_floats;
        return p;
    }
    p.brick = !relu && g.lg >= 4 && g.taps == 27 &&
              (g.c2 == 0 || g.c1s % 16 == 0) &&
              ((g.cin >= 8 && (g.coutp == 16 || g.coutp == 32)) || (g.cin >= 16 && g.coutp == 64));
    if (p.brick) {
        p.rs = g.coutp / 16;
        p.chunks = ceil_div(g.cin, 16);
        const int64_t nbricks = M / 256;  // 16 x 4 x 4 voxels
        const int64_t blk_floats = (int64_t)27 * g.coutp * 16;
        // one generation of resident blocks (64 output channels: two a range)
        const int64_t blocks = p.rs == 4 ? resident.two / 2 : p.rs == 2 ? resident.two : resident.one;
        const int64_t cap = std::max<int64_t>(
            1, std::min<int64_t>(blocks, kPartFloats / blk_floats) / p.chunks);
        const int64_t groups = std::max<int64_t>(1, std::min<int64_t>(nbricks, cap));
        p.per = (nbricks + groups - 1) / groups;
        p.groups = ceil_div(nbricks, p.per);
        p.bias_off = (int64_t)p.groups * p.chunks * blk_floats;
        p.part_floats = p.bias_off + (int64_t)p.groups * g.coutp;
        p.rows = p.groups;
        p.wwidth = (int64_t)p.chunks * blk_floats;
        p.bwidth = g.coutp;
        p.slices = false;  // one pass (k_brick_partials_sum)
        p.scratch_floats = p.part_floats;
        return p;
    }
    p.rs = g.coutp >= 64 ? 4 : g.coutp >= 32 ? 2 : 1;
    p.cs = 8 / p.rs;
    p.ct = ceil_div(g.coutp, 16 * p.rs);
    p.kt = ceil_div(g.K, 16 * p.cs);
    const int64_t steps = (M + 31) / 32;
    const int64_t blk_floats = (int64_t)p.rs * 16 * p.cs * 16;
    const int64_t tiles = (int64_t)p.kt * p.ct;
    const int64_t cap = std::max<int64_t>(
        1, std::min<int64_t>(2 * kPartBlocks, kPartFloats / blk_floats) / tiles);
    const int64_t chunks = std::max<int64_t>(1, std::min<int64_t>(steps, cap));
    p.vchunk = (steps + chunks - 1) / chunks * 32;
    p.nz = ceil_div(M, p.vchunk);
    p.bias_off = (int64_t)p.nz * tiles * blk_floats;
    p.part_floats = p.bias_off + (int64_t)p.nz * p.ct * p.rs * 16;
    p.rows = p.nz;
    p.wwidth = tiles * blk_floats;
    p.bwidth = (int64_t)p.ct * p.rs * 16;
    finish_plan(&p);
    return p;
}

// Scratch floats of conv_backward_weight for every call of up to g.n samples.
// A plan rounds its bricks or voxels a block up, so a smaller batch can have
// more blocks and need more than the full one: on an 8-cell grid dec1a needs
// 4.2 M floats for 11 samples and 2.3 M for 12.
inline int64_t wgrad_scratch_floats(const ConvGeom& g, const WgradBlocks& resident) {
    int64_t most = 0;
    for (ConvGeom s = g; s.n >= 1; --s.n)
        for (int relu = 0; relu < 2; ++relu)
            most = std::max(most, wgrad_plan(s, relu, resident).scratch_floats);
    return most;
}

}  // namespace lbmnn
