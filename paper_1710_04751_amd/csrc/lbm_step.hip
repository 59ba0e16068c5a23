// gfx950 kernels of the cascaded double-distribution lattice Boltzmann
// update (arXiv:1710.04751) and the observables around it.
//
// Step kernel: one thread per cell, one pass per time step (A -> B); boxes of
// few cells take three steps a pass (k_step3).
//   * pull streaming (eq. 2b, 13b): population a of cell x is read from
//     x - e_a in the previous post-collision state; each value is read once
//     and written once, so the kernel moves (15 + q) values in and out per
//     cell and is bound by HBM bandwidth;
//   * row groups interleaved: each group of consecutive x-rows holds one
//     run per population, x fastest, so a wave reads 64 consecutive cells
//     of one population, shifted by at most one element (coalesced), and
//     the streams of one block lie within a few runs of ~32 KB;
//   * walls (Sec. 3): a link whose source lies outside the box takes the
//     opposite population of the cell itself (half-way bounce-back for the
//     flow; anti-bounce-back -g + 2 w T_wall across the two Dirichlet walls,
//     which take precedence on edges; bounce-back across the adiabatic ones);
//   * T = sum g (eq. 25), F = g beta (T - T0) z (Boussinesq), then the flow
//     collision and the scalar collision with the same step's velocity, all
//     in registers, then the stores of the post-collision state, under the
//     block's cache policy (Policy);
//   * blocks are numbered so that each of the 8 XCDs works on a contiguous
//     range of tiles: neighbouring tiles of a row share the partly-read
//     cache lines of the x-shifted populations in the same L2.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include <algorithm>
#include <type_traits>

#include "lbm_dispatch.hpp"
#include "lbm_step.hpp"

namespace lbm {

namespace kern {

// Block number -> tile number, so that XCD k (hardware places block b on XCD
// b mod 8) receives the contiguous tile range [start_k, start_k + count_k).
__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t nb) {
    const uint32_t q = nb >> 3, r = nb & 7u, k = b & 7u;
    return k * q + (k < r ? k : r) + (b >> 3);
}

struct CellPos {
    int x, y, z, y0, z0;  // (z0, y0): first row of the block
    bool ok;
};

// The block's cells: bx * by consecutive ones (tiles_x = 0) or a bx x by tile
// of one plane.  set_geom chooses; see there.
__device__ __forceinline__ CellPos tile_cell(const Geom& g) {
    const uint32_t t = xcd_tile(blockIdx.x, gridDim.x);
    CellPos c;
    if (g.tiles_x == 0) {
        const idx::FlatStart f = idx::flat_start(t * (blockDim.x * blockDim.y), g.nx, g.ny);
        idx::flat_cell(f, threadIdx.y * blockDim.x + threadIdx.x, g.nx, g.ny, g.mx, g.my, &c.x,
                       &c.y, &c.z);
        c.y0 = (int)f.y0;
        c.z0 = (int)f.z0;
        c.ok = c.z < g.nz;
        return c;
    }
    const uint32_t per_z = (uint32_t)g.tiles_x * (uint32_t)g.tiles_y;
    const uint32_t tz = t / per_z;
    const uint32_t rem = t - tz * per_z;
    const uint32_t ty = rem / (uint32_t)g.tiles_x;
    const uint32_t tx = rem - ty * (uint32_t)g.tiles_x;
    c.x = (int)(tx * blockDim.x + threadIdx.x);
    c.y = (int)(ty * blockDim.y + threadIdx.y);
    c.z = c.z0 = (int)tz;
    c.y0 = (int)(ty * blockDim.y);
    c.ok = c.x < g.nx && c.y < g.ny;
    return c;
}

// Single cavity: one thread per cell, blocks of bx * by cells.  WAYS: the cache
// policies the blocks take (update_cell_policy, ways_of).
template <typename R, typename S, int QT, bool HG, int WAYS>
__global__ void __launch_bounds__(1024)
k_step(const S* __restrict__ in, S* __restrict__ out, Geom g, KCoef<R> k) {
    const CellPos p = tile_cell(g);
    if (!p.ok) return;
    update_cell_policy<R, S, QT, HG, WAYS>(blockIdx.x, g.keep16, g.stream_loads, in, out, p.x, p.y, p.z,
                                     p.y0, p.z0, g.nx, g.ny, g.nz, g.gs, k, k.seed);
}

// Three steps of a small box in one launch.  A block computes the first step
// of 8 x 8 x 8 cells from the state into LDS, the second of the 6 x 6 x 6
// inside them from LDS, the third of its own 4 x 4 x 4 from LDS into the other
// state: the same cell update, over a window of LDS whose rows are 8 cells.
// A small box leaves most of the chip idle and a launch is a chain of
// start, loads that miss, arithmetic and stores; the cells computed several
// times cost less than two more such chains.  Three steps change states once,
// as one does, so which state is current stays the parity of the steps.
// Bound by three updates' latency on one or two waves a SIMD.  Us a step, one
// step a launch -> three: 16^3 FP64 4.0 -> 2.8, FP32 3.75 -> 2.16, FP16 3.97 ->
// 2.22, FP32 D3Q15 4.7 -> 2.9; 32^3 FP32 4.2 -> 3.5.
constexpr int kTripleEdge = 8, kTripleCells = 512;

template <typename R, typename S, int QT, bool HG>
__global__ void __launch_bounds__(kTripleCells)
k_step3(const S* __restrict__ in, S* __restrict__ out, Geom g, KCoef<R> k) {
    __shared__ S lds[(15 + QT) * kTripleCells];
    const int t = threadIdx.x, lx = t & 7, ly = (t >> 3) & 7, lz = t >> 6;
    const int X0 = (int)blockIdx.x * kTripleTile - 2, Y0 = (int)blockIdx.y * kTripleTile - 2,
              Z0 = (int)blockIdx.z * kTripleTile - 2;
    const int x = X0 + lx, y = Y0 + ly, z = Z0 + lz;
    const bool inside = x >= 0 && x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz;
    const uint32_t cell = ((uint32_t)z * (uint32_t)g.ny + (uint32_t)y) * (uint32_t)g.nx + (uint32_t)x;
    // whether the cell is at least m cells inside the block's 8 x 8 x 8
    auto within = [&](int m) __attribute__((always_inline)) {
        return inside && lx >= m && lx < 8 - m && ly >= m && ly < 8 - m && lz >= m && lz < 8 - m;
    };
    // the states' window (as update_cell's: rows from the block's first on)
    // and that of LDS: own cell, walls where the box has them
    const idx::Window w = idx::window_of(Z0 < 0 ? 0 : Z0, Y0 < 0 ? 0 : Y0, g.nx, g.ny, g.nz, g.gs,
                                         15 + QT, (int)sizeof(S));
    const idx::CellAt c = idx::cell_at(w, x, y, z, g.nx, g.ny, g.nz);
    idx::Window wl = {};
    wl.nx = wl.ny = kTripleEdge;
    wl.gs = 6;
    wl.gmask = 63;
    wl.run = kTripleCells;
    idx::CellAt cl = c;
    cl.x = lx;
    cl.y = ly;
    cl.z = lz;
    cl.r = (uint32_t)(t >> 3);
    cl.own = (uint32_t)t;
    auto load = [&](uint32_t i) __attribute__((always_inline)) { return (R)lds[i]; };
    auto keep = [&](uint32_t i, R v) __attribute__((always_inline)) { lds[i] = (S)v; };
    R d[15], gq[QT];
    if (inside) {
        const __amdgpu_buffer_rsrc_t ri = pop_rsrc(in + (size_t)w.g0 * w.glen, w.bytes);
        gather_collide<R, QT, HG>(w, c, [&](uint32_t i) __attribute__((always_inline)) {
            return Buf<S>::template ld<R, kKeep>(ri, i); }, k, d, gq);
        put_cell<R, S, QT>(wl, cl, keep, k, k.seed, cell, d, gq);
    }
    __syncthreads();
    if (within(1)) gather_collide<R, QT, HG>(wl, cl, load, k, d, gq);
    __syncthreads();
    if (within(1)) put_cell<R, S, QT>(wl, cl, keep, k, k.seed + 1, cell, d, gq);
    __syncthreads();
    if (within(2)) {
        const __amdgpu_buffer_rsrc_t ro = pop_rsrc(out + (size_t)w.g0 * w.glen, w.bytes);
        gather_collide<R, QT, HG>(wl, cl, load, k, d, gq);
        put_cell<R, S, QT>(w, c, [&](uint32_t i, R v) __attribute__((always_inline)) {
            Buf<S>::template st<kKeep>(ro, i, v); }, k, k.seed + 2, cell, d, gq);
    }
}

template <typename R, typename S, int QT, bool HG>
hipError_t step3_impl(const Geom& g, StateBuf in, StateBuf out, const Coefs& c, hipStream_t s) {
    const KCoef<R> k = make_kcoef<R>(c, QT);
    const dim3 grid((unsigned)triple_tiles(g.nx), (unsigned)triple_tiles(g.ny),
                    (unsigned)triple_tiles(g.nz));
    hipLaunchKernelGGL((k_step3<R, S, QT, HG>), grid, dim3(kTripleCells), 0, s, (const S*)in.F, (S*)out.F, g, k);
    return hipGetLastError();
}

// The cache policies a box's blocks take: update_cell_policy's WAYS.
int ways_of(const Geom& g) {
    if (g.keep16 == 16) return 1 << kKeep;
    return (g.keep16 ? 1 << kKeep : 0) | (g.stream_loads ? 1 << kStreamLoads : 1 << kStream);
}

template <typename R, typename S, int QT, bool HG>
hipError_t step_impl(const Geom& g, StateBuf in, StateBuf out, const Coefs& c, hipStream_t s) {
    const KCoef<R> k = make_kcoef<R>(c, QT);
    const dim3 block(g.bx, g.by, 1);
    const int64_t ncell = (int64_t)g.nx * g.ny * g.nz, threads = (int64_t)g.bx * g.by;
    const dim3 grid((unsigned)(g.tiles_x ? (int64_t)g.tiles_x * g.tiles_y * g.nz
                                         : (ncell + threads - 1) / threads), 1, 1);
    auto launch = [&](auto ways) {
        hipLaunchKernelGGL((k_step<R, S, QT, HG, decltype(ways)::value>), grid, block, 0, s,
                           (const S*)in.F, (S*)out.F, g, k);
    };
    constexpr int keep = 1 << kKeep, plain = 1 << kStream, loads = 1 << kStreamLoads;
    switch (ways_of(g)) {
        case keep: launch(std::integral_constant<int, keep>{}); break;
        case plain: launch(std::integral_constant<int, plain>{}); break;
        case keep | plain: launch(std::integral_constant<int, keep | plain>{}); break;
        default:
            if constexpr (sizeof(S) > 2) {  // (streams_loads)
                if (g.keep16 == 0)
                    launch(std::integral_constant<int, loads>{});
                else
                    launch(std::integral_constant<int, keep | loads>{});
            }
    }
    return hipGetLastError();
}

}  // namespace kern
using namespace kern;

hipError_t launch_step(Prec p, int qt, bool general, const Geom& g, StateBuf in,
                       StateBuf out, const Coefs& c, hipStream_t s) {
    if (general) {
        LBM_DISPATCH_PQ(p, qt, return (step_impl<R, S, Q, true>(g, in, out, c, s)));
    } else {
        LBM_DISPATCH_PQ(p, qt, return (step_impl<R, S, Q, false>(g, in, out, c, s)));
    }
}

hipError_t launch_step3(Prec p, int qt, bool general, const Geom& g, StateBuf in, StateBuf out,
                        const Coefs& c, hipStream_t s) {
    if (general) {
        LBM_DISPATCH_PQ(p, qt, return (step3_impl<R, S, Q, true>(g, in, out, c, s)));
    } else {
        LBM_DISPATCH_PQ(p, qt, return (step3_impl<R, S, Q, false>(g, in, out, c, s)));
    }
}

const char* step_kernel_name(Prec p, int qt, bool general, bool threes, const Geom& g) {
    struct Names {
        char of[3][2][2][8][56];  // precision, lattice, collision; ways, 0: k_step3
        Names() {
            const char* types[3] = {"double, double", "float, float", "float, _Float16"};
            for (int t = 0; t < 3; ++t)
                for (int q = 0; q < 2; ++q)
                    for (int c = 0; c < 2; ++c)
                        for (int w = 0; w < 8; ++w) {
                            const char ways[] = {',', ' ', (char)('0' + w), 0};
                            snprintf(of[t][q][c][w], sizeof of[t][q][c][w], "lbm::kern::k_step%s<%s, %d, %s%s>",
                                     w ? "" : "3", types[t], q ? 15 : 7, c ? "true" : "false",
                                     w ? ways : "");
                        }
        }
    };
    static const Names names;
    return names.of[(int)p][qt == 15][general ? 1 : 0][threes ? 0 : ways_of(g)];
}

}  // namespace lbm
