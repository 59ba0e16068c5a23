// Host-side declarations shared by the C ABI (lbm_api.cpp) and the kernel
// launchers (lbm_kernels.hip).  Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

// Geometry of one cavity and the tiling of its step launch.
struct Geom {
    int32_t nx, ny, nz;
    int32_t bx, by;           // threads per block along x, y
    int32_t tiles_x, tiles_y; // blocks per row / per plane (0: blocks of bx * by
                              // consecutive cells)
    uint32_t mx, my;          // idx::small_magic of nx and ny
    uint32_t keep16;          // keep_sixteenths of the two states
    int32_t stream_loads;     // streams_loads of the rows
    int32_t gs;               // log2 of the rows per population run (PopLay)
};

// Lattice-unit coefficients, in double; launchers convert to the arithmetic
// type of the kernel.
struct Coefs {
    double omega, omega_bulk, omega_hi;  // flow
    double omega_T, omega_hiT, cs2;      // scalar
    double gbeta, T_ref, T_hot, T_cold;
    double src;                          // uniform scalar source R
    double alpha;                        // for the Nusselt number
    int32_t fourth_maxwell;
    int32_t sr;                          // FP16 storage: stochastic rounding
    uint32_t seed;                       // step index, the random stream's key
    int32_t spec;                        // scalar adiabatic faces: specular reflection
};

// Layout of one stored state (A or B), row groups interleaved.  The x-rows
// r = z*ny + y are taken in groups of R = 2^gs consecutive rows; a group is
// stored as rq = 15 + q runs of R*nx values, one run per population (flow
// 0..14, then scalar 0..q-1), each run holding its R rows one after another,
// x fastest.  Flow population a of cell (x, y, z) sits at
// F[((r >> gs)*rq + a)*R*nx + (r & (R-1))*nx + x]; G points 15 runs past F,
// so scalar population a sits at the same position from G.  The state is
// padded to a whole number of groups.
struct PopLay {
    int32_t nx;  // values per row
    int32_t rq;  // runs per group: 15 + q
    int32_t gs;  // log2 of the rows per group
};

// One stored state: base of the flow runs and of the scalar runs.
struct StateBuf {
    void* F;
    void* G;
};

enum class Prec : int32_t { FP64 = 0, FP32 = 1, FP32_S16 = 2 };

int value_bytes(Prec p);

// Whether blocks that stream also load past the caches: rows of whole 128-byte
// lines of values of 4 bytes or more, so that a wave shares at most the lines
// at its ends with its neighbours (512^3: FP32 3.75 against 3.81 ms a step
// with ordinary loads, FP64 2.5% better; but FP16 2.05 against 1.98 ms, and
// rows of odd length 301^3 0.92 against 0.89 ms, D3Q15 333^3 1.72 against 1.67).
inline bool streams_loads(int64_t nx, int vbytes) {
    return vbytes >= 4 && nx * vbytes % 128 == 0;
}

// Of 16 blocks of the step, how many leave their results in the 256 MB
// memory-side cache (Policy, lbm_step.hpp), for states of `bytes` in all (A
// and B): all of them while everything fits, else the share that holds about
// 170 MB, none once that is below 1/16 (2/16 in FP16, where the registers of
// the mix cost more than it saves: 256^3 D3Q15 with a source 407 us a step
// without, 416 with 1/16).
inline uint32_t keep_sixteenths(uint64_t bytes, int vbytes) {
    constexpr uint64_t MB = 1 << 20;
    if (bytes <= 240 * MB) return 16;
    const uint32_t share = (uint32_t)(16 * 170 * MB / bytes);
    return vbytes == 2 && share < 2 ? 0 : share;
}

hipError_t launch_step(Prec p, int qt, bool general, const Geom& g, StateBuf in,
                       StateBuf out, const Coefs& c, hipStream_t s);
// Three steps (keyed c.seed, + 1, + 2) in one launch, for boxes where
// steps_in_threes.
constexpr int kTripleTile = 4;
inline int64_t triple_tiles(int64_t n) { return (n + kTripleTile - 1) / kTripleTile; }

// Whether a box goes three steps a launch, on a device of `units` compute
// units: while every block of k_step3 runs at once, one a unit, or two where two
// fit and share a unit well.  FP64: one, for its 90-123 KB of LDS.  Two: D3Q7
// without stochastic rounding; with one of D3Q15 and stochastic rounding (which
// make the update longer than a launch's latency) while rows are whole tiles and
// short, so that the blocks' stores share few lines; else one.  Us a step, one
// a launch / three, 256 units (blocks in brackets):
//   FP64 24^3 (216) D3Q7 4.17 / 3.48, D3Q15 with a source 5.29 / 4.88, 28^3 (343)
//     D3Q7 4.36 / 5.75
//   FP32 D3Q7 32^3 (512) 4.23 / 3.50, with a source 30^3 (512) 4.30 / 4.07, 40^3
//     (1000) 4.53 / 5.52
//   FP32 D3Q15 32^3 4.95 / 4.77, 40x28x28 (490) 4.93 / 4.72, but 64x16x32 (512)
//     5.06 / 5.26, 30^3 4.90 / 5.29, 32^3 with a source 5.12 / 5.20
//   FP16 D3Q7 stochastic 32^3 3.99 / 3.76, 25^3 (343) 3.92 / 4.32; D3Q15 32^3 4.81
//     / 4.38, 25^3 4.73 / 4.91; D3Q15 stochastic 32^3 5.08 / 5.35, 24^3 (216) 5.00 /
//     3.72
// D3Q15 boxes whose rows end one or two cells into a tile go singly where the
// blocks are few or a row has 2, 4, 8, .. of them (so that every XCD, which takes
// each eighth block, always has the same part of the rows) and they are a tile
// thick in y or, in FP64 and FP16, the update is longer still (a source, specular
// faces, stochastic rounding): those lose, by time between the blocks' work that
// the counters do not attribute:
//   FP64 with a source 13^3 5.30 / 6.26, 13x24x24 5.28 / 5.59, 9^3 5.23 / 6.20, but
//     12x24x24 5.38 / 4.40, 15x20x24 5.26 / 4.50, 18^3 5.22 / 4.82
//   FP64 plain 17x4x40 5.10 / 5.57, 13^3 5.20 / 5.27; FP16 stochastic 13^3 5.37 / 5.69
inline bool steps_in_threes(Prec p, int qt, bool general, bool stochastic, bool specular,
                            const Geom& g, int units) {
    const int64_t row = triple_tiles(g.nx), blocks = row * triple_tiles(g.ny) * triple_tiles(g.nz);
    const int over = g.nx % kTripleTile;
    if (qt == 15 && (over == 1 || over == 2) && (blocks < 100 || (row & (row - 1)) == 0) &&
        (g.ny <= kTripleTile || (p != Prec::FP32 && (general || stochastic || specular))))
        return false;
    const bool q15 = qt == 15;
    bool two = false;
    if (p != Prec::FP64) {
        if (!q15 && !stochastic)
            two = true;
        else if (!(q15 && (stochastic || (general && p == Prec::FP32))))
            two = g.nx % kTripleTile == 0 && g.nx <= 48;
    }
    return blocks <= (two ? 2 : 1) * (int64_t)units;
}
hipError_t launch_step3(Prec p, int qt, bool general, const Geom& g, StateBuf in, StateBuf out,
                        const Coefs& c, hipStream_t s);
hipError_t launch_fill_zero(void* ptr, size_t bytes, hipStream_t s);
// Rest state: zero-fills state_bytes at state (both buffers), then, with a
// scalar source, writes the scalar equilibrium at T = -R/2 into st.
hipError_t launch_init_rest(Prec p, int qt, const Geom& g, PopLay pl, void* state,
                            size_t state_bytes, StateBuf st, const Coefs& c, hipStream_t s);
// stag: 4 doubles of device memory for the staggered sums; scratch: device
// memory of scratch_doubles >= 4 doubles for the blocks' partial sums
hipError_t launch_init_macros(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st,
                              const float* ux, const float* uy, const float* uz, const float* T,
                              double* stag, double* scratch, int64_t scratch_doubles,
                              const Coefs& c, hipStream_t s);
hipError_t launch_macros(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st, void* rho,
                         void* ux, void* uy, void* uz, void* T, bool fp64, const Coefs& c,
                         hipStream_t s);
hipError_t launch_nusselt(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st,
                          double* local_hot, double* local_cold, double* result,
                          const Coefs& c, hipStream_t s);
hipError_t launch_centerlines(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st,
                              double* u_line, double* w_line, const Coefs& c, double u0,
                              hipStream_t s);
hipError_t launch_symmetrize(const Geom& g, float* ux, float* uy, float* uz, float* T, double T0,
                             hipStream_t s);
hipError_t launch_residual(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st, void* snapshot,
                           bool compare, unsigned long long* max_bits, unsigned int* bad_flag,
                           hipStream_t s);
hipError_t launch_get_pops(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st, double* F,
                           double* G, hipStream_t s);
hipError_t launch_set_pops(Prec p, int qt, const Geom& g, PopLay pl, StateBuf st,
                           const double* F, const double* G, hipStream_t s);
hipError_t launch_gather_cells(Prec p, int qt, int64_t ncell, PopLay pl, StateBuf st,
                               const int64_t* cells, int64_t n, double* F, double* G,
                               hipStream_t s);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s);
const char* step_kernel_name(Prec p, int qt, bool general, bool threes, const Geom& g);

}  // namespace lbm
