// Index arithmetic of the weight gradient on bricks (k_wgrad_tr): which brick
// a number names, where each copied 16-byte item comes from and goes in LDS,
// how far ahead the copies run, and which LDS byte each lane reads.  Host and
// device functions, so the same code the kernel runs can be enumerated on the
// CPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbmnn {

constexpr int kWtHaloRow = 20;                 // voxels per LDS halo row (18 + 2 padding)
constexpr int kWtPlaneItems = 256;             // 16-byte items per plane slot: 6 rows, padding

// RS: 16-channel output groups of a block.
template <int RS>
struct WgShape {
    static constexpr int dy_row = RS == 1 ? 40 : 66;   // 16-byte items per output-gradient row (padded)
    static constexpr int dy_items = 16 * dy_row;       // 4 planes x 4 rows
    static constexpr int dy_buf = (dy_items + 63) / 64 * 64;
    static constexpr int dy_copies = dy_buf / 64;
    static constexpr int dy_it = (dy_copies + 1) / 2;  // per copying wave, at most
    static constexpr int dy_min = dy_copies / 2;       // and at least
    static constexpr int ahead = RS == 1 ? 4 : 3;      // bricks copied ahead
    static constexpr int ring = 6 + 4 * ahead;         // plane slots
    static constexpr int halo = ring * kWtPlaneItems;
    static constexpr int lds_items = halo + (ahead + 1) * dy_buf;
    static_assert(lds_items * 16 <= 160 * 1024, "one block's LDS");

    __host__ __device__ static int slot(int s) { return s >= ring ? s - ring : s; }  // s < 2 ring
    __host__ __device__ static int next_buf(int buf) { return buf == ahead ? 0 : buf + 1; }
};

// Offsets with bit 31 set lie past every buffer's end (samples are below 2^31
// bytes), so these items read zeros.
constexpr uint32_t kWgOutside = 0x80000000u;

__host__ __device__ inline uint32_t wg_negative(int v) { return (uint32_t)v >> 31; }

// Brick b (z fastest, then x, y, sample: powers of two) of 16 x 4 x 4 voxels.
struct WgBrick {
    int x0, y0, z0, smp;
};
__host__ __device__ inline WgBrick wg_brick(int b, int lg) {
    WgBrick o;
    o.z0 = (b & ((1 << (lg - 2)) - 1)) * 4;
    b >>= lg - 2;
    o.x0 = (b & ((1 << (lg - 4)) - 1)) * 16;
    b >>= lg - 4;
    o.y0 = (b & ((1 << (lg - 2)) - 1)) * 4;
    o.smp = b >> (lg - 2);
    return o;
}
// Whether brick b, of a range from b0 on, follows its z neighbour: then the two
// share the halo's first two planes.
__host__ __device__ inline bool wg_follows(int b, int b0, int lg) {
    return b > b0 && (b & ((1 << (lg - 2)) - 1)) != 0;
}

// Halo item t of a plane: slot t / 2 of 20 x 6, channel half t % 2.  from: its
// byte from the plane's first voxel in a tensor of `chans` channels on the
// layer's grid (lo) or, at its parent, on the grid of half the cells; side: the
// sides of the halo it lies on, 64 for padding and for channel halves past the
// input (half1: the second half exists), 128 in all (for a plane outside the grid).
struct WgHaloItem {
    uint32_t from, side;
};
__host__ __device__ inline WgHaloItem wg_halo_item(int t, bool lo, int lg, int chans, int cloc,
                                                   bool half1) {
    const int half = t & 1, hv = t >> 1, h = lg - 1;
    const int hx = hv % kWtHaloRow, hy = hv / kWtHaloRow;
    const bool never = hy >= 6 || hx >= 18 || (half && !half1);
    const int v = lo ? (hy << lg) + hx : ((hy + 1) >> 1 << h) + ((hx + 1) >> 1);
    WgHaloItem o;
    o.from = (uint32_t)(v * chans + cloc + half * 8) * 2u;
    o.side = (uint32_t)((hx == 0) | (hx == 17) << 1 | (hy == 0) << 2 | (hy == 5) << 3 | never << 6 | 128);
    return o;
}
// The sides of the grid the brick's halo reaches past (with the padding's), and
// those of its plane zz; the plane's first voxel's byte.
__host__ __device__ inline uint32_t wg_sides(const WgBrick& o, int lg) {
    const int G = 1 << lg;
    return wg_negative(o.x0 - 1) | wg_negative(G - 17 - o.x0) << 1 | wg_negative(o.y0 - 1) << 2 |
           wg_negative(G - 5 - o.y0) << 3 | 64u;
}
__host__ __device__ inline uint32_t wg_plane_sides(int zz, int lg) {
    return (wg_negative(zz) | wg_negative((1 << lg) - 1 - zz)) << 7;
}
__host__ __device__ inline uint32_t wg_plane_first(const WgBrick& o, int zz, bool lo, int lg, int chans) {
    const int hl = lo ? lg : lg - 1, sh = lo ? 0 : 1;
    const int row0 = (((o.y0 >> sh) - 1) << hl) + (o.x0 >> sh) - 1;
    return (uint32_t)(((zz >> sh) << (2 * hl)) + row0) * (uint32_t)chans * 2u;
}
__host__ __device__ inline uint32_t wg_halo_offset(const WgHaloItem& i, uint32_t sides, uint32_t first) {
    const uint32_t v = i.from + first;
    return i.side & sides ? kWgOutside : v;
}

// Output-gradient item t: row t / dy_row (4 plane + row), voxel and 8 channels
// of item t % dy_row, from output channel co0 on: its byte from the brick's
// first voxel (added to kWgOutside for padding and channels past ys).
template <int RS>
__host__ __device__ inline uint32_t wg_dy_item(int t, int lg, int ys, int co0) {
    using W = WgShape<RS>;
    const int row = t / W::dy_row, it = t - row * W::dy_row;
    const int px = it / (2 * RS), co = co0 + (it % (2 * RS)) * 8;
    const int v = ((row >> 2) << (2 * lg)) + ((row & 3) << lg) + px;
    const bool ok = t < W::dy_items && px < 16 && co < ys;
    return ok ? (uint32_t)(v * ys + co) * 2u : kWgOutside;
}
__host__ __device__ inline uint32_t wg_dy_first(const WgBrick& o, int lg, int ys) {
    return (uint32_t)((o.z0 << (2 * lg)) + (o.y0 << lg) + o.x0) * (uint32_t)ys * 2u;
}

// How far ahead the copies run: the next brick to copy, the ring position
// (counting up) and slot after the last plane copied, its output-gradient
// buffer, and the position of the current brick's first plane.
template <int RS>
struct WgAhead {
    int next, end = 0, wslot = 0, wbuf = 0, base = 0;
    __host__ __device__ explicit WgAhead(int b0) : next(b0) {}
    // Whether the next brick can be copied while brick b is the current one:
    // as far as the ring and the buffers go.  planes: its new ones.
    __host__ __device__ bool can(int b, int b1, int planes) const {
        return next < b1 && next - b <= WgShape<RS>::ahead && end + planes - base <= WgShape<RS>::ring;
    }
    __host__ __device__ void copied(int planes) {
        end += planes;
        wslot = WgShape<RS>::slot(wslot + planes);
        wbuf = WgShape<RS>::next_buf(wbuf);
        ++next;
    }
};

// The LDS bytes lane (r, q) = (lane % 16, lane / 16) of a product wave (plane,
// dy + 1) reads, of buffer 0 and slot 0: k value 8 q + 4 i + e of a step (i:
// which piece, e = r / 4) is the voxel (row 2 rp + q % 2, cell 8 (q / 2) + 4 i +
// e) of its plane; the lane reads channels 4 (r % 4) .. + 3 of it.
template <int RS>
__host__ __device__ inline uint32_t wg_lane_dy(int lane, int plane) {
    using W = WgShape<RS>;
    const int r = lane & 15, q = lane >> 4, e = r >> 2, ac = r & 3;
    return (uint32_t)(W::halo * 16 + ((q & 1) * W::dy_row + (8 * (q >> 1) + e) * 2 * RS) * 16 + ac * 8 +
                      plane * 4 * W::dy_row * 16);
}
template <int RS>
__host__ __device__ constexpr uint32_t wg_dy_read(int rp, int m, int piece) {  // added to it
    return (uint32_t)(2 * rp * WgShape<RS>::dy_row * 16 + m * 32 + piece * 4 * 32 * RS);
}
__host__ __device__ inline uint32_t wg_lane_halo(int lane, int dyw) {
    const int r = lane & 15, q = lane >> 4, e = r >> 2, ac = r & 3;
    return (uint32_t)((((q & 1) + dyw) * kWtHaloRow + 8 * (q >> 1) + e) * 32 + ac * 8);
}
__host__ __device__ constexpr uint32_t wg_halo_read(int rp, int piece) {  // added to it and the slot's
    return (uint32_t)((2 * rp * kWtHaloRow + 4 * piece) * 32);
}

}  // namespace lbmnn
