// gfx950 kernels of the warm-start network: 3D convolutions as implicit
// GEMMs on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16, FP32
// accumulation), the 1 x 1 x 1 head with the loss on the vector units,
// pooling, upsampling and Adam.
//
// Matrix-core fragments (64 lanes, r = lane % 16, q = lane / 16):
//   A (16 x 32): lane holds row r, k = 8q .. 8q+7;
//   B (32 x 16): lane holds column r, k = 8q .. 8q+7;
//   D (16 x 16, FP32): lane holds rows 4q .. 4q+3 of column r.
// Forward: rows are output channels, columns 16 voxels, k runs over
// (tap, input channel) with the channels of one tap contiguous, so a lane's
// 8 k values are one 16-byte load of a channels-last voxel, and its 4 results
// are 4 consecutive channels of one voxel: one 8-byte store (and one 8-byte
// load of the ReLU mask).  With voxels as rows and channels as columns the
// products are the same but each lane stored four 2-byte values.  The input
// gradient is the same kernel run on the output gradient with the
// transposed, tap-flipped weight.  The weight gradient takes rows = output
// channels, columns = (tap, input channel) and k = voxels; each block sums
// a range of voxels and writes its partial sums, and a second kernel adds
// the partials of all ranges in a fixed order (no atomics, so gradients are
// bit-reproducible).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>

#include "lbm_units.hpp"
#include "nn_internal.hpp"
#include "nn_wgrad_index.hpp"

namespace lbmnn {

using lbm::compute_units;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void_ptr;  // LDS destination of direct loads

namespace {

// Per-sample scalars passed by value (at most kMaxBatch samples).
struct SampleFloats {
    float v[kMaxBatch];
};
struct SampleInts {
    int32_t v[kMaxBatch];
};

// One layer of the weight packing: destinations, the layer's offset in the
// master parameters and its geometry.
struct PackLayer {
    __bf16* wp;
    __bf16* wt;
    int64_t woff;
    int32_t coutp, kpad, cout, K, cin, c1, c1s, taps, cin_real, cinp, kpad_t, ys;
};
struct PackTable {
    PackLayer l[kMaxPackLayers];
    int64_t blk[2 * kMaxPackLayers];  // cumulative blocks of 256 over the segments
};

struct ConvArgs {
    const __bf16* x1;
    const __bf16* x2;
    const __bf16* w;
    const float* bias;
    __bf16* out;
    const __bf16* omask;  // outputs where omask <= 0 are written as 0
    int32_t n, lg, taps, c1s, c2, cin, K, kpad, cout, ys, relu;
    int32_t wrows;        // rows of the packed weight w (set by launch_conv)
    // The brick kernel's second result, on the grid of half the cells (null:
    // none).  With a bias: the averages of 2 x 2 x 2 results.  Without: the
    // sums over 2 x 2 x 2 of the channels from `split` on (a multiple of 16),
    // 0 where lowmask is not positive; out then has the first `split` only.
    __bf16* low = nullptr;
    const __bf16* lowmask = nullptr;
    int32_t split = 0;
};

// The convolutions' results: lane (r, q) has channels co .. co + 3 (co a
// multiple of 4) of one voxel, acc + bias, ReLU, 0 where the mask is not
// positive and for padding channels co >= cout; nothing for co >= ys.
// bias_quad: the lane's four biases, loaded ahead.
__device__ __forceinline__ floatx4 bias_quad(const ConvArgs& a, int co) {
    floatx4 b = {0.f, 0.f, 0.f, 0.f};
    if (a.bias) {
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = co + i < a.cout ? a.bias[co + i] : 0.f;
    }
    return b;
}

__device__ __forceinline__ void store_quad(const ConvArgs& a, int64_t vo, int co, floatx4 acc,
                                           floatx4 bias, bf16x4 mask) {
    if (co >= a.ys) return;
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float val = acc[i] + bias[i];
        if (a.relu) val = fmaxf(val, 0.f);
        if (co + i >= a.cout || (a.omask && !((float)mask[i] > 0.f))) val = 0.f;
        o[i] = (__bf16)val;
    }
    *(bf16x4*)(a.out + vo * a.ys + co) = o;
}

__device__ __forceinline__ bf16x4 mask_quad(const ConvArgs& a, int64_t vo, int co) {
    return a.omask && co < a.ys ? *(const bf16x4*)(a.omask + vo * a.ys + co) : bf16x4{};
}

// One block: 16 voxels x (NSUB * 16) output channels, channel group
// blockIdx.y.  The KS waves of a block split the k range (wave w takes every
// KS-th step of 32 from step w) and add their partial sums through LDS; this
// keeps enough waves in flight on the coarse grids.
//
// Each wave is one chain of loads (one voxel and NSUB weight fragments a step,
// from the memory-side cache: about 0.6 us), so kDepth steps' fragments are in
// flight in as many register sets.  With two sets and four output groups a
// wave the 4-cell layers of 128 channels took 17-19 us a launch, the
// concatenated layer on 8 cells 26 (each step waited for its loads).
// WIDE: the input channels are a multiple of 32 and the tensors are below 2 GB,
// so a step lies in one tap and its addresses are a lane register plus scalars
// (range-checked buffer loads; a tap outside the grid reads past the end, as
// zeros).
constexpr int conv_depth(int nsub) { return nsub == 1 ? 8 : nsub == 2 ? 6 : 3; }

template <int NSUB, int KS, bool WIDE>
__global__ void __launch_bounds__(64 * KS) k_conv(ConvArgs a) {
    constexpr int kDepth = conv_depth(NSUB);
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lg = a.lg, G = 1 << lg;
    const int64_t V = (int64_t)1 << (3 * lg);
    const int64_t M = (int64_t)a.n * V;
    const int64_t vo = (int64_t)blockIdx.x * 16 + r;  // the lane's voxel
    const int cobase = blockIdx.y * NSUB * 16;
    const bool vok = vo < M;
    const int64_t vc = vok ? vo : 0;
    const int vs = (int)(vc >> (3 * lg));
    const int rem = (int)(vc & (V - 1));
    const int vz = rem >> (2 * lg), vy = (rem >> lg) & (G - 1), vx = rem & (G - 1);
    floatx4 acc[NSUB];
#pragma unroll
    for (int j = 0; j < NSUB; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Wave w takes the k steps w, w + KS, ...: nst of them; at step s the
    // lane's 8 k values start at kw + 32 KS s.  The fragments of a step are
    // the voxels (8 channels of one tap per lane) and NSUB weight tiles.  The
    // loop body has no branches (a lane outside the grid loads voxel 0 and
    // takes zeros; a step past the last takes zero voxels and zero weights, so
    // its products add 0 whatever the weights are), so the compiler keeps the
    // loads ahead of the products and the waits cover only the step in use.
    const int kw = q * 8 + 32 * wave;
    const int nst = 32 * wave < a.kpad ? (a.kpad / 32 - 1 - wave) / KS + 1 : 0;  // (kpad: whole steps)
    const float icin = 1.f / (float)a.cin;
    const int h = lg - 1;
    auto load_any = [&](int st, bf16x8& av, bf16x8* bv) __attribute__((always_inline)) {
        const bool live = st < nst;
        const int k = kw + (live ? st : nst - 1) * (32 * KS);
        // tap = k / cin (exact: k < 2^13, so (k + 0.5) / cin is far from an integer)
        const int tap = (int)(((float)k + 0.5f) * icin), c = k - tap * a.cin;
        const bool t27 = a.taps == 27;
        const int dz = t27 ? tap / 9 - 1 : 0, dy = t27 ? (tap / 3) % 3 - 1 : 0,
                  dx = t27 ? tap % 3 - 1 : 0;
        const bool lo = c < a.c1s;
        const __bf16* base = lo ? a.x1 : a.x2;
        const int zz = vz + dz, yy = vy + dy, xx = vx + dx;
        const bool ok = live && vok && k < a.K && (unsigned)zz < (unsigned)G &&
                        (unsigned)yy < (unsigned)G && (unsigned)xx < (unsigned)G;
        const int zc = ok ? zz : 0, yc = ok ? yy : 0, xc = ok ? xx : 0;
        const int64_t off =
            lo ? (((int64_t)vs << (3 * lg)) + (zc << (2 * lg)) + (yc << lg) + xc) * a.c1s + c
               : (((int64_t)vs << (3 * h)) + ((zc >> 1) << (2 * h)) + ((yc >> 1) << h) + (xc >> 1)) *
                         a.c2 + (c - a.c1s);
        const bf16x8 v = *(const bf16x8*)(base + off);
#pragma unroll
        for (int i = 0; i < 8; ++i) av[i] = ok ? v[i] : (__bf16)0.f;
#pragma unroll
        for (int j = 0; j < NSUB; ++j)
            bv[j] = live ? *(const bf16x8*)(a.w + (int64_t)(cobase + j * 16 + r) * a.kpad + k) : bf16x8{};
    };
    // bit t: tap t of this voxel lies in the grid
    uint32_t inside = 0;
    const __bf16 *x1 = a.x1, *x2 = a.c2 ? a.x2 : a.x1;
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(x1), (short)0, (int)(uint32_t)(M * a.c1s * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(x2), (short)0, (int)(uint32_t)((M >> 3) * a.c2 * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(a.w), (short)0, (int)(uint32_t)((cobase + NSUB * 16) * a.kpad * 2),
        0x00020000);
    const uint32_t wbase = (uint32_t)((cobase + r) * a.kpad + q * 8) * 2u;
    const uint32_t vbase = (uint32_t)(vc * a.c1s + q * 8) * 2u;
    if constexpr (WIDE) {
        if (a.taps == 27) {
            for (int t = 0; t < 27; ++t) {
                const int zz = vz + t / 9 - 1, yy = vy + (t / 3) % 3 - 1, xx = vx + t % 3 - 1;
                const bool ok = vok && (unsigned)zz < (unsigned)G && (unsigned)yy < (unsigned)G &&
                                (unsigned)xx < (unsigned)G;
                inside |= (uint32_t)ok << t;
            }
        } else {
            inside = vok;
        }
    }
    const int nall = a.kpad / 32;  // (WIDE: K = kpad)
    auto load_wide = [&](int st, bf16x8& av, bf16x8* bv) __attribute__((always_inline)) {
        const bool live = st < nst;
        const int k = 32 * (live ? wave + KS * st : nall - 1);
        const int tap = (int)(((float)k + 0.5f) * icin), c = k - tap * a.cin;
        const bool t27 = a.taps == 27;
        const int dz = t27 ? tap / 9 - 1 : 0, dy = t27 ? (tap / 3) % 3 - 1 : 0,
                  dx = t27 ? tap % 3 - 1 : 0;
        const bool ok = live && (inside >> tap & 1u);
        typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
        uintx4 v;
        if (c < a.c1s) {
            const uint32_t off = vbase + (uint32_t)(((dz << (2 * lg)) + (dy << lg) + dx) * a.c1s + c) * 2u;
            const uint32_t o = ok ? off : 0x80000000u;
            v = __builtin_amdgcn_raw_buffer_load_b128(r1, o, 0, 0);
        } else {
            const uint32_t par = ((uint32_t)vs << (3 * h)) + ((uint32_t)(vz + dz) >> 1 << (2 * h)) +
                                 ((uint32_t)(vy + dy) >> 1 << h) + ((uint32_t)(vx + dx) >> 1);
            const uint32_t off = (par * (uint32_t)a.c2 + (uint32_t)(c - a.c1s + q * 8)) * 2u;
            const uint32_t o = ok ? off : 0x80000000u;
            v = __builtin_amdgcn_raw_buffer_load_b128(r2, o, 0, 0);
        }
        av = __builtin_bit_cast(bf16x8, v);
#pragma unroll
        for (int j = 0; j < NSUB; ++j) {
            const uint32_t o = wbase + (live ? (uint32_t)(j * 16 * a.kpad + k) * 2u : 0x80000000u);
            bv[j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, o, 0, 0));
        }
    };
    auto load_step = [&](int st, bf16x8& av, bf16x8* bv) __attribute__((always_inline)) {
        if constexpr (WIDE)
            load_wide(st, av, bv);
        else
            load_any(st, av, bv);
    };
    if (nst > 0) {
        bf16x8 av[kDepth], bv[kDepth][NSUB];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) load_step(d, av[d], bv[d]);
        for (int st = 0; st < nst; st += kDepth) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
#pragma unroll
                for (int j = 0; j < NSUB; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv[d][j], av[d], acc[j], 0, 0, 0);
                load_step(st + d + kDepth, av[d], bv[d]);
            }
        }
    }
    if constexpr (KS > 1) {
        __shared__ floatx4 part[KS - 1][NSUB][64];
        if (wave > 0) {
#pragma unroll
            for (int j = 0; j < NSUB; ++j) part[wave - 1][j][lane] = acc[j];
        }
        __syncthreads();
        if (wave > 0) return;
#pragma unroll
        for (int w = 0; w < KS - 1; ++w)
#pragma unroll
            for (int j = 0; j < NSUB; ++j) acc[j] += part[w][j][lane];
    }
    // D rows 4q .. 4q+3 are output channels, column r the voxel
    if (!vok) return;
#pragma unroll
    for (int j = 0; j < NSUB; ++j) {
        const int co = cobase + j * 16 + q * 4;
        store_quad(a, vo, co, acc[j], bias_quad(a, co), mask_quad(a, vo, co));
    }
}

struct WgradArgs {
    const __bf16* x1;
    const __bf16* x2;
    const __bf16* dy;
    const __bf16* y;
    float* part;    // partial sums: weights of every block, then the bias partials
    int64_t bias_off;  // floats from part to the bias partials
    int32_t n, lg, taps, c1, c1s, c2, cin, K, cout, coutp, ys, relu, cin_real;
    int64_t vchunk;
};

// LDS layouts follow what the part's LDS serves without bank conflicts
// (measured with a probe over 768 layouts): for 16-byte reads where lane
// (r, q) = (lane % 16, lane / 16) reads byte r S + (q & 1) H + (q >> 1) T, T
// never matters; S = 16 is conflict-free for any H; S = 32 (mod 64) for H = 16
// or 48; S = 16 or 48 (mod 64) only for H a multiple of 256 (or S = H = 48);
// S = 0 (mod 64) never.  The fragments here have H = 16 (the lane's second 8
// channels or k values), so row strides are 32 (mod 64) bytes.
constexpr int kTileRow = 48;   // 32-voxel tile rows, in elements (96 bytes)

// B fragment of ones: an A fragment times it gives its row sums in every
// column (the bias gradient's sum over voxels, on the matrix cores).
__device__ __forceinline__ bf16x8 ones_frag() {
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)1.f;
    return o;
}

// Weight gradient, one block of 4 waves per (row tile, column tile, voxel
// chunk): rows are RS * 16 output channels, columns CS * 16 (tap, channel)
// pairs with RS * CS = 8, so each wave owns two 16 x 16 accumulators.  Per
// 32 voxels the block loads the masked output gradient and the input patch
// with 16-byte loads (8 channels of one voxel) and writes them transposed
// into LDS ([channel][voxel]), where each fragment (8 consecutive voxels) is
// one 16-byte read.  Blocks of the first column tile also sum the output
// gradient into the bias gradient (one more matrix-core product, against
// ones).  Every block writes its partial sums to part (block b = (z * ct +
// y) * kt + x: RS * 16 rows x CS * 16 columns; bias partials [z * ct + y][RS
// * 16] at bias_off); k_wgrad_reduce adds them up.
template <int RS>
__global__ void __launch_bounds__(256) k_wgrad(WgradArgs a) {
    constexpr int CS = 8 / RS;
    __shared__ __attribute__((aligned(16))) __bf16 dT[RS * 16][kTileRow];
    __shared__ __attribute__((aligned(16))) __bf16 xT[CS * 16][kTileRow];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int lg = a.lg, G = 1 << lg;
    const int64_t V = (int64_t)1 << (3 * lg);
    const int64_t M = (int64_t)a.n * V;
    const int row0 = blockIdx.y * RS * 16, col0 = blockIdx.x * CS * 16;
    const int wr = wave % RS, wc = 2 * (wave / RS);
    floatx4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    floatx4 accb = {0.f, 0.f, 0.f, 0.f};
    const bool bias_wave = blockIdx.x == 0 && wave < RS;  // wc == 0
    const int64_t v0 = (int64_t)blockIdx.z * a.vchunk;
    const int64_t v1 = std::min(M, v0 + a.vchunk);
    for (int64_t vb = v0; vb < v1; vb += 32) {
        // output gradient: RS*2 groups of 8 channels x 32 voxels
        for (int t = tid; t < RS * 2 * 32; t += 256) {
            const int g8 = t >> 5, vi = t & 31;
            const int c0 = row0 + g8 * 8;
            const int64_t vv = vb + vi;
            bf16x8 d;
#pragma unroll
            for (int i = 0; i < 8; ++i) d[i] = (__bf16)0.f;
            if (vv < v1 && c0 < a.ys) {
                d = *(const bf16x8*)(a.dy + vv * a.ys + c0);
                if (a.relu) {
                    const bf16x8 m = *(const bf16x8*)(a.y + vv * a.ys + c0);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (!((float)m[i] > 0.f)) d[i] = (__bf16)0.f;
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) dT[g8 * 8 + i][vi] = d[i];
        }
        // input patches: CS*2 groups of 8 (tap, channel) columns x 32 voxels
        for (int t = tid; t < CS * 2 * 32; t += 256) {
            const int g8 = t >> 5, vi = t & 31;
            const int k0 = col0 + g8 * 8;
            const int64_t vv = vb + vi;
            bf16x8 xv;
#pragma unroll
            for (int i = 0; i < 8; ++i) xv[i] = (__bf16)0.f;
            if (vv < v1 && k0 < a.K) {
                const int tap = k0 / a.cin, c = k0 - tap * a.cin;
                const int s = (int)(vv >> (3 * lg));
                const int rem = (int)(vv & (V - 1));
                int z = rem >> (2 * lg), y = (rem >> lg) & (G - 1), x = rem & (G - 1);
                if (a.taps == 27) {
                    z += tap / 9 - 1;
                    y += (tap / 3) % 3 - 1;
                    x += tap % 3 - 1;
                }
                if ((unsigned)z < (unsigned)G && (unsigned)y < (unsigned)G &&
                    (unsigned)x < (unsigned)G) {
                    if (c < a.c1s) {
                        const int64_t vi2 = ((int64_t)s << (3 * lg)) + ((int64_t)z << (2 * lg)) +
                                            ((int64_t)y << lg) + x;
                        xv = *(const bf16x8*)(a.x1 + vi2 * a.c1s + c);
                    } else {
                        const int h = lg - 1;
                        const int64_t vi2 = ((int64_t)s << (3 * h)) +
                                            ((int64_t)(z >> 1) << (2 * h)) +
                                            ((int64_t)(y >> 1) << h) + (x >> 1);
                        xv = *(const bf16x8*)(a.x2 + vi2 * a.c2 + (c - a.c1s));
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) xT[g8 * 8 + i][vi] = xv[i];
        }
        __syncthreads();
        const bf16x8 av = *(const bf16x8*)&dT[wr * 16 + r][q * 8];
        const bf16x8 b0 = *(const bf16x8*)&xT[wc * 16 + r][q * 8];
        const bf16x8 b1 = *(const bf16x8*)&xT[(wc + 1) * 16 + r][q * 8];
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b0, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b1, acc1, 0, 0, 0);
        if (bias_wave) accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, ones_frag(), accb, 0, 0, 0);
        __syncthreads();
    }
    const int64_t blk = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
    float* pb = a.part + blk * (RS * 16) * (CS * 16);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const floatx4 acc = j ? acc1 : acc0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            pb[(wr * 16 + q * 4 + i) * (CS * 16) + (wc + j) * 16 + r] = acc[i];
    }
    if (bias_wave && r == 0) {
        float* bb = a.part + a.bias_off + ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * (RS * 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) bb[wr * 16 + q * 4 + i] = accb[i];
    }
}

// First pass of the partial-sum reduction: for the weight partials (rows x
// ww floats at in) and then the bias partials (rows x bw floats at in +
// boff), out[j][w] = sum of in[g][w] over the rows g of slice j (kRowSlice
// consecutive rows, fewer in the last), in order.  One thread per (slice,
// column), so the loads of many rows are in flight at once; the weight
// slices go to out, the bias slices after them.
__global__ void k_sum_row_slices(const float* __restrict__ in, int64_t boff, int64_t rows,
                                 int64_t ww, int64_t bw, float* __restrict__ out) {
    const int64_t slices = (rows + kRowSlice - 1) / kRowSlice;
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t width = ww;
    if (i >= slices * ww) {
        i -= slices * ww;
        if (i >= slices * bw) return;
        in += boff;
        out += slices * ww;
        width = bw;
    }
    const int64_t j = i / width, w = i - j * width;
    const int64_t g0 = j * kRowSlice;
    const int n = (int)(rows - g0 < kRowSlice ? rows - g0 : kRowSlice);
    float v[kRowSlice];
#pragma unroll
    for (int k = 0; k < kRowSlice; ++k) v[k] = k < n ? in[(g0 + k) * width + w] : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < kRowSlice; ++k) sum += v[k];
    out[i] = sum;
}

// Sum over the rows of a partial-sum table by L consecutive lanes per
// gradient entry (L = 8 for tables of many rows, 1 for few): lane j adds rows
// j, j + L, ... in order, then a fixed xor butterfly adds the L lane sums
// (lane 0's result is written), so the order of every addition is fixed and,
// for many rows, many loads are in flight.
template <int L>
__device__ __forceinline__ float lane_group_sum(float v) {
    if constexpr (L >= 2) v += __shfl_xor(v, 1, L);
    if constexpr (L >= 4) v += __shfl_xor(v, 2, L);
    if constexpr (L >= 8) v += __shfl_xor(v, 4, L);
    return v;
}
constexpr int kRedManyRows = 32;  // rows from which a table takes 8 lanes per entry

// Sum of the k_wgrad partials over the voxel chunks, into the master layout
// dw[co][tap][ci] (zero padding channels dropped) and db.  One group of L
// lanes per (row, column) of the gradient matrix or per bias entry.
template <int L>
__global__ void k_wgrad_reduce(WgradArgs a, int kt, int ct, int nz, int rs, int cs, float* dw,
                               float* db) {
    // 32-bit index arithmetic: the host launches fewer than 2^31 lanes
    const uint32_t rows = (uint32_t)(ct * rs * 16), cols = (uint32_t)(kt * cs * 16);
    const uint32_t i = (blockIdx.x * blockDim.x + threadIdx.x) / L;
    const int j = threadIdx.x % L;
    if (i < rows * cols) {
        const uint32_t row = i / cols, col = i - row * cols;
        const uint32_t cty = row / (uint32_t)(rs * 16), rl = row - cty * (uint32_t)(rs * 16);
        const uint32_t ktx = col / (uint32_t)(cs * 16), cl = col - ktx * (uint32_t)(cs * 16);
        if (row >= (uint32_t)a.cout || col >= (uint32_t)a.K) return;
        const uint32_t t = col / (uint32_t)a.cin, cc = col - t * (uint32_t)a.cin;
        if (cc < (uint32_t)a.c1s && cc >= (uint32_t)a.c1) return;  // zero padding channels of x1
        const uint32_t ci = cc < (uint32_t)a.c1s ? cc : a.c1 + (cc - a.c1s);
        const int64_t per = (int64_t)rs * 16 * cs * 16;
        float sum = 0.f;
#pragma unroll 4
        for (int z = j; z < nz; z += L)
            sum += a.part[(((int64_t)z * ct + cty) * kt + ktx) * per + rl * (cs * 16) + cl];
        sum = lane_group_sum<L>(sum);
        if (j == 0) dw[((int64_t)row * a.taps + t) * a.cin_real + ci] = sum;
    } else if (i < rows * cols + (uint32_t)a.cout) {
        const uint32_t co = i - rows * cols;
        const uint32_t cty = co / (uint32_t)(rs * 16), rl = co - cty * (uint32_t)(rs * 16);
        float sum = 0.f;
        for (int z = j; z < nz; z += L)
            sum += a.part[a.bias_off + ((int64_t)z * ct + cty) * (rs * 16) + rl];
        sum = lane_group_sum<L>(sum);
        if (j == 0) db[co] = sum;
    }
}

// Direct-to-LDS copy of 16 bytes per lane, from byte off of the buffer (zeros
// past its end) to LDS byte `lds` (the wave's, in a scalar) plus 16 times the
// lane.  Written as an instruction because the compiler, which cannot tell the
// two halo buffers apart across the loop, would wait for the copies of the
// next step before every LDS read of this one; it has no register result.
// The waits are the caller's: copies_landed.
typedef int intx4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ intx4 buffer_words(const void* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    intx4 words = {__builtin_amdgcn_readfirstlane((int)(uint32_t)p),
                   __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32) & 0xFFFF),
                   __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
    // the five wait states a buffer instruction needs after a vector
    // instruction wrote its descriptor, which the compiler does not count
    // for an instruction in inline assembly
    __asm__ volatile("s_nop 4" : "+s"(words));
    return words;
}
__device__ __forceinline__ void copy_to_lds(intx4 rsrc, uint32_t lds, uint32_t off) {
    __asm__ volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :
                     : "s"(lds), "v"(off), "s"(rsrc)
                     : "memory", "m0");
}
// Waits until at most `later` of this wave's vector-memory operations are
// outstanding (they finish in order) and its LDS reads are done, then for the
// block's other waves.
template <int later>
__device__ __forceinline__ void copies_outstanding() {
    static_assert(later < 64, "the counter's range");
    __asm__ volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(later) : "memory");
}
__device__ __forceinline__ void block_barrier() { __asm__ volatile("s_barrier" : : : "memory"); }
template <int later>
__device__ __forceinline__ void copies_landed() {
    copies_outstanding<later>();
    block_barrier();
}

// Weight gradient on 16 x 4 x 4 bricks through transposing LDS reads, for
// grids of at least 16 cells and unmasked output gradients.  dW[tap][co][ci]
// sums dY[v][co] X[v + tap][ci] over voxels v, so both matrix-core operands
// need 8 consecutive voxels of one channel per lane, while the tensors are
// stored channels-last.  The block copies the brick's output gradient and the
// 18 x 6 x 6 input halo of one 16-channel group into LDS as they are stored
// (direct-to-LDS loads, 32 bytes per voxel and 16 channels), and
// ds_read_b64_tr_b16 transposes on the way out: within each 16 lanes, lane
// 4a + b receives element b of the 8-byte pieces addressed by lanes a, a + 4,
// a + 8, a + 12.  So when lane L of a group addresses voxel k0 + L / 4,
// channels 4 (L % 4) .. + 3, lane n gets voxels k0 .. k0 + 3 of channel n: two
// such reads give an operand fragment.
//
// Twelve waves make the products: wave w the taps with dy = w % 3 - 1 (nine of
// them) on plane w / 3 of the brick.  A wave reads its plane's output gradient
// once, and each row of its three halo planes once, as three 4-voxel pieces
// from which the fragments of dx = -1, 0, +1 are shifted together in registers:
// 22 reads for 18 products (26 for 36 with 32 output channels); one wave per
// (dz, dy) with a read per fragment took 64 for 24.
//
// Four more waves make the copies (two the halo, two the output gradient): the
// scalar work of their addresses, done by every wave, had cost more issue slots
// than the products (174 scalar instructions a wave and brick beside 18
// products: 51 us for a 16-channel layer at 64^3).  They have the higher wave
// priority (16 channels at 64^3 45 -> 40 us, 48 -> 16 122 -> 106).
//
// Lane groups q and q ^ 1 of a k step take neighbouring rows, and the LDS rows
// are padded so that their reads fall in opposite halves of the banks (a row of
// the halo or of a one-group output gradient holds 20 voxels, 640 bytes; of a
// two-group output gradient 1056 bytes).  A block (one per compute unit) walks
// a range of bricks in z order within each (x, y) column.  The halo planes sit
// in a ring of slots: a brick after its z neighbour keeps the two planes they
// share and copies its 4 new ones.  The copies of up to `ahead` bricks are in
// flight (26 KB a brick against about 0.4 us of products).  blockIdx.z: 32 of
// the output channels.
//
// Measured, 8 samples, before (nine waves, one brick copied ahead by all of
// them, four blocks a compute unit) -> now: 16 -> 16 channels at 64^3
// 55 -> 40 us (134 MB: 3.3 TB/s; copies alone 31, products alone 31), 48 -> 16
// at 64^3 155 -> 106, 32 -> 32 at 32^3 25 -> 21, 96 -> 32 at 32^3 58 -> 45,
// 192 -> 64 at 16^3 52 -> 29; slower: 16 -> 32 at 32^3 and 32 -> 64 at 16^3
// (few bricks a block), 14.6 -> 15.5.
constexpr int kWtWaves = 9;                    // k_wgrad_small
constexpr int kWgWaves = 16;                   // k_wgrad_tr: 12 for the products, 4 for the copies
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4* lds_shortx4_ptr;

__device__ __forceinline__ bf16x8 tr_fragment(const char* lds, uint32_t byte0, uint32_t byte1) {
    const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_ptr)(lds + byte0));
    const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_shortx4_ptr)(lds + byte1));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int RS>
__global__ void __launch_bounds__(64 * kWgWaves) k_wgrad_tr(WgradArgs a, int64_t bricks_per_block) {
    using W = WgShape<RS>;
    __shared__ __attribute__((aligned(16))) __bf16 set[W::lds_items * 8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int lg = a.lg;
    // XCD-grouped order: the dispatcher deals consecutive blocks to the 8 XCDs
    // in turn, so logical block (lin mod 8) (total / 8) + lin / 8 puts runs of
    // consecutive (range, channel group) pairs on one XCD: the channel groups
    // of a range share its output gradient, neighbouring ranges their halo
    // rows, in that XCD's L2
    const uint32_t total = gridDim.x * gridDim.y, lin = blockIdx.y * gridDim.x + blockIdx.x;
    const uint32_t lblk = total % 8 ? lin : (lin % 8) * (total / 8) + lin / 8;
    const int chunk = (int)(lblk % gridDim.x), grp = (int)(lblk / gridDim.x);
    const int c0 = chunk * 16, co0 = (int)blockIdx.z * RS * 16;
    const int nbricks = a.n << (3 * lg - 8);
    const int per = (int)bricks_per_block;
    const int b0 = grp * per, b1 = b0 + per < nbricks ? b0 + per : nbricks;
    const bool lo = c0 < a.c1s;  // the group's channels lie in x1 (else x2; c1s is then a multiple of 16)
    const int chans = lo ? a.c1s : a.c2;
    const int cloc = lo ? c0 : c0 - a.c1s;
    const int64_t sample_x = (int64_t)chans << (3 * (lo ? lg : lg - 1)), sample_d = (int64_t)a.ys << (3 * lg);
    const __bf16 *xin = lo ? a.x1 : a.x2, *dyin = a.dy;
    __asm__ volatile("" : "+s"(xin), "+s"(dyin));  // held in scalars, not fetched again each brick
    // Waves 12 and 13 copy the halo (items 128 (w % 2) .. + 127 of each plane),
    // waves 14 and 15 the output gradient in turn; a lane's items are decoded
    // once (nn_wgrad_index.hpp).
    const int copier = wave - 12;
    uint32_t dyfrom[W::dy_it];
    WgHaloItem item[2] = {};
    if (copier == 0 || copier == 1) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            item[i] = wg_halo_item(copier * 128 + i * 64 + lane, lo, lg, chans, cloc, c0 + 8 < a.cin);
    } else if (copier > 1) {
#pragma unroll
        for (int i = 0; i < W::dy_it; ++i)
            dyfrom[i] = wg_dy_item<RS>((2 * i + copier - 2) * 64 + lane, lg, a.ys, co0);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_ptr)&set[0];
    // The copies of brick b: the halo planes from z0 - 1 + p0 on into the slots
    // from `to` on (p0: 0, or 2 for a brick that follows its z neighbour), the
    // output gradient into buffer buf.
    auto issue = [&](int b, int p0, int to, int buf) __attribute__((always_inline)) {
        const WgBrick o = wg_brick(b, lg);
        if (copier < 2) {
            const intx4 rx = buffer_words(xin + o.smp * sample_x, (uint32_t)(sample_x * 2));
            const uint32_t edges = wg_sides(o, lg);
            for (int p = p0; p < 6; ++p) {
                const int zz = o.z0 - 1 + p;
                const uint32_t sides = edges | wg_plane_sides(zz, lg);
                const uint32_t first = wg_plane_first(o, zz, lo, lg, chans);
                const uint32_t dst =
                    lds0 + (uint32_t)(W::slot(to + p - p0) * kWtPlaneItems + copier * 128) * 16u;
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    copy_to_lds(rx, dst + i * 1024, wg_halo_offset(item[i], sides, first));
            }
        } else {
            const intx4 rd = buffer_words(dyin + o.smp * sample_d, (uint32_t)(sample_d * 2));
            const uint32_t first = wg_dy_first(o, lg, a.ys);
            const uint32_t dst = lds0 + (uint32_t)(W::halo + buf * W::dy_buf) * 16u;
#pragma unroll
            for (int i = 0; i < W::dy_it; ++i) {
                const int c = 2 * i + copier - 2;
                if (c >= W::dy_copies) continue;
                copy_to_lds(rd, dst + (uint32_t)c * 1024u, dyfrom[i] + first);
            }
        }
    };
    const int dyw = wave % 3, plane = wave / 3;  // this wave's dy + 1 and plane (waves 0 .. 11)
    const uint32_t laneA = wg_lane_dy<RS>(lane, plane), laneB = wg_lane_halo(lane, dyw);
    floatx4 acc[3][3][RS];
#pragma unroll
    for (int z = 0; z < 3; ++z)
#pragma unroll
        for (int x = 0; x < 3; ++x)
#pragma unroll
            for (int m = 0; m < RS; ++m) acc[z][x][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    floatx4 accb[RS];
#pragma unroll
    for (int m = 0; m < RS; ++m) accb[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    const bool bias_wave = chunk == 0 && dyw == 0;
    auto products = [&](int base, int buf) __attribute__((always_inline)) {
        const char* sb = (const char*)set;
        const uint32_t la = laneA + (uint32_t)(buf * W::dy_buf * 16);
        bf16x8 av[2][RS];
#pragma unroll
        for (int rp = 0; rp < 2; ++rp)
#pragma unroll
            for (int m = 0; m < RS; ++m) {
                av[rp][m] = tr_fragment(sb, la + wg_dy_read<RS>(rp, m, 0), la + wg_dy_read<RS>(rp, m, 1));
            }
        if (bias_wave) {
#pragma unroll
            for (int rp = 0; rp < 2; ++rp)
#pragma unroll
                for (int m = 0; m < RS; ++m)
                    accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[rp][m], ones_frag(), accb[m],
                                                                      0, 0, 0);
        }
#pragma unroll
        for (int z = 0; z < 3; ++z) {  // dz + 1: halo plane `plane` + z
            const uint32_t lb = laneB + (uint32_t)(W::slot(base + plane + z) * kWtPlaneItems * 16);
#pragma unroll
            for (int rp = 0; rp < 2; ++rp) {
                typedef uint32_t uintx2 __attribute__((ext_vector_type(2)));
                typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
                uint32_t w[6];  // 12 voxels of the row, two a word
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const uintx2 d = __builtin_bit_cast(
                        uintx2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                    (lds_shortx4_ptr)(sb + lb + wg_halo_read(rp, i))));
                    w[2 * i] = d[0];
                    w[2 * i + 1] = d[1];
                }
                uintx4 f[3];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    f[0][i] = w[i];
                    f[1][i] = __builtin_amdgcn_alignbit(w[i + 1], w[i], 16);
                    f[2][i] = w[i + 1];
                }
#pragma unroll
                for (int x = 0; x < 3; ++x)
#pragma unroll
                    for (int m = 0; m < RS; ++m)
                        acc[z][x][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            av[rp][m], __builtin_bit_cast(bf16x8, f[x]), acc[z][x][m], 0, 0, 0);
            }
        }
    };
    // A brick's first halo plane is 4 ring slots on from its z neighbour's, 6 on
    // at the start of a column; its slots are free again once the next brick's
    // products start.
    auto follows = [&](int b) { return wg_follows(b, b0, lg); };
    if (copier >= 0) {
        __builtin_amdgcn_s_setprio(3);  // the next bricks' copies go out before the products' work
        WgAhead<RS> at(b0);
        for (int b = b0; b < b1; ++b) {
            // copy ahead as far as the ring and the buffers go: once under way,
            // one brick (whose slots the last brick has left)
            auto fill = [&]() __attribute__((always_inline)) {
                for (;;) {
                    const bool f = follows(at.next);
                    const int planes = f ? 4 : 6;
                    if (!at.can(b, b1, planes)) break;
                    issue(at.next, f ? 2 : 0, at.wslot, at.wbuf);
                    at.copied(planes);
                }
            };
            if (b == b0) fill();
            // the brick's copies have landed: later ones of this wave, at least
            // 8 (dy_min) for each brick copied after it, may be outstanding
            const int later = at.next - b - 1;
            if (copier < 2) {
                if (later >= 4) copies_outstanding<32>();
                else if (later == 3) copies_outstanding<24>();
                else if (later == 2) copies_outstanding<16>();
                else if (later == 1) copies_outstanding<8>();
                else copies_outstanding<0>();
            } else {
                if (later >= 4) copies_outstanding<4 * W::dy_min>();
                else if (later == 3) copies_outstanding<3 * W::dy_min>();
                else if (later == 2) copies_outstanding<2 * W::dy_min>();
                else if (later == 1) copies_outstanding<W::dy_min>();
                else copies_outstanding<0>();
            }
            block_barrier();
            if (b > b0) fill();
            at.base += follows(b + 1) ? 4 : 6;
        }
    } else {
        int bslot = 0, bbuf = 0;
        for (int b = b0; b < b1; ++b) {
            copies_landed<0>();  // (none of its own: its LDS reads are done)
            products(bslot, bbuf);
            bslot = W::slot(bslot + (follows(b + 1) ? 4 : 6));
            bbuf = W::next_buf(bbuf);
        }
    }
    // The four planes' sums: planes 2 and 3 through LDS to 0 and 1, then 1 to 0.
    constexpr int kSums = 9 * RS + RS;
    static_assert(6 * kSums * 64 <= W::lds_items, "the sums fit");
    floatx4* red = (floatx4*)set;
    auto put = [&](int at) __attribute__((always_inline)) {
        floatx4* p = red + (at * 3 + dyw) * kSums * 64 + lane;
#pragma unroll
        for (int z = 0; z < 3; ++z)
#pragma unroll
            for (int x = 0; x < 3; ++x)
#pragma unroll
                for (int m = 0; m < RS; ++m) p[((z * 3 + x) * RS + m) * 64] = acc[z][x][m];
#pragma unroll
        for (int m = 0; m < RS; ++m) p[(9 * RS + m) * 64] = accb[m];
    };
    auto add = [&](int at) __attribute__((always_inline)) {
        const floatx4* p = red + (at * 3 + dyw) * kSums * 64 + lane;
#pragma unroll
        for (int z = 0; z < 3; ++z)
#pragma unroll
            for (int x = 0; x < 3; ++x)
#pragma unroll
                for (int m = 0; m < RS; ++m) acc[z][x][m] += p[((z * 3 + x) * RS + m) * 64];
#pragma unroll
        for (int m = 0; m < RS; ++m) accb[m] += p[(9 * RS + m) * 64];
    };
    __syncthreads();
    if (plane == 2 || plane == 3) put(plane - 2);
    __syncthreads();
    if (plane < 2) add(plane);
    __syncthreads();
    if (plane == 1) put(0);
    __syncthreads();
    if (plane != 0) return;
    add(0);
    const int rst = a.coutp / 16, m0 = (int)blockIdx.z * RS;
    const int64_t blk = (int64_t)grp * gridDim.x + chunk;
    float* pb = a.part + blk * (27 * rst * 16 * 16);
#pragma unroll
    for (int z = 0; z < 3; ++z)
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const int t = z * 9 + dyw * 3 + x;
#pragma unroll
            for (int m = 0; m < RS; ++m)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    pb[((t * rst + m0 + m) * 16 + q * 4 + k) * 16 + r] = acc[z][x][m][k];
        }
    if (bias_wave && r == 0) {
        float* bb = a.part + a.bias_off + (int64_t)grp * (rst * 16) + m0 * 16;
#pragma unroll
        for (int m = 0; m < RS; ++m)
#pragma unroll
            for (int k = 0; k < 4; ++k) bb[m * 16 + q * 4 + k] = accb[m][k];
    }
}

// Weight gradient on grids of 8 cells (the bottleneck layers), by the
// transposing LDS reads of k_wgrad_tr: a block takes one sample, one
// 16-channel input group and 32 output channels, copies the sample's
// 10 x 10 x 10 input halo (rows padded to 12 voxels) and the 32 channels of
// its output gradient (rows of 8 voxels padded to 544 bytes) into LDS, and
// nine waves (wave w the taps with dz = w / 3 - 1, dy = w % 3 - 1) walk the
// 16 k steps of 32 voxels (plane s / 2, rows 4 (s % 2) + q for lane group q).
// Partials per (sample, input group): the layout k_brick_partials_sum adds up
// (samples as its rows).
constexpr int kWsHaloRow = 12;                       // voxels per padded halo row
constexpr int kWsHaloItems = 2 * kWsHaloRow * 10 * 10;  // 2400
constexpr int kWsHaloBuf = 38 * 64;                  // whole waves
constexpr int kWsDyRow = 34;                         // 16-byte items per output-gradient row
constexpr int kWsDyItems = 64 * kWsDyRow;            // 2176 = 34 waves
constexpr int kWsCopies = (kWsHaloBuf + kWsDyItems) / 64 / kWtWaves;  // 8 per wave

__global__ void __launch_bounds__(64 * kWtWaves) k_wgrad_small(WgradArgs a) {
    static_assert((kWsHaloBuf + kWsDyItems) / 64 == kWsCopies * kWtWaves, "uniform copies");
    __shared__ __attribute__((aligned(16))) __bf16 set[(kWsHaloBuf + kWsDyItems) * 8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int chunk = blockIdx.x, smp = blockIdx.y, cp = blockIdx.z;
    const int c0 = chunk * 16;
    const int rsg = a.coutp / 16;  // output-channel tiles of the layer
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(a.x1 + (int64_t)smp * 512 * a.c1s), (short)0, 512 * a.c1s * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(a.dy + (int64_t)smp * 512 * a.ys), (short)0, 512 * a.ys * 2, 0x00020000);
#pragma unroll
    for (int j = 0; j < kWsCopies; ++j) {
        const int tb = (j * kWtWaves + wv) * 64;
        const int t0 = tb + lane;
        uint32_t off;
        __amdgpu_buffer_rsrc_t rsrc;
        if (tb < kWsHaloBuf) {
            // halo item t: slot t / 2 of 12 x 10 x 10, channel half t % 2
            const int half = t0 & 1, hv = t0 >> 1;
            const int hx = hv % kWsHaloRow, hy = (hv / kWsHaloRow) % 10, hz = hv / (10 * kWsHaloRow);
            const int xx = hx - 1, yy = hy - 1, zz = hz - 1;
            const bool ok = t0 < kWsHaloItems && hx < 10 && c0 + half * 8 < a.cin && (unsigned)xx < 8u &&
                            (unsigned)yy < 8u && (unsigned)zz < 8u;
            const uint32_t vox = ((uint32_t)zz << 6) + ((uint32_t)yy << 3) + (uint32_t)xx;
            off = ((vox * (uint32_t)a.c1s + (uint32_t)(c0 + half * 8)) * 2u) | ((uint32_t)!ok << 31);
            rsrc = rx;
        } else {
            // output-gradient item t: row t / 34 (8 z + y), voxel and 8 channels of item t % 34
            const int t = t0 - kWsHaloBuf;
            const int row = t / kWsDyRow, it = t - row * kWsDyRow;
            const int px = it >> 2, c8 = it & 3;
            const int co = cp * 32 + c8 * 8;
            const bool ok = it < 32 && co < a.ys;
            const uint32_t vox = ((uint32_t)row << 3) + (uint32_t)(px & 7);
            off = ((vox * (uint32_t)a.ys + (uint32_t)co) * 2u) | ((uint32_t)!ok << 31);
            rsrc = rd;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)&set[tb * 8], 16, off, 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt 0: this wave's copies landed
    __syncthreads();
    floatx4 acc[3][2], accb[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        accb[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int d = 0; d < 3; ++d) acc[d][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const bool bias_wave = chunk == 0 && wave == 0;
    const int e = r >> 2, ac = r & 3;
    const int dzw = wave / 3, dyw = wave % 3;
    const uint32_t laneA = (uint32_t)(kWsHaloBuf * 16 + (q * kWsDyRow + e * 4) * 16 + ac * 8);
    const uint32_t laneB = (uint32_t)(((q + dyw) * kWsHaloRow + dzw * 10 * kWsHaloRow + e) * 32 + ac * 8);
    const char* sb = (const char*)set;
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const int ra = ((s >> 1) * 8 + 4 * (s & 1)) * kWsDyRow * 16;  // the step's first row
        const int vb = ((s >> 1) * 10 + 4 * (s & 1)) * kWsHaloRow;   // halo slot of its first cell
        bf16x8 av[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) av[m] = tr_fragment(sb, laneA + ra + m * 32, laneA + ra + 4 * 64 + m * 32);
        if (bias_wave) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
                accb[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[m], ones_frag(), accb[m], 0, 0, 0);
        }
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
            const bf16x8 bv = tr_fragment(sb, laneB + (vb + dx) * 32, laneB + (vb + dx + 4) * 32);
#pragma unroll
            for (int m = 0; m < 2; ++m)
                acc[dx][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[m], bv, acc[dx][m], 0, 0, 0);
        }
    }
    const int chunks = gridDim.x;
    float* pb = a.part + ((int64_t)smp * chunks + chunk) * (27 * rsg * 256);
#pragma unroll
    for (int dx = 0; dx < 3; ++dx) {
        const int t = wave * 3 + dx;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                pb[((t * rsg + cp * 2 + m) * 16 + q * 4 + k) * 16 + r] = acc[dx][m][k];
    }
    if (bias_wave && r == 0) {
        float* bb = a.part + a.bias_off + (int64_t)smp * a.coutp + cp * 32;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int k = 0; k < 4; ++k) bb[m * 16 + q * 4 + k] = accb[m][k];
    }
}

// Sum of the brick kernels' partials over the brick ranges in one pass, into
// dw[co][tap][ci] (zero padding channels dropped) and db.  A block takes E
// entries (consecutive in a partial row) and L row lanes: lane j adds rows j,
// j + L, ... in order, then a fixed tree adds the L lane sums, so every sum
// has one fixed order.  Blocks past the weight entries take the bias.  Tables
// of few rows take L = 1 (256 entries a block, each thread its entry's rows
// in order, several loads in flight), tall ones that give fewer than two
// blocks per CU L = 32 (32 entries, 128 bytes of a row), the rest L = 8.
constexpr int kPsShortRows = 32, kPsTallRows = 256, kPsFewBlocks = 512;

template <int kPsLanes, int kEnt>
__global__ void __launch_bounds__(kEnt * kPsLanes)
k_brick_partials_sum(WgradArgs a, int chunks, int rows, int rs, float* dw, float* db) {
    const uint32_t per = (uint32_t)(27 * rs * 16 * 16);  // entries of one channel group
    const uint32_t W = per * (uint32_t)chunks;           // weight entries of a row
    const uint32_t nbw = (W + kEnt - 1) / kEnt;
    const int el = threadIdx.x % kEnt, j = threadIdx.x / kEnt;
    const bool bias = blockIdx.x >= nbw;
    const uint32_t e = (bias ? blockIdx.x - nbw : blockIdx.x) * kEnt + el;
    const bool valid = bias ? e < (uint32_t)a.cout : e < W;
    const float* base = bias ? a.part + a.bias_off : a.part;
    const uint32_t stride = bias ? (uint32_t)(rs * 16) : W;
    float v = 0.f;
    if constexpr (kPsLanes == 1) {
        if (!valid) return;
#pragma unroll 8
        for (int g = 0; g < rows; ++g) v += base[(int64_t)g * stride + e];
    } else {
        __shared__ float red[kPsLanes][kEnt + 1];
        float sum = 0.f;
        if (valid) {
#pragma unroll 4
            for (int g = j; g < rows; g += kPsLanes) sum += base[(int64_t)g * stride + e];
        }
        red[j][el] = sum;
        __syncthreads();
#pragma unroll
        for (int h = kPsLanes / 2; h > 0; h >>= 1) {
            if (j < h) red[j][el] += red[j + h][el];
            __syncthreads();
        }
        if (j != 0 || !valid) return;
        v = red[0][el];
    }
    if (bias) {
        db[e] = v;
        return;
    }
    const uint32_t chunk = e / per, r0 = e - chunk * per;
    const uint32_t t = r0 / (uint32_t)(rs * 256), rem = r0 - t * (uint32_t)(rs * 256);
    const uint32_t co = rem >> 4, cc = chunk * 16 + (rem & 15);
    if (co >= (uint32_t)a.cout || cc >= (uint32_t)a.cin || (cc < (uint32_t)a.c1s && cc >= (uint32_t)a.c1))
        return;
    const uint32_t ci = cc < (uint32_t)a.c1s ? cc : a.c1 + (cc - a.c1s);
    dw[((int64_t)co * 27 + t) * a.cin_real + ci] = v;
}

// Packed weight element idx of wp[coutp][kpad] (k = tap * cin + stored
// channel; zero padding channels and k >= K hold 0).
__device__ __forceinline__ float pack_w_elem(const PackLayer& L, int64_t idx,
                                             const float* __restrict__ w) {
    const int co = (int)(idx / L.kpad), k = (int)(idx - (int64_t)co * L.kpad);
    if (co >= L.cout || k >= L.K) return 0.f;
    const int t = k / L.cin, cc = k - t * L.cin;
    if (cc < L.c1s) return cc < L.c1 ? w[((int64_t)co * L.taps + t) * L.cin_real + cc] : 0.f;
    return w[((int64_t)co * L.taps + t) * L.cin_real + L.c1 + (cc - L.c1s)];
}

// Transposed, tap-flipped element idx of wt[cinp][kpad_t] (k = tap * ys + co).
__device__ __forceinline__ float pack_wt_elem(const PackLayer& L, int64_t idx,
                                              const float* __restrict__ w) {
    const int ci = (int)(idx / L.kpad_t), k = (int)(idx - (int64_t)ci * L.kpad_t);
    if (ci >= L.cin || k >= L.taps * L.ys) return 0.f;
    const int t = k / L.ys, co = k - t * L.ys;
    const bool real = ci >= L.c1s || ci < L.c1;
    if (co >= L.cout || !real) return 0.f;
    const int cir = ci < L.c1s ? ci : L.c1 + (ci - L.c1s);
    return w[((int64_t)co * L.taps + (L.taps - 1 - t)) * L.cin_real + cir];
}

// The transposed copy is written in tiles of 16 input channels x 64 k
// entries through LDS: the master weights are read along the input channels
// (16 consecutive floats per k entry) and wt is written along k (8 bytes per
// lane, 128 bytes per channel row), instead of one gather per element at the
// stride of a whole output channel.
constexpr int kWtTileCi = 16, kWtTileK = 64;

// Every layer's packed and transposed weights in one launch.  Segment 2l is
// layer l's wp (8 elements per thread), segment 2l + 1 its wt (one tile per
// block); each block serves one segment (the first whose cumulative block
// count exceeds blockIdx.x), so the table is read with block-uniform indices.
__global__ void __launch_bounds__(256) k_pack_all(PackTable t, const float* __restrict__ theta) {
    __shared__ float tile[kWtTileK][kWtTileCi + 1];
    int seg = 0;
    while ((int64_t)blockIdx.x >= t.blk[seg]) ++seg;
    const int64_t first = seg ? t.blk[seg - 1] : 0;
    const int64_t b = (int64_t)blockIdx.x - first;
    const PackLayer& L = t.l[seg >> 1];
    const float* w = theta + L.woff;
    if (!(seg & 1)) {
        // 8 consecutive k entries per thread (one tap: cin is a multiple of 8), 16 bytes
        const int64_t i = (b * 256 + threadIdx.x) * 8;
        if (i >= (int64_t)L.coutp * L.kpad) return;
        bf16x8 o;
#pragma unroll
        for (int u = 0; u < 8; ++u) o[u] = (__bf16)pack_w_elem(L, i + u, w);
        *(bf16x8*)(L.wp + i) = o;
        return;
    }
    const int nkt = (L.kpad_t + kWtTileK - 1) / kWtTileK;
    const int ci0 = (int)(b / nkt) * kWtTileCi, k0 = (int)(b % nkt) * kWtTileK;
    {
        // 4 lanes per k entry, 4 consecutive input channels each
        const int kk = threadIdx.x >> 2, c4 = (threadIdx.x & 3) * 4;
        const int k = k0 + kk;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            tile[kk][c4 + u] = k < L.kpad_t ? pack_wt_elem(L, (int64_t)(ci0 + c4 + u) * L.kpad_t + k, w)
                                            : 0.f;
    }
    __syncthreads();
    // 16 lanes per input channel, 4 consecutive k entries (8 bytes) each
    const int cl = threadIdx.x >> 4, k4 = (threadIdx.x & 15) * 4;
    if (k0 + k4 >= L.kpad_t) return;  // kpad_t is a multiple of 4: whole groups
    bf16x4 o;
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = (__bf16)tile[k4 + u][cl];
    *(bf16x4*)(L.wt + (int64_t)(ci0 + cl) * L.kpad_t + k0 + k4) = o;
}

__device__ __forceinline__ int64_t fine_index(int s, int z, int y, int x, int lg) {
    return ((int64_t)s << (3 * lg)) + ((int64_t)z << (2 * lg)) + ((int64_t)y << lg) + x;
}

// thread per (coarse cell, group of 8 channels)
__global__ void k_pool(int n, int lg, int c, const __bf16* __restrict__ x, __bf16* __restrict__ y) {
    const int h = lg - 1, cg = c / 8;
    const int64_t Vc = (int64_t)1 << (3 * h);
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n * Vc * cg) return;
    const int g = (int)(idx % cg);
    const int64_t vc = idx / cg;
    const int s = (int)(vc >> (3 * h));
    const int rem = (int)(vc & (Vc - 1));
    const int Z = rem >> (2 * h), Y = (rem >> h) & ((1 << h) - 1), X = rem & ((1 << h) - 1);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const int64_t vf = fine_index(s, 2 * Z + dz, 2 * Y + dy, 2 * X + dx, lg);
                const bf16x8 t = *(const bf16x8*)(x + vf * c + g * 8);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (float)t[i];
            }
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)(acc[i] * 0.125f);
    *(bf16x8*)(y + vc * c + g * 8) = o;
}

// thread per (fine cell, group of 8 channels)
__global__ void k_pool_bwd_add(int n, int lg, int c, const __bf16* __restrict__ dy,
                               const __bf16* __restrict__ skip, int ctot,
                               const __bf16* __restrict__ ymask, __bf16* __restrict__ dx) {
    const int h = lg - 1, cg = c / 8, G = 1 << lg;
    const int64_t V = (int64_t)1 << (3 * lg);
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n * V * cg) return;
    const int g = (int)(idx % cg);
    const int64_t v = idx / cg;
    const int s = (int)(v >> (3 * lg));
    const int rem = (int)(v & (V - 1));
    const int z = rem >> (2 * lg), y = (rem >> lg) & (G - 1), x = rem & (G - 1);
    const int64_t vc = ((int64_t)s << (3 * h)) + ((int64_t)(z >> 1) << (2 * h)) +
                       ((int64_t)(y >> 1) << h) + (x >> 1);
    const bf16x8 p = *(const bf16x8*)(dy + vc * c + g * 8);
    bf16x8 o;
    if (skip) {
        const bf16x8 k = *(const bf16x8*)(skip + v * ctot + g * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (__bf16)((float)p[i] * 0.125f + (float)k[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (__bf16)((float)p[i] * 0.125f);
    }
    if (ymask) {
        const bf16x8 mk = *(const bf16x8*)(ymask + v * c + g * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (!((float)mk[i] > 0.f)) o[i] = (__bf16)0.f;
    }
    *(bf16x8*)(dx + v * c + g * 8) = o;
}

// thread per (coarse cell, group of 8 channels)
__global__ void k_up_bwd(int n, int lg, int c, const __bf16* __restrict__ dcat, int ctot, int coff,
                         const __bf16* __restrict__ ymask, __bf16* __restrict__ dlow) {
    const int h = lg - 1, cg = c / 8;
    const int64_t Vc = (int64_t)1 << (3 * h);
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n * Vc * cg) return;
    const int g = (int)(idx % cg);
    const int64_t vc = idx / cg;
    const int s = (int)(vc >> (3 * h));
    const int rem = (int)(vc & (Vc - 1));
    const int Z = rem >> (2 * h), Y = (rem >> h) & ((1 << h) - 1), X = rem & ((1 << h) - 1);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) {
                const int64_t vf = fine_index(s, 2 * Z + dz, 2 * Y + dy, 2 * X + dx, lg);
                const bf16x8 t = *(const bf16x8*)(dcat + vf * ctot + coff + g * 8);
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] += (float)t[i];
            }
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)acc[i];
    if (ymask) {
        const bf16x8 mk = *(const bf16x8*)(ymask + vc * c + g * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (!((float)mk[i] > 0.f)) o[i] = (__bf16)0.f;
    }
    *(bf16x8*)(dlow + vc * c + g * 8) = o;
}

__global__ void k_inputs(int n, int lg, SampleFloats lra, __bf16* __restrict__ x) {
    const int G = 1 << lg;
    const int64_t V = (int64_t)1 << (3 * lg);
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= (int64_t)n * V) return;
    const int s = (int)(v >> (3 * lg));
    const int rem = (int)(v & (V - 1));
    const int z = rem >> (2 * lg), y = (rem >> lg) & (G - 1), xx = rem & (G - 1);
    const float inv = 2.0f / (float)G;
    bf16x8 o;
    o[0] = (__bf16)((lra.v[s] - 4.0f) * 0.5f);
    o[1] = (__bf16)((xx + 0.5f) * inv - 1.0f);
    o[2] = (__bf16)((y + 0.5f) * inv - 1.0f);
    o[3] = (__bf16)((z + 0.5f) * inv - 1.0f);
    o[4] = o[5] = o[6] = o[7] = (__bf16)0.f;
    *(bf16x8*)(x + v * 8) = o;
}

// The 1 x 1 x 1 head on the vector units (it reads 32 bytes and writes 16
// per voxel, far too little work for the matrix cores): kHeadIn BF16
// channels-last inputs -> kHeadOut FP32 outputs, channel-first, with the
// FP32 master weights w[co][ci] and bias b[co].  One thread per voxel.
constexpr int kHeadIn = 16, kHeadOut = 4, kHeadGrad = kHeadOut * kHeadIn + kHeadOut;

__device__ __forceinline__ void widen_head_input(bf16x8 lo, bf16x8 hi, float* xf) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        xf[i] = (float)lo[i];
        xf[8 + i] = (float)hi[i];
    }
}

__device__ __forceinline__ void load_head_input(const __bf16* __restrict__ x, int64_t v,
                                                float* xf) {
    widen_head_input(*(const bf16x8*)(x + v * kHeadIn), *(const bf16x8*)(x + v * kHeadIn + 8), xf);
}

__global__ void __launch_bounds__(256) k_head_forward(int n, int lg, const __bf16* __restrict__ x,
                                                      const float* __restrict__ w,
                                                      const float* __restrict__ b, float4 sc,
                                                      float* __restrict__ out) {
    const int64_t V = (int64_t)1 << (3 * lg);
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= (int64_t)n * V) return;
    const int64_t s = v >> (3 * lg), vin = v & (V - 1);
    float xf[kHeadIn];
    load_head_input(x, v, xf);
    const float scale[kHeadOut] = {sc.x, sc.y, sc.z, sc.w};
#pragma unroll
    for (int c = 0; c < kHeadOut; ++c) {
        float acc = b[c];
#pragma unroll
        for (int i = 0; i < kHeadIn; ++i) acc = fmaf(w[c * kHeadIn + i], xf[i], acc);
        out[(s * kHeadOut + c) * V + vin] = acc * scale[c];
    }
}

// Sum over the 64 lanes of a wave with DPP lane moves (no LDS): pairs and
// quads by quad permutes, rows of 16 by rotations by 4 and 8, then row 0's
// sum into row 1 and row 2's into row 3 by the lane-15 broadcast, and row
// 1's into rows 2 and 3 by the lane-31 broadcast.  Lane 63 receives the
// total, summed in the same order every time.  Rows left out of a move add 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_moved(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xF, false));
}

__device__ __forceinline__ float wave_sum_in_last_lane(float v) {
    v += dpp_moved<0xB1, 0xF>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_moved<0x4E, 0xF>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_moved<0x124, 0xF>(v);  // row_ror 4
    v += dpp_moved<0x128, 0xF>(v);  // row_ror 8
    v += dpp_moved<0x142, 0xA>(v);  // row_bcast 15 (rows 1 and 3)
    v += dpp_moved<0x143, 0xC>(v);  // row_bcast 31 (rows 2 and 3)
    return v;
}

// Loss and the whole backward step of the head in one pass: per voxel the
// head's output out = b + w x (the FMA sequence of k_head_forward, so the
// same values), the output gradient d = 2 (out - t) / count (t = target
// times its scale), the
// input gradient dx[ci] = sum_co w[co][ci] d[co] (0 where the ReLU output x
// <= 0; written as BF16), and the contributions d[co] x[ci] and d[co] to the
// weight and bias gradients.  Block b takes voxels [b chunk, (b + 1) chunk);
// its sums (squared error in FP64, the kHeadGrad gradient entries in FP32)
// are added over the block in a fixed order and written to lpart[b] and
// gpart[b][kHeadGrad].
//
// A voxel's 32 bytes of input and 16 of targets are loaded while the one
// before is computed; the sample, one for the 256 voxels of a turn, is a
// scalar (a lane's own index into idx was a load that the targets' loads
// waited for).  8 samples: 64^3 54 -> 40 us (168 MB: 4.2 TB/s; 2048 blocks 42),
// 32^3 25 -> 13 with blocks of 512 voxels (2048 before; 1024: 13.3).
__global__ void __launch_bounds__(256) k_head_backward(
    int n, int lg, const float* __restrict__ tg, SampleInts idx, int64_t stride, float4 ts,
    const __bf16* __restrict__ x, const float* __restrict__ w, const float* __restrict__ b,
    int64_t chunk, __bf16* __restrict__ dx, double* __restrict__ lpart,
    float* __restrict__ gpart) {
    __shared__ float gred[4][kHeadGrad];
    __shared__ double lred[256];
    const int64_t V = (int64_t)1 << (3 * lg);
    const int64_t M = (int64_t)n * V;
    const float inv = (float)(2.0 / ((double)n * 4.0 * (double)V));
    const float tsc[kHeadOut] = {ts.x, ts.y, ts.z, ts.w};
    float g[kHeadGrad];
#pragma unroll
    for (int j = 0; j < kHeadGrad; ++j) g[j] = 0.f;
    double lsum = 0.0;
    const int64_t v0 = (int64_t)blockIdx.x * chunk;
    const int64_t v1 = v0 + chunk < M ? v0 + chunk : M;
    // (M, chunk and V are multiples of 256: every thread takes every turn)
    bf16x8 xlo, xhi;
    float tv[kHeadOut];
    auto load = [&](int64_t first) __attribute__((always_inline)) {
        const int64_t v = first + threadIdx.x;
        const float* t = tg + (int64_t)idx.v[first >> (3 * lg)] * stride + (v & (V - 1));
        xlo = *(const bf16x8*)(x + v * kHeadIn);
        xhi = *(const bf16x8*)(x + v * kHeadIn + 8);
#pragma unroll
        for (int c = 0; c < kHeadOut; ++c) tv[c] = t[c * V];
    };
    if (v0 < v1) load(v0);
    for (int64_t first = v0; first < v1; first += 256) {
        const int64_t v = first + threadIdx.x;
        float xf[kHeadIn], t[kHeadOut];
        widen_head_input(xlo, xhi, xf);
#pragma unroll
        for (int c = 0; c < kHeadOut; ++c) t[c] = tv[c] * tsc[c];
        if (first + 256 < v1) load(first + 256);
        float d[kHeadOut];
#pragma unroll
        for (int c = 0; c < kHeadOut; ++c) {
            float ov = b[c];
#pragma unroll
            for (int i = 0; i < kHeadIn; ++i) ov = fmaf(w[c * kHeadIn + i], xf[i], ov);
            const double e = (double)ov - (double)t[c];
            lsum += e * e;
            d[c] = (float)e * inv;
        }
        bf16x8 lo, hi;
#pragma unroll
        for (int i = 0; i < kHeadIn; ++i) {
            float acc = 0.f;
#pragma unroll
            for (int c = 0; c < kHeadOut; ++c) acc = fmaf(w[c * kHeadIn + i], d[c], acc);
            const __bf16 r = (__bf16)(xf[i] > 0.f ? acc : 0.f);
            if (i < 8)
                lo[i] = r;
            else
                hi[i - 8] = r;
        }
        *(bf16x8*)(dx + v * kHeadIn) = lo;
        *(bf16x8*)(dx + v * kHeadIn + 8) = hi;
#pragma unroll
        for (int c = 0; c < kHeadOut; ++c) {
#pragma unroll
            for (int i = 0; i < kHeadIn; ++i) g[c * kHeadIn + i] = fmaf(d[c], xf[i], g[c * kHeadIn + i]);
            g[kHeadOut * kHeadIn + c] += d[c];
        }
    }
    // the wave's 64 lanes by DPP moves, then the 4 waves in order
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < kHeadGrad; ++j) {
        const float val = wave_sum_in_last_lane(g[j]);
        if (lane == 63) gred[wave][j] = val;
    }
    lred[threadIdx.x] = lsum;
    __syncthreads();
    for (int m = 128; m > 0; m >>= 1) {
        if ((int)threadIdx.x < m) lred[threadIdx.x] += lred[threadIdx.x + m];
        __syncthreads();
    }
    if (threadIdx.x < kHeadGrad)
        gpart[(int64_t)blockIdx.x * kHeadGrad + threadIdx.x] =
            ((gred[0][threadIdx.x] + gred[1][threadIdx.x]) + gred[2][threadIdx.x]) +
            gred[3][threadIdx.x];
    if (threadIdx.x == 0) lpart[blockIdx.x] = lred[0];
}

// The head's block sums in one launch.  Blocks j < width: out[j] = sum over
// rows r of in[r][j] (rows x width, FP32); the last block: loss = sum of the
// rows FP64 partials lp.  Thread t adds rows t, t + 256, ... in order, then a
// fixed tree adds the 256 thread sums.
template <typename T>
__device__ __forceinline__ T block_tree_sum(T* red, T v) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int m = 128; m > 0; m >>= 1) {
        if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
        __syncthreads();
    }
    return red[0];
}

__global__ void __launch_bounds__(256) k_head_sums(const float* __restrict__ in, int rows,
                                                   int width, float* __restrict__ out,
                                                   const double* __restrict__ lp,
                                                   double* __restrict__ loss) {
    __shared__ float redf[256];
    __shared__ double redd[256];
    const int j = blockIdx.x;
    if (j < width) {
        float acc = 0.f;
        for (int r = threadIdx.x; r < rows; r += 256) acc += in[(int64_t)r * width + j];
        const float t = block_tree_sum(redf, acc);
        if (threadIdx.x == 0) out[j] = t;
    } else {
        double acc = 0.0;
        for (int r = threadIdx.x; r < rows; r += 256) acc += lp[r];
        const double t = block_tree_sum(redd, acc);
        if (threadIdx.x == 0) loss[0] = t;
    }
}

__global__ void k_adam(int64_t count, float* __restrict__ th, float* __restrict__ m,
                       float* __restrict__ v, const float* __restrict__ g, float lr, float b1,
                       float b2, float eps, float c1, float c2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    th[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void k_zero(float* __restrict__ p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0.f;
}

__global__ void k_bf16_to_f32(const __bf16* __restrict__ x, int64_t cells, int cs, int c,
                              float* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cells * c) return;
    const int64_t v = i / c;
    const int ch = (int)(i - v * c);
    y[i] = (float)x[v * cs + ch];
}

__global__ void k_cf_to_cl(const float* __restrict__ x, int n, int64_t V, int c,
                           float* __restrict__ y) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n * V * c) return;
    const int ch = (int)(i % c);
    const int64_t v = (i / c) % V;
    const int64_t s = i / (c * V);
    y[i] = x[(s * c + ch) * V + v];
}

// Forward / input-gradient convolution on LDS-staged bricks (3x3x3 taps,
// BF16 output, grids of at least 16 cells, input channels a multiple of 16,
// or 8 with no second tensor).  A block of 8 WY waves computes bricks of 16 x
// 4 WY x 8 output voxels (wave w the plane z0 + w % 8, the four 16-voxel row
// tiles from y0 + 4 (w / 8), whose taps share most of their halo rows; where
// 2 x 2 x 2 cells are added up, rows y0 + 2 (w / 4), + 1 of planes z0 + 2 (w %
// 4), + 1) for NSUB * 16 output channels.  A step takes 16
// input channels of a brick: the 18 x (4 WY + 2) x 10 input halo
// (channels-last, 32 bytes per voxel: lane r reads voxel r and its second 8
// channels sit 16 bytes on, which the LDS serves without bank conflicts) and
// the chunk's weights, copied into LDS with direct-to-LDS buffer loads, so
// every fragment is one LDS read.  A k step of 32 takes two taps of the 16
// channels, paired so that the second lies a fixed displacement from the first
// within each group of steps (two planes on, two rows on, two voxels on, or a
// slot of zero weights): a lane's LDS addresses are then a base register per
// group plus a compile-time offset, with no per-step index arithmetic.
//
// A block walks a range of bricks with two halo buffers: the copies of step
// s + 1 are in flight during the products of step s.  What had bound the
// one-brick-a-block form of this kernel was each block's chain of launch,
// address decode, copy round trip and stores (64^3, batch 8, 16 -> 16
// channels: 46 us, of which 28 with neither copies nor products), at 25% of
// the matrix cores, 25% of the LDS and 46% of HBM.
constexpr int kCvVox = 16;                  // LDS elements per voxel
constexpr int kCvPlanes = 8;                // output planes per brick
constexpr int kCvSlots = 28;                // 27 taps + a zero-weight slot
constexpr int kCvWItemsRow = 2 * kCvSlots + 2;  // 16-byte weight items per row (+ 32 B pad)
constexpr int kCvWRow = 8 * kCvWItemsRow;   // elements per LDS weight row (928 B, 32 mod 64)

// Step p (0..13) of the k loop takes tap p in lanes q < 2 and tap
// cv_pair_tap(p) in lanes q >= 2 (-1: the zero slot), two planes, two rows or
// two voxels on (or anywhere, with zero weights).
__device__ constexpr int cv_pair_tap(int p) {
    return p <= 8 ? p + 18 : p <= 11 ? p + 6 : p == 12 ? 14 : -1;
}

template <int NSUB, int WY, bool ONE>
struct CvShape {
    static constexpr int rows = 4 * WY + 2;        // halo rows
    static constexpr int plane = 18 * rows;        // halo voxels per plane
    static constexpr int items = 2 * plane * (kCvPlanes + 2);  // 16-byte halo items
    static constexpr int buf = (items + 63) / 64 * 64;
    static constexpr int threads = 64 * kCvPlanes * WY;
    static constexpr int halo_it = (items + threads - 1) / threads;
    static constexpr int witems = NSUB * 16 * kCvWItemsRow;
    static constexpr int wbuf = (witems + 63) / 64 * 64;
    static constexpr int weight_it = (wbuf + threads - 1) / threads;
    static constexpr int wsets = ONE ? 1 : 2;      // weight buffers
    static constexpr int lds_items = 2 * buf + wsets * wbuf;
    static_assert(lds_items * 16 <= 160 * 1024, "one block's LDS");
};

// ONE: one step a brick (at most 16 input channels), so the weights are
// copied once.  EPI: what the results take (kPlain; kBias: bias and ReLU;
// kMask: 0 where the mask is not positive; kBiasPool: kBias, and averages over
// 2 x 2 x 2 to a.low; kUp: the first a.split channels as kPlain, of the others
// only their sums over 2 x 2 x 2 to a.low, 0 where a.lowmask is not positive).
// work: bricks in all, per: bricks per block.  The output channels are a
// multiple of 16.
//
// kBiasPool and kUp take the pooling and the gradient of the upsampling out of
// their own passes over memory, for the sums of four tiles of a wave and of
// lane pairs: the additions are those passes', of the rounded results and in
// their order.  8 samples: at 64^3 with the pooling 37 us (32 and 13 apart), 16
// -> 16 + 32 with the upsampling's gradient 72 us (71 and 35 apart: 134 MB less
// written and read, now the products' and sums' issue slots), 32 -> 32 + 64 at
// 32^3 48 (45 and 10); the skip's gradient, now dense, is read in 35 us (63).
//
// Everything outside the products is kept short, for it takes the issue slots
// of all waves in step: addresses are a lane register plus scalars, and the
// results have no branches.  (With general results and per-item address
// arithmetic, 184 vector and 272 scalar instructions a wave and step beside
// the 56 products, the same walk took 41-43 us instead of 30-33.)
enum { kPlain, kBias, kMask, kBiasPool, kUp };

template <int NSUB, int WY, bool ONE, int EPI>
__global__ void __launch_bounds__(64 * kCvPlanes * WY)
k_conv_brick(ConvArgs a, int work, int per) {
    using C = CvShape<NSUB, WY, ONE>;
    typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) __bf16 lds[C::lds_items * 8];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4, hi = q >> 1;
    const int lg = a.lg, h = lg - 1, G = 1 << lg;
    // blocks i, i + 8, ... run on one XCD (dispatch is round-robin over the
    // eight): give each XCD contiguous ranges of bricks, whose halos overlap
    // in its L2
    const int nb = (int)gridDim.x;
    const int range = nb % 8 ? (int)blockIdx.x : (int)(blockIdx.x % 8) * (nb / 8) + (int)blockIdx.x / 8;
    const int b0 = range * per, b1 = b0 + per < work ? b0 + per : work;
    if (b0 >= b1) return;
    const int cobase = blockIdx.y * NSUB * 16;
    const int chunks = ONE ? 1 : a.cin / 16;
    // The lane's copy items, decoded once: item i is voxel tid / 2 + i threads
    // / 2 of the halo (channel half tid % 2).  fine, coarse: its byte in x1 (in
    // x2, at its parent) from the halo's first voxel; side: the sides of the
    // halo it lies on (a brick at that side of the grid reads zeros there).
    // Items that read zeros take offsets with bit 31 set (samples are below
    // 2^31 bytes): past the buffer's end.
    constexpr int kHalf = C::threads / 2;
    constexpr uint32_t kOutside = 0x80000000u;
    const int half = tid & 1;
    uint32_t fine[C::halo_it], coarse[C::halo_it], side[C::halo_it], wofs[C::weight_it];
    {
        int hx = (tid >> 1) % 18, hy = ((tid >> 1) / 18) % C::rows, hz = (tid >> 1) / C::plane;
#pragma unroll
        for (int i = 0; i < C::halo_it; ++i) {
            const bool never = i * C::threads + tid >= C::items || half * 8 >= a.cin;
            const int v1 = (hz << (2 * lg)) + (hy << lg) + hx;
            const int v2 = ((hz + 1) >> 1 << (2 * h)) + ((hy + 1) >> 1 << h) + ((hx + 1) >> 1);
            fine[i] = never ? kOutside : (uint32_t)(v1 * a.c1s + half * 8) * 2u;
            coarse[i] = never ? kOutside : (uint32_t)(v2 * a.c2 + half * 8) * 2u;
            side[i] = (uint32_t)((hx == 0) | (hx == 17) << 1 | (hy == 0) << 2 |
                                 (hy == C::rows - 1) << 3 | (hz == 0) << 4 |
                                 (hz == kCvPlanes + 1) << 5 | never << 6);
            hx += kHalf % 18;
            if (hx >= 18) hx -= 18, ++hy;
            hy += kHalf % C::plane / 18;
            if (hy >= C::rows) hy -= C::rows, ++hz;
            hz += kHalf / C::plane;
        }
        // weight item t: row t / 58 (output channel cobase + row), slot s =
        // (t % 58) / 2 (tap s / 2 for even s, the paired tap for odd s), 8
        // channels of half t % 2; items 56, 57 of a row are padding.  (With 8
        // input channels the upper half holds the next tap's weights, which
        // meet zero inputs, and stays inside the row since 27 * 8 + 8 <= kpad.)
#pragma unroll
        for (int i = 0; i < C::weight_it; ++i) {
            const int t = i * C::threads + tid;
            const int row = t / kCvWItemsRow, rem = t - row * kCvWItemsRow;
            const int slot = rem >> 1, p = slot >> 1;
            const int tap = (slot & 1) ? cv_pair_tap(p) : p;
            const bool ok = t < C::witems && rem < 2 * kCvSlots && tap >= 0;
            wofs[i] = ok ? (uint32_t)((cobase + row) * a.kpad + tap * a.cin + (rem & 1) * 8) * 2u
                         : kOutside;
        }
    }
    // What a brick's copies and results take from its place, in scalars: the
    // sample, the first voxel (out: of the brick; fine, coarse: of the halo, in
    // x1 and x2) and the sides of the grid it lies at.  Bricks run x fastest,
    // then y, z, sample.  (Comparisons as sign bits: as truth values the
    // compiler takes them through vector registers.)
    struct Place {
        int smp, out, fine, coarse;
        uint32_t sides;
    };
    auto place = [&](int b) __attribute__((always_inline)) {
        constexpr int ly = WY == 2 ? 3 : 2;
        const int x0 = (b & ((1 << (lg - 4)) - 1)) * 16;
        b >>= lg - 4;
        const int y0 = (b & ((1 << (lg - ly)) - 1)) * (4 * WY);
        b >>= lg - ly;
        const int z0 = (b & ((1 << (lg - 3)) - 1)) * kCvPlanes;
        auto negative = [](int v) { return (uint32_t)v >> 31; };
        Place o;
        o.smp = b >> (lg - 3);
        o.out = (z0 << (2 * lg)) + (y0 << lg) + x0;
        o.fine = ((z0 - 1) << (2 * lg)) + ((y0 - 1) << lg) + x0 - 1;
        o.coarse = ((z0 / 2 - 1) << (2 * h)) + ((y0 / 2 - 1) << h) + x0 / 2 - 1;
        o.sides = negative(x0 - 1) | negative(G - 17 - x0) << 1 | negative(y0 - 1) << 2 |
                  negative(G - 4 * WY - 1 - y0) << 3 | negative(z0 - 1) << 4 |
                  negative(G - kCvPlanes - 1 - z0) << 5 | 64u;
        return o;
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_ptr)&lds[0];
    const intx4 rw = buffer_words(a.w, (uint32_t)((int64_t)a.wrows * a.kpad * 2));
    const __bf16 *x1 = a.x1, *x2 = a.x2;  // held in scalars, not fetched again each step
    __asm__ volatile("" : "+s"(x1), "+s"(x2));
    const int64_t sample1 = (int64_t)a.c1s << (3 * lg), sample2 = (int64_t)a.c2 << (3 * h);
    // the copies of a step into halo buffer (and weight buffer) `to`
    auto issue = [&](const Place& o, int chunk, int to, bool weights) __attribute__((always_inline)) {
        const int c0 = chunk * 16;
        const uint32_t dst = lds0 + (uint32_t)(to * C::buf) * 16u;
        auto halo = [&](const uint32_t (&item)[C::halo_it], const __bf16* x, int64_t sample,
                        int first, int chans, int c) __attribute__((always_inline)) {
            const intx4 rs = buffer_words(x + o.smp * sample, (uint32_t)(sample * 2));
            const uint32_t from = (uint32_t)(first * chans + c) * 2u;
#pragma unroll
            for (int i = 0; i < C::halo_it; ++i) {
                const int tb = i * C::threads + wave * 64;
                if (tb >= C::items) continue;
                const uint32_t v = item[i] + from;
                const uint32_t off = side[i] & o.sides ? kOutside : v;
                copy_to_lds(rs, dst + (uint32_t)tb * 16u, off);
            }
        };
        if (ONE || c0 < a.c1s)  // x1's channels, else x2's (c1s is then a multiple of 16)
            halo(fine, x1, sample1, o.fine, a.c1s, c0);
        else
            halo(coarse, x2, sample2, o.coarse, a.c2, c0 - a.c1s);
        if (!weights) return;
        const uint32_t wdst = lds0 + (uint32_t)(2 * C::buf + (ONE ? 0 : to * C::wbuf)) * 16u;
#pragma unroll
        for (int i = 0; i < C::weight_it; ++i) {
            const int tb = i * C::threads + wave * 64;
            if (tb >= C::wbuf) continue;
            const uint32_t off = wofs[i] + (uint32_t)c0 * 2u;
            copy_to_lds(rw, wdst + (uint32_t)tb * 16u, off);
        }
    };
    floatx4 acc[4][NSUB];
    const int ch = (q & 1) * 8;
    // LDS byte addresses of this lane: A (weights), B (halo) per shift group
    constexpr bool kCells = EPI == kBiasPool || EPI == kUp;
    const int wz = kCells ? (wave & 3) * 2 : wave & 7, wy = kCells ? (wave >> 2) * 2 : (wave >> 3) * 4;
    auto row = [](int m) { return kCells ? m & 1 : m; };  // of tile m, from the wave's first
    auto plane = [](int m) { return kCells ? m >> 1 : 0; };
    const uint32_t lb = (uint32_t)(wz * C::plane + wy * 18 + r);
    const uint32_t vB0 = ((lb + hi * 2 * C::plane) * kCvVox + ch) * 2;
    const uint32_t vB1 = ((lb + hi * 2 * 18) * kCvVox + ch) * 2;
    const uint32_t vB2 = ((lb + hi * 2) * kCvVox + ch) * 2;
    const uint32_t vB3 = (lb * kCvVox + ch) * 2;
    uint32_t vA = (uint32_t)(2 * C::buf * 16 + (r * kCvWRow + hi * 16 + ch) * 2);
    __asm__ volatile("" : "+v"(vA));  // (as a constant it would pass the reads' 16-bit offsets)
    // D rows 4q .. 4q+3 are output channels, column r the voxel x0 + r: the
    // lane's byte from the brick's first voxel (tile 0)
    const uint32_t vout =
        (uint32_t)((((wz << (2 * lg)) + (wy << lg) + r) * a.ys) + cobase + 4 * q) * 2u;
    const uint32_t row_bytes = (uint32_t)a.ys * 2u << lg, plane_bytes = row_bytes << lg;
    const int64_t sample_out = (int64_t)a.ys << (3 * lg);
    // in a.low: the even lanes' byte from the brick's first coarse voxel
    const int lows = EPI == kUp ? a.cout - a.split : a.cout;
    const uint32_t vlow =
        r & 1 ? kOutside
              : (uint32_t)((((wave & 3) << (2 * h)) + ((wave >> 2) << h) + (r >> 1)) * lows + 4 * q) * 2u;
    const int64_t sample_low = (int64_t)lows << (3 * h);
    floatx4 bias[NSUB];
    if constexpr (EPI == kBias || EPI == kBiasPool) {
#pragma unroll
        for (int j = 0; j < NSUB; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) bias[j][i] = a.bias[cobase + j * 16 + 4 * q + i];
    }
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int j = 0; j < NSUB; ++j) acc[m][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    int chunk = 0, set = 0;
    bool stored = false;  // whether the step before ended a brick
    Place o = place(b0);
    issue(o, 0, 0, true);
    for (int b = b0; b < b1;) {
        // this step's copies have landed (only the last brick's stores were
        // issued after them), and every wave is done with the other buffer
        if (!stored)
            copies_landed<0>();
        else if (EPI == kUp && cobase >= a.split)
            copies_landed<NSUB>();
        else
            copies_landed<EPI == kUp ? NSUB + 3 : EPI == kBiasPool ? 5 * NSUB : 4 * NSUB>();
        const bool last = ONE || chunk + 1 == chunks;
        const uint32_t first = vout + (uint32_t)o.out * (uint32_t)a.ys * 2u;
        // the mask is loaded ahead of the products
        uintx2 mask[EPI == kMask ? 4 * NSUB : NSUB];
        const int olow = o.coarse + (1 << (2 * h)) + (1 << h) + 1;  // the brick's first coarse voxel
        const uint32_t first_low = vlow + (uint32_t)olow * (uint32_t)lows * 2u;
        if constexpr (EPI == kMask) {
            if (last) {
                const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<__bf16*>(a.omask + o.smp * sample_out), (short)0,
                    (int)(uint32_t)(sample_out * 2), 0x00020000);
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int j = 0; j < NSUB; ++j) {
                        const uint32_t off = first + row(m) * row_bytes + plane(m) * plane_bytes + j * 32;
                        mask[m * NSUB + j] = __builtin_amdgcn_raw_buffer_load_b64(rm, off, 0, 0);
                    }
            }
        }
        if constexpr (EPI == kUp) {
            if (last) {
                const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<__bf16*>(a.lowmask + o.smp * sample_low), (short)0,
                    (int)(uint32_t)(sample_low * 2), 0x00020000);
#pragma unroll
                for (int j = 0; j < NSUB; ++j) {
                    const int c = cobase + j * 16 - a.split;  // (of a.out's channels: not used)
                    const uint32_t off = first_low + (uint32_t)(c < 0 ? 0 : c) * 2u;
                    mask[j] = __builtin_amdgcn_raw_buffer_load_b64(rm, off, 0, 0);
                }
            }
        }
        const char* xsb = (const char*)lds + set * C::buf * 16;
        const char* wlb = (const char*)lds + (ONE ? 0 : set * C::wbuf * 16);
        auto products = [&](int p0, int p1) __attribute__((always_inline)) {
#pragma unroll
            for (int p = p0; p < p1; ++p) {
                const uint32_t vb = p <= 8 ? vB0 : p <= 11 ? vB1 : p == 12 ? vB2 : vB3;
                // tap p's halo position
                const int toff = (p / 9) * C::plane + ((p / 3) % 3) * 18 + p % 3;
                bf16x8 av[NSUB], bv[4];
#pragma unroll
                for (int j = 0; j < NSUB; ++j)
                    av[j] = *(const bf16x8*)(wlb + vA + (j * 16 * kCvWRow + p * 32) * 2);
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    bv[m] = *(const bf16x8*)(xsb + vb + (toff + row(m) * 18 + plane(m) * C::plane) * kCvVox * 2);
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int j = 0; j < NSUB; ++j)
                        acc[m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[j], bv[m], acc[m][j],
                                                                            0, 0, 0);
                // (reads of many k steps ahead would spill with three groups' results)
                if constexpr (NSUB == 3) __builtin_amdgcn_sched_barrier(0);
            }
        };
        // With several chunks a brick the next step's copies are issued after
        // the first products, so that the scalar work for them runs beside the
        // matrix cores (48 channels at 64^3 88 -> 86 us); with one, where the
        // stores of every step make memory the bound, before them (16 -> 48
        // channels 73 us, 78 after); not with kUp, which stores less (75 us
        // before, 72 after).
        constexpr int kAhead = ONE && EPI != kUp ? 0 : 2;
        products(0, kAhead);
        int nbk = b, nch = chunk + 1;
        Place on = o;
        if (last) {
            nbk = b + 1;
            nch = 0;
            on = place(nbk);
        }
        if (nbk < b1) issue(on, nch, set ^ 1, !ONE);
        products(kAhead, 14);
        if (last) {
            const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
                a.out + o.smp * sample_out, (short)0, (int)(uint32_t)(sample_out * 2), 0x00020000);
            auto result = [&](int m, int j) __attribute__((always_inline)) {
                bf16x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float t = acc[m][j][i];
                    if constexpr (EPI == kBias || EPI == kBiasPool) t = fmaxf(t + bias[j][i], 0.f);
                    if constexpr (EPI == kMask) {
                        const bf16x4 k = __builtin_bit_cast(bf16x4, mask[m * NSUB + j]);
                        t = (float)k[i] > 0.f ? t : 0.f;
                    }
                    v[i] = (__bf16)t;
                }
                return v;
            };
            auto store = [&](int m, int j, bf16x4 v) __attribute__((always_inline)) {
                const uint32_t off = first + row(m) * row_bytes + plane(m) * plane_bytes + j * 32;
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v), ro, off, 0, 0);
            };
            // a coarse voxel's sum, in the even lanes: the lane's value and its
            // neighbour's in x, tile after tile (y, then z)
            auto add = [&](floatx4& sum, bf16x4 v) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float t = (float)v[i];
                    sum[i] += t;
                    sum[i] += dpp_moved<0xF5, 0xF>(t);  // quad_perm [1, 1, 3, 3]
                }
            };
            auto store_low = [&](bf16x4 v, int c) __attribute__((always_inline)) {
                const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(
                    a.low + o.smp * sample_low, (short)0, (int)(uint32_t)(sample_low * 2), 0x00020000);
                const uint32_t off = first_low + (uint32_t)c * 2u;
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v), rl, off, 0, 0);
            };
            if constexpr (EPI == kBiasPool) {
#pragma unroll
                for (int j = 0; j < NSUB; ++j) {
                    floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const bf16x4 v = result(m, j);
                        store(m, j, v);
                        add(sum, v);
                    }
                    bf16x4 p;
#pragma unroll
                    for (int i = 0; i < 4; ++i) p[i] = (__bf16)(sum[i] * 0.125f);
                    store_low(p, cobase + j * 16);
                }
            } else if constexpr (EPI == kUp) {
#pragma unroll
                for (int j = 0; j < NSUB; ++j) {
                    const int c = cobase + j * 16 - a.split;
                    if (c < 0) {
#pragma unroll
                        for (int m = 0; m < 4; ++m) store(m, j, result(m, j));
                    } else {
                        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int m = 0; m < 4; ++m) add(sum, result(m, j));
                        const bf16x4 k = __builtin_bit_cast(bf16x4, mask[j]);
                        bf16x4 v;
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = (float)k[i] > 0.f ? (__bf16)sum[i] : (__bf16)0.f;
                        store_low(v, c);
                    }
                }
            } else {
#pragma unroll
                for (int m = 0; m < 4; ++m)
#pragma unroll
                    for (int j = 0; j < NSUB; ++j) store(m, j, result(m, j));
            }
            clear();
        }
        stored = last;
        o = on;
        b = nbk;
        chunk = nch;
        set ^= 1;
    }
}

// Forward / input-gradient convolution on grids of 8 cells (3x3x3 taps,
// input channels a multiple of 16, one input tensor), split over the input
// channel groups: a block of 8 waves computes one sample's 8 x 8 x 8 outputs
// (wave w the plane z = w: four 16-voxel tiles of two 8-cell rows) for 16
// output channels from one 16-channel input group and writes FP32 partial
// sums, which k_conv_small_sum adds in a fixed order (with the bias, ReLU and
// mask).  Split this way a 128-channel layer of batch 8 has 512 blocks
// instead of 64.  The 10 x 10 x 10 halo (channels-last, 32 bytes a voxel)
// and the group's weights (in the brick convolution's tap-pair order) are
// copied with direct-to-LDS loads; the pairs' displacements are two planes
// (200 voxels), two rows (20) or two voxels.
constexpr int kSmHaloItems = 2 * 1000;   // 16-byte halo items
constexpr int kSmHaloBuf = 32 * 64;      // whole waves of items

__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(6)))
k_conv_small(ConvArgs a, float* __restrict__ part) {
    constexpr int kThreads = 512;
    constexpr int kWItems = 16 * kCvWItemsRow;
    constexpr int kWBuf = (kWItems + 63) / 64 * 64;
    __shared__ __attribute__((aligned(16))) __bf16 xs[kSmHaloBuf * 8];
    __shared__ __attribute__((aligned(16))) __bf16 wl[kWBuf * 8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, q = lane >> 4, hi = q >> 1;
    const int nch = a.cin / 16;
    const int smp = blockIdx.x / nch, chunk = blockIdx.x % nch;
    const int c0 = chunk * 16;
    const int cobase = blockIdx.y * 16;
    const int ch = (q & 1) * 8;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    // halo item t (voxel t / 2 of 10 x 10 x 10, channel half t % 2) -> LDS byte 16 t;
    // positions outside the grid, channel halves past cin and the padding items read zeros
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(a.x1 + (int64_t)smp * 512 * a.c1s), (short)0, 512 * a.c1s * 2,
        0x00020000);
#pragma unroll
    for (int i = 0; i < kSmHaloBuf / kThreads; ++i) {
        const int tb = i * kThreads + wv * 64;
        const int t = tb + lane;
        const int half = t & 1, hv = t >> 1;
        const int xx = hv % 10 - 1, yy = (hv / 10) % 10 - 1, zz = hv / 100 - 1;
        const bool ok = t < kSmHaloItems && c0 + half * 8 < a.cin && (unsigned)xx < 8u &&
                        (unsigned)yy < 8u && (unsigned)zz < 8u;
        const uint32_t vox = ((uint32_t)zz << 6) + ((uint32_t)yy << 3) + (uint32_t)xx;
        const uint32_t off = ((vox * (uint32_t)a.c1s + (uint32_t)(c0 + half * 8)) * 2u) |
                             ((uint32_t)!ok << 31);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_ptr)&xs[tb * 8], 16, off, 0, 0, 0);
    }
    // weight item t: row t / 58 (output channel cobase + row), tap-pair slot
    // (t % 58) / 2, channel half t % 2; items 56, 57 of a row pad
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<__bf16*>(a.w), (short)0, (int)(uint32_t)((int64_t)a.wrows * a.kpad * 2), 0x00020000);
#pragma unroll
    for (int i = 0; i < (kWBuf + kThreads - 1) / kThreads; ++i) {
        const int tb = i * kThreads + wv * 64;
        if (tb >= kWBuf) continue;
        const int t = tb + lane;
        const int row = t / kCvWItemsRow, rem = t - row * kCvWItemsRow;
        const int slot = rem >> 1, half = rem & 1, p = slot >> 1;
        const int tap = (slot & 1) ? cv_pair_tap(p) : p;
        const bool ok = t < kWItems && rem < 2 * kCvSlots && tap >= 0 && cobase + row < a.wrows;
        const uint32_t off =
            ((uint32_t)((cobase + row) * a.kpad + tap * a.cin + c0 + half * 8) * 2u) |
            ((uint32_t)!ok << 31);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void_ptr)&wl[tb * 8], 16, off, 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));  // vmcnt 0: this wave's copies landed
    __syncthreads();
    // lane r of tile m is the output voxel (z = w, y = 2 m + r / 8, x = r % 8)
    const uint32_t lb = (uint32_t)(wave * 100 + (r >> 3) * 10 + (r & 7));
    const uint32_t vA0 = ((lb + hi * 200) * kCvVox + ch) * 2;
    const uint32_t vA1 = ((lb + hi * 20) * kCvVox + ch) * 2;
    const uint32_t vA2 = ((lb + hi * 2) * kCvVox + ch) * 2;
    const uint32_t vA3 = (lb * kCvVox + ch) * 2;
    const uint32_t vB = (uint32_t)(r * kCvWRow + hi * 16 + ch) * 2;
    const char* xsb = (const char*)xs;
    const char* wlb = (const char*)wl;
    floatx4 acc[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < 14; ++p) {
        const uint32_t va = p <= 8 ? vA0 : p <= 11 ? vA1 : p == 12 ? vA2 : vA3;
        const int toff = (p / 9) * 100 + ((p / 3) % 3) * 10 + p % 3;  // halo position of tap p
        const bf16x8 bv = *(const bf16x8*)(wlb + vB + p * 64);
        bf16x8 av[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) av[m] = *(const bf16x8*)(xsb + va + (toff + m * 20) * kCvVox * 2);
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bv, av[m], acc[m], 0, 0, 0);
    }
    // D rows 4q .. 4q+3 of tile m are output channels, column r the plane's voxel 16 m + r
    const int Cp = gridDim.y * 16;
    float* pp = part + ((int64_t)chunk * a.n + smp) * 512 * Cp;
#pragma unroll
    for (int m = 0; m < 4; ++m)
        *(floatx4*)(pp + (int64_t)(wave * 64 + 16 * m + r) * Cp + cobase + 4 * q) = acc[m];
}

// out[v][co] = (ReLU)(bias + sum over the nch input groups of the partials,
// in group order), 0 where omask <= 0 and for co >= cout; one thread per output.
__global__ void k_conv_small_sum(const float* __restrict__ part, int nch, int64_t cells, int Cp,
                                 const float* __restrict__ bias, int relu,
                                 const __bf16* __restrict__ omask, int cout, int ys,
                                 __bf16* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= cells * ys) return;
    const int64_t v = i / ys;
    const int co = (int)(i - v * ys);
    float val = 0.f;
    if (co < cout) {
        float sum = 0.f;
        for (int c = 0; c < nch; ++c) sum += part[((int64_t)c * cells + v) * Cp + co];
        val = sum + (bias ? bias[co] : 0.f);
        if (relu) val = fmaxf(val, 0.f);
        if (omask && !((float)omask[i] > 0.f)) val = 0.f;
    }
    out[i] = (__bf16)val;
}

// Partial-sum floats k_conv_small needs for the convolution a describes
// (coutp output rows), or 0 if it does not apply.
int64_t conv_small_floats(const ConvArgs& a, int coutp) {
    if (a.lg != 3 || a.taps != 27 || a.c2 != 0 || a.cin % 16 != 0 || a.kpad < 27 * a.cin)
        return 0;
    return (int64_t)(a.cin / 16) * a.n * 512 * coutp;
}

// Output groups a wave: one while the waves are few (each is then a short
// chain with eight steps in flight), more where the blocks already fill the
// chip and a voxel fragment should serve several groups.
template <int KS>
hipError_t launch_conv_ks(const ConvArgs& a, int coutp, hipStream_t s) {
    const int64_t tiles = ceil_div((int64_t)a.n << (3 * a.lg), 16);
    const int sub = coutp / 16;
    const int64_t waves = tiles * sub * KS;
    const int nsub = waves > 2048 && sub % 4 == 0 ? 4 : waves > 1024 && sub % 2 == 0 ? 2 : 1;
    const int64_t M = (int64_t)a.n << (3 * a.lg);
    const bool wide = a.cin % 32 == 0 && a.c1s % 32 == 0 && a.K == a.kpad &&
                      M * std::max(a.c1s, a.c2) * 2 < ((int64_t)1 << 31);
    const dim3 grid((unsigned)tiles, sub / nsub), block(64 * KS);
#define LBMNN_CONV(N)                                                                        \
    if (wide)                                                                                \
        hipLaunchKernelGGL((k_conv<N, KS, true>), grid, block, 0, s, a);                     \
    else                                                                                     \
        hipLaunchKernelGGL((k_conv<N, KS, false>), grid, block, 0, s, a)
    switch (nsub) {
        case 4: LBMNN_CONV(4); break;
        case 2: LBMNN_CONV(2); break;
        default: LBMNN_CONV(1); break;
    }
#undef LBMNN_CONV
    return hipGetLastError();
}

// Bricks of 8 rows (1024 threads) when they give every compute unit one, else
// of 4 rows; about one block per compute unit (its LDS holds one), each
// walking the same number of bricks.
template <int NSUB, int WY, bool ONE>
hipError_t launch_conv_wy(const ConvArgs& a, int groups, int64_t bricks, hipStream_t s) {
    const int64_t most = std::max<int64_t>(1, compute_units() / groups);
    const int64_t per = (bricks + most - 1) / most;
    const dim3 grid((unsigned)((bricks + per - 1) / per), groups), block(64 * kCvPlanes * WY);
    const int w = (int)bricks, p = (int)per;
    if (a.low && !a.bias) {
        hipLaunchKernelGGL((k_conv_brick<NSUB, WY, ONE, kUp>), grid, block, 0, s, a, w, p);
    } else if constexpr (NSUB < 3) {
        if (a.low)
            hipLaunchKernelGGL((k_conv_brick<NSUB, WY, ONE, kBiasPool>), grid, block, 0, s, a, w, p);
        else if (a.omask)
            hipLaunchKernelGGL((k_conv_brick<NSUB, WY, ONE, kMask>), grid, block, 0, s, a, w, p);
        else if (a.bias)
            hipLaunchKernelGGL((k_conv_brick<NSUB, WY, ONE, kBias>), grid, block, 0, s, a, w, p);
        else if constexpr (!ONE)
            hipLaunchKernelGGL((k_conv_brick<NSUB, WY, ONE, kPlain>), grid, block, 0, s, a, w, p);
        else  // (every layer of at most 16 output channels masks its input gradient)
            return hipErrorInvalidValue;
    } else {  // (three groups: launch_conv_brick)
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Whether the brick kernel covers the convolution.  (8 input channels, the
// first layer, take a 16-channel group whose upper half reads zeros; its
// weight rows there hold the next tap's weights, which multiply those zeros,
// and stay inside the row since 27 * 8 + 8 <= kpad.)
bool conv_brick_covers(const ConvArgs& a, int coutp) {
    return a.taps == 27 && a.lg >= 4 && a.kpad >= 27 * a.cin &&
           (a.cin % 16 == 0 || (a.cin == 8 && a.c2 == 0)) && (a.c2 == 0 || a.c1s % 16 == 0) &&
           a.cout == coutp && a.ys == coutp && !(a.omask && a.bias) && !a.bias == !a.relu;
}

hipError_t launch_conv_brick(const ConvArgs& args, int coutp, hipStream_t s) {
    ConvArgs a = args;
    a.wrows = coutp;
    const int sub = coutp / 16;
    const bool up = a.low && !a.bias;
    const int64_t G = (int64_t)1 << a.lg, tall = a.n * (G / 16) * (G / 8) * (G / kCvPlanes);
    if (a.cin <= 16) {
        // three output groups share a step's halo in the gradients of
        // concatenated inputs (48, 96, 192 channels)
        if (up && sub % 3 == 0 && tall * (sub / 3) >= compute_units())
            return launch_conv_wy<3, 2, true>(a, sub / 3, tall, s);
        if (tall * sub >= compute_units()) return launch_conv_wy<1, 2, true>(a, sub, tall, s);
        return launch_conv_wy<1, 1, true>(a, sub, 2 * tall, s);
    }
    if (up && sub % 3 == 0 && 2 * tall * (sub / 3) >= compute_units())
        return launch_conv_wy<3, 1, false>(a, sub / 3, 2 * tall, s);
    if (tall * sub >= compute_units()) return launch_conv_wy<1, 2, false>(a, sub, tall, s);
    return launch_conv_wy<1, 1, false>(a, sub, 2 * tall, s);
}

// The tiled kernel's k range is split over 2 or 4 waves per block when there
// are fewer than 4096 or 1024 (voxel tile, up to four output groups) pairs and
// at least two steps of 32 per wave (8 waves were measured no faster on the
// 8^3 layers).
hipError_t launch_conv(const ConvArgs& a, int coutp, float* scratch, int64_t scratch_floats,
                       hipStream_t s) {
    const int64_t M = (int64_t)a.n << (3 * a.lg);
    const int sub = coutp / 16;
    const int64_t small = conv_small_floats(a, coutp);
    if (small > 0 && scratch && small <= scratch_floats) {
        // grids of 8 cells: split over the input channel groups, then summed
        ConvArgs b = a;
        b.wrows = coutp;
        hipLaunchKernelGGL(k_conv_small, dim3(a.n * (a.cin / 16), sub), dim3(512), 0, s, b, scratch);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const int64_t outs = M * a.ys;
        hipLaunchKernelGGL(k_conv_small_sum, dim3((unsigned)ceil_div(outs, 256)), dim3(256), 0, s,
                           scratch, a.cin / 16, M, coutp, a.bias, a.relu, a.omask, a.cout, a.ys,
                           a.out);
        return hipGetLastError();
    }
    if (conv_brick_covers(a, coutp)) return launch_conv_brick(a, coutp, s);
    const int nsub = sub % 4 == 0 ? 4 : sub % 3 == 0 ? 3 : sub % 2 == 0 ? 2 : 1;
    const int64_t waves1 = (int64_t)ceil_div(M, 16) * (sub / nsub);
    const int ksteps = a.kpad / 32;
    if (waves1 < 1024 && ksteps >= 8) return launch_conv_ks<4>(a, coutp, s);
    if (waves1 < 4096 && ksteps >= 4) return launch_conv_ks<2>(a, coutp, s);
    return launch_conv_ks<1>(a, coutp, s);
}

}  // namespace

hipError_t pack_weights(int layers, const ConvGeom* g, const float* theta, const int64_t* woff,
                        __bf16* const* wp, __bf16* const* wt, hipStream_t s) {
    if (layers < 1 || layers > kMaxPackLayers) return hipErrorInvalidValue;
    PackTable t;
    int64_t blocks = 0;
    for (int l = 0; l < kMaxPackLayers; ++l) {
        PackLayer& L = t.l[l];
        if (l >= layers) {
            L = PackLayer{};
            t.blk[2 * l] = t.blk[2 * l + 1] = blocks;
            continue;
        }
        L.wp = wp[l];
        L.wt = wt[l];
        L.woff = woff[l];
        L.coutp = g[l].coutp;
        L.kpad = g[l].kpad;
        L.cout = g[l].cout;
        L.K = g[l].K;
        L.cin = g[l].cin;
        L.c1 = g[l].c1;
        L.c1s = g[l].c1s;
        L.taps = g[l].taps;
        L.cin_real = g[l].c1 + g[l].c2;
        L.cinp = g[l].cinp;
        L.kpad_t = g[l].kpad_t;
        L.ys = g[l].ys;
        blocks += ceil_div((int64_t)L.coutp * L.kpad, 256 * 8);
        t.blk[2 * l] = blocks;
        // (kpad is a multiple of 8, cinp of kWtTileCi, kpad_t of 4)
        if (L.kpad % 8 || L.cinp % kWtTileCi || L.kpad_t % 4) return hipErrorInvalidValue;
        blocks += (int64_t)(L.cinp / kWtTileCi) * ceil_div((int64_t)L.kpad_t, kWtTileK);
        t.blk[2 * l + 1] = blocks;
    }
    hipLaunchKernelGGL(k_pack_all, dim3((unsigned)blocks), dim3(256), 0, s, t, theta);
    return hipGetLastError();
}

hipError_t conv_forward(const ConvGeom& g, const __bf16* x1, const __bf16* x2, const __bf16* wp,
                        const float* bias, int relu, __bf16* out, __bf16* pool, float* scratch,
                        int64_t scratch_floats, hipStream_t s) {
    if (!x1 || !wp || !out || (g.c2 > 0 && (!x2 || g.lg < 1)) || g.c1s % 8 || g.c2 % 8)
        return hipErrorInvalidValue;
    ConvArgs a;
    a.x1 = x1;
    a.x2 = x2;
    a.w = wp;
    a.bias = bias;
    a.out = out;
    a.omask = nullptr;
    a.n = g.n;
    a.lg = g.lg;
    a.taps = g.taps;
    a.c1s = g.c1s;
    a.c2 = g.c2;
    a.cin = g.cin;
    a.K = g.K;
    a.kpad = g.kpad;
    a.cout = g.cout;
    a.ys = g.ys;
    a.relu = relu;
    if (pool && conv_brick_covers(a, g.coutp)) {
        a.low = pool;
        pool = nullptr;
    }
    const hipError_t e = launch_conv(a, g.coutp, scratch, scratch_floats, s);
    return e == hipSuccess && pool ? pool_forward(g.n, g.lg, g.ys, out, pool, s) : e;
}

namespace {

ConvArgs backward_args(const ConvGeom& g, const __bf16* dy, const __bf16* wt, const __bf16* dxmask,
                       __bf16* dx) {
    ConvArgs a;
    a.x1 = dy;
    a.x2 = nullptr;
    a.w = wt;
    a.bias = nullptr;
    a.out = dx;
    a.omask = dxmask;
    a.n = g.n;
    a.lg = g.lg;
    a.taps = g.taps;
    a.c1s = g.ys;
    a.c2 = 0;
    a.cin = g.ys;
    a.K = g.taps * g.ys;
    a.kpad = g.kpad_t;
    a.cout = g.cin;
    a.ys = g.cin;
    a.relu = 0;
    return a;
}

// Whether the brick kernel sums the upsampled channels' gradients itself.
bool concat_fused(const ConvGeom& g) {
    return g.c1s % 16 == 0 && conv_brick_covers(backward_args(g, nullptr, nullptr, nullptr, nullptr), g.cinp);
}

}  // namespace

hipError_t conv_backward_data(const ConvGeom& g, const __bf16* dy, const __bf16* wt,
                              const __bf16* dxmask, __bf16* dx, float* scratch,
                              int64_t scratch_floats, hipStream_t s) {
    if (!dy || !wt || !dx) return hipErrorInvalidValue;
    return launch_conv(backward_args(g, dy, wt, dxmask, dx), g.cinp, scratch, scratch_floats, s);
}

int concat_skip_channels(const ConvGeom& g) { return concat_fused(g) ? g.c1s : g.cin; }

hipError_t conv_backward_concat(const ConvGeom& g, const __bf16* dy, const __bf16* wt,
                                const __bf16* upmask, __bf16* dcat, __bf16* dup, float* scratch,
                                int64_t scratch_floats, hipStream_t s) {
    if (!dy || !wt || !upmask || !dcat || !dup || g.c2 < 1) return hipErrorInvalidValue;
    ConvArgs a = backward_args(g, dy, wt, nullptr, dcat);
    if (concat_fused(g)) {
        a.low = dup;
        a.lowmask = upmask;
        a.split = a.ys = g.c1s;
        return launch_conv_brick(a, g.cinp, s);
    }
    const hipError_t e = launch_conv(a, g.cinp, scratch, scratch_floats, s);
    if (e != hipSuccess) return e;
    return upsample_backward(g.n, g.lg, g.c2, dcat, g.cin, g.c1s, upmask, dup, s);
}

int64_t conv_scratch_floats(const ConvGeom& g) {
    ConvArgs f = {};
    f.n = g.n, f.lg = g.lg, f.taps = g.taps, f.c2 = g.c2, f.cin = g.cin, f.kpad = g.kpad;
    ConvArgs b = f;
    b.c2 = 0, b.cin = g.ys, b.kpad = g.kpad_t;
    return std::max(conv_small_floats(f, g.coutp), conv_small_floats(b, g.cinp));
}

namespace {

// First reduction pass over the partials of plan p, when they have more
// than 2 kRowSlice rows (more than the second pass's lane groups read
// quickly).
// Returns the arguments of the second pass: the partials, or their slice
// sums with rows replaced by slices.
hipError_t sum_slices(const WgradPlan& p, const WgradArgs& a, WgradArgs* b, int64_t* rows,
                      hipStream_t s) {
    *b = a;
    *rows = p.rows;
    if (!p.slices) return hipSuccess;
    const int64_t sl = (p.rows + kRowSlice - 1) / kRowSlice;
    float* out = a.part + p.part_floats;
    hipLaunchKernelGGL(k_sum_row_slices, dim3(ceil_div(sl * (p.wwidth + p.bwidth), 256)),
                       dim3(256), 0, s, (const float*)a.part, p.bias_off, p.rows, p.wwidth,
                       p.bwidth, out);
    b->part = out;
    b->bias_off = sl * p.wwidth;
    *rows = sl;
    return hipGetLastError();
}

}  // namespace

// Blocks of k_wgrad_tr for one generation on the current device: the compute
// units times the blocks each holds at once (one: the ring of halo planes takes
// 140 KB of LDS; at most 2 if that ever shrinks, since fewer blocks each walking
// more bricks share halo cells and output rows in L2).  512 if the runtime
// cannot say.  Asked once per device; an answer it did not give is not kept.
WgradBlocks wgrad_blocks() {
    static std::atomic<int64_t> known[64][2];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return {512, 512};
    int64_t blocks[2];
    for (int two = 0; two < 2; ++two) {
        blocks[two] = known[dev][two].load(std::memory_order_relaxed);
        if (blocks[two] > 0) continue;
        int cus = 0, per = 0;
        hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = two ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_wgrad_tr<2>, 64 * kWgWaves, 0)
                    : hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_wgrad_tr<1>, 64 * kWgWaves, 0);
        if (e != hipSuccess || cus <= 0 || per <= 0) return {512, 512};
        blocks[two] = (int64_t)cus * std::min(per, 2);
        known[dev][two].store(blocks[two], std::memory_order_relaxed);
    }
    return {blocks[0], blocks[1]};
}

// One pass over a brick or 8-cell partial table (rows x W weight entries,
// then the bias rows).
hipError_t launch_partials_sum(const WgradArgs& a, int chunks, int rows, int rs, float* dw,
                               float* db, hipStream_t s) {
    const int64_t W = (int64_t)27 * rs * 16 * 16 * chunks;
    auto blocks = [&](int ent) { return ceil_div(W, ent) + ceil_div(a.cout, ent); };
    if (W >= ((int64_t)1 << 31) || blocks(32) * 32 >= ((int64_t)1 << 31))
        return hipErrorInvalidValue;  // 32-bit entry index
    if (rows <= kPsShortRows)
        hipLaunchKernelGGL((k_brick_partials_sum<1, 256>), dim3((unsigned)blocks(256)), dim3(256), 0,
                           s, a, chunks, rows, rs, dw, db);
    else if (rows >= kPsTallRows && blocks(32) < kPsFewBlocks)
        hipLaunchKernelGGL((k_brick_partials_sum<32, 32>), dim3((unsigned)blocks(32)), dim3(1024), 0,
                           s, a, chunks, rows, rs, dw, db);
    else
        hipLaunchKernelGGL((k_brick_partials_sum<8, 32>), dim3((unsigned)blocks(32)), dim3(256), 0,
                           s, a, chunks, rows, rs, dw, db);
    return hipGetLastError();
}

hipError_t conv_backward_weight(const ConvGeom& g, const __bf16* x1, const __bf16* x2,
                                const __bf16* dy, const __bf16* y, int relu, float* dw,
                                float* db, const WgradBlocks& resident, float* scratch,
                                int64_t scratch_floats, hipStream_t s) {
    if (!x1 || !dy || !dw || !db || !scratch || (relu && !y) || (g.c2 > 0 && (!x2 || g.lg < 1)))
        return hipErrorInvalidValue;
    const WgradPlan p = wgrad_plan(g, relu, resident);
    if (p.scratch_floats > scratch_floats) return hipErrorInvalidValue;
    WgradArgs a;
    a.x1 = x1;
    a.x2 = x2;
    a.dy = dy;
    a.y = y;
    a.part = scratch;
    a.bias_off = p.bias_off;
    a.n = g.n;
    a.lg = g.lg;
    a.taps = g.taps;
    a.c1 = g.c1;
    a.c1s = g.c1s;
    a.c2 = g.c2;
    a.cin = g.cin;
    a.K = g.K;
    a.cout = g.cout;
    a.coutp = g.coutp;
    a.ys = g.ys;
    a.relu = relu;
    a.cin_real = g.c1 + g.c2;
    a.vchunk = p.vchunk;
    if (p.small) {
        hipLaunchKernelGGL(k_wgrad_small, dim3(p.chunks, g.n, g.coutp / 32), dim3(64 * kWtWaves), 0,
                           s, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_partials_sum(a, p.chunks, p.groups, p.rs, dw, db, s);
    }
    if (p.brick) {
        const dim3 grid(p.chunks, p.groups, p.rs == 4 ? 2 : 1), block(64 * kWgWaves);
        if (p.rs == 1)
            hipLaunchKernelGGL(k_wgrad_tr<1>, grid, block, 0, s, a, p.per);
        else
            hipLaunchKernelGGL(k_wgrad_tr<2>, grid, block, 0, s, a, p.per);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_partials_sum(a, p.chunks, p.groups, p.rs, dw, db, s);
    }
    const dim3 grid(p.kt, p.ct, p.nz);
    switch (p.rs) {
        case 4: hipLaunchKernelGGL(k_wgrad<4>, grid, dim3(256), 0, s, a); break;
        case 2: hipLaunchKernelGGL(k_wgrad<2>, grid, dim3(256), 0, s, a); break;
        default: hipLaunchKernelGGL(k_wgrad<1>, grid, dim3(256), 0, s, a); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    WgradArgs b;
    int64_t rows = 0;
    e = sum_slices(p, a, &b, &rows, s);
    if (e != hipSuccess) return e;
    const int64_t nred = (int64_t)p.ct * p.rs * 16 * p.kt * p.cs * 16 + g.cout;
    if (nred * 8 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;  // 32-bit lane index
    if (rows >= kRedManyRows)
        hipLaunchKernelGGL(k_wgrad_reduce<8>, dim3(ceil_div(nred * 8, 256)), dim3(256), 0, s, b,
                           p.kt, p.ct, (int)rows, p.rs, p.cs, dw, db);
    else
        hipLaunchKernelGGL(k_wgrad_reduce<1>, dim3(ceil_div(nred, 256)), dim3(256), 0, s, b, p.kt,
                           p.ct, (int)rows, p.rs, p.cs, dw, db);
    return hipGetLastError();
}

hipError_t pool_forward(int n, int lg, int c, const __bf16* x, __bf16* y, hipStream_t s) {
    if (lg < 1 || c % 8 || !x || !y) return hipErrorInvalidValue;
    const int64_t t = ((int64_t)n << (3 * (lg - 1))) * (c / 8);
    hipLaunchKernelGGL(k_pool, dim3(ceil_div(t, 256)), dim3(256), 0, s, n, lg, c, x, y);
    return hipGetLastError();
}

hipError_t pool_backward_add(int n, int lg, int c, const __bf16* dy, const __bf16* skip, int ctot,
                             const __bf16* ymask, __bf16* dx, hipStream_t s) {
    if (lg < 1 || c % 8 || !dy || !dx || (skip && (ctot < c || ctot % 8))) return hipErrorInvalidValue;
    const int64_t t = ((int64_t)n << (3 * lg)) * (c / 8);
    hipLaunchKernelGGL(k_pool_bwd_add, dim3(ceil_div(t, 256)), dim3(256), 0, s, n, lg, c, dy, skip,
                       ctot, ymask, dx);
    return hipGetLastError();
}

hipError_t upsample_backward(int n, int lg, int c, const __bf16* dcat, int ctot, int coff,
                             const __bf16* ymask, __bf16* dlow, hipStream_t s) {
    if (lg < 1 || c % 8 || coff % 8 || coff + c > ctot || !dcat || !dlow)
        return hipErrorInvalidValue;
    const int64_t t = ((int64_t)n << (3 * (lg - 1))) * (c / 8);
    hipLaunchKernelGGL(k_up_bwd, dim3(ceil_div(t, 256)), dim3(256), 0, s, n, lg, c, dcat, ctot, coff,
                       ymask, dlow);
    return hipGetLastError();
}

hipError_t make_inputs(int n, int lg, const float* log10_ra, __bf16* x, hipStream_t s) {
    if (n < 1 || n > kMaxBatch || !log10_ra || !x) return hipErrorInvalidValue;
    SampleFloats lra;
    for (int i = 0; i < kMaxBatch; ++i) lra.v[i] = i < n ? log10_ra[i] : 0.f;
    const int64_t t = (int64_t)n << (3 * lg);
    hipLaunchKernelGGL(k_inputs, dim3(ceil_div(t, 256)), dim3(256), 0, s, n, lg, lra, x);
    return hipGetLastError();
}

bool head_geometry(const ConvGeom& g) {
    return g.taps == 1 && g.c1 == kHeadIn && g.c1s == kHeadIn && g.c2 == 0 && g.cout == kHeadOut;
}

hipError_t head_forward(const ConvGeom& g, const __bf16* x, const float* w, const float* b,
                        const float* scale4, float* out, hipStream_t s) {
    if (!head_geometry(g) || !x || !w || !b || !out) return hipErrorInvalidValue;
    const float4 sc = scale4 ? make_float4(scale4[0], scale4[1], scale4[2], scale4[3])
                             : make_float4(1.f, 1.f, 1.f, 1.f);
    const int64_t M = (int64_t)g.n << (3 * g.lg);
    hipLaunchKernelGGL(k_head_forward, dim3(ceil_div(M, 256)), dim3(256), 0, s, g.n, g.lg, x, w, b,
                       sc, out);
    return hipGetLastError();
}

int head_backward_blocks(const ConvGeom& g) {
    const int64_t M = (int64_t)g.n << (3 * g.lg);
    return (int)std::min<int64_t>(kHeadBlocks, ceil_div(M, 512));
}

int64_t head_scratch_floats(const ConvGeom& g) {
    return (int64_t)head_backward_blocks(g) * kHeadGrad;
}

hipError_t head_backward(const ConvGeom& g, const float* targets, const int32_t* idx,
                         int64_t stride, const float* tscale4, const __bf16* x, const float* w,
                         const float* b, __bf16* dx, float* grad, float* scratch,
                         double* lpartial, double* loss, hipStream_t s) {
    if (!head_geometry(g) || g.n < 1 || g.n > kMaxBatch || !targets || !idx || !x || !w || !b ||
        !dx || !grad || !scratch || !lpartial || !loss)
        return hipErrorInvalidValue;
    SampleInts ix;
    for (int i = 0; i < kMaxBatch; ++i) ix.v[i] = i < g.n ? idx[i] : 0;
    const int64_t M = (int64_t)g.n << (3 * g.lg);
    const int nb = head_backward_blocks(g);
    const int64_t chunk = (int64_t)ceil_div(M, (int64_t)nb * 256) * 256;
    const float4 ts = make_float4(tscale4[0], tscale4[1], tscale4[2], tscale4[3]);
    hipLaunchKernelGGL(k_head_backward, dim3(nb), dim3(256), 0, s, g.n, g.lg, targets, ix, stride,
                       ts, x, w, b, chunk, dx, lpartial, scratch);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_head_sums, dim3(kHeadGrad + 1), dim3(256), 0, s, (const float*)scratch,
                       nb, kHeadGrad, grad, (const double*)lpartial, loss);
    return hipGetLastError();
}

hipError_t adam_update(int64_t count, float* theta, float* m, float* v, const float* g, int t,
                       float lr, float beta1, float beta2, float eps, hipStream_t s) {
    const float c1 = 1.f - powf(beta1, (float)t), c2 = 1.f - powf(beta2, (float)t);
    hipLaunchKernelGGL(k_adam, dim3(ceil_div(count, 256)), dim3(256), 0, s, count, theta, m, v, g,
                       lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t fill_zero_f32(float* p, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero, dim3(ceil_div(count, 256)), dim3(256), 0, s, p, count);
    return hipGetLastError();
}

hipError_t bf16_to_f32(const __bf16* x, int64_t cells, int cs, int c, float* y, hipStream_t s) {
    const int64_t t = cells * c;
    hipLaunchKernelGGL(k_bf16_to_f32, dim3(ceil_div(t, 256)), dim3(256), 0, s, x, cells, cs, c, y);
    return hipGetLastError();
}

hipError_t cf_to_cl(const float* x, int n, int64_t v, int c, float* y, hipStream_t s) {
    const int64_t t = (int64_t)n * v * c;
    hipLaunchKernelGGL(k_cf_to_cl, dim3(ceil_div(t, 256)), dim3(256), 0, s, x, n, v, c, y);
    return hipGetLastError();
}

}  // namespace lbmnn
