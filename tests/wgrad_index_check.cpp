// CPU check of the weight gradient's copies and LDS reads (nn_wgrad_index.hpp,
// the functions k_wgrad_tr runs): replays every block of a launch on a model of
// LDS.  Every copy must come from inside its sample and go to a slot or buffer
// the current brick does not use, and every lane of every product wave must
// read the voxel and channels its place in the product asks for, zeros outside
// the grid and the channels.
//
// Usage: wgrad_index_check groups grid samples per c1s c2 ys
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1710_04751_amd/csrc/nn_wgrad_index.hpp"

using namespace lbmnn;

struct Item {  // 8 channels from c of a voxel of a sample; kind 0: never written, 1: zeros
    int kind = 0, smp = 0, z = 0, y = 0, x = 0, c = 0;
    bool operator==(const Item& o) const {
        return kind == o.kind && (kind < 2 || (smp == o.smp && z == o.z && y == o.y && x == o.x && c == o.c));
    }
};
constexpr int kZero = 1, kHalo = 2, kDy = 3;

void fail(const char* what, int b, int wave, int lane) {
    std::printf("FAIL %s: brick %d wave %d lane %d\n", what, b, wave, lane);
    std::exit(1);
}

Item source(int kind, uint32_t off, int smp, int lg, int chans) {
    Item i;
    i.kind = kZero;
    if (off >= kWgOutside) return i;
    const uint32_t v = off / 2 / chans;
    if (off % 16 || v >= 1u << (3 * lg)) fail("source outside the sample", smp, 0, 0);
    const int m = (1 << lg) - 1;
    return Item{kind, smp, (int)(v >> (2 * lg)), (int)(v >> lg) & m, (int)v & m, (int)(off / 2 % chans)};
}

template <int RS>
long replay(int lg, int n, int per, int c1s, int c2, int ys) {
    using W = WgShape<RS>;
    const int nbricks = n << (3 * lg - 8), cin = c1s + c2, G = 1 << lg;
    long reads = 0;
    for (int co0 = 0; co0 < ys; co0 += 16 * RS)
        for (int c0 = 0; c0 < cin; c0 += 16)
            for (int b0 = 0; b0 < nbricks; b0 += per) {
                const int b1 = std::min(b0 + per, nbricks);
                const bool lo = c0 < c1s;
                const int chans = lo ? c1s : c2, cloc = lo ? c0 : c0 - c1s, lgx = lo ? lg : lg - 1;
                std::vector<Item> lds(W::lds_items);
                WgAhead<RS> at(b0);
                int bslot = 0, bbuf = 0;
                auto issue = [&](int cur, int b, int p0, int to, int buf) {
                    const WgBrick o = wg_brick(b, lg);
                    for (int copier = 0; copier < 2; ++copier)
                        for (int p = p0; p < 6; ++p) {
                            const int slot = W::slot(to + p - p0), zz = o.z0 - 1 + p;
                            for (int k = 0; k < 6; ++k)
                                if (cur >= b0 && slot == W::slot(bslot + k)) fail("slot in use", b, copier, p);
                            for (int i = 0; i < 2; ++i)
                                for (int lane = 0; lane < 64; ++lane) {
                                    const int t = copier * 128 + i * 64 + lane;
                                    const uint32_t off = wg_halo_offset(
                                        wg_halo_item(t, lo, lg, chans, cloc, c0 + 8 < cin),
                                        wg_sides(o, lg) | wg_plane_sides(zz, lg),
                                        wg_plane_first(o, zz, lo, lg, chans));
                                    lds.at(slot * kWtPlaneItems + t) = source(kHalo, off, o.smp, lgx, chans);
                                }
                        }
                    if (cur >= b0 && buf == bbuf) fail("buffer in use", b, 0, 0);
                    for (int t = 0; t < W::dy_buf; ++t)
                        lds.at(W::halo + buf * W::dy_buf + t) = source(
                            kDy, wg_dy_item<RS>(t, lg, ys, co0) + wg_dy_first(o, lg, ys), o.smp, lg, ys);
                };
                for (int b = b0; b < b1; ++b) {
                    auto fill = [&](int cur) {
                        for (;;) {
                            const bool f = wg_follows(at.next, b0, lg);
                            if (!at.can(b, b1, f ? 4 : 6)) break;
                            issue(cur, at.next, f ? 2 : 0, at.wslot, at.wbuf);
                            at.copied(f ? 4 : 6);
                        }
                    };
                    if (b == b0) fill(-1);
                    if (at.next <= b) fail("not copied in time", b, 0, 0);
                    if (b > b0) fill(b);
                    const WgBrick o = wg_brick(b, lg);
                    auto check = [&](uint32_t byte, Item want, int ac, int wave, int lane) {
                        if (byte % 8 || byte / 16 >= (uint32_t)W::lds_items) fail("address", b, wave, lane);
                        if ((byte % 16) / 8 != (uint32_t)(ac & 1)) fail("channel half", b, wave, lane);
                        if (!(lds[byte / 16] == want)) fail("value", b, wave, lane);
                        ++reads;
                    };
                    for (int wave = 0; wave < 12; ++wave)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int dyw = wave % 3, plane = wave / 3, r = lane & 15, q = lane >> 4;
                            const int e = r >> 2, ac = r & 3;
                            const uint32_t la = wg_lane_dy<RS>(lane, plane) + bbuf * W::dy_buf * 16;
                            for (int rp = 0; rp < 2; ++rp) {
                                for (int m = 0; m < RS; ++m)
                                    for (int i = 0; i < 2; ++i) {
                                        const int co = co0 + m * 16 + ac / 2 * 8;
                                        Item want{kDy, o.smp, o.z0 + plane, o.y0 + 2 * rp + (q & 1),
                                                  o.x0 + 8 * (q >> 1) + 4 * i + e, co};
                                        if (co >= ys) want = Item{kZero};
                                        check(la + wg_dy_read<RS>(rp, m, i), want, ac, wave, lane);
                                    }
                                for (int z = 0; z < 3; ++z)
                                    for (int i = 0; i < 3; ++i) {
                                        const int hx = 8 * (q >> 1) + 4 * i + e, x = o.x0 - 1 + hx;
                                        const int y = o.y0 - 1 + 2 * rp + (q & 1) + dyw;
                                        const int zz = o.z0 - 1 + plane + z, half = ac / 2;
                                        const int sh = lo ? 0 : 1;
                                        Item want{kHalo, o.smp, zz >> sh, y >> sh, x >> sh, cloc + half * 8};
                                        if (hx >= 18 || x < 0 || x >= G || y < 0 || y >= G || zz < 0 || zz >= G ||
                                            c0 + half * 8 >= cin)
                                            want = Item{kZero};
                                        check(wg_lane_halo(lane, dyw) + wg_halo_read(rp, i) +
                                                  W::slot(bslot + plane + z) * kWtPlaneItems * 16,
                                              want, ac, wave, lane);
                                    }
                            }
                        }
                    const int planes = wg_follows(b + 1, b0, lg) ? 4 : 6;
                    at.base += planes;
                    bslot = W::slot(bslot + planes);
                    bbuf = W::next_buf(bbuf);
                }
            }
    return reads;
}

int main(int argc, char** argv) {
    if (argc != 8) return 2;
    int v[8], lg = 0;
    for (int i = 1; i < 8; ++i) v[i] = std::atoi(argv[i]);
    while ((1 << lg) < v[2]) ++lg;
    const long reads = v[1] == 1 ? replay<1>(lg, v[3], v[4], v[5], v[6], v[7])
                                 : replay<2>(lg, v[3], v[4], v[5], v[6], v[7]);
    std::printf("ok %ld\n", reads);
    return 0;
}
