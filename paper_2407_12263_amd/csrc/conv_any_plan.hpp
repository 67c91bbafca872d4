// Launch shape of conv3d_any_kernel (sur.hip): host arithmetic, free of HIP, so
// that it can be checked over all sizes without a GPU.
#pragma once
#include <algorithm>
#include <cstddef>

constexpr size_t kMaxLds = 160 * 1024;  // of a block, and of a CU

// 16-byte weight pieces that each of the 256 threads holds for the next stage,
// for 16 nc input channels and nt output tiles: six, or what the smallest
// stage, three taps, needs (seven for 96 channels and three tiles).
constexpr int any_pieces(int nc, int nt) {
    const int three = (3 * 16 * nt * 2 * nc + 255) / 256;
    return three > 6 ? three : 6;
}

// Points of the tiles 2^ltx x (16 mt / 2^ltx) x 4 that cover a grid.
inline long any_padded(int mt, int ltx, int nx, int ny, int nz) {
    const long tx = 1 << ltx, ty = 16 * mt >> ltx;
    return (nx + tx - 1) / tx * tx * ((ny + ty - 1) / ty * ty) * ((nz + 3) / 4 * 4);
}

// mt runs of 16 points and nt output tiles per block, tiles 2^ltx wide, taps
// weight taps per stage, ntile tiles, lds bytes. mt = 0: the kernel does not
// take these channels.
struct AnyPlan {
    int mt, nt, ltx, taps;
    long ntile;
    size_t lds;
};

inline AnyPlan any_plan(int cin, int cout, int nx, int ny, int nz, long cus) {
    // the widest block tile (most products per fragment read, least halo)
    // that still gives one and a half blocks per CU; below that the time is
    // one block's chain, shortest with one run and one output tile
    AnyPlan p{};
    if (cin > 128) return p;
    const int no = cout / 16;
    const int cand[6][2] = {{4, 3}, {4, 2}, {2, 2}, {4, 1}, {2, 1}, {1, 1}};
    size_t halo = 0, tap = 0;
    for (const auto &c : cand) {
        if (no % c[1]) continue;
        // tile width: the fewest points that cover the grid, of equals the
        // widest; two blocks on a CU do half as much again as one (48 -> 64
        // on 90^3, 16 or 8 wide: 425 us with one, 260 with two), for up to a
        // quarter more points
        const size_t t = (size_t)16 * c[1] * (2 * cin + 16);
        long least = 0;
        for (int l = 4; l >= 2; --l) {
            const long pts = any_padded(c[0], l, nx, ny, nz);
            if (least == 0 || pts < least) least = pts;
        }
        double best = 0;
        for (int l = 4; l >= 2; --l) {
            const size_t h = (size_t)((1 << l) + 2) * ((16 * c[0] >> l) + 2) * 6 * (2 * cin + 16);
            const long pts = any_padded(c[0], l, nx, ny, nz), blocks = pts / (64 * c[0]) * (no / c[1]);
            if (h + 3 * t > kMaxLds || 4 * pts > 5 * least) continue;
            const double cost = (double)pts * (2 * blocks >= 3 * cus && 2 * (h + 3 * t) <= kMaxLds ? 2 : 3);
            if (best > 0 && cost >= best) continue;
            best = cost;
            p.mt = c[0];
            p.nt = c[1];
            p.ltx = l;
            p.ntile = pts / (64 * c[0]);
            halo = h;
            tap = t;
        }
        if (best > 0 && 2 * p.ntile * (no / p.nt) >= 3 * cus) break;
    }
    if (p.mt == 0) return p;
    // taps per weight stage: the most that cost no block per CU (a block
    // alone on its CU leaves it idle while it stages: 48 -> 16 channels on
    // 104 x 88 x 120, 141 us with 3 taps and two blocks, 214 with all 27 and
    // one) and that the threads' registers hold
    const long need = (p.ntile * (no / p.nt) + cus - 1) / cus;
    auto per_cu = [&](int g) { return std::min(need, (long)(kMaxLds / (halo + g * tap))); };
    const int held = 256 * any_pieces(cin / 16, p.nt);
    p.taps = 27;
    while (p.taps > 3 && (per_cu(p.taps) < per_cu(3) || (p.taps < 27 && p.taps * 2 * p.nt * cin > held)))
        p.taps /= 3;
    p.lds = halo + p.taps * tap;
    return p;
}

// Microseconds of conv3d_any_kernel in plan p: the points that the tiles cover,
// at 0.10 to 0.23 ps per point and product of channels with one, two or three
// output tiles and one or two blocks on a CU (measured on grids of 0.4 to 2
// million points: 48 -> 16 0.16, 112 -> 48 0.22; 48 -> 64 0.10, 64 -> 64 0.15;
// 16 -> 48 0.10, 96 -> 48 0.11), at least one block on every CU.
inline double any_us(const AnyPlan &p, int cin, int cout, long cus) {
    const double blocks = (double)p.ntile * (cout / 16 / p.nt);
    const bool two = 2 * p.lds <= kMaxLds;
    const double ps = p.nt == 1 ? (two ? 0.17 : 0.23) : (p.nt == 2 ? (two ? 0.10 : 0.155) : (two ? 0.10 : 0.115));
    return 4.0 + std::max(blocks, (double)cus) * (64 * p.mt) * (16 * p.nt) * cin * ps * 1e-6;
}

// Microseconds of conv3d_kernel, towards the lower end of what it measured: a
// block's chain of gathers on small grids (16 -> 16 23, 96 -> 16 62, 80 -> 32 81,
// 48 -> 64 63, 112 -> 48 126; 64 -> 48 92), and per million points and input
// channel 6 (16 output channels) to 14 us on large ones, 17 to 23 with 64 or 128
// input channels.
inline double general_us(int cin, int cout, long points) {
    const int nc = cin / 16;
    const double chain = (cout == 16 ? 7.8 * nc + 15 : (cout == 32 ? 14.0 : 16.0) * nc + 8) *
                         (cin % 64 == 0 && cout > 16 ? 1.2 : 1.0);
    auto block = [&](int co) {  // us per million points and input channel
        if (co == 0) return 0.0;
        if (co == 16) return 6.3;
        if (cin % 64 == 0) return co == 32 ? 16.5 : (co == 48 ? 19.5 : 22.0);
        return cin > 64 ? (co == 32 ? 10.3 : 14.0) : 10.5;
    };
    return std::max(chain, (cout / 64 * block(64) + block(cout % 64)) * cin * (double)points * 1e-6);
}
