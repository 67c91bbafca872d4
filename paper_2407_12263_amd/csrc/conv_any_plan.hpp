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

// Tile width of conv3d_any_kernel: the one that covers the grid with the
// fewest points, the widest of equals.
inline int any_ltx(int mt, int nx, int ny, int nz) {
    int best = 4;
    for (int l = 3; l >= 2; --l)
        if (any_padded(mt, l, nx, ny, nz) < any_padded(mt, best, nx, ny, nz)) best = l;
    return best;
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
        const int l = any_ltx(c[0], nx, ny, nz);
        const size_t h = (size_t)((1 << l) + 2) * ((16 * c[0] >> l) + 2) * 6 * (2 * cin + 16);
        const size_t t = (size_t)16 * c[1] * (2 * cin + 16);
        if (h + 3 * t > kMaxLds) continue;
        p.mt = c[0];
        p.nt = c[1];
        p.ltx = l;
        p.ntile = any_padded(c[0], l, nx, ny, nz) / (64 * c[0]);
        halo = h;
        tap = t;
        if (2 * p.ntile * (no / p.nt) >= 3 * cus) break;
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
