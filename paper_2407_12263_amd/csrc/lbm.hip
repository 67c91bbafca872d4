// lbm.hip -- host side of the C ABI declared in include/lbm.h.
//
// The context holds two ping-pong population buffers A, B carved from the
// caller's workspace. The state "at time t" is the post-collision buffer
// cur, whose propagation gives the post-propagation PDFs at t + 1; the other
// buffer still holds what the last step read, so the moments at t are
// obtained by propagating it again (or, right after lbm_init / lbm_set_pdfs,
// by reading it in place, since it then holds the post-propagation PDFs at t).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>

#include "lbm.h"
#include "lbm_kernels.hpp"

using namespace cpf;

namespace {

// Discards an error that an earlier HIP call of another library left pending
// in this thread, so that the check after an entry point's launches
// (hipGetLastError) reports only that entry point's own failures.
inline void clear_stale_error() { (void)hipGetLastError(); }


constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

size_t elem_bytes(int precision) {
    switch (precision) {
        case LBM_FP64: return 8;
        case LBM_FP32: return 4;
        default: return 2;
    }
}

bool is16(int precision) {
    return precision == LBM_FP32_FP16STORE || precision == LBM_FP32_BF16STORE;
}

// Populations per field: 19 (D3Q19; lattice = 0 means the same) or 27.
int num_pop(const lbm_params *P) { return P->lattice == 27 ? 27 : 19; }

// Launch shape: one block per tile of w x th nodes of one z-plane.
// LBM_TILE_X_LOG2, LBM_TILE_ORDER and LBM_TILE_BAND override the choice
// (tuning only; results do not depend on it; a width whose tiles outnumber the
// rows of the phase-mass partials is not taken).
struct TileCfg {
    int w, th, threads, order, band;
};

int env_int(const char *name, int dflt) {
    const char *v = std::getenv(name);
    return v && *v ? std::atoi(v) : dflt;
}

// Tiles of one z-plane.
size_t plane_tiles(const lbm_params *P, int w, int th) {
    return (size_t)((P->nx + w - 1) / w) * (size_t)((P->ny + th - 1) / th);
}

// log2 of the tile width that LBM_TILE_X_LOG2 asks for; -1 for the default. A
// block of a launch that sums the phase mass writes two values; the partials
// hold NSUM for each tile of width 1.
int tile_override(const lbm_params *P) {
    const int l = env_int("LBM_TILE_X_LOG2", -1);
    if (l < 0 || l > 8 || 2 * plane_tiles(P, 1 << l, BLOCK >> l) > NSUM * plane_tiles(P, 1, BLOCK)) return -1;
    return l;
}

// base: a power of two that spans whole x-rows up to 128 nodes (a row's
// periodic wrap stays inside the tile; 128 measured best among 32, 64 and 128
// on the 128 x 512 x 128 Rayleigh-Taylor lattice). Otherwise the row itself:
// - up to 128 nodes where its fewer tiles are fewer rounds of 256 CUs (16
//   steps: 75 x 61 x 43 FP32 374 -> 311 us, 6 rounds -> 4, 50^3 FP64 420 -> 337,
//   3 -> 2; with the same two rounds 20 x 70 x 50 D3Q27 FP32 203 -> 217);
// - up to 224 where it spares a row's second, partial tile (133 x 110 x 90
//   FP16 1484 -> 1187, 150^3 FP64 12670 -> 10401, 210 x 60 x 60 FP32 1.10 times;
//   230 x 60 x 60 D3Q27 FP16 0.98, 250 x 50 x 30 0.97 times).
// Even shares of a row, 50 of 100, are 20% slower than the row for their
// unaligned segments. Rows beyond a block's threads
// take 64 where that leaves fewer lanes idle and the state is small (300 x 200
// FP64 248 -> 161 us, 300 x 90 x 30 FP16 887 -> 749; but D3Q27 FP32 1962 ->
// 2036).
TileCfg tile_cfg(const lbm_params *P, int threads, bool base) {
    TileCfg t;
    t.threads = threads;
    const int nx = P->nx, lx = tile_override(P);
    int l = 0;
    while ((1 << l) < nx && l < (threads == 64 ? 6 : 7)) ++l;
    t.w = 1 << l;
    const size_t idle = ((size_t)(nx + 127) / 128 * 128 - (nx + 63) / 64 * 64) / 64;
    const size_t bytes = (size_t)P->nx * P->ny * P->nz * elem_bytes(P->precision) * 2 * num_pop(P);
    auto rounds = [&](int w) { return (plane_tiles(P, w, threads / w) * P->nz + 255) / 256; };
    if (lx >= 0 && threads == BLOCK) t.w = 1 << lx;
    else if (base) ;
    else if (nx <= threads && (rounds(nx) < rounds(t.w) || (nx > t.w && nx <= 224)))
        t.w = nx;
    else if (nx > threads && t.w == 128 && idle && bytes < (size_t)100 << 20) t.w = 64;
    t.th = threads / t.w;
    // default: XCD runs of the z-banded order with bands of 32 tile rows (the
    // y/z taps of a band stay in L2; on RT: FP32 14.6 against 13.9 GLUPS and
    // FP16 25.6 against 24.3 in the plain order)
    const int dflt_order = 2;
    t.order = env_int("LBM_TILE_ORDER", dflt_order);
    if (t.order < 0 || t.order > 2) t.order = dflt_order;
    // a band of whole-row tiles is at most 64 rows of nodes, as that of tiles
    // of two: with 32 tiles of three or more rows the planes of some lattices
    // fall on each other in the caches (16 steps: 80^3 FP64 1533 -> 1278 us, D3Q27
    // 2237 -> 1859, 20 x 160 x 160 FP64 1532 -> 1279; 75 x 61 x 43 the same)
    const int dflt_band = !base && t.w == nx && (nx & (nx - 1)) ? std::max(1, std::min(32, 64 / t.th)) : 32;
    t.band = env_int("LBM_TILE_BAND", dflt_band);
    if (t.band < 1) t.band = dflt_band;
    return t;
}

// Bytes from one population plane to the next: N elements (16-bit storage:
// the 32-bit f/g words) rounded up to 256 B, plus a pad of 64 KiB + 256 B.
// With power-of-two strides (the usual lattice sizes) the 19 planes of a
// node fall on the same L2 sets and channels and evict each other's tap
// lines: unpadded, 256^3 FP16 steps fetch 1.6x the algorithmic bytes. The
// pad was measured best over 256 B .. 128 KiB on the Rayleigh-Taylor,
// rising-bubble and 256^3 lattices. LBM_PLANE_PAD (bytes) overrides it
// (tuning only; results do not depend on it).
size_t plane_pitch(const lbm_params *P) {
    const size_t N = (size_t)P->nx * P->ny * P->nz;
    const size_t pe = is16(P->precision) ? 4 : (size_t)elem_bytes(P->precision);
    const int pad = env_int("LBM_PLANE_PAD", 65536 + 256);
    return align_up(N * pe) + align_up((size_t)(pad > 0 ? pad : 0));
}

struct Layout {
    size_t pdf_bytes;      // f (16-bit storage: f and g words), Q planes
    size_t g_bytes;        // g, Q planes (0 for 16-bit storage)
    size_t phis_bytes;     // N floats (16-bit storage) or 0
    size_t buf_bytes;      // f + g + phis of one ping-pong buffer
    size_t partial_bytes;  // NSUM doubles per reduction block
    size_t result_bytes;
    size_t flag_bytes;
    size_t mf_bytes;
    size_t phifd_bytes;    // phi field of the finite-difference variant (or 0)
    size_t total;
};

Layout layout_of(const lbm_params *P) {
    Layout L;
    const size_t N = (size_t)P->nx * P->ny * P->nz;
    // rows of the reduction partials: the tile count at tile width 1. Some
    // sizes have more tiles at the width in use (133 x 154: 154 against 133 a
    // plane); the diagnostics then take their tile rows in parts (reduce_diag).
    // The phase-mass partials are 2 values a block, not NSUM: they fit at up
    // to 8.5 times this count. No size has more than twice it at its default
    // width, and other widths are taken only where they fit (tile_override).
    const size_t nblocks = plane_tiles(P, 1, BLOCK) * (size_t)P->nz;
    L.pdf_bytes = align_up((size_t)num_pop(P) * plane_pitch(P));
    L.g_bytes = is16(P->precision) ? 0 : L.pdf_bytes;
    L.phis_bytes = is16(P->precision) ? align_up(N * sizeof(float)) : 0;
    L.buf_bytes = L.pdf_bytes + L.g_bytes + L.phis_bytes;
    L.partial_bytes = align_up(nblocks * NSUM * sizeof(double));
    L.result_bytes = align_up(NSUM * sizeof(double));
    L.flag_bytes = kAlign;
    L.mf_bytes = kAlign;  // M0, coef
    L.phifd_bytes = P->normal_fd ? align_up(N * sizeof(double)) : 0;
    L.total = 2 * L.buf_bytes + L.partial_bytes + L.result_bytes + L.flag_bytes + L.mf_bytes +
              L.phifd_bytes;
    return L;
}

int validate(const lbm_params *P) {
    if (!P) return LBM_EINVAL;
    if (P->nx < 1 || P->ny < 1 || P->nz < 1) return LBM_EINVAL;
    if (P->lattice != 0 && P->lattice != 19 && P->lattice != 27) return LBM_EINVAL;
    // the finite-difference comparison scheme is built for D3Q19 only
    if (P->lattice == 27 && P->normal_fd) return LBM_EINVAL;
    // wetting walls act on the K1 normal; not combined with the FD scheme
    if (P->wetting != 0 && P->wetting != 1) return LBM_EINVAL;
    if (P->wetting && P->normal_fd) return LBM_EINVAL;
    if (P->wetting && !(std::isfinite(P->cos_theta) && P->cos_theta >= -1.0 && P->cos_theta <= 1.0))
        return LBM_EINVAL;
    const double N = (double)P->nx * P->ny * P->nz;
    const double Q = num_pop(P);
    if (Q * N >= 2147483647.0) return LBM_EINVAL;
    if (P->precision < LBM_FP64 || P->precision > LBM_FP32_BF16STORE) return LBM_EINVAL;
    // every population field is addressed through one 32-bit buffer range
    // (16-bit storage keeps f and g of a population in one 32-bit plane)
    if (Q * (double)plane_pitch(P) >= 4294967295.0) return LBM_EINVAL;
    const int nn[3] = {P->nx, P->ny, P->nz};
    for (int a = 0; a < 3; ++a) {
        if (P->wall[a] != 0 && P->wall[a] != 1) return LBM_EINVAL;
        if (P->wall[a] && nn[a] < 2) return LBM_EINVAL;
    }
    for (int k = 0; k < 2; ++k)
        if (P->store_log2[k] < -24 || P->store_log2[k] > 24) return LBM_EINVAL;
    if (P->check_every < 0 || P->mass_fix_every < 0) return LBM_EINVAL;
    if (P->normal_fd != 0 && P->normal_fd != 1) return LBM_EINVAL;
    auto fin = [](double x) { return std::isfinite(x); };
    if (!(fin(P->courant) && P->courant > 0.0 && P->courant <= 1.0)) return LBM_EINVAL;
    if (!(fin(P->rho1) && fin(P->rho2) && P->rho1 > 0.0 && P->rho2 > 0.0)) return LBM_EINVAL;
    if (!(fin(P->tau_rho1) && fin(P->tau_rho2) && P->tau_rho1 > 0.0 && P->tau_rho2 > 0.0))
        return LBM_EINVAL;
    if (!(fin(P->tau_phi) && P->tau_phi > 0.0)) return LBM_EINVAL;
    if (!(fin(P->sigma) && P->sigma >= 0.0)) return LBM_EINVAL;
    if (!(fin(P->delta) && P->delta > 0.0)) return LBM_EINVAL;
    if (!(fin(P->G[0]) && fin(P->G[1]) && fin(P->G[2]))) return LBM_EINVAL;
    if (!(fin(P->k1_eps) && P->k1_eps >= 0.0)) return LBM_EINVAL;
    if (!fin(P->p_ref)) return LBM_EINVAL;
    return LBM_OK;
}

FastDiv make_fastdiv(uint32_t d) {
    FastDiv f{0u, 0u, d < 1u ? 1u : d};
    if (f.d == 1u) return f;
    uint32_t l = 0;
    while ((1ull << l) < f.d) ++l;  // 2^(l-1) < d <= 2^l
    const unsigned __int128 num = (unsigned __int128)1 << (31 + l);
    f.m = (uint32_t)((num + f.d - 1) / f.d);
    f.s = l - 1;
    return f;
}

// Rows y0 .. y0 + rows - 1 (and the same `ystep` further where two), planes
// z0 + k zstep (k < nz), in tiles of shape tc.
Box make_box(const lbm_params *P, const TileCfg &tc, int y0, int rows, int ystep, int z0, int nz, int zstep) {
    Box b;
    b.th = tc.th;
    b.tw_log2 = -1;
    for (int l = 0; l <= 8; ++l)
        if (tc.w == 1 << l) b.tw_log2 = l;
    b.nsub = (rows + tc.th - 1) / tc.th;
    const int ntx = (P->nx + tc.w - 1) / tc.w, nty = b.nsub * (ystep > 0 ? 2 : 1), ntiles = ntx * nty * nz;
    const int band = tc.band < nty ? tc.band : nty;
    b.nz = nz;
    b.y0 = y0;
    b.ystep = ystep;
    b.rows = rows;
    b.z0 = z0;
    b.zstep = zstep;
    b.order = tc.order;
    b.nfull = nty / band;
    b.xq = ntiles / 8;
    b.xr = ntiles % 8;
    const int rem = nty - b.nfull * band;
    b.d_tw = make_fastdiv((uint32_t)tc.w);
    b.d_ntx = make_fastdiv((uint32_t)ntx);
    b.d_nty = make_fastdiv((uint32_t)nty);
    b.d_band = make_fastdiv((uint32_t)band);
    b.d_perband = make_fastdiv((uint32_t)(band * nz));
    b.d_rem = make_fastdiv((uint32_t)(rem > 0 ? rem : 1));
    return b;
}

Box full_box(const lbm_params *P, const TileCfg &tc) { return make_box(P, tc, 0, P->ny, 0, 0, P->nz, 1); }

// How a step covers the lattice. Periodic lattices: the wall-free instance
// everywhere. Walls in y and/or z: the wall-free instance on the interior, the
// wall-aware one on the slabs of rows and planes that touch a wall. A y slab is
// slab_rows rows from the bottom, and from the last multiple of them to the
// top: a tile's height at a power-of-two width. Walls in x touch every row,
// and slabs that meet leave no interior: the wall-aware instance everywhere.
struct Cover {
    int threads;
    bool split, walls;
    int n;               // boxes in use
    Box b[3];            // the whole lattice; or interior and slabs
    int blocks;
};

Cover make_cover(const lbm_params *P, const TileCfg &tc) {
    Cover v;
    v.threads = tc.threads;
    const int *w = P->wall;
    v.walls = w[0] || w[1] || w[2];
    int l = 0;
    while ((1 << l) < P->nx && l < 7) ++l;
    const int lx = tile_override(P);
    if (lx >= 0) l = lx;
    const int h = BLOCK >> l, top = (P->ny - 1) / h * h;  // slab rows, first row of the upper slab
    const int ylo = w[1] ? h : 0, yhi = w[1] ? top : P->ny;
    const int zlo = w[2] ? 1 : 0, zhi = w[2] ? P->nz - 1 : P->nz;
    v.split = v.walls && !w[0] && yhi > ylo && zhi > zlo;
    if (!v.split) {
        v.n = 1;
        v.b[0] = full_box(P, tc);
    } else {
        v.n = 1;
        v.b[0] = make_box(P, tc, ylo, yhi - ylo, 0, zlo, zhi - zlo, 1);
        if (w[1]) v.b[v.n++] = make_box(P, tc, 0, h, top, 0, P->nz, 1);
        if (w[2]) v.b[v.n++] = make_box(P, tc, ylo, yhi - ylo, 0, 0, 2, P->nz - 1);
    }
    v.blocks = 0;
    for (int k = 0; k < v.n; ++k) v.blocks += v.b[k].ntiles();
    return v;
}

template <class R>
DevParams<R> make_params(const lbm_params *P) {
    DevParams<R> d;
    d.nx = P->nx;
    d.ny = P->ny;
    d.nz = P->nz;
    d.N = P->nx * P->ny * P->nz;
    d.plane_bytes = (uint32_t)plane_pitch(P);
    for (int a = 0; a < 3; ++a) d.wall[a] = P->wall[a];
    const double c = P->courant, cs2 = c * c / 3.0;
    const double eta1 = P->rho1 * cs2 * P->tau_rho1, eta2 = P->rho2 * cs2 * P->tau_rho2;
    d.c = R(c);
    d.h = R(0.5 * c * (1.0 - c));
    d.lwA = R(0.5 * c * (1.0 + c));
    d.lwD = R(-0.5 * c * (1.0 - c));
    d.cs2 = R(cs2);
    d.inv_cs2 = R(1.0 / cs2);
    d.half_inv_cs4 = R(0.5 / (cs2 * cs2));
    d.rho2 = R(P->rho2);
    d.drho = R(P->rho1 - P->rho2);
    d.eta2 = R(eta2);
    d.deta = R(eta1 - eta2);
    d.omega_g = R(1.0 / (P->tau_phi + 0.5));
    d.tau_phi_c = R(P->tau_phi * c);
    d.tau_phi_cs2 = R(P->tau_phi * cs2);
    d.inv_tp = R(1.0 / ((P->tau_phi + 0.5) * cs2));
    d.sigma = R(P->sigma);
    d.four_over_delta = R(4.0 / P->delta);
    for (int a = 0; a < 3; ++a) d.G[a] = R(P->G[a]);
    d.k1_eps = R(P->k1_eps);
    d.rho0 = R(P->p_ref / cs2);
    d.scale_f = R(std::ldexp(1.0, P->store_log2[0]));
    d.iscale_f = R(std::ldexp(1.0, -P->store_log2[0]));
    d.scale_g = R(std::ldexp(1.0, P->store_log2[1]));
    d.iscale_g = R(std::ldexp(1.0, -P->store_log2[1]));
    const double lwA = 0.5 * c * (1.0 + c), lwD = -0.5 * c * (1.0 - c), lwB = 1.0 - c * c;
    d.wA_f = R(std::ldexp(lwA, -P->store_log2[0]));
    d.wB_f = R(std::ldexp(lwB, -P->store_log2[0]));
    d.wD_f = R(std::ldexp(lwD, -P->store_log2[0]));
    d.wA_g = R(std::ldexp(lwA, -P->store_log2[1]));
    d.wB_g = R(std::ldexp(lwB, -P->store_log2[1]));
    d.wD_g = R(std::ldexp(lwD, -P->store_log2[1]));
    d.phi_fd = nullptr;
    return d;
}

template <class R>
Wet<R> make_wet(const lbm_params *P) {
    Wet<R> w;
    w.on = P->wetting;
    w.cos_theta = R(P->wetting ? P->cos_theta : 0.0);
    w.sin_theta = R(P->wetting ? std::sqrt(1.0 - P->cos_theta * P->cos_theta) : 1.0);
    return w;
}

}  // namespace

struct lbm_ctx {
    lbm_params P;
    Layout L;
    hipStream_t stream;
    char *ws;
    char *buf[2];
    double *partials;
    double *result;
    int *flag;
    double *mf;         // M0, coef of the phase-mass bookkeeping
    void *phifd;        // phi field of the finite-difference variant (or NULL)
    bool mf_pending;    // the next step applies coef
    TileCfg base;       // shape of the launches that sum over the lattice
    Cover cover;        // a step
    Cover sums;         // a step that reports the phase mass, in shape base: its
                        // blocks group the sum, so the correction does not
                        // follow the step's shape
    Box full, full_base;   // the whole lattice, in the step's shape and in base
    DevParams<float> pf;   // launch parameters
    DevParams<double> pd;
    int cur;            // buffer holding the post-collision state
    bool prev_local;    // the other buffer holds post-propagation PDFs at t
    int64_t t;
    int status;
};

namespace {

template <class St>
Buf<St> buf_of(lbm_ctx *c, int k) {
    Buf<St> b;
    b.f = (typename St::T *)c->buf[k];
    b.g = (typename St::T *)(c->buf[k] + c->L.pdf_bytes);
    b.phis = c->L.phis_bytes ? (float *)(c->buf[k] + c->L.pdf_bytes + c->L.g_bytes) : nullptr;
    return b;
}

template <class St>
CBuf<St> cbuf_of(lbm_ctx *c, int k) {
    Buf<St> b = buf_of<St>(c, k);
    return CBuf<St>{b.f, b.g, b.phis};
}

int check_launch(lbm_ctx *c) {
    if (hipGetLastError() != hipSuccess) {
        if (c) c->status = LBM_EDEVICE;
        return LBM_EDEVICE;
    }
    return LBM_OK;
}

template <class St, Mode M, bool W, bool FD>
void launch_step(lbm_ctx *c, int src, int dst, const DevParams<typename St::R> &P, const Box &b,
                 int threads, MassFix mf, int &block_off) {
    mf.block_off = block_off;
    if constexpr (St::DEV && !W && !FD && St::Q == 19)
        hipLaunchKernelGGL((step_kernel_o5<St, M, W, FD>), dim3((unsigned)b.ntiles()), dim3(threads), 0,
                           c->stream, cbuf_of<St>(c, src), buf_of<St>(c, dst), P, b, mf);
    else
        hipLaunchKernelGGL((step_kernel<St, M, W, FD>), dim3((unsigned)b.ntiles()), dim3(threads), 0,
                           c->stream, cbuf_of<St>(c, src), buf_of<St>(c, dst), P, b, mf,
                           make_wet<typename St::R>(&c->P));
    block_off += b.ntiles();
}

// Parameters of a launch, with the phi field of the finite-difference variant.
template <class R>
const DevParams<R> &launch_params(lbm_ctx *c) {
    if constexpr (sizeof(R) == 8) return c->pd;
    else return c->pf;
}

// First pass of the finite-difference variant: phi of the state the next
// launch reads from buffer src, split into interior and wall slabs as the
// step is.
template <class St, Mode M>
void launch_phi(lbm_ctx *c, int src, const MassFix &mf) {
    const DevParams<typename St::R> &P = launch_params<typename St::R>(c);
    const Cover &v = c->cover;
    for (int k = 0; k < v.n; ++k) {
        const dim3 grid((unsigned)v.b[k].ntiles()), block(v.threads);
        if (v.split ? k > 0 : v.walls)
            hipLaunchKernelGGL((phi_kernel<St, M, true>), grid, block, 0, c->stream, cbuf_of<St>(c, src), P, v.b[k], mf);
        else
            hipLaunchKernelGGL((phi_kernel<St, M, false>), grid, block, 0, c->stream, cbuf_of<St>(c, src), P, v.b[k], mf);
    }
}

template <class St, Mode M, bool FD>
void launch_step_w(lbm_ctx *c, int src, int dst, const MassFix &mf) {
    using R = typename St::R;
    const DevParams<R> &P = launch_params<R>(c);
    const Cover &v = (mf.mode & 1) ? c->sums : c->cover;
    int off = 0;
    // One launch for the interior and the slabs: on small lattices the launches
    // set the time (16 steps, walls in y, two launches -> one: 32^3 FP16 187 ->
    // 113 us, 75 x 61 x 43 FP32 407 -> 361, D3Q27 BF16 430 -> 345); on large
    // ones the wall instance's registers cost the interior more than the slab
    // launch takes (128 x 512 x 128 FP32 8241 -> 8443, 100 x 96 x 70 D3Q27 BF16
    // 911 -> 928), except in FP64, whose step is no wider for it (19351 -> 19005).
    if constexpr (!FD && M != LOCAL) {
        const int most = St::Q == 27 ? 500000 : (sizeof(R) == 8 ? P.N : 1250000);
        if (v.split && P.N <= most) {
            Boxes B;
            B.b[0] = v.b[0];
            B.b[1] = v.b[1];
            B.b[2] = v.b[v.n - 1];
            B.n0 = (uint32_t)v.b[0].ntiles();
            B.n1 = B.n0 + (uint32_t)v.b[1].ntiles();
            hipLaunchKernelGGL((step_all_kernel<St, M>), dim3((unsigned)v.blocks), dim3(v.threads), 0,
                               c->stream, cbuf_of<St>(c, src), buf_of<St>(c, dst), P, B, mf,
                               make_wet<R>(&c->P));
            return;
        }
    }
    for (int k = 0; k < v.n; ++k) {
        if (v.split ? k > 0 : v.walls) launch_step<St, M, true, FD>(c, src, dst, P, v.b[k], v.threads, mf, off);
        else launch_step<St, M, false, FD>(c, src, dst, P, v.b[k], v.threads, mf, off);
    }
}

template <class St, Mode M>
void launch_step_fd(lbm_ctx *c, int src, int dst, const MassFix &mf) {
    if constexpr (St::Q == 19) {
        if (c->P.normal_fd) {
            MassFix apply = mf;
            apply.mode &= 2;
            launch_phi<St, M>(c, src, apply);
            launch_step_w<St, M, true>(c, src, dst, mf);
            return;
        }
    }
    launch_step_w<St, M, false>(c, src, dst, mf);
}

template <class St>
void step_dispatch(lbm_ctx *c, Mode m, int src, int dst, const MassFix &mf) {
    switch (m) {
        case LOCAL: launch_step_fd<St, LOCAL>(c, src, dst, mf); break;
        case SHIFT: launch_step_fd<St, SHIFT>(c, src, dst, mf); break;
        default: launch_step_fd<St, LW>(c, src, dst, mf); break;
    }
}

// Calls F::template run<St>(args...) with the storage type of the context's
// precision and lattice.
template <class F, class... A>
void with_storage(const lbm_ctx *c, A &&...args) {
    const bool q27 = num_pop(&c->P) == 27;
    switch (c->P.precision) {
        case LBM_FP64:
            q27 ? F::template run<Q27<SF64>>(args...) : F::template run<SF64>(args...);
            break;
        case LBM_FP32:
            q27 ? F::template run<Q27<SF32>>(args...) : F::template run<SF32>(args...);
            break;
        case LBM_FP32_FP16STORE:
            q27 ? F::template run<Q27<SH16>>(args...) : F::template run<SH16>(args...);
            break;
        default:
            q27 ? F::template run<Q27<SB16>>(args...) : F::template run<SB16>(args...);
            break;
    }
}

struct StepOp {
    template <class St>
    static void run(lbm_ctx *c, Mode m, int src, int dst, const MassFix &mf) {
        step_dispatch<St>(c, m, src, dst, mf);
    }
};

void step_any(lbm_ctx *c, Mode m, int src, int dst, int mf_mode = 0) {
    const MassFix mf{mf_mode, c->partials, c->mf + 1, 0};
    with_storage<StepOp>(c, c, m, src, dst, mf);
}

Mode prop_mode(const lbm_ctx *c) { return c->P.courant == 1.0 ? SHIFT : LW; }

template <class St, Mode M, bool W>
void launch_moments(lbm_ctx *c, const FieldOut &o, const Box &b, int threads) {
    using R = typename St::R;
    const DevParams<R> &P = launch_params<R>(c);
    const dim3 grid((unsigned)b.ntiles()), block(threads);
    if constexpr (St::Q == 19) {
        if (c->P.normal_fd) {
            launch_phi<St, M>(c, c->cur ^ 1, MassFix{0, nullptr, nullptr, 0});
            hipLaunchKernelGGL((moments_kernel<St, M, W, true>), grid, block, 0, c->stream,
                               cbuf_of<St>(c, c->cur ^ 1), P, b, o, make_wet<R>(&c->P));
            return;
        }
    }
    hipLaunchKernelGGL((moments_kernel<St, M, W, false>), grid, block, 0, c->stream,
                       cbuf_of<St>(c, c->cur ^ 1), P, b, o, make_wet<R>(&c->P));
}

template <class St, Mode M>
void moments_w(lbm_ctx *c, const FieldOut &o, const Box &b, int threads) {
    const bool walls = c->P.wall[0] || c->P.wall[1] || c->P.wall[2];
    if (walls) launch_moments<St, M, true>(c, o, b, threads);
    else launch_moments<St, M, false>(c, o, b, threads);
}

template <class St>
void moments_dispatch(lbm_ctx *c, const FieldOut &o, const Box &b, int threads) {
    if (c->prev_local) moments_w<St, LOCAL>(c, o, b, threads);
    else if (prop_mode(c) == SHIFT) moments_w<St, SHIFT>(c, o, b, threads);
    else moments_w<St, LW>(c, o, b, threads);
}

struct MomentsOp {
    template <class St>
    static void run(lbm_ctx *c, const FieldOut &o, const Box &b, int threads) {
        moments_dispatch<St>(c, o, b, threads);
    }
};

void moments_any(lbm_ctx *c, const FieldOut &o, const Box &b, int threads) { with_storage<MomentsOp>(c, c, o, b, threads); }
void moments_any(lbm_ctx *c, const FieldOut &o) { moments_any(c, o, c->full, c->cover.threads); }

// The state at the current time from fields: post-propagation populations
// into dst and their collision into post, in one launch (the
// finite-difference variant collides in its own two passes).
template <class St>
void launch_init(lbm_ctx *c, const double *phi0, const double *u0, const double *p0, int dst, int post) {
    using R = typename St::R;
    const DevParams<double> &PD = c->pd;
    const DevParams<R> &PR = launch_params<R>(c);
    const Cover &v = c->cover;
    const bool step = !c->P.normal_fd;
    // the sum of phi in the groups of full_base: in the same launch where that
    // is the launch
    const bool sum_here = v.n == 1 && v.threads == BLOCK && v.b[0].tw() == c->full_base.tw();
    if (!sum_here)
        hipLaunchKernelGGL(field_sum_kernel, dim3((unsigned)c->full_base.ntiles()), dim3(BLOCK), 0, c->stream,
                           phi0, PD, c->full_base, c->partials);
    auto launch = [&](const Box &b, auto W, auto S) {
        hipLaunchKernelGGL((init_kernel<St, decltype(W)::value, decltype(S)::value>), dim3((unsigned)b.ntiles()),
                           dim3(v.threads), 0, c->stream, phi0, u0, p0, PD, PR, b, buf_of<St>(c, dst),
                           c->flag, sum_here ? c->partials : nullptr, buf_of<St>(c, post), make_wet<R>(&c->P));
    };
    for (int k = 0; k < v.n; ++k) {
        const bool w = v.split ? k > 0 : v.walls;
        if (step && w) launch(v.b[k], std::true_type{}, std::true_type{});
        else if (step) launch(v.b[k], std::false_type{}, std::true_type{});
        if constexpr (St::Q == 19) {
            if (!step && w) launch(v.b[k], std::true_type{}, std::false_type{});
            else if (!step) launch(v.b[k], std::false_type{}, std::false_type{});
        }
    }
    if constexpr (St::Q == 19)
        if (!step) launch_step_fd<St, LOCAL>(c, dst, post, MassFix{0, c->partials, c->mf + 1, 0});
}

struct InitOp {
    template <class St>
    static void run(lbm_ctx *c, const double *phi0, const double *u0, const double *p0, int dst, int post) {
        launch_init<St>(c, phi0, u0, p0, dst, post);
    }
};

void init_any(lbm_ctx *c, const double *phi0, const double *u0, const double *p0, int dst, int post) {
    with_storage<InitOp>(c, c, phi0, u0, p0, dst, post);
}

template <class St>
void launch_load(lbm_ctx *c, const double *f, const double *g, int dst) {
    using R = typename St::R;
    const DevParams<R> &P = launch_params<R>(c);
    hipLaunchKernelGGL((load_kernel<St>), dim3((unsigned)c->full.ntiles()), dim3(c->cover.threads), 0, c->stream,
                       f, g, P, c->full, buf_of<St>(c, dst));
}

struct LoadOp {
    template <class St>
    static void run(lbm_ctx *c, const double *f, const double *g, int dst) {
        launch_load<St>(c, f, g, dst);
    }
};

void load_any(lbm_ctx *c, const double *f, const double *g, int dst) {
    with_storage<LoadOp>(c, c, f, g, dst);
}

// Folds the first `rows` partial rows, in order, into c->result (or into row 0).
void fold_partials(lbm_ctx *c, int rows, bool last) {
    int stride = 1;
    if (rows > 4 * RRUN) {  // runs of rows by many blocks first
        const int nb = (rows + RRUN - 1) / RRUN;
        hipLaunchKernelGGL(reduce_partials_kernel, dim3(nb), dim3(256), 0, c->stream, c->partials,
                           rows, 1, RRUN, (double *)nullptr);
        rows = nb;
        stride = RRUN;
    }
    hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(256), 0, c->stream, c->partials, rows,
                       stride, rows, last ? c->result : (double *)nullptr);
}

// Runs the diagnostics reduction of the state at t into c->result (device).
// Where the tiles outnumber the rows of the partials, their rows go in parts:
// row 0 keeps the parts before, the others take the next tile rows.
int reduce_diag(lbm_ctx *c, const double *phi_ref) {
    FieldOut o{};
    o.phi_ref = phi_ref;
    o.partials = c->partials;
    const Box &all = c->full_base;
    const int per = all.ntx() * all.nz;  // blocks of a tile row
    const int cap = (int)(c->L.partial_bytes / (NSUM * sizeof(double)));
    if (all.ntiles() <= cap) {
        moments_any(c, o, all, BLOCK);
        fold_partials(c, all.ntiles(), true);
        return check_launch(c);
    }
    for (int ty = 0; ty < all.nty();) {
        o.row0 = ty > 0 ? 1 : 0;
        const int n = std::min(all.nty() - ty, (cap - 1) / per);
        if (n < 1) return LBM_EDEVICE;
        const int y0 = ty * all.th, rows = std::min(n * all.th, c->P.ny - y0);
        moments_any(c, o, make_box(&c->P, c->base, y0, rows, 0, 0, c->P.nz, 1), BLOCK);
        ty += n;
        fold_partials(c, o.row0 + n * per, ty == all.nty());
    }
    return check_launch(c);
}

// State at the current time from fields (device FP64): post-propagation
// PDFs into buffer 1, M0 = sum phi (FP64) for the phase-mass bookkeeping, one
// collision into buffer 0; checks the inputs (synchronises the stream).
int build_state(lbm_ctx *c, const double *d_phi, const double *d_u, const double *d_p) {
    hipLaunchKernelGGL(clear_int_kernel, dim3(1), dim3(1), 0, c->stream, c->flag);
    init_any(c, d_phi, d_u, d_p, 1, 0);
    hipLaunchKernelGGL(massfix_kernel, dim3(1), dim3(RBLOCK), 0, c->stream,
                       (const double *)c->partials, c->full_base.ntiles(), c->mf, c->mf + 1, 1);
    c->cur = 0;
    c->prev_local = true;
    c->mf_pending = false;
    int bad = 0;
    if (check_launch(c) != LBM_OK ||
        hipMemcpyAsync(&bad, c->flag, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess)
        return LBM_EDEVICE;
    return bad ? LBM_EINVAL : LBM_OK;
}

}  // namespace

extern "C" {

void lbm_lattice(int32_t e[57], double t[19]) { lbm_lattice_q(19, e, t); }

int lbm_lattice_q(int32_t q, int32_t *e, double *t) {
    if ((q != 19 && q != 27) || !e || !t) return LBM_EINVAL;
    for (int i = 0; i < q; ++i) {
        const int ex = q == 27 ? LatQ<27>::EX[i] : LatQ<19>::EX[i];
        const int ey = q == 27 ? LatQ<27>::EY[i] : LatQ<19>::EY[i];
        const int ez = q == 27 ? LatQ<27>::EZ[i] : LatQ<19>::EZ[i];
        e[3 * i + 0] = ex;
        e[3 * i + 1] = ey;
        e[3 * i + 2] = ez;
        const int cl = ex * ex + ey * ey + ez * ez;
        if (q == 27)
            t[i] = cl == 0 ? 8.0 / 27.0 : (cl == 1 ? 2.0 / 27.0 : (cl == 2 ? 1.0 / 54.0 : 1.0 / 216.0));
        else
            t[i] = cl == 0 ? 1.0 / 3.0 : (cl == 1 ? 1.0 / 18.0 : 1.0 / 36.0);
    }
    return LBM_OK;
}

int lbm_workspace_bytes(const lbm_params *P, size_t *bytes) {
    if (!bytes) return LBM_EINVAL;
    const int rc = validate(P);
    if (rc != LBM_OK) return rc;
    *bytes = layout_of(P).total;
    return LBM_OK;
}

int lbm_init(const lbm_params *P, void *d_workspace, size_t bytes, void *stream,
             const double *d_phi0, const double *d_u0, const double *d_p0, lbm_ctx **out) {
    clear_stale_error();
    if (!out) return LBM_EINVAL;
    *out = nullptr;
    int rc = validate(P);
    if (rc != LBM_OK) return rc;
    if (!d_workspace || !d_phi0) return LBM_EINVAL;
    if (((uintptr_t)d_workspace) % kAlign != 0) return LBM_EINVAL;
    const Layout L = layout_of(P);
    if (bytes < L.total) return LBM_ENOMEM;

    lbm_ctx *c = new (std::nothrow) lbm_ctx;
    if (!c) return LBM_ENOMEM;
    std::memset(c, 0, sizeof(*c));
    c->P = *P;
    c->L = L;
    c->stream = (hipStream_t)stream;
    c->ws = (char *)d_workspace;
    c->buf[0] = c->ws;
    c->buf[1] = c->ws + L.buf_bytes;
    c->partials = (double *)(c->ws + 2 * L.buf_bytes);
    c->result = (double *)(c->ws + 2 * L.buf_bytes + L.partial_bytes);
    c->flag = (int *)(c->ws + 2 * L.buf_bytes + L.partial_bytes + L.result_bytes);
    c->mf = (double *)(c->ws + 2 * L.buf_bytes + L.partial_bytes + L.result_bytes + L.flag_bytes);
    c->phifd = L.phifd_bytes ? (void *)(c->ws + 2 * L.buf_bytes + L.partial_bytes + L.result_bytes +
                                        L.flag_bytes + L.mf_bytes)
                             : nullptr;
    c->base = tile_cfg(P, BLOCK, true);
    TileCfg tc = tile_cfg(P, BLOCK, false);
    // blocks of one wavefront where 256-thread blocks would leave half the CUs
    // without one (16 steps: 100 x 100 FP64 113 -> 84 us, 32^3 FP64 124 -> 104,
    // FP16 90 -> 86; 48^3 FP16 121 -> 143)
    const int64_t N = (int64_t)P->nx * P->ny * P->nz;
    if (2 * N <= 256 * BLOCK) tc = tile_cfg(P, 64, false);
    c->cover = make_cover(P, tc);
    c->sums = make_cover(P, c->base);
    c->full = full_box(P, tc);
    c->full_base = full_box(P, c->base);
    c->pf = make_params<float>(P);
    c->pd = make_params<double>(P);
    c->pf.phi_fd = (float *)c->phifd;
    c->pd.phi_fd = (double *)c->phifd;
    c->mf_pending = false;
    c->status = LBM_OK;

    c->t = 0;
    const int rc2 = build_state(c, d_phi0, d_u0, d_p0);
    if (rc2 != LBM_OK) {
        delete c;
        return rc2;
    }
    *out = c;
    return LBM_OK;
}

int lbm_reset(lbm_ctx *c, const double *d_phi, const double *d_u, const double *d_p, int64_t t) {
    clear_stale_error();
    if (!c || !d_phi || t < 0) return LBM_EINVAL;
    if (c->status == LBM_EDEVICE) return LBM_ESTATE;
    const int rc = build_state(c, d_phi, d_u, d_p);
    if (rc == LBM_OK) {
        c->t = t;
        c->status = LBM_OK;
    } else {
        // the buffers now hold the rejected fields' state: refuse lbm_step
        // until a reset succeeds
        c->status = rc == LBM_EDEVICE ? LBM_EDEVICE : LBM_ESTATE;
    }
    return rc;
}

int lbm_step(lbm_ctx *c, int64_t n) {
    clear_stale_error();
    if (!c || n < 0) return LBM_EINVAL;
    if (c->status != LBM_OK) return LBM_ESTATE;
    const Mode m = prop_mode(c);
    const int mfe = c->P.mass_fix_every;
    for (int64_t k = 0; k < n; ++k) {
        int mf_mode = c->mf_pending ? 2 : 0;
        if (mfe > 0 && (c->t + 1) % mfe == 0) mf_mode |= 1;
        step_any(c, m, c->cur, c->cur ^ 1, mf_mode);
        c->mf_pending = false;
        if (mf_mode & 1) {
            hipLaunchKernelGGL(massfix_kernel, dim3(1), dim3(RBLOCK), 0, c->stream,
                               (const double *)c->partials, c->sums.blocks, c->mf, c->mf + 1, 0);
            c->mf_pending = true;
        }
        c->cur ^= 1;
        c->prev_local = false;
        c->t += 1;
        if (c->P.check_every > 0 && c->t % c->P.check_every == 0) {
            if (reduce_diag(c, nullptr) != LBM_OK) return LBM_EDEVICE;
            double r[NSUM];
            if (hipMemcpyAsync(r, c->result, sizeof(r), hipMemcpyDeviceToHost, c->stream) !=
                    hipSuccess ||
                hipStreamSynchronize(c->stream) != hipSuccess) {
                c->status = LBM_EDEVICE;
                return LBM_EDEVICE;
            }
            const double cs = c->P.courant / std::sqrt(3.0);
            bool ok = true;
            for (int k2 = 0; k2 < NSUM; ++k2) ok = ok && std::isfinite(r[k2]);
            if (!ok || r[6] >= cs) {
                c->status = LBM_EUNSTABLE;
                return LBM_EUNSTABLE;
            }
        }
    }
    return check_launch(c);
}

int lbm_fields(lbm_ctx *c, void *d_phi, void *d_u, void *d_p, int32_t dtype) {
    return lbm_fields_twice(c, d_phi, d_u, d_p, nullptr, nullptr, nullptr, dtype);
}

int lbm_fields_twice(lbm_ctx *c, void *d_phi, void *d_u, void *d_p, void *d_phi2, void *d_u2, void *d_p2,
                     int32_t dtype) {
    clear_stale_error();
    if (!c || (dtype != 0 && dtype != 1) || (d_phi2 && !d_phi) || (d_u2 && !d_u) || (d_p2 && !d_p))
        return LBM_EINVAL;
    if (c->status == LBM_EDEVICE) return LBM_ESTATE;
    FieldOut o{};
    o.phi = d_phi;
    o.u = d_u;
    o.p = d_p;
    o.phi2 = d_phi2;
    o.u2 = d_u2;
    o.p2 = d_p2;
    o.dtype = dtype;
    moments_any(c, o);
    return check_launch(c);
}

int lbm_diagnostics(lbm_ctx *c, const double *d_phi_ref, lbm_diag *out) {
    clear_stale_error();
    if (!c || !out) return LBM_EINVAL;
    if (c->status == LBM_EDEVICE) return LBM_ESTATE;
    if (reduce_diag(c, d_phi_ref) != LBM_OK) return LBM_EDEVICE;
    double r[NSUM];
    if (hipMemcpyAsync(r, c->result, sizeof(r), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess) {
        c->status = LBM_EDEVICE;
        return LBM_EDEVICE;
    }
    out->step = c->t;
    out->sum_phi = r[0];
    out->mass = r[1];
    out->mom[0] = r[2];
    out->mom[1] = r[3];
    out->mom[2] = r[4];
    out->ekin = r[5];
    out->umax = r[6];
    out->phi_min = r[7];
    out->phi_max = r[8];
    for (int a = 0; a < 3; ++a) {
        out->com[a] = r[9 + a];
        out->phiu[a] = r[12 + a];
    }
    out->l2_num = r[15];
    out->l2_den = r[16];
    return LBM_OK;
}

int lbm_get_pdfs(lbm_ctx *c, double *d_f, double *d_g) {
    clear_stale_error();
    if (!c || !d_f || !d_g) return LBM_EINVAL;
    if (c->status == LBM_EDEVICE) return LBM_ESTATE;
    FieldOut o{};
    o.pdf_f = d_f;
    o.pdf_g = d_g;
    moments_any(c, o);
    return check_launch(c);
}

int lbm_set_pdfs(lbm_ctx *c, const double *d_f, const double *d_g) {
    clear_stale_error();
    if (!c || !d_f || !d_g) return LBM_EINVAL;
    if (c->status == LBM_EDEVICE) return LBM_ESTATE;
    const int prev = c->cur ^ 1;
    load_any(c, d_f, d_g, prev);
    // collide in place of a step; the loaded state's sum of phi becomes the
    // target of the phase-mass bookkeeping
    step_any(c, LOCAL, prev, c->cur, 1);
    hipLaunchKernelGGL(massfix_kernel, dim3(1), dim3(RBLOCK), 0, c->stream,
                       (const double *)c->partials, c->sums.blocks, c->mf, c->mf + 1, 1);
    c->mf_pending = false;
    c->prev_local = true;
    c->status = LBM_OK;
    return check_launch(c);
}

int64_t lbm_time(const lbm_ctx *c) { return c ? c->t : -1; }

void lbm_destroy(lbm_ctx *c) { delete c; }

const char *lbm_strerror(int status) {
    switch (status) {
        case LBM_OK: return "ok";
        case LBM_EINVAL: return "invalid argument";
        case LBM_ENOMEM: return "workspace too small";
        case LBM_EDEVICE: return "HIP device error";
        case LBM_EUNSTABLE: return "simulation became unstable";
        case LBM_ESTATE: return "context is in an error state";
        default: return "unknown status";
    }
}

}  // extern "C"
