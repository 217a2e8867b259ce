// Reactive porosity waves (thesis article 3; the appendix reactive script):
// the fused pseudo-transient sweep, the pseudo-step reduction and the host
// side of the C ABI declared in include/ptwaves.h.
//
// One launch is one PT iteration on the four iterated cell fields (Xs, Pf,
// phi, dPf/dt) from iteration-k values.  The only neighbour data are Pf and
// the permeability k(phi) of the six face neighbours (the Darcy flux of each
// face), so a W x H block owns a (W-2) x (H-2) column of cells plus a
// one-cell halo ring and marches up a chunk of planes: per plane it stages
// Pf and k in LDS (double-buffered: one barrier per plane), keeps the plane
// above of its own column and the flux from the one below in registers, and
// updates its tile cells.  Bound by HBM on large grids, by a wave's chain of
// instructions on small ones; loads and stores go through buffer descriptors
// whose range check replaces the edges' branches, so that a step waits for
// its own plane's loads alone (see the two-phase sweep, iter_kernel.hip).
// The check variant (every nup-th iteration) also takes the maximum of
// k/beta_P over its output porosity, which the next pseudo step needs, so
// that only the first pseudo step of a physical step reads the porosity
// in a pass of its own.
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "plane.h"
#include "pt_internal.h"
#include "ptwaves.h"

// Multiply-adds are fused where an expression of the source has one: every
// tile and the check variant round alike.
#pragma clang fp contract(on)

namespace ptk {
namespace {

// Tiles of the sweep and their cost (pick_tile, constants in us; rms error 14 %
// over 340 measured launches from 8 x 8 x 32 to 95 x 95 x 380, where the tile
// picked is the fastest measured or within 1 % of it).  Where the fields outgrow the
// last-level cache, one block at a time on each compute unit: two interleave
// their planes' accesses in memory (255 x 255 x 1020 1118 -> 1080 us, 506 x
// 506 x 2042 1 % less; the request for LDS keeps the second one away).
// Measured, one tile of 66 x 12 threads -> these: 31 x 31 x 124 10.7 -> 5.5 us,
// 64 x 60 x 250 19.8 -> 15.7, 95 x 95 x 380 78 -> 60, 127 x 127 x 508 170 -> 137,
// 255 x 255 x 1020 1451 -> 1080, 506 x 506 x 2042 9.34 -> 8.75 ms.
constexpr TileShape WAVE_TILES[] = {{66, 10}, {34, 14}, {34, 10}, {34, 6}, {34, 4}};
constexpr unsigned ONE_BLOCK_LDS = 80 * 1024;   // bytes, beside the kernel's own
inline TileShape waves_tile(const Geom& g) {
    const SweepCost cost{0.31, 0.089, 0.135, 0.195, 0.73, 88.0};
    const bool cached = (double)g.nx * g.ny * g.nz * cost.cell_bytes <= LAST_LEVEL_CACHE;
    // (past the cache the two larger tiles, unless their rows are too wide)
    const int n = cached || !rows_fit(g, WAVE_TILES[0].h, 8) ? 5 : 2;
    return pick_tile(
        g, cost, WAVE_TILES, n, 8, [](const TileShape&, bool fits) { return fits ? 28 : 1; },
        [](const TileShape&, bool) { return 1.0; });
}
constexpr int RB = 256;  // threads of the reduction kernels

struct WavesCoef {
    double dxi, dyi, dzi, rfg;           // 1/dx, ..., rho_f g
    double hxx, hyy;                     // -1/(2 dx^2), -1/(2 dy^2)
    double phi0_inv, k_muf0, eta_inv;
    double beta_d, beta_s, beta_f;
    double tau_inv, beta_x, xs_half, xs_max;
    double dt, dti, phi_min, phi_max;
    double onepdx, rho_term;             // 1 + dX, 1 - rho_s/(rho_f (1 + dX))
    double h2_cpf;                       // h^2 / c_pf
};

struct WavesPtrs {
    const double *xs, *pf, *phi, *dp, *xso, *pfo, *phio;
    double *xs_o, *pf_o, *phi_o, *dp_o;
    const double* dtau;                  // pseudo step (device scalar)
    double* partials;                    // [blocks][8]: the block's error, max k/beta_P of its output
};
struct WavesArgs {
    Geom g;
    WavesCoef c;
    WavesPtrs p;
};

__device__ __forceinline__ double perm(const WavesCoef& c, double phi) {
    const double r = phi * c.phi0_inv;
    return c.k_muf0 * r * r * r;
}
__device__ __forceinline__ double beta_p(const WavesCoef& c, double phi) {
    return phi * c.beta_f + c.beta_d - (1.0 + phi) * c.beta_s;
}

template <bool NORMS, int W, int H, bool STREAM>
__global__ __launch_bounds__(W * H) void k_waves_sweep(WavesArgs args) {
    __shared__ double lds[4 * W * H + 2 * (W + 1)];   // Pf and k of two planes, a margin for the rim's reads
    const Geom& g = args.g;
    const WavesCoef& c = args.c;
    const int gx = (g.nx + W - 3) / (W - 2);
    const int gy = (g.ny + H - 3) / (H - 2);
    const int64_t Tt = xcd_tile(blockIdx.x, (int64_t)gridDim.x);
    const int bx = (int)(Tt % gx), by = (int)((Tt / gx) % gy), bz = (int)(Tt / ((int64_t)gx * gy));
    int tx, ty;
    tile_thread<W, H>(tx, ty);
    const int i = bx * (W - 2) - 1 + tx;
    const int j = by * (H - 2) - 1 + ty;
    const int kz0 = bz * g.kz, kz1 = min(g.nz, kz0 + g.kz);
    const bool in_tile = tx >= 1 && tx <= W - 2 && ty >= 1 && ty <= H - 2;
    const bool tile = in_tile && i < g.nx && j < g.ny;
    const bool tile_wave = __builtin_amdgcn_ballot_w64(in_tile) != 0;

    // Byte offsets in the tile's rows: every column takes the nearest cell's
    // Pf and k (no flux comes out through the walls), only tile cells the rest.
    const int row0 = max(by * (H - 2) - 1, 0), rows = min(by * (H - 2) + H - 2, g.ny) - row0 + 1;
    const int64_t tile0 = (int64_t)row0 * g.P;
    const u32 o_near = ((u32)(min(max(j, 0), g.ny - 1) - row0) * (u32)g.P + (u32)min(max(i, 0), g.nx - 1)) * 8u;
    const u32 o_out = tile ? o_near : OFF_NONE;
    const u32 bytes = (u32)rows * (u32)g.P * 8u;
    const double dtau = *args.p.dtau;

    using KPtrs = const __attribute__((address_space(4))) WavesPtrs;
    KPtrs* const kargs = (KPtrs*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                                  offsetof(WavesArgs, p));
    auto ptrs = [&]() {
        KPtrs* q = kargs;
        asm volatile("" : "+s"(q));   // pointers read at each step (see the two-phase sweep)
        return q;
    };

    // (as in the two-phase sweep: past the last-level cache's size, what is
    // read once and what is written bypass the caches)
    constexpr int ONCE = STREAM ? NONTEMPORAL : 0;
    struct QSet { double pf, phi; };              // plane p+1 of the own column
    struct CSet { double xs, dp, xso, pfo, phio; };   // tile-only values of plane p
    struct OSet { double xs, pf, phi, dp; };
    auto load_q = [&](KPtrs* p, int k, QSet& q) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = (k >= 0 && k < g.nz) ? bytes : 0u;
        q.pf = ldp(p->pf + o, nb, o_near);
        q.phi = ldp(p->phi + o, nb, o_near);
    };
    auto load_c = [&](KPtrs* p, int k, CSet& q) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = k < kz1 ? bytes : 0u;
        q.xs = ldp<ONCE>(p->xs + o, nb, o_out);
        q.dp = ldp<ONCE>(p->dp + o, nb, o_out);
        q.xso = ldp<ONCE>(p->xso + o, nb, o_out);
        q.pfo = ldp<ONCE>(p->pfo + o, nb, o_out);
        q.phio = ldp<ONCE>(p->phio + o, nb, o_out);
    };
    auto store = [&](KPtrs* p, int k, u32 nb, const OSet& v) {
        const int64_t o = (int64_t)k * g.S + tile0;
        stp<ONCE>(p->xs_o + o, nb, o_out, v.xs);
        stp<ONCE>(p->pf_o + o, nb, o_out, v.pf);
        stp<ONCE>(p->phi_o + o, nb, o_out, v.phi);
        stp<ONCE>(p->dp_o + o, nb, o_out, v.dp);
    };

    double* const me = lds + (W + 1) + ty * W + tx;
    auto sh = [&](int pl, int dx, int dy) -> double& { return me[pl * (W * H) + dy * W + dx]; };

    // own column: Pf, k and phi of plane p, the Darcy flux through the level below it
    double pf_c, kc_c, phi_c, qz_c;
    double err = 0.0, kmax = 0.0;

    auto flux_z = [&](int lev, double pf_lo, double k_lo, double pf_hi, double k_hi) {
        // through the level between planes lev-1 and lev, zero through the walls;
        // rounded before it enters a difference
#pragma clang fp contract(off)
        const double h = (lev > 0 && lev < g.nz) ? -0.5 : 0.0;
        return h * (k_lo + k_hi) * ((pf_hi - pf_lo) * c.dzi - c.rfg);
    };

    auto step = [&](int pz, const QSet& qn, QSet& qnn, const CSet& cc, CSet& cn) __attribute__((always_inline)) {
        const int b = 2 * (pz & 1);
        KPtrs* const p = ptrs();
        load_q(p, pz + 2, qnn);
        load_c(p, pz + 1, cn);
        sh(b, 0, 0) = pf_c;
        sh(b + 1, 0, 0) = kc_c;
        const double pf_n = qn.pf, phi_n = qn.phi;
        const double kc_n = perm(c, phi_n);
        __syncthreads();
        OSet out{};
        if (tile_wave) {
            // Darcy flux of the six faces (zero through the walls), eq (8)'s divergence
            double qx, qy;
            {
#pragma clang fp contract(off)
                qx = (kc_c + sh(b + 1, 1, 0)) * (sh(b, 1, 0) - pf_c) - (sh(b + 1, -1, 0) + kc_c) * (pf_c - sh(b, -1, 0));
                qy = (kc_c + sh(b + 1, 0, 1)) * (sh(b, 0, 1) - pf_c) - (sh(b + 1, 0, -1) + kc_c) * (pf_c - sh(b, 0, -1));
            }
            const double qz_n = flux_z(pz + 1, pf_c, kc_c, pf_n, kc_n);
            const double divq = c.hxx * qx + c.hyy * qy + (qz_n - qz_c) * c.dzi;
            qz_c = qz_n;

            const double xs = cc.xs, dp = cc.dp;
            const double xseq = fmin(fmax(c.beta_x * pf_c + c.xs_half, 0.0), c.xs_max);
            const double bp = beta_p(c, phi_c);
            const double s = 1.0 - phi_c, s_inv = quot(1.0, s);
            const double bphi = c.beta_d - c.beta_s * s_inv;
            const double dxsdt = (xseq - xs) * c.tau_inv;
            const double compaction = -pf_c * c.eta_inv * s_inv;
            const double react = quot(c.onepdx, 1.0 - xs) * dxsdt;
            out.xs = cc.xso + c.dt * dxsdt;
            out.pf = pf_c + dtau * dp - dtau * (pf_c - cc.pfo) * c.dti;
            const double dphidt = s * (bphi * dp - compaction - react);
            out.phi = fmin(fmax(cc.phio + c.dt * dphidt, c.phi_min), c.phi_max);
            out.dp = quot(-divq + compaction + c.rho_term * s * react, bp);
            if (NORMS && tile) {
                err = nanmax(err, fabs(out.phi - phi_c));
                err = nanmax(err, fabs(out.pf - pf_c) / 10.0);
                err = nanmax(err, fabs(out.xs - xs));
                // the next pseudo step's maximum, over this iteration's output
                kmax = nanmax(kmax, perm(c, out.phi) / beta_p(c, out.phi));
            }
        }
        store(ptrs(), pz, bytes, out);
        pf_c = fresh(pf_n);
        kc_c = kc_n;
        phi_c = fresh(phi_n);
    };

    QSet qa, qb;
    CSet ca, cb;
    {
        KPtrs* const p = ptrs();
        QSet q0, q1;
        load_q(p, kz0 - 1, q0);
        load_q(p, kz0, q1);
        load_q(p, kz0 + 1, qa);
        load_c(p, kz0, ca);
        // as many (empty) stores as a step ends with, so that the first step
        // waits for its loads as every other does
        store(p, kz0, 0u, OSet{});
        pf_c = q1.pf;
        phi_c = q1.phi;
        kc_c = perm(c, q1.phi);
        qz_c = flux_z(kz0, q0.pf, perm(c, q0.phi), pf_c, kc_c);
    }
    for (int pz = kz0; pz < kz1; pz += 2) {
        step(pz, qa, qb, ca, cb);
        if (pz + 1 >= kz1) break;
        step(pz + 1, qb, qa, cb, ca);
    }

    if constexpr (NORMS) {
        // wave64 butterfly in each of the waves of whole tile rows (the halo
        // wave holds no tile cell), then across them through LDS
        constexpr int NW = (W - 2) * H / 64;
        __shared__ double red[2][NW];
        const int L = threadIdx.x, wave = L >> 6, lane = L & 63;
        if (wave < NW) {
            double v = err, u = kmax;
            for (int off = 32; off >= 1; off >>= 1) {
                v = nanmax(v, __shfl_xor(v, off, 64));
                u = nanmax(u, __shfl_xor(u, off, 64));
            }
            if (lane == 0) {
                red[0][wave] = v;
                red[1][wave] = u;
            }
        }
        __syncthreads();
        if (L < NNORM) {
            double r = 0.0;
            if (L < 2)
                for (int w = 0; w < NW; ++w) r = nanmax(r, red[L][w]);
            args.p.partials[(int64_t)blockIdx.x * NNORM + L] = r;
        }
    }
}

// Per-block maxima of k/beta_P over the cells (grid-stride), into partials.
__global__ __launch_bounds__(RB) void k_waves_kmax(Geom g, WavesCoef c, const double* __restrict__ phi,
                                                   double* __restrict__ partials) {
    __shared__ double red[RB / 64];
    const int64_t ncell = (int64_t)g.nx * g.ny * g.nz;
    double m = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * RB + threadIdx.x; t < ncell; t += (int64_t)gridDim.x * RB) {
        const int i = (int)(t % g.nx), j = (int)((t / g.nx) % g.ny), k = (int)(t / ((int64_t)g.nx * g.ny));
        const double f = phi[(int64_t)k * g.S + (int64_t)j * g.P + i];
        m = nanmax(m, perm(c, f) / beta_p(c, f));
    }
    for (int off = 32; off >= 1; off >>= 1) m = nanmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = 0.0;
        for (int w = 0; w < RB / 64; ++w) r = nanmax(r, red[w]);
        partials[blockIdx.x] = r;
    }
}

// dtau = h^2 / c_pf / max over the block maxima (one block).
__global__ __launch_bounds__(RB) void k_waves_dtau(const double* __restrict__ partials, int64_t nb, double h2_cpf,
                                                   double* __restrict__ dtau) {
    __shared__ double red[RB / 64];
    double m = 0.0;
    for (int64_t b = threadIdx.x; b < nb; b += RB) m = nanmax(m, partials[b]);
    for (int off = 32; off >= 1; off >>= 1) m = nanmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = 0.0;
        for (int w = 0; w < RB / 64; ++w) r = nanmax(r, red[w]);
        *dtau = h2_cpf / r;
    }
}

constexpr int64_t KMAX_BLOCKS = 2048;

}  // namespace
}  // namespace ptk

using namespace ptk;

struct pt_waves {
    Geom geom;
    pt_waves_params prm;
    WavesCoef coef;
    double* f[PT_W_NFIELDS][2];
    int cur[PT_W_NPING];
    void* ws = nullptr;
    size_t ws_bytes = 0;
    hipStream_t stream = nullptr;
    int64_t iter = 0;
    bool checked = false;
    bool kmax_fresh = false;   // the last sweep was a check: max k/beta_P of the present porosity is in hand
    TileShape tile;            // the sweep's tile on this grid
    int64_t blocks = 0;        // its blocks
    std::string err;
};

namespace {

// [sweep partials: blocks x 8][error: 8][dtau: 1][k/beta_P partials: KMAX_BLOCKS]
size_t waves_ws_needed(const pt_waves* w) {
    const int64_t n = w->blocks * NNORM + NNORM + 1 + KMAX_BLOCKS;
    return (size_t)((n + 31) / 32 * 32) * sizeof(double);
}
double* ws_partials(pt_waves* w) { return static_cast<double*>(w->ws); }
double* ws_error(pt_waves* w) { return ws_partials(w) + w->blocks * NNORM; }
double* ws_dtau(pt_waves* w) { return ws_error(w) + NNORM; }
double* ws_kmax(pt_waves* w) { return ws_dtau(w) + 1; }

pt_status wfail(pt_waves* w, pt_status s, const char* msg) {
    if (w) w->err = msg;
    return s;
}
pt_status whip(pt_waves* w, hipError_t e, const char* where) {
    if (w) w->err = std::string(where) + ": " + hipGetErrorString(e);
    return PT_EDEVICE;
}

bool waves_valid(const pt_waves_params* p) {
    if (!p || p->version != PT_WAVES_ABI_VERSION || p->nup < 1) return false;
    const double pos[] = {p->lx, p->ly, p->lz, p->phi0, p->k_muf0, p->eta, p->rho_f, p->tau, p->dt, p->c_pf};
    for (double v : pos)
        if (!(v > 0.0) || !std::isfinite(v)) return false;
    if (!(p->phi_min > 0.0 && p->phi_min <= p->phi_max && p->phi_max <= 1.0)) return false;
    if (!(p->xs_max > 0.0 && p->xs_max < 1.0) || !(p->delta_x > -1.0)) return false;
    return true;
}

void waves_coef(pt_waves* w) {
    const pt_waves_params& p = w->prm;
    WavesCoef& c = w->coef;
    const double dx = p.lx / w->geom.nx, dy = p.ly / w->geom.ny, dz = p.lz / w->geom.nz;
    const double h = std::fmin(dx, std::fmin(dy, dz));
    c.dxi = 1.0 / dx; c.dyi = 1.0 / dy; c.dzi = 1.0 / dz;
    c.rfg = p.rho_f * p.g;
    c.phi0_inv = 1.0 / p.phi0;
    c.k_muf0 = p.k_muf0;
    c.hxx = -0.5 * c.dxi * c.dxi;
    c.hyy = -0.5 * c.dyi * c.dyi;
    c.eta_inv = 1.0 / p.eta;
    c.beta_d = p.beta_d; c.beta_s = p.beta_s; c.beta_f = p.beta_f;
    c.tau_inv = 1.0 / p.tau;
    c.beta_x = p.beta_x;
    c.xs_half = 0.5 * p.xs_max;
    c.xs_max = p.xs_max;
    c.dt = p.dt; c.dti = 1.0 / p.dt;
    c.phi_min = p.phi_min; c.phi_max = p.phi_max;
    c.onepdx = 1.0 + p.delta_x;
    c.rho_term = 1.0 - p.rho_s / (p.rho_f * (1.0 + p.delta_x));
    c.h2_cpf = h * h / p.c_pf;
}

pt_status waves_ready(pt_waves* w) {
    for (int f = 0; f < PT_W_NFIELDS; ++f) {
        if (!w->f[f][0]) return wfail(w, PT_EINVAL, "not every field is bound");
        if (f < PT_W_NPING && !w->f[f][1]) return wfail(w, PT_EINVAL, "both copies of the iterated fields must be bound");
    }
    if (!w->ws || w->ws_bytes < waves_ws_needed(w)) return wfail(w, PT_EINVAL, "workspace not bound or too small");
    return PT_OK;
}

double* wcur(pt_waves* w, int f) { return f < PT_W_NPING ? w->f[f][w->cur[f]] : w->f[f][0]; }
double* walt(pt_waves* w, int f) { return w->f[f][1 - w->cur[f]]; }

template <bool NORMS, int W, int H, bool STREAM>
hipError_t launch_waves_tile(pt_waves* w, const WavesPtrs& p) {
    if (!rows_fit(w->geom, H, sizeof(double))) return hipErrorInvalidValue;
    WavesArgs a{w->geom, w->coef, p};
    a.g.kz = w->tile.kz;
    hipLaunchKernelGGL((k_waves_sweep<NORMS, W, H, STREAM>), dim3((unsigned)w->blocks), dim3(W * H),
                       STREAM ? ONE_BLOCK_LDS : 0, w->stream, a);
    return hipGetLastError();
}
template <bool NORMS>
hipError_t launch_waves(pt_waves* w, const WavesPtrs& p) {
    const int wh = w->tile.w * 100 + w->tile.h;
    if (w->tile.stream) {
        if (wh == 6610) return launch_waves_tile<NORMS, 66, 10, true>(w, p);
        if (wh == 3414) return launch_waves_tile<NORMS, 34, 14, true>(w, p);
    }
    switch (wh) {
        case 6610: return launch_waves_tile<NORMS, 66, 10, false>(w, p);
        case 3414: return launch_waves_tile<NORMS, 34, 14, false>(w, p);
        case 3410: return launch_waves_tile<NORMS, 34, 10, false>(w, p);
        case 3406: return launch_waves_tile<NORMS, 34, 6, false>(w, p);
        case 3404: return launch_waves_tile<NORMS, 34, 4, false>(w, p);
    }
    return hipErrorInvalidValue;
}

pt_status waves_iteration(pt_waves* w, bool refresh_dtau, bool norms) {
    hipError_t e = hipSuccess;
    if (refresh_dtau) {
        if (w->kmax_fresh) {
            // the check sweep just before took the maximum over its output
            hipLaunchKernelGGL(k_waves_dtau, dim3(1), dim3(RB), 0, w->stream, ws_error(w) + 1, (int64_t)1,
                               w->coef.h2_cpf, ws_dtau(w));
        } else {
            const int64_t ncell = (int64_t)w->geom.nx * w->geom.ny * w->geom.nz;
            const int64_t nb = std::min<int64_t>(KMAX_BLOCKS, (ncell + RB - 1) / RB);
            hipLaunchKernelGGL(k_waves_kmax, dim3((unsigned)nb), dim3(RB), 0, w->stream, w->geom, w->coef,
                               wcur(w, PT_W_PHI), ws_kmax(w));
            hipLaunchKernelGGL(k_waves_dtau, dim3(1), dim3(RB), 0, w->stream, ws_kmax(w), nb, w->coef.h2_cpf,
                               ws_dtau(w));
        }
        e = hipGetLastError();
        if (e != hipSuccess) return whip(w, e, "pseudo step");
    }
    WavesPtrs p{};
    p.xs = wcur(w, PT_W_XS); p.pf = wcur(w, PT_W_PF); p.phi = wcur(w, PT_W_PHI); p.dp = wcur(w, PT_W_DPFDT);
    p.xso = wcur(w, PT_W_XSO); p.pfo = wcur(w, PT_W_PFO); p.phio = wcur(w, PT_W_PHIO);
    p.xs_o = walt(w, PT_W_XS); p.pf_o = walt(w, PT_W_PF); p.phi_o = walt(w, PT_W_PHI); p.dp_o = walt(w, PT_W_DPFDT);
    p.dtau = ws_dtau(w);
    p.partials = ws_partials(w);
    e = norms ? launch_waves<true>(w, p) : launch_waves<false>(w, p);
    if (e != hipSuccess) return whip(w, e, "waves sweep");
    if (norms) {
        e = launch_reduce_max(ws_partials(w), w->blocks, ws_error(w), w->stream);
        if (e != hipSuccess) return whip(w, e, "waves error");
        w->checked = true;
    }
    w->kmax_fresh = norms;
    for (int f = 0; f < PT_W_NPING; ++f) w->cur[f] ^= 1;
    w->iter += 1;
    return PT_OK;
}

pt_status waves_read_error(pt_waves* w, double* err) {
    double host = 0.0;
    hipError_t e = hipMemcpyAsync(&host, ws_error(w), sizeof(double), hipMemcpyDeviceToHost, w->stream);
    const hipError_t es = hipStreamSynchronize(w->stream);
    if (e == hipSuccess) e = es;
    if (e != hipSuccess) return whip(w, e, "error copy");
    *err = host;
    if (!std::isfinite(host)) return wfail(w, PT_EDIVERGED, "non-finite stopping quantity");
    return PT_OK;
}

}  // namespace

extern "C" {

pt_status pt_waves_create(int32_t nx, int32_t ny, int32_t nz, int64_t row_pitch, const pt_waves_params* params,
                          pt_waves** out) {
    if (!out) return PT_EINVAL;
    *out = nullptr;
    if (nx < 2 || ny < 2 || nz < 2 || row_pitch < (int64_t)nx + 1 || !waves_valid(params)) return PT_EINVAL;
    pt_waves* w = new (std::nothrow) pt_waves();
    if (!w) return PT_EINVAL;
    w->geom.nx = nx; w->geom.ny = ny; w->geom.nz = nz;
    w->geom.P = row_pitch;
    w->geom.S = row_pitch * (int64_t)(ny + 1);
    w->geom.kz = KZ_MAX;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
        w->geom.cus = cus;
    (void)hipGetLastError();
    w->tile = waves_tile(w->geom);
    w->blocks = sweep_blocks(w->geom, w->tile);
    w->prm = *params;
    std::memset(w->f, 0, sizeof(w->f));
    std::memset(w->cur, 0, sizeof(w->cur));
    waves_coef(w);
    *out = w;
    return PT_OK;
}

pt_status pt_waves_destroy(pt_waves* w) {
    delete w;
    return PT_OK;
}

int64_t pt_waves_field_elems(const pt_waves* w) { return w ? w->geom.S * (int64_t)(w->geom.nz + 1) : 0; }

pt_status pt_waves_bind_field(pt_waves* w, int32_t field, int32_t copy, void* dev_ptr) {
    if (!w) return PT_EINVAL;
    if (field < 0 || field >= PT_W_NFIELDS) return wfail(w, PT_EINVAL, "bad field id");
    if (copy < 0 || copy > 1 || (copy == 1 && field >= PT_W_NPING)) return wfail(w, PT_EINVAL, "bad copy index");
    if (!dev_ptr || (reinterpret_cast<uintptr_t>(dev_ptr) & 255u)) return wfail(w, PT_EINVAL, "null or unaligned pointer");
    w->f[field][copy] = static_cast<double*>(dev_ptr);
    return PT_OK;
}

pt_status pt_waves_workspace_size(const pt_waves* w, size_t* bytes) {
    if (!w || !bytes) return PT_EINVAL;
    *bytes = waves_ws_needed(w);
    return PT_OK;
}

pt_status pt_waves_bind_workspace(pt_waves* w, void* dev_ptr, size_t bytes) {
    if (!w) return PT_EINVAL;
    if (!dev_ptr || (reinterpret_cast<uintptr_t>(dev_ptr) & 255u) || bytes < waves_ws_needed(w))
        return wfail(w, PT_EINVAL, "workspace missing, unaligned or too small");
    w->ws = dev_ptr;
    w->ws_bytes = bytes;
    return PT_OK;
}

pt_status pt_waves_set_stream(pt_waves* w, void* hip_stream) {
    if (!w) return PT_EINVAL;
    w->stream = static_cast<hipStream_t>(hip_stream);
    return PT_OK;
}

pt_status pt_waves_current(const pt_waves* w, int32_t field, int32_t* copy) {
    if (!w || !copy || field < 0 || field >= PT_W_NFIELDS) return PT_EINVAL;
    *copy = field < PT_W_NPING ? w->cur[field] : 0;
    return PT_OK;
}

pt_status pt_waves_begin_step(pt_waves* w) {
    if (!w) return PT_EINVAL;
    pt_status st = waves_ready(w);
    if (st != PT_OK) return st;
    const int64_t n = w->geom.S * (int64_t)(w->geom.nz + 1);
    const int pairs[3][2] = {{PT_W_XS, PT_W_XSO}, {PT_W_PF, PT_W_PFO}, {PT_W_PHI, PT_W_PHIO}};
    for (auto& pr : pairs) {
        hipError_t e = launch_copy(wcur(w, pr[0]), w->f[pr[1]][0], n, w->stream);
        if (e != hipSuccess) return whip(w, e, "old values");
    }
    w->iter = 0;
    w->kmax_fresh = false;
    return PT_OK;
}

pt_status pt_waves_iterate(pt_waves* w, int64_t n) {
    if (!w || n < 0) return PT_EINVAL;
    pt_status st = waves_ready(w);
    if (st != PT_OK) return st;
    const int64_t nup = w->prm.nup;
    for (int64_t m = 0; m < n; ++m) {
        const int64_t it = w->iter + 1;
        st = waves_iteration(w, (it - 1) % nup == 0, it % nup == 0);
        if (st != PT_OK) return st;
    }
    return PT_OK;
}

pt_status pt_waves_last_error(pt_waves* w, double* err) {
    if (!w || !err) return PT_EINVAL;
    if (!w->checked) return wfail(w, PT_EINVAL, "no stopping quantity computed yet");
    return waves_read_error(w, err);
}

pt_status pt_waves_solve_step(pt_waves* w, double eps, int64_t iter_max, int64_t* iters, double* err) {
    if (!w || !(eps > 0.0) || iter_max < 1) return PT_EINVAL;
    pt_status st = waves_ready(w);
    if (st != PT_OK) return st;
    const int64_t nup = w->prm.nup;
    double e = INFINITY;
    while (w->iter < iter_max) {
        const int64_t chunk = std::min<int64_t>(nup - (w->iter % nup), iter_max - w->iter);
        st = pt_waves_iterate(w, chunk);
        if (st != PT_OK) return st;
        if (w->iter % nup == 0) {
            st = waves_read_error(w, &e);
            if (st != PT_OK) break;
            if (e < eps) break;
        }
    }
    if (iters) *iters = w->iter;
    if (err) *err = e;
    if (st != PT_OK) return st;
    return (e < eps) ? PT_OK : PT_ENOTCONV;
}

const char* pt_waves_last_message(const pt_waves* w) { return w ? w->err.c_str() : "null handle"; }

}  // extern "C"
