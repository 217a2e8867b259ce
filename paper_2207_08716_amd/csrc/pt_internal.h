// Internal definitions shared by the kernels and the host side of the library.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdint.h>

#include "ptporo.h"

namespace ptk {

// Compute units assumed when the device cannot be queried (MI355X: 256).
constexpr int DEFAULT_CUS = 256;

// Index layout common to every field: (k * (ny+1) + j) * P + i.
struct Geom {
    int nx, ny, nz;
    int64_t P;   // row pitch (elements)
    int64_t S;   // plane pitch = (ny + 1) * P
    int kz;      // planes per z chunk of a sweep (set per sweep variant at launch)
    int cus = DEFAULT_CUS;   // compute units of the device (one sweep block each)
    int tall32 = 0;          // FP32 correction sweep: always the 14-row tiles
};

// Physical and numerical constants, in the form the kernels use them.
struct Coef {
    double dxi, dyi, dzi;          // 1/dx, 1/dy, 1/dz
    double dt, dti;                // dt, 1/dt
    double beta_d, alpha, B, beta_phi;
    double rhofg, rhosg;           // fluid / solid density x g
    double rhobg;                  // background density x g
    double buoy;                   // rhofg - rhobg (Darcy flux term, z up)
    double gdts_inv;               // 1 / (G dtS)
    double beta_n;
    double rho_i_inv;
    double dtauv_c;                // rho_i h^2 / (c_v (1 + beta_n)):  dtau_V = dtauv_c / mu_s
    double dtaupt_c;               // (1 + beta_n) / n_max:          dtau_Pt = dtaupt_c * mu_s
    double dtaupf_c;               // h^2 (1 + beta_d B/alpha) / c_pf: dtau_Pf = dtaupf_c / k_loc
    double dampx, dampy, dampz;    // 1 - damp_c / n
    double ab;                     // alpha / B
    double third;                  // 1/3
    double gbg_half;               // half the background shear rate (xy strain rate of eq (32)), 0: none
    int mech_off;
    // FP64 sweeps: the rx..rz inputs hold the stored damped residual R
    // (rform) or the previous velocity iterate; rwrite: store R' (see the
    // sweep's header).  The correction sweeps always read and store R.
    int rform = 1;
    int rwrite = 1;
    int undamped = 0;              // linear sweep without damping (the multigrid smoother): no R at all
};

// Sweep modes (see iter_kernel.hip).
constexpr int MD_THESIS = 0;   // FP64, porosity updated
constexpr int MD_LINEAR = 1;   // FP64, porosity frozen
constexpr int MD_RESID = 2;    // FP64, residuals of the present state only
constexpr int MD_CORR = 3;     // FP32 correction sweep

// Pointers of one sweep (inputs at iteration k, outputs at k + 1).  In the
// correction mode the slots carry: vx..rz = correction d and its damped
// residual; pto = r_Pt(x), pfo = r_Pf(x), fox..foz = momentum residual f(x);
// eta = 1/((1-phi) eta_phi); kc, mus = FP32 copies of the coefficients.
template <typename T>
struct SweepPtrs {
    const T *vx, *vy, *vz, *pt, *pf, *lp, *rx, *ry, *rz;
    const T *fox, *foy, *foz, *pto, *pfo, *lpo, *kc, *eta, *mus;
    T *vx_o, *vy_o, *vz_o, *pt_o, *pf_o, *lp_o, *rx_o, *ry_o, *rz_o;
    float *res_fx, *res_fy, *res_fz, *res_rpt, *res_rpf;   // residual mode outputs
    double* partials;              // [n_blocks][8] maxima (norm variants)
    double* domain;                // set to 1 where ln(1-phi)' leaves (-inf, 0) (thesis mode)
    const double* gate;            // not 0 there: the solve this sweep belongs to has ended (null: no gate)
};

constexpr int NNORM = 8;

// Tiles of the z-marching kernels: a W x H thread block covers a (W-2) x
// (H-2) output tile plus one halo column/row on every side and marches in z.
// W = 66 makes the output tile 64 columns wide: its rows start on 512-byte
// boundaries of the padded rows (whole cache lines written) and n = 2^k - 1
// grids fill their last tile; each row's 64 interior columns are one wave,
// the side halo columns of all rows one more (partial) wave.  Every cell's
// arithmetic is the same in every tiling.  The sweeps choose theirs per
// grid (sweep_shape).
constexpr int BX = 66;
constexpr int BY = 10;         // FP64 sweeps on large grids
constexpr int BY_CORR32 = 14;  // FP32 correction sweep (large grids)
constexpr int BY_CORR32_SHORT = 10;   // FP32 correction sweep where its tiling costs less
constexpr int KZ_MAX = 256;

constexpr int KZ_MIN = 4;

inline int64_t tiles_xy(const Geom& g, int bx = BX, int by = BY) {
    return (int64_t)((g.nx + bx - 3) / (bx - 2)) * ((g.ny + by - 3) / (by - 2));
}

// Planes per z chunk for a tiling: the sweep blocks occupy one CU each, so a
// launch takes ceil(blocks / CUs) rounds of (chunk + 2) plane steps (two
// planes of halo and prefetch per chunk); the chunk minimising that wins,
// the longer one on ties.  (Serves the preference among the FP32 tiles and the
// grids that the static scratch refuses; the launches take pick_tile's chunks.)
inline int choose_kz(const Geom& g, int bx, int by, int64_t* cost_out = nullptr) {
    const int64_t t = tiles_xy(g, bx, by);
    int best = KZ_MAX;
    int64_t best_cost = -1;
    for (int kz = KZ_MAX; kz >= KZ_MIN; kz /= 2) {
        const int64_t blocks = t * ((g.nz + kz - 1) / kz);
        const int64_t cus = g.cus > 0 ? g.cus : DEFAULT_CUS;
        const int64_t cost = ((blocks + cus - 1) / cus) * (std::min(kz, g.nz) + 2);
        if (best_cost < 0 || cost < best_cost) {
            best = kz;
            best_cost = cost;
        }
    }
    if (cost_out) *cost_out = best_cost;
    return best;
}

// Cost of a tiling in units of row-plane steps: a block's plane step is
// proportional to its rows, so the best chunk's cost times the block height.
inline int64_t tiling_cost(const Geom& g, int bx, int by) {
    int64_t c = 0;
    choose_kz(g, bx, by, &c);
    return c * by;
}

// Whether the FP32 correction sweep's 10-row tiling costs less rows than its
// 14-row one (see sweep_shape).
inline bool corr32_short(const Geom& g) {
    if (g.tall32) return false;
    return tiling_cost(g, BX, BY_CORR32_SHORT) < tiling_cost(g, BX, BY_CORR32);
}

// The geometry of one sweep variant: its z chunk set.
inline Geom sweep_geom(const Geom& g, int bx, int by) {
    Geom v = g;
    v.kz = choose_kz(g, bx, by);
    return v;
}

inline int64_t iter_grid_blocks(const Geom& g, int bx, int by) {
    const Geom v = sweep_geom(g, bx, by);
    return tiles_xy(v, bx, by) * ((v.nz + v.kz - 1) / v.kz);
}

// Tile order of the z-marching kernels: consecutive tiles go to the same XCD
// (blocks are dealt to the eight XCDs round robin), so tiles that share halo
// planes share an L2.
__device__ __forceinline__ int64_t xcd_tile(int64_t L, int64_t total) {
    const int64_t nx = 8;
    int64_t xcd = L % nx, idx = L / nx;
    int64_t q = total / nx, r = total % nx;
    return (xcd < r) ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// Thread layout of a W x H tile block (one-dimensional launch of W*H
// threads): first the W-2 interior columns of every row, row after row, then
// the two side halo columns of all rows.  In 66-wide blocks wave r (r < H) so
// takes the 64 interior columns of row r: every load and store of a row is
// one whole, aligned 512-byte segment.
template <int W, int H>
__device__ __forceinline__ void tile_thread(int& tx, int& ty) {
    static_assert(W == 66 || W == 34, "tiles are 64 or 32 columns wide");
    constexpr int C = W - 2;
    const int L = threadIdx.x;
    if (L < C * H) {
        tx = 1 + L % C;
        ty = L / C;
    } else {
        const int r = L - C * H;
        tx = (r < H) ? 0 : W - 1;
        ty = (r < H) ? r : r - H;
    }
}

// ---- tile of a sweep launch ----------------------------------------------------
// Blocks of w x h threads (w - 2 by h - 2 output columns and rows) over
// chunks of kz planes.
struct TileShape {
    int w = 0, h = 0, kz = 0;
    bool stream = false;   // the grid's fields outgrow the last-level cache
};

// Waves per SIMD that a sweep block of n threads is compiled for: what it has
// itself, but three for small blocks, of which several share a compute unit.
// (The FP64 sweeps with norms need more registers: two.)
constexpr int sweep_waves(int n, bool norms = false) {
    return n > 768 ? 4 : (norms || (n > 448 && n <= 512)) ? 2 : 3;
}

// Sweep variants by what their blocks take of a compute unit.
enum SweepKind { SK_F64, SK_F32, SK_NORM64, SK_NORM32 };

// A launch's time, for choosing its tiles.  A compute unit runs its share of
// the blocks, as many at a time as its registers hold; a plane step of n
// resident waves takes max(step + wave n, full n): at first latency, then
// the vector units or, for grids whose fields outgrow the last-level cache,
// memory; a block's march takes its chunk's planes and `lead` more.  The
// constants (in us) fit 900 measured launches (12 tiles, 2 to 12 chunk
// lengths, grids of 8^3 to 255^3, thesis, linear and FP32 correction
// sweeps) within 10 %; the tile it picks is within 1.5 % of the fastest of
// all those measured in FP64 and 2.2 % in FP32 (geometric mean), against
// 40 % for one tile of 66 x 10 threads: linear sweep 20.6 -> 6.7 us at 16^3,
// 20.7 -> 7.5 at 32^3, 23.5 -> 16.7 at 64^3, 68.6 -> 40.1 at 95^3,
// 121 -> 97 at 173 x 131 x 97.
// (Fitted before the loads were spread over the plane step; since then, on 14
// grids of 16^3 to 150 x 128 x 101, the tile it picks was within 3 % of the
// fastest of all, at 40^3 within 10 % (11.9 us on 66 x 10 threads, 11.1 on
// 66 x 6), and the linear sweep takes 6.4 us at 16^3, 7.0 at 32^3, 14.0 at
// 64^3, 31.4 at 95^3, 65.8 at 127^3.)
struct SweepCost {
    double step, wave, full_cached, full_memory, lead;
    double cell_bytes;   // streamed per cell
};
inline SweepCost sweep_cost(SweepKind k) {
    if (k == SK_F32 || k == SK_NORM32) return {0.65, 0.105, 0.126, 0.20, 1.4, 84.0};
    return {1.1, 0.2, 0.28, 0.38, 1.8, 192.0};
}
constexpr double LAST_LEVEL_CACHE = 256.0e6;   // bytes

// Tiles each variant is built for, larger ones first.
constexpr int SWEEP_SHAPES = 5;
inline const TileShape* sweep_shapes(SweepKind k, int& n) {
    static constexpr TileShape f64[SWEEP_SHAPES] = {{66, 10}, {66, 6}, {34, 14}, {34, 6}, {34, 4}};
    static constexpr TileShape f32[SWEEP_SHAPES] = {{66, 14}, {66, 10}, {66, 6}, {34, 14}, {34, 6}};
    static constexpr TileShape norms[4] = {{66, 7}, {34, 14}, {34, 6}, {34, 4}};
    if (k == SK_F64) { n = 5; return f64; }
    if (k == SK_F32) { n = 5; return f32; }
    n = 4;
    return norms;
}

// Blocks of a launch with a tile shape.
inline int64_t sweep_blocks(const Geom& g, const TileShape& t) {
    return tiles_xy(g, t.w, t.h) * ((g.nz + t.kz - 1) / t.kz);
}

// Whether the rows that a tile of h rows holds of a plane (of the box's ny + 1
// at most) lie within 2 GiB, which the kernels' 32-bit offsets reach.
inline bool rows_fit(const Geom& g, int h, int elem_bytes) {
    return g.P <= (int64_t)0x7fffffff / ((int64_t)std::min(h, g.ny + 1) * elem_bytes);
}

// The cheapest tile and chunk by the model above, over those of the n shapes
// given whose rows fit and, for each, the chunks that fill 1 to 16 blocks per
// compute unit (no more than 4096 blocks beyond the first).  held: waves of a
// shape's blocks that a compute unit's registers hold; weight: a factor on a
// shape's cost.  (Where no shape's rows fit, the last shape, whose launch is
// refused.)
template <typename Held, typename Weight>
inline TileShape pick_tile(const Geom& g, const SweepCost& sc, const TileShape* shapes, int n, int elem_bytes, Held held,
                           Weight weight) {
    const int cus = g.cus > 0 ? g.cus : DEFAULT_CUS;
    const bool cached = (double)g.nx * g.ny * g.nz * sc.cell_bytes <= LAST_LEVEL_CACHE;
    const double full = cached ? sc.full_cached : sc.full_memory;
    TileShape best = shapes[n - 1];
    best.kz = std::min(g.nz, KZ_MAX);
    double best_cost = -1.0;
    for (int q = 0; q < n; ++q) {
        if (!rows_fit(g, shapes[q].h, elem_bytes)) continue;
        TileShape t = shapes[q];
        t.stream = !cached;
        const int64_t tiles = tiles_xy(g, t.w, t.h);
        const int nw = (t.w * t.h + 63) / 64;
        const int res = std::max(1, held(t, cached) / nw);
        const double fac = weight(t, cached);
        auto step = [&](int64_t blocks) { return std::max(sc.step + sc.wave * blocks * nw, full * blocks * nw); };
        int last = 0;
        for (int m = 1; m <= 16; ++m) {
            const int64_t chunks = std::min<int64_t>(std::max<int64_t>(m * (int64_t)cus / tiles, 1), g.nz);
            t.kz = std::min((int)((g.nz + chunks - 1) / chunks), KZ_MAX);
            if (t.kz != last) {
                last = t.kz;
                const int64_t blocks = tiles * ((g.nz + t.kz - 1) / t.kz);
                if (m > 1 && blocks > 4096) break;
                const int64_t per_cu = (blocks + cus - 1) / cus;
                const int64_t rounds = per_cu / res, rest = per_cu % res;
                const double cost = fac * (t.kz + sc.lead) * (rounds * step(res) + (rest ? step(rest) : 0.0));
                if (best_cost < 0.0 || cost < best_cost * (1.0 - 1e-9)) {
                    best = t;
                    best_cost = cost;
                }
            }
            if (t.kz == 1) break;
        }
    }
    return best;
}

// The tile of a sweep.  Tiles half as wide cost 15 % more where the fields
// come from memory (rows of 256 bytes; 34 x 14 against 66 x 10 threads at
// 180^3: 284 and 255 us, at 383^3: 2.32 and 2.15 ms, at equal model cost).  Of
// the FP32 sweep's 64-column tiles, the 14-row ones are preferred where their
// tiling costs less rows (corr32_short: it decides where the model has both
// nearly equal, as at 200^3, 168 us against 171 on 10 rows), and run alone if
// asked for.  Measured, 14 and 10 rows, where the rule takes 14: 150^3 70 and
// 74 us, 300^3 498 and 537, 383^3 1.02 and 1.09 ms, 511^3 2.42 and 2.55; where
// it takes 10: 64^3 11.2 and 9.7 us, 255^3 300 and 272, 127^3 34 either way;
// at 173 x 131 x 97 43.7 on the 34 x 14 it takes, 42.0 on 14 rows (per sweep,
// the check after every 15th included).
inline TileShape sweep_shape(const Geom& g, SweepKind kind) {
    int n = 0;
    const TileShape* shapes = sweep_shapes(kind, n);
    const int elem_bytes = kind == SK_F32 || kind == SK_NORM32 ? 4 : 8;
    if (kind == SK_F32 && g.tall32 && rows_fit(g, BY_CORR32, elem_bytes)) n = 1;
    const int other = kind == SK_F32 ? (corr32_short(g) ? BY_CORR32 : BY_CORR32_SHORT) : 0;
    return pick_tile(
        g, sweep_cost(kind), shapes, n, elem_bytes,
        [&](const TileShape& t, bool) {
            return kind == SK_F32 ? 24 : kind == SK_NORM32 ? 16 : 4 * sweep_waves(t.w * t.h, kind == SK_NORM64);
        },
        [&](const TileShape& t, bool cached) { return t.w != BX ? (cached ? 1.0 : 1.15) : t.h == other ? 1.05 : 1.0; });
}

// The tiles of a grid's sweeps, chosen once per grid, and the blocks that
// write per-block norm maxima: of the sweeps with norms and of the residual
// sweep (which runs the plain sweeps' tiles).
struct Tiling {
    TileShape shape[4];
    int64_t norms64 = 0, norms32 = 0, resid = 0;
    int64_t most = 0;   // of these three (size of the partials area)
};
inline Tiling make_tiling(const Geom& g) {
    Tiling t;
    for (int k = 0; k < 4; ++k) t.shape[k] = sweep_shape(g, (SweepKind)k);
    t.norms64 = sweep_blocks(g, t.shape[SK_NORM64]);
    t.norms32 = sweep_blocks(g, t.shape[SK_NORM32]);
    t.resid = sweep_blocks(g, t.shape[SK_F64]);
    t.most = std::max(t.resid, std::max(t.norms64, t.norms32));
    return t;
}

// Launchers (defined in the .hip files).
hipError_t launch_iteration(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int mode,
                            int norms, hipStream_t s);
hipError_t launch_correction(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<float>& p, int norms,
                             hipStream_t s);
hipError_t launch_correction64(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int norms,
                               hipStream_t s);
hipError_t launch_reduce_max(const double* partials, int64_t nblocks, double* out8, hipStream_t s);

// When a solve by PT sweeps ends.  A check reduces the norms and, by the
// rule here, closes the solve's gate: rho = max(f / ref_v, max(r_Pt, r_Pf) /
// ref_p) at most tol, or its value with the second references at most tol2,
// or (stall > 0) no new minimum of rho by 1 % in `stall` checks, or a
// non-finite norm or a set domain flag.  Sweeps and checks behind a closed
// gate do nothing, so the host may launch the sweeps up to the next check
// before it has seen this one: with the host in between, the device idled
// 20 to 36 us per check (15 sweeps of 7.5 us at 32^3).
struct CheckRule {
    double ref_v, ref_p, tol;
    double ref_v2, ref_p2, tol2;
    int stall;
    int first;          // the solve's first check
};
// Doubles of a gate: closed (0 or 1), the least rho, checks since then.
constexpr int GATE_DOUBLES = 3;
// What a check leaves in host memory (slot, if not null): the norms, the
// domain flag, whether the gate is closed, and last the check's number.
constexpr int SLOT_DOUBLES = NNORM + 3;
hipError_t launch_check(const double* partials, int64_t nblocks, double* out8, const double* domain, double* gate,
                        const CheckRule& r, double* slot, double number, hipStream_t s);

struct AuxPtrs {
    // state (present copies)
    const double *vx, *vy, *vz, *pt, *pf, *lp;
    double *pto, *pfo, *lpo;
    double *sxx, *syy, *szz, *sxy, *sxz, *syz;
    double *fox, *foy, *foz;
    double *mn, *kc, *eta, *mus;
    const double* k0;
    double* lp_o;                  // porosity step output
    double* domain;                // set to 1 where ln(1-phi) leaves (-inf, 0)
};

struct RefreshCoef {
    double phi0, kmuf0, eta0, mu0, cmu, R0;
    double n_pow, tau0_inv, coh_cos, sin_f, tau_y_min;
    double r_eta, r_mu;
    int first, powerlaw, dpcap, k0field;
};

hipError_t launch_begin_step(const Geom& g, const Coef& c, const AuxPtrs& a, int update_history,
                             hipStream_t s);
// t: the tile of the grid's plain FP64 sweeps (refresh with the stress
// invariant, history divergence).
hipError_t launch_refresh(const Geom& g, const TileShape& t, const Coef& c, const RefreshCoef& r, const AuxPtrs& a,
                          hipStream_t s);
hipError_t launch_refresh_tiled(const Geom& g, const TileShape& t, const Coef& c, const RefreshCoef& r, const AuxPtrs& a,
                                hipStream_t s);
hipError_t launch_fo_tiled(const Geom& g, const TileShape& t, const Coef& c, const RefreshCoef& r, const AuxPtrs& a,
                           hipStream_t s);
hipError_t launch_porosity_step(const Geom& g, const Coef& c, const AuxPtrs& a, hipStream_t s);
hipError_t launch_copy(const double* src, double* dst, int64_t n, hipStream_t s);
// ln(1-phi) and its old value from a porosity field; domain <- 1 where phi is
// not in (0, 1).
hipError_t launch_set_porosity(const Geom& g, const double* phi, double* lp, double* lpo, double* domain,
                               hipStream_t s);
// Damped residual R = (V - V_prev) / dtau_V on the interior faces (dtau_V =
// dtauv_c / the larger mu_s of the face's two cells).
hipError_t launch_damped_residual(const Geom& g, const Coef& c, const double* vx, const double* vy, const double* vz,
                                  const double* vx_p, const double* vy_p, const double* vz_p, const double* mus,
                                  double* rx, double* ry, double* rz, hipStream_t s);
// n doubles <- v (a kernel, so that the clear can sit in a captured graph).
hipError_t launch_fill(double* dst, double v, int64_t n, hipStream_t s);

// Mixed precision helpers.
struct MixedPtrs {
    // FP64 state (present copies) and coefficients
    double *vx, *vy, *vz, *pt, *pf;
    const double *lp, *kc, *eta, *mus;
    // FP32 correction (present copies) and coefficient copies
    const float *dvx, *dvy, *dvz, *dpt, *dpf;
    float *kc32, *mus32, *chi32;
};
hipError_t launch_prepare_mixed(const Geom& g, const MixedPtrs& m, hipStream_t s);

// Adjoint of a linear Picard stage.
hipError_t launch_gather(const double* src, const int64_t* offs, int n, double* out, hipStream_t s);
hipError_t launch_scatter(const double* vals, const int64_t* offs, int n, double* dst, hipStream_t s);
hipError_t launch_chi64(const Geom& g, const double* eta, const double* lp, double* chi, hipStream_t s);
hipError_t launch_adjoint_gradient(const Geom& g, const Coef& c, const double* kc, const double* pf,
                                   const double* lam_pf, double* grad, hipStream_t s);
hipError_t launch_exp_cells(const Geom& g, const double* src, double* dst, hipStream_t s);
hipError_t launch_apply_correction(const Geom& g, const MixedPtrs& m, hipStream_t s);

// Multigrid transfers between a fine grid gf and its coarse grid gc
// (mg_kernels.hip).
// Normalised restriction rows of one axis (fine nf, coarse nc points; face:
// faces normal to the axis): MG_TAB doubles per coarse index (first fine
// index, count, weights), nc + face rows.
constexpr int MG_TAPS = 4;
constexpr int MG_TAB = 2 + MG_TAPS;
hipError_t launch_mg_taps(double* tab, int nf, int nc, int face, hipStream_t s);
// The fine grid's FP32 residual (momentum rows on the x, y, z faces, r_Pt,
// r_Pf) restricted to the coarse grid's constant terms: dst[0..2] the
// momentum rows, dst[3] = m[0] a + m[1] b, dst[4] = m[2] a + m[3] b of the
// restricted r_Pt, r_Pf (a, b).  tab[axis][face]: the rows of each axis.
hipError_t launch_mg_residual_restrict(const Geom& gf, const Geom& gc, const float* const res[5], double* const dst[5],
                                       const double m[4], const double* const tab[3][2], hipStream_t s);
// Four cell fields averaged onto the coarse grid (mean 0: arithmetic, 1:
// harmonic, 2: geometric).
hipError_t launch_mg_coef_restrict(const Geom& gf, const Geom& gc, const double* const src[4], double* const dst[4],
                                   const int mean[4], const double* const tab[3], hipStream_t s);
// dst (fine V, Pt, Pf) += interpolated src (coarse); the walls' normal faces
// are kept.
hipError_t launch_mg_prolong_add(const Geom& gf, const Geom& gc, const double* const src[5], double* const dst[5],
                                 hipStream_t s);
// n damped linear PT sweeps from the zero state on a grid of at most 1024
// cells, in one launch; the result (V, Pt, Pf) to out.
bool mg_coarsest_fits(const Geom& g);
hipError_t launch_mg_coarsest(const Geom& g, const Coef& c, const SweepPtrs<double>& p, double* const out[5], int n,
                              hipStream_t s);

// Krylov acceleration of the multigrid cycle (krylov_kernels.hip): the
// cycles' iterates recombined over a subspace of their own steps.
// Vectors are the fine grid's five unknowns or five residuals in their
// padded boxes; only entries that carry an equation are read or written.
constexpr int KRY_MAX = 8;         // stored directions at most
constexpr int KRY_SLOTS = 16;      // partial sums per block (>= 2 KRY_MAX)
constexpr int KRY_BLOCKS = 2048;
constexpr int KRY_VW = 4;          // columns per work item (the row pitch a multiple of it)   // blocks of the reduction kernels at most
struct KryVecs {
    const float* rk[5];            // residual of the iterate x_k
    const float* ry[5];            // residual of the cycle's result y
    double* x[5];                  // saved x_k (boxes of the fine geometry)
    double* y[5];                  // the fine fields' present copies
    const double* p[KRY_MAX][5];   // stored directions p_s and images A p_s, s < na
    const float* ap[KRY_MAX][5];
    double* p_new[5];              // the new direction and its image
    float* ap_new[5];
    double gamma[KRY_MAX];         // x' = y + sum gamma_s p_s
    double beta[KRY_MAX];          // p = (y - x) - sum beta_s p_s
    double wv2, wp2;               // squared weights of momentum and pressure rows
    int na;
};
// Partial sums go to part[0 .. KRY_BLOCKS * KRY_SLOTS), their totals to the
// KRY_SLOTS doubles after them.
// dots: totals s = <r_k, A p_s>_W, KRY_MAX + s = <r_y, A p_s>_W, s < na.
hipError_t launch_kry_dots(const Geom& g, const KryVecs& v, double* part, hipStream_t s);
// update: x, y <- y + sum gamma_s p_s; p_new = y - x - sum beta_s p_s,
// ap_new = r_k - r_y - sum beta_s A p_s; total 0 = <ap_new, ap_new>_W.
hipError_t launch_kry_update(const Geom& g, const KryVecs& v, double* part, hipStream_t s);
// save: x <- y.
hipError_t launch_kry_save(const Geom& g, const KryVecs& v, hipStream_t s);

// Adjoint of a Picard run (adjoint_kernels.hip).  rhs holds -xbar, the
// right-hand side of the transposed stage solve in the slots of the
// correction sweep (momentum rows on the faces, r_Pt and r_Pf in the cells).
struct AdjPtrs {
    // recorded stage (incoming ln(1-phi), coefficients, solution)
    const double *vx, *vy, *vz, *pt, *pf, *lp, *kc, *eta, *mus;
    // transposed-solve solution lambda
    const double *lvx, *lvy, *lvz, *lpt, *lpf;
    double *rvx, *rvy, *rvz, *rpt, *rpf;   // -xbar
    const double* lbar;                    // adjoint of the stage's outgoing ln(1-phi)
    double* lbar_out;                      // adjoint of its incoming ln(1-phi)
    double *eta_bar, *s_bar;               // porosity-step adjoints of eta and s
    double *pto_bar, *pfo_bar, *lo_bar;    // adjoints of the step's old values
    double *fbx, *fby, *fbz;               // adjoint of the history term div(a So)
    double *sbxx, *sbyy, *sbzz, *sbxy, *sbxz, *sbyz;   // adjoint of the history So
    double* grad;                          // dJ/d(ln k0), accumulated
};
hipError_t launch_adj_porosity(const Geom& g, const Coef& c, const AdjPtrs& a, hipStream_t s);
hipError_t launch_adj_coef(const Geom& g, const Coef& c, const AdjPtrs& a, hipStream_t s);
hipError_t launch_adj_step(const Geom& g, const Coef& c, const AdjPtrs& a, hipStream_t s);
hipError_t launch_adj_history(const Geom& g, const Coef& c, const AdjPtrs& a, hipStream_t s);
hipError_t launch_adj_oldvalues(const Geom& g, const Coef& c, const double* rpt, const double* rpf, double* pto,
                                double* pfo, hipStream_t s);
hipError_t launch_absmax5(const Geom& g, const double* const* f, double* partials, int64_t nblocks,
                          hipStream_t s);
// Per-block maxima of a cell field (its cell extent only) into partials[b * 8]
// (the other seven slots 0), nblocks blocks.
hipError_t launch_cell_max(const Geom& g, const double* f, double* partials, int64_t nblocks, hipStream_t s);

}  // namespace ptk
