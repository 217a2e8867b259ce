// Grid transfers of the geometric multigrid solver for the linear Picard
// stage (the thesis's outlook: geometric multigrid with weighted-Jacobi
// smoothing, which the PT iteration becomes without damping).
//
// A coarse grid has ceil(n/2) cells per axis on the same domain, so grids
// with odd counts (511 -> 256 -> 128 ...) are not nested.  Transfers are
// tensor products of one-dimensional linear interpolation between the two
// grids' point positions, per staggering: cell centres (i + 1/2) h, taken
// constant beyond the outermost coarse centres, and faces i h, which both
// grids have at the walls.  Prolongation P interpolates a coarse correction
// to the fine points; restriction is P's transpose with every row
// normalised to weight sum 1 (an average of the fine values around a coarse
// point).  Normal faces on the walls carry no equation: the restriction
// skips them and gives zero there, the prolongation leaves them alone.
#include "pt_internal.h"

namespace ptk {
namespace {

constexpr int TB = 256;

// Fine index i of an axis with nf fine and nc coarse cells, in coarse
// units: the coarse index j0 and the weight t of j0 + 1 (1 - t of j0).
__device__ __forceinline__ void pw(int i, int nf, int nc, bool face, int& j0, double& t) {
    if (face) {
        const double u = (double)i * nc / nf;
        j0 = min((int)floor(u), nc - 1);
        t = u - j0;
    } else {
        const double u = ((double)i + 0.5) * nc / nf - 0.5;
        if (u <= 0.0) {
            j0 = 0;
            t = 0.0;
        } else if (u >= (double)(nc - 1)) {
            j0 = nc - 1;
            t = 0.0;
        } else {
            j0 = (int)floor(u);
            t = u - j0;
        }
    }
}

// P's entry (fine i, coarse J) of one axis.
__device__ __forceinline__ double pweight(int i, int J, int nf, int nc, bool face) {
    int j0;
    double t;
    pw(i, nf, nc, face, j0, t);
    return J == j0 ? 1.0 - t : (J == j0 + 1 ? t : 0.0);
}

// Fine indices whose interpolation can involve coarse index J.
__device__ __forceinline__ void prange(int J, int nf, int nc, bool face, int& lo, int& hi) {
    const double r = (double)nf / nc;
    if (face) {
        lo = max(0, (int)floor((J - 1) * r));
        hi = min(nf, (int)ceil((J + 1) * r));
    } else {
        lo = max(0, (int)floor((J - 0.5) * r - 0.5));
        hi = min(nf - 1, (int)ceil((J + 1.5) * r - 0.5));
    }
}

// Candidate taps of coarse index J: P's entries for the fine indices lo ..
// lo + n - 1 (a coarse grid has ceil(n/2) cells, so the ratio is at most 2
// and the candidates span at most 7 fine points).
constexpr int MAXT = 8;
struct Taps {
    int lo, n;
    double w[MAXT];
    double sum;
};
__device__ __forceinline__ void taps(int J, int nf, int nc, bool face, bool skip_walls, Taps& t) {
    int lo, hi;
    prange(J, nf, nc, face, lo, hi);
    if (skip_walls) {
        lo = max(lo, 1);
        hi = min(hi, nf - 1);
    }
    t.lo = lo;
    t.n = min(hi - lo + 1, MAXT);
    t.sum = 0.0;
#pragma unroll
    for (int q = 0; q < MAXT; ++q) {
        const double w = (q < t.n) ? pweight(lo + q, J, nf, nc, face) : 0.0;
        t.w[q] = w;
        t.sum += w;
    }
}

struct Ext {
    int nx, ny, nz;     // cells of the grid
    int64_t P, S;       // row and plane pitch
};
__host__ __device__ inline Ext ext(const Geom& g) { return Ext{g.nx, g.ny, g.nz, g.P, g.S}; }

// The normalised restriction rows of one axis (fine nf, coarse nc points;
// face: the field sits on faces normal to it, whose wall faces carry no
// equation: skipped as inputs, rows of no tap for the coarse walls).  A row is
// the first fine index, the number of taps and MG_TAPS weights.  The weights
// of linear interpolation at a ratio of at most 2 are zero outside an open
// interval 4 fine points wide, so at most MG_TAPS of them are not.  A row
// starts MG_TAPS points before the end of the axis at the latest (taps of
// weight 0 in front), so that the MG_TAPS values from its first index on
// always belong to the field (a fine grid has at least 4 cells per axis).
__global__ __launch_bounds__(TB) void k_mg_taps(double* __restrict__ tab, int nf, int nc, bool face) {
    const int J = blockIdx.x * TB + threadIdx.x;
    if (J > nc - 1 + face) return;
    double* row = tab + (int64_t)J * MG_TAB;
    Taps tt;
    taps(J, nf, nc, face, face, tt);
    const bool none = (face && (J == 0 || J == nc)) || !(tt.sum > 0.0);
    int first = 0, last = -1;
#pragma unroll
    for (int q = 0; q < MAXT; ++q)
        if (tt.w[q] != 0.0) {
            if (last < 0) first = q;
            last = q;
        }
    const int at = min(max(tt.lo + first, 0), nf + face - MG_TAPS), pad = tt.lo + first - at;
    const int n = none ? 0 : min(last - first + 1 + pad, MG_TAPS);
    row[0] = at;
    row[1] = n;
#pragma unroll
    for (int q = 0; q < MG_TAPS; ++q) row[2 + q] = 0.0;
#pragma unroll
    for (int q = 0; q < MAXT; ++q)
        if (!none && q >= first && q - first + pad < n) row[2 + q - first + pad] = tt.w[q] / tt.sum;
}

// Restriction of several fields in one launch.  The restriction is a tensor
// product of one-dimensional rows of at most four weights, each normalised to
// sum 1.  A thread owns a coarse column (I, J) of one field (or of a pair of
// fields whose combinations are wanted) and marches up a chunk of coarse
// planes: it averages each fine plane around (I, J) once (up to 16 values
// through the caches) and keeps the last four of these averages, from which
// every coarse plane takes its own; neighbouring threads read the same lines,
// so the fine field comes from memory about once.  Bound by the latency of
// these reads: a row's four values come as one load, two fine planes' are in
// flight at once, columns are dealt out along the rows without gaps (a coarse
// row seldom fills whole wavefronts), and the chunk's z rows are in LDS.  The five residuals of 300x255x201 in
// 133 us, of 127^3 in 28 us, of 16^3 in 6.3 us (251, 43 and 7.5 us with a load
// per value; 820, 210 and 21 us with one plane's loads behind a branch at a
// time).
// mean (cells): 0 arithmetic, 1 harmonic, 2 geometric, by averaging v, 1/v
// or ln v.
struct RestrictField {
    const void* src;
    double* dst;
    const double* tab[3];
    int ex, ey, ez;      // coarse extent
    int mean;
};
struct RestrictArgs {
    RestrictField f[4];
    // with a pair: field 3 and src2 give dst = m[0] f + m[1] f2, dst2 = m[2] f + m[3] f2
    const void* src2;
    double* dst2;
    double m[4];
    int64_t fP, fS, cP, cS;
    int kc;              // coarse planes per chunk (at most MAX_KC)
};
constexpr int MAX_KC = 16;

template <typename TI, bool PAIR>
__device__ __forceinline__ void restrict_column(const RestrictArgs& a, const RestrictField& f, int I, int J, int K0, int K1,
                                                const double (*rows)[MG_TAB]) {
    constexpr int NS = PAIR ? 2 : 1, T = MG_TAPS;
    const TI* __restrict__ src[2] = {static_cast<const TI*>(f.src), static_cast<const TI*>(a.src2)};
    const double* rx = f.tab[0] + (int64_t)I * MG_TAB;
    const double* ry = f.tab[1] + (int64_t)J * MG_TAB;
    const int nx = (int)rx[1], ny = (int)ry[1];
    double wx[T], wy[T];
    int64_t oy[T];
#pragma unroll
    for (int q = 0; q < T; ++q) {
        wx[q] = rx[2 + q];
        wy[q] = ry[2 + q];
        oy[q] = (int64_t)((int)ry[0] + q) * a.fP + (int)rx[0];
    }
    const bool any = nx > 0 && ny > 0;
    double s[NS][T] = {};      // averages of the fine planes base .. base + have - 1
    int base = 0, have = 0;
    for (int K = K0; K < K1; ++K) {
        const double* rz = rows[K - K0];
        const int lo = (int)rz[0], nz = (int)rz[1];
        double r[NS] = {};
        if (any && nz > 0) {
            // drop what lies below lo
            const int drop = have ? min(lo - base, have) : 0;
            for (int d = 0; d < drop; ++d)
#pragma unroll
                for (int n = 0; n < NS; ++n) {
                    s[n][0] = s[n][1]; s[n][1] = s[n][2]; s[n][2] = s[n][3];
                }
            have -= drop;
            base = lo;
            while (have < nz) {
                TI raw[NS][2][T][T];
#pragma unroll
                for (int n = 0; n < NS; ++n)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const int64_t o = (int64_t)(lo + min(have + p, nz - 1)) * a.fS;
#pragma unroll
                        for (int y = 0; y < T; ++y) __builtin_memcpy(raw[n][p][y], src[n] + o + oy[y], sizeof raw[n][p][y]);
                    }
#pragma unroll
                for (int n = 0; n < NS; ++n)
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        double v = 0.0;
#pragma unroll
                        for (int y = 0; y < T; ++y) {
                            double t = 0.0;
#pragma unroll
                            for (int x = 0; x < T; ++x) {
                                double u = (double)raw[n][p][y][x];
                                if (!PAIR && f.mean) u = f.mean == 1 ? 1.0 / u : log(u);
                                t += wx[x] * u;
                            }
                            v += wy[y] * t;
                        }
#pragma unroll
                        for (int q = 0; q < T; ++q)
                            if (q == have + p) s[n][q] = v;
                    }
                have += 2;
            }
            have = nz;
#pragma unroll
            for (int n = 0; n < NS; ++n)
#pragma unroll
                for (int q = 0; q < T; ++q)
                    if (q < nz) r[n] += rz[2 + q] * s[n][q];
            if (!PAIR && f.mean) r[0] = f.mean == 1 ? 1.0 / r[0] : exp(r[0]);
        } else {
            have = 0;
        }
        const int64_t o = (int64_t)K * a.cS + (int64_t)J * a.cP + I;
        if (PAIR) {
            f.dst[o] = a.m[0] * r[0] + a.m[1] * r[NS - 1];
            a.dst2[o] = a.m[2] * r[0] + a.m[3] * r[NS - 1];
        } else {
            f.dst[o] = r[0];
        }
    }
}

template <typename TI, bool PAIR>
__global__ __launch_bounds__(TB) void k_mg_restrict(RestrictArgs a) {
    __shared__ double rows[MAX_KC][MG_TAB];
    const RestrictField& f = a.f[blockIdx.y];
    const int K0 = (int)blockIdx.z * a.kc, K1 = min(f.ez, K0 + a.kc);
    if (K0 >= K1) return;
    for (int t = threadIdx.x; t < (K1 - K0) * MG_TAB; t += TB) rows[t / MG_TAB][t % MG_TAB] = f.tab[2][(int64_t)K0 * MG_TAB + t];
    __syncthreads();
    const unsigned t = blockIdx.x * TB + threadIdx.x;
    const int J = (int)(t / (unsigned)f.ex), I = (int)(t - (unsigned)J * f.ex);
    if (J >= f.ey) return;
    if (PAIR && blockIdx.y == 3)
        restrict_column<TI, PAIR>(a, f, I, J, K0, K1, rows);
    else
        restrict_column<TI, false>(a, f, I, J, K0, K1, rows);
}

// fine += P coarse for the three velocities and the two pressures, one launch
// (a block's field in its second index, its chunk of fine planes in the
// third); the walls' normal faces keep their values.  A thread owns a fine
// column and keeps the interpolations within the two coarse planes around
// its plane, so that a fine value costs its own read and write and about two
// reads through the caches; four planes' reads are in flight.  Onto
// 300x255x201 in 274 us, 4.9 TB/s of the fine fields' reads and writes, onto
// 127^3 in 42 us (about 480 and 70 us for a thread per fine point, which read
// eight coarse values and divided for its weights).
struct ProlongArgs {
    Ext f, c;
    const double* src[5];
    double* dst[5];
    int kc;              // fine planes per chunk (at most MAX_PC)
};
constexpr int MAX_PC = 64;
__global__ __launch_bounds__(TB) void k_mg_prolong_add(ProlongArgs a) {
    __shared__ double st[MAX_PC];
    __shared__ int sz[MAX_PC];
    const Ext& f = a.f;
    const Ext& c = a.c;
    const int q = blockIdx.y;
    const bool fx = q == 0, fy = q == 1, fz = q == 2;
    const int K0 = (int)blockIdx.z * a.kc, K1 = min(f.nz + fz, K0 + a.kc);
    if (K0 >= K1) return;
    if ((int)threadIdx.x < K1 - K0) pw(K0 + threadIdx.x, f.nz, c.nz, fz, sz[threadIdx.x], st[threadIdx.x]);
    __syncthreads();
    const unsigned ex = f.nx + fx, t = blockIdx.x * TB + threadIdx.x;
    const int j = (int)(t / ex), i = (int)(t - (unsigned)j * ex);
    if (j >= f.ny + fy || (fx && (i == 0 || i == f.nx)) || (fy && (j == 0 || j == f.ny))) return;
    int x0, y0;
    double tx, ty;
    pw(i, f.nx, c.nx, fx, x0, tx);
    pw(j, f.ny, c.ny, fy, y0, ty);
    // the second point of an axis: inside the coarse extent (its weight
    // is zero where the first point is the last one)
    const int x1 = min(x0 + 1, c.nx - 1 + fx), y1 = min(y0 + 1, c.ny - 1 + fy), zmax = c.nz - 1 + fz;
    const double* __restrict__ src = a.src[q];
    double* __restrict__ dst = a.dst[q] + (int64_t)j * f.P + i;
    const int64_t o00 = (int64_t)y0 * c.P + x0, o01 = (int64_t)y0 * c.P + x1;
    const int64_t o10 = (int64_t)y1 * c.P + x0, o11 = (int64_t)y1 * c.P + x1;
    auto plane = [&](int z) {
        const double* p = src + (int64_t)z * c.S;
        const double v0 = (1.0 - tx) * p[o00] + tx * p[o01];
        const double v1 = (1.0 - tx) * p[o10] + tx * p[o11];
        return (1.0 - ty) * v0 + ty * v1;
    };
    int zc = sz[0];
    double c0 = plane(zc), c1 = plane(min(zc + 1, zmax));
    for (int k = K0; k < K1; k += 4) {
        double d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d[u] = dst[(int64_t)min(k + u, K1 - 1) * f.S];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (k + u >= K1) break;
            const int z0 = sz[k + u - K0];
            const double tz = st[k + u - K0];
            // (the coarse grid is the coarser one: z0 rises by at most 1)
            if (z0 != zc) {
                zc = z0;
                c0 = c1;
                c1 = plane(min(zc + 1, zmax));
            }
            if (fz && (k + u == 0 || k + u == f.nz)) continue;
            dst[(int64_t)(k + u) * f.S] = d[u] + ((1.0 - tz) * c0 + tz * c1);
        }
    }
}

// ---- the coarsest grid's damped PT sweeps, in one launch -------------------------
// n sweeps of the linear PT iteration from the zero state on a grid of at
// most 1024 cells, by one block with one thread per cell (and the three
// faces at its low sides).  The state stays in registers, neighbours are read
// from LDS planes with a rim of zeros, every coefficient, including the
// quotients of the pseudo steps, is formed once; two barriers per sweep.
// Bound by the latency of a sweep's chain through LDS: fifty sweeps of the
// 8^3 grid take 44 us, where fifty launches of the sweep kernel on its
// smallest tile took 7 us each (22 us each on the 66 x 10 tile that every
// grid once had).
struct CoarseArgs {
    int nx, ny, nz, n;
    int64_t P, S;
    double dxi, dyi, dzi;
    double bdt, alpha, ab;          // beta_d/dt, alpha, alpha/B
    double gdts, beta_n, rho_i_inv;
    double dtauv_c, dtaupt_c, dtaupf_c, dampx, dampy, dampz;
    const double *lp, *kc, *eta, *mus, *fox, *foy, *foz, *pto, *pfo;
    double *vx, *vy, *vz, *pt, *pf;
};

// FROZEN: mechanics off, V and Pt keep their zero whatever the forces.
template <bool FROZEN>
__global__ __launch_bounds__(1024) void k_mg_coarsest(CoarseArgs a) {
    extern __shared__ double lds[];
    const int X = a.nx + 2, XY = X * (a.ny + 2), N = XY * (a.nz + 2);   // a plane of the rimmed grid
    double *vx = lds, *vy = vx + N, *vz = vy + N, *pf = vz + N, *sx = pf + N, *sy = sx + N, *sz = sy + N, *txy = sz + N,
           *txz = txy + N, *tyz = txz + N;
    for (int t = threadIdx.x; t < 10 * N; t += blockDim.x) lds[t] = 0.0;
    const int cells = a.nx * a.ny * a.nz;
    const bool on = (int)threadIdx.x < cells;
    const int c = on ? threadIdx.x : 0;
    const int i = c % a.nx, j = (c / a.nx) % a.ny, k = c / (a.nx * a.ny);
    const int64_t o = (int64_t)k * a.S + (int64_t)j * a.P + i;
    const int me = (k + 1) * XY + (j + 1) * X + i + 1;
    const bool lx = i >= 1, ly = j >= 1, lz = k >= 1;
    __syncthreads();
    // coefficients of neighbours through two of the planes
    const double mu = a.mus[o], kc = a.kc[o];
    if (on) {
        sx[me] = mu;
        sy[me] = kc;
    }
    __syncthreads();
    const double mw = sx[me - 1], ms = sx[me - X], mb = sx[me - XY];
    auto maxwell = [&](double m) { return 2.0 * m / (1.0 + m * a.gdts); };
    const double b = maxwell(mu);
    // half the edge coefficients (the strain rates come without their 1/2); zero on the walls
    const double exy = lx && ly ? 0.5 * maxwell(0.25 * (sx[me - X - 1] + ms + mw + mu)) : 0.0;
    const double exz = lx && lz ? 0.5 * maxwell(0.25 * (sx[me - XY - 1] + mb + mw + mu)) : 0.0;
    const double eyz = ly && lz ? 0.5 * maxwell(0.25 * (sx[me - XY - X] + mb + ms + mu)) : 0.0;
    const double dvx = lx ? a.dtauv_c / fmax(mu, mw) : 0.0, dvy = ly ? a.dtauv_c / fmax(mu, ms) : 0.0,
                 dvz = lz ? a.dtauv_c / fmax(mu, mb) : 0.0;
    const double kw = sy[me - 1], ke = sy[me + 1], ks = sy[me - X], kn = sy[me + X], kb = sy[me - XY], kt = sy[me + XY];
    const double qx = 0.5 * a.dxi * a.dxi, qy = 0.5 * a.dyi * a.dyi, qz = 0.5 * a.dzi * a.dzi;
    const double cw = lx ? qx * (kw + kc) : 0.0, ce = i + 1 < a.nx ? qx * (kc + ke) : 0.0;
    const double cs = ly ? qy * (ks + kc) : 0.0, cn = j + 1 < a.ny ? qy * (kc + kn) : 0.0;
    const double cb = lz ? qz * (kb + kc) : 0.0, ct = k + 1 < a.nz ? qz * (kc + kt) : 0.0;
    const double kl = fmax(fmax(fmax(kc, kw), fmax(ke, ks)), fmax(fmax(kn, kb), kt));   // zero outside the domain
    const double chi = 1.0 / (a.eta[o] * exp(a.lp[o]));
    const double dtp = a.dtaupt_c * mu, dtf = a.dtaupf_c / kl;
    const double tp = dtp / (1.0 + dtp * (a.bdt + chi)), tf = dtf / (1.0 + dtf * (a.bdt * a.ab + chi));
    const double pto = a.pto[o], pfo = a.pfo[o];
    // r_Pt = div V + rp0 + Pt rpp - Pf cross, r_Pf = div q + rf0 + Pf rff - Pt cross
    const double rp0 = a.bdt * (a.alpha * pfo - pto), rf0 = a.bdt * (a.alpha * pto - a.ab * pfo);
    const double rpp = a.bdt + chi, rff = a.bdt * a.ab + chi, cross = a.bdt * a.alpha + chi;
    const double fox = lx ? a.fox[o] : 0.0, foy = ly ? a.foy[o] : 0.0, foz = lz ? a.foz[o] : 0.0;
    __syncthreads();
    if (on) sx[me] = sy[me] = 0.0;
    __syncthreads();
    double u = 0.0, v = 0.0, w = 0.0, p = 0.0, f = 0.0, ru = 0.0, rv = 0.0, rw = 0.0;
    for (int it = 0; it < a.n; ++it) {
        // (the planes written here are read before the second barrier, those
        // written between the barriers after it: no third barrier is needed)
        if (on) {
            vx[me] = u; vy[me] = v; vz[me] = w; pf[me] = f;
        }
        __syncthreads();
        const double ex = (vx[me + 1] - u) * a.dxi, ey = (vy[me + X] - v) * a.dyi, ez = (vz[me + XY] - w) * a.dzi;
        const double div = ex + ey + ez;
        const double rpt = div + rp0 + p * rpp - f * cross;
        const double divq = cw * (f - pf[me - 1]) - ce * (pf[me + 1] - f) + cs * (f - pf[me - X]) - cn * (pf[me + X] - f) +
                            cb * (f - pf[me - XY]) - ct * (pf[me + XY] - f);
        const double rpf = divq + rf0 + f * rff - p * cross;
        const double ptn = p - tp * rpt;
        const double m = a.beta_n * rpt - div * (1.0 / 3.0);
        const double nx = b * (ex + m) - ptn, ny = b * (ey + m) - ptn, nz = b * (ez + m) - ptn;
        const double hxy = exy * ((u - vx[me - X]) * a.dyi + (v - vy[me - 1]) * a.dxi);
        const double hxz = exz * ((u - vx[me - XY]) * a.dzi + (w - vz[me - 1]) * a.dxi);
        const double hyz = eyz * ((v - vy[me - XY]) * a.dzi + (w - vz[me - X]) * a.dyi);
        if (on) {
            sx[me] = nx; sy[me] = ny; sz[me] = nz;
            txy[me] = hxy; txz[me] = hxz; tyz[me] = hyz;
        }
        f -= tf * rpf;
        if constexpr (!FROZEN) p = ptn;
        __syncthreads();
        if constexpr (FROZEN) continue;
        const double gx = (nx - sx[me - 1]) * a.dxi + (txy[me + X] - hxy) * a.dyi + (txz[me + XY] - hxz) * a.dzi + fox;
        const double gy = (txy[me + 1] - hxy) * a.dxi + (ny - sy[me - X]) * a.dyi + (tyz[me + XY] - hyz) * a.dzi + foy;
        const double gz = (txz[me + 1] - hxz) * a.dxi + (tyz[me + X] - hyz) * a.dyi + (nz - sz[me - XY]) * a.dzi + foz;
        ru = gx * a.rho_i_inv + a.dampx * ru;
        rv = gy * a.rho_i_inv + a.dampy * rv;
        rw = gz * a.rho_i_inv + a.dampz * rw;
        u += dvx * ru;
        v += dvy * rv;
        w += dvz * rw;
    }
    if (on) {
        // (wall faces hold their zero)
        a.vx[o] = u; a.vy[o] = v; a.vz[o] = w;
        a.pt[o] = p;
        a.pf[o] = f;
    }
}

}  // namespace

hipError_t launch_mg_taps(double* tab, int nf, int nc, int face, hipStream_t s) {
    hipLaunchKernelGGL(k_mg_taps, dim3((unsigned)((nc + 1 + TB - 1) / TB)), dim3(TB), 0, s, tab, nf, nc, face != 0);
    return hipGetLastError();
}

namespace {

// Planes per chunk: a chunk starts with reads that its neighbour below also
// makes (two fine planes more than the two per coarse plane), so long chunks
// read less; short ones give a small grid enough blocks, four per compute
// unit while a chunk has a plane.
int chunk(const Geom& g, int64_t planes, int64_t blocks, int most) {
    const int cus = g.cus > 0 ? g.cus : DEFAULT_CUS;
    return (int)std::min<int64_t>(most, std::max<int64_t>(1, planes * blocks / (4 * cus)));
}
unsigned column_blocks(const Geom& g) { return (unsigned)(((int64_t)(g.nx + 1) * (g.ny + 1) + TB - 1) / TB); }

template <typename TI, bool PAIR>
hipError_t launch_restrict(const Geom& gf, const Geom& gc, RestrictArgs& a, hipStream_t s) {
    a.fP = gf.P; a.fS = gf.S; a.cP = gc.P; a.cS = gc.S;
    const unsigned cols = column_blocks(gc);
    a.kc = chunk(gf, gc.nz + 1, (int64_t)cols * 4, MAX_KC);
    hipLaunchKernelGGL((k_mg_restrict<TI, PAIR>), dim3(cols, 4, (unsigned)((gc.nz + a.kc) / a.kc)), dim3(TB), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_mg_residual_restrict(const Geom& gf, const Geom& gc, const float* const res[5], double* const dst[5],
                                       const double m[4], const double* const tab[3][2], hipStream_t s) {
    RestrictArgs a{};
    for (int q = 0; q < 4; ++q) {
        RestrictField& f = a.f[q];
        f.src = res[q];
        f.dst = dst[q];
        f.ex = gc.nx + (q == 0); f.ey = gc.ny + (q == 1); f.ez = gc.nz + (q == 2);
        for (int x = 0; x < 3; ++x) f.tab[x] = tab[x][x == q];
    }
    a.src2 = res[4];
    a.dst2 = dst[4];
    for (int q = 0; q < 4; ++q) a.m[q] = m[q];
    return launch_restrict<float, true>(gf, gc, a, s);
}

hipError_t launch_mg_coef_restrict(const Geom& gf, const Geom& gc, const double* const src[4], double* const dst[4],
                                   const int mean[4], const double* const tab[3], hipStream_t s) {
    RestrictArgs a{};
    for (int q = 0; q < 4; ++q) {
        RestrictField& f = a.f[q];
        f.src = src[q];
        f.dst = dst[q];
        f.ex = gc.nx; f.ey = gc.ny; f.ez = gc.nz;
        for (int x = 0; x < 3; ++x) f.tab[x] = tab[x];
        f.mean = mean[q];
    }
    return launch_restrict<double, false>(gf, gc, a, s);
}

hipError_t launch_mg_prolong_add(const Geom& gf, const Geom& gc, const double* const src[5], double* const dst[5],
                                 hipStream_t s) {
    ProlongArgs a{};
    a.f = ext(gf);
    a.c = ext(gc);
    for (int q = 0; q < 5; ++q) {
        a.src[q] = src[q];
        a.dst[q] = dst[q];
    }
    const unsigned cols = column_blocks(gf);
    a.kc = chunk(gf, gf.nz + 1, (int64_t)cols * 5, MAX_PC);
    hipLaunchKernelGGL(k_mg_prolong_add, dim3(cols, 5, (unsigned)((gf.nz + a.kc) / a.kc)), dim3(TB), 0, s, a);
    return hipGetLastError();
}

namespace {
size_t coarsest_lds(const Geom& g) { return (size_t)10 * (g.nx + 2) * (g.ny + 2) * (g.nz + 2) * sizeof(double); }
}  // namespace

bool mg_coarsest_fits(const Geom& g) {
    return (int64_t)g.nx * g.ny * g.nz <= 1024 && coarsest_lds(g) <= 150 * 1024;
}

hipError_t launch_mg_coarsest(const Geom& g, const Coef& c, const SweepPtrs<double>& p, double* const out[5], int n,
                              hipStream_t s) {
    CoarseArgs a{};
    a.nx = g.nx; a.ny = g.ny; a.nz = g.nz; a.n = n;
    a.P = g.P; a.S = g.S;
    a.dxi = c.dxi; a.dyi = c.dyi; a.dzi = c.dzi;
    a.bdt = c.beta_d * c.dti; a.alpha = c.alpha; a.ab = c.ab;
    a.gdts = c.gdts_inv; a.beta_n = c.beta_n; a.rho_i_inv = c.rho_i_inv;
    a.dtauv_c = c.dtauv_c; a.dtaupt_c = c.dtaupt_c; a.dtaupf_c = c.dtaupf_c;
    a.dampx = c.dampx; a.dampy = c.dampy; a.dampz = c.dampz;
    a.lp = p.lp; a.kc = p.kc; a.eta = p.eta; a.mus = p.mus;
    a.fox = p.fox; a.foy = p.foy; a.foz = p.foz; a.pto = p.pto; a.pfo = p.pfo;
    a.vx = out[0]; a.vy = out[1]; a.vz = out[2]; a.pt = out[3]; a.pf = out[4];
    const int threads = (g.nx * g.ny * g.nz + 63) / 64 * 64;
    if (c.mech_off) hipLaunchKernelGGL(k_mg_coarsest<true>, dim3(1), dim3(threads), coarsest_lds(g), s, a);
    else hipLaunchKernelGGL(k_mg_coarsest<false>, dim3(1), dim3(threads), coarsest_lds(g), s, a);
    return hipGetLastError();
}

}  // namespace ptk
