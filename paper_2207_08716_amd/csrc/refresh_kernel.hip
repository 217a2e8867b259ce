// Picard refresh with the stress invariant, and the divergence of the stress
// history, as z-marching tile kernels.
//
// The refresh of the lagged coefficients (thesis article 1, eqs (23)-(26))
// needs, when the viscosity depends on stress (power law, yield cap), the
// second invariant of the present deviatoric stress at every cell: the three
// normal stresses at the cell and the shear stresses of the twelve edges
// around it, averaged per component (eq (21) for the stresses, without the
// numerical compressibility term).  A W x H block owns a (W-2) x (H-2) column
// of cells plus a one-cell halo ring and marches upward through a chunk of
// planes, like the PT sweep: per plane it stages viscosities and velocities
// in LDS, computes each edge's shear stress once (xy edges of the plane, xz
// and yz edges of the level above, the level below carried from the previous
// plane), then updates k/mu_f, eta_phi and Mn of the tile cells in place.
// Edge stresses never touch memory.
//
// Both kernels take the tile chosen for the plain FP64 sweeps of the grid,
// which march alike (of the tiles and chunks measured for them it was the
// fastest or within 4 % on eight grids from 32^3 to 511^3).  As in the sweeps,
// loads and stores go through buffer descriptors, so that a step waits for its
// loads alone and not for stores, and the sets loaded ahead alternate between
// two register sets.  The refresh is bound by its vector instructions (three
// exponentials, four logarithms and a dozen quotients per cell: 4 us of a
// 66 x 10 block's plane step) as much as by memory (3.6 us), the divergence
// by memory on large grids, both by a step's latency on small ones.  Refresh
// and divergence together, before (fixed tiles of 66 x 10 and 66 x 14 threads,
// branches around the stores) and now: 511^3 8.4 and 6.9 ms, 255x255x510 2.24
// and 1.70 ms, 173x131x97 215 and 140 us, 127^3 155 and 117 us, 32^3 38 and
// 14 us.
#include "plane.h"
#include "pt_internal.h"

#pragma clang fp contract(on)

namespace ptk {

namespace {

// Maxwell coefficients of eq (21): a = xi/(1+xi), b = 2 mu/(1+xi), xi = mu/(G dtS).
__device__ __forceinline__ double maxwell_a(double mu, double gdts_inv) {
    const double xi = mu * gdts_inv;
    return quot(xi, 1.0 + xi);
}
__device__ __forceinline__ void maxwell(double mu, double gdts_inv, double& a, double& b) {
    const double xi = mu * gdts_inv;
    quot2(xi, 2.0 * mu, 1.0 + xi, a, b);
}

struct RefreshArgs {
    Geom g;
    Coef c;
    RefreshCoef r;
    AuxPtrs a;
};
// The field pointers from the argument segment (read where they are used:
// kept in registers they exceed the scalar file).
using KAux = const __attribute__((address_space(4))) AuxPtrs;
__device__ __forceinline__ KAux* fields() {
    KAux* q = (KAux*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                      offsetof(RefreshArgs, a));
    asm volatile("" : "+s"(q));
    return q;
}
using KRef = const __attribute__((address_space(4))) RefreshCoef;
__device__ __forceinline__ KRef* coefficients() {
    KRef* q = (KRef*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                      offsetof(RefreshArgs, r));
    asm volatile("" : "+s"(q));
    return q;
}

// A thread's place: its column, the block's chunk of planes, the rows of the
// tile in a plane.
template <int W, int H>
struct Place {
    int tx, ty, i, j, kz0, kz1;
    int64_t tile0;
    u32 off, bytes;
    __device__ explicit Place(const Geom& g) {
        const int gx = (g.nx + W - 3) / (W - 2);
        const int gy = (g.ny + H - 3) / (H - 2);
        const int64_t t = xcd_tile(blockIdx.x, (int64_t)gridDim.x);
        const int bx = (int)(t % gx), by = (int)((t / gx) % gy), bz = (int)(t / ((int64_t)gx * gy));
        tile_thread<W, H>(tx, ty);
        i = bx * (W - 2) - 1 + tx;
        j = by * (H - 2) - 1 + ty;
        kz0 = bz * g.kz;
        kz1 = min(g.nz, kz0 + g.kz);
        const int row0 = max(by * (H - 2) - 1, 0), rows = min(by * (H - 2) + H - 2, g.ny) - row0 + 1;
        tile0 = (int64_t)row0 * g.P;
        off = ((u32)(j - row0) * (u32)g.P + (u32)i) * 8u;
        bytes = (u32)rows * (u32)g.P * 8u;
    }
};

template <int W, int H, bool STREAM>
__global__ __launch_bounds__(W * H, sweep_waves(W * H)) void k_refresh_tiled(RefreshArgs args) {
    enum { L_MU0, L_MU1, L_VX, L_VY, L_VZ1, L_TXY, L_TXZ, L_TYZ = L_TXZ + 2, NPL = L_TYZ + 2 };
    constexpr int WH = W * H, ONCE = STREAM ? NONTEMPORAL : 0;
    // (a margin on either side: every thread reads its neighbours' places)
    __shared__ double lds[NPL * WH + 2 * (W + 1)];
    const Geom& g = args.g;
    const Coef& c = args.c;
    const bool k0field = args.r.k0field != 0;
    const Place<W, H> at(g);
    const int tx = at.tx, ty = at.ty, i = at.i, j = at.j;

    const bool ci = i >= 0 && i < g.nx, cj = j >= 0 && j < g.ny;
    const bool edge = tx >= 1 && ty >= 1;   // LDS neighbours at tx-1, ty-1 exist
    const bool outc = ci && cj && tx >= 1 && tx <= W - 2 && ty >= 1 && ty <= H - 2;
    // edges computed by this thread (interior edges; boundary edges are zero
    // except for xy edges under the background shear of eq (32))
    const bool exy = edge && i >= 1 && i < g.nx && j >= 1 && j < g.ny;
    const bool bxy = edge && c.gbg_half != 0.0 && !exy && i >= 0 && i <= g.nx && j >= 0 && j <= g.ny;
    const bool exz = edge && i >= 1 && i < g.nx && cj;
    const bool eyz = edge && j >= 1 && j < g.ny && ci;
    const u32 o_cell = ci && cj ? at.off : OFF_NONE;
    const u32 o_vx = i >= 0 && i <= g.nx && cj ? at.off : OFF_NONE;
    const u32 o_vy = ci && j >= 0 && j <= g.ny ? at.off : OFF_NONE;
    const u32 o_xy = exy || bxy ? at.off : OFF_NONE;
    const u32 o_xz = exz ? at.off : OFF_NONE;
    const u32 o_yz = eyz ? at.off : OFF_NONE;
    const u32 o_out = outc ? at.off : OFF_NONE;

    // values of level/plane k along the own column
    struct QSet { double mu, vx, vy, vz, sxz, syz; };
    // cell and xy-edge values of plane k
    struct CSet { double sxy, sxx, syy, szz, lp, k0, pt, pf, mn, eta; };
    auto load_q = [&](KAux* p, int k, QSet& v) {
        const int64_t o = (int64_t)k * g.S + at.tile0;
        const u32 nb = k >= 0 && k < g.nz ? at.bytes : 0u;
        const u32 nbz = k >= 0 && k <= g.nz ? at.bytes : 0u;
        v.mu = ldp(p->mus + o, nb, o_cell);
        v.vx = ldp(p->vx + o, nb, o_vx);
        v.vy = ldp(p->vy + o, nb, o_vy);
        v.vz = ldp(p->vz + o, nbz, o_cell);
        v.sxz = ldp(p->sxz + o, nb, o_xz);
        v.syz = ldp(p->syz + o, nb, o_yz);
    };
    auto load_c = [&](KAux* p, int k, CSet& v) {
        const int64_t o = (int64_t)k * g.S + at.tile0;
        const u32 nb = k >= at.kz0 && k < at.kz1 ? at.bytes : 0u;
        v.sxy = ldp(p->sxy + o, nb, o_xy);
        v.sxx = ldp<ONCE>(p->sxx + o, nb, o_out);
        v.syy = ldp<ONCE>(p->syy + o, nb, o_out);
        v.szz = ldp<ONCE>(p->szz + o, nb, o_out);
        v.lp = ldp<ONCE>(p->lp + o, nb, o_out);
        v.k0 = ldp<ONCE>(p->k0 + o, k0field ? nb : 0u, o_out);
        v.pt = ldp<ONCE>(p->pt + o, nb, o_out);
        v.pf = ldp<ONCE>(p->pf + o, nb, o_out);
        v.mn = ldp<ONCE>(p->mn + o, nb, o_out);
        v.eta = ldp<ONCE>(p->eta + o, nb, o_out);
    };
    struct OSet { double kc, eta, mn; };
    auto store = [&](KAux* p, int k, bool live, const OSet& v) {
        const int64_t o = (int64_t)k * g.S + at.tile0;
        const u32 nb = live ? at.bytes : 0u;
        stp<ONCE>(p->kc + o, nb, o_out, v.kc);
        stp<ONCE>(p->eta + o, nb, o_out, v.eta);
        stp<ONCE>(p->mn + o, nb, o_out, v.mn);
    };
    double* const me = lds + (W + 1) + ty * W + tx;   // own place in a plane
    auto sh = [&](int pl, int dx, int dy) -> double& { return me[pl * WH + dy * W + dx]; };

    double mu_c, vx_c, vy_c, vz_c;             // own column, plane pz
    double txz_c = 0.0, tyz_c = 0.0;           // xz/yz-edge stresses of level pz

    // One plane step: the loads of the next go to qnn and cn, plane pz + 1 of
    // the queue is in qn, the cell set of plane pz in cc.
    auto step = [&](int pz, const QSet& qn, QSet& qnn, const CSet& cc, CSet& cn) __attribute__((always_inline)) {
        const bool live = pz >= at.kz0;
        KAux* const p = fields();
        load_q(p, pz + 2, qnn);
        load_c(p, pz + 1, cn);

        const double mu_n = qn.mu, vx_n = qn.vx, vy_n = qn.vy, vz_n = qn.vz;
        sh(L_MU0, 0, 0) = mu_c;
        sh(L_MU1, 0, 0) = mu_n;
        sh(L_VX, 0, 0) = vx_c;
        sh(L_VY, 0, 0) = vy_c;
        sh(L_VZ1, 0, 0) = vz_n;
        __syncthreads();

        // edge stresses: xy edges of plane pz, xz/yz edges of level pz+1
        double txy = 0.0, txz_n = 0.0, tyz_n = 0.0, ma, mb;
        const int lv = pz + 1;
        if (live && exy) {
            const double mue = 0.25 * (sh(L_MU0, -1, -1) + sh(L_MU0, 0, -1) + sh(L_MU0, -1, 0) + mu_c);
            const double e = 0.5 * ((vx_c - sh(L_VX, 0, -1)) * c.dyi + (vy_c - sh(L_VY, -1, 0)) * c.dxi) + c.gbg_half;
            maxwell(mue, c.gdts_inv, ma, mb);
            txy = ma * cc.sxy + mb * e;
        } else if (live && bxy) {
            // boundary edge: background strain rate only, viscosity averaged
            // over the cells inside
            double sum = 0.0;
            if (j >= 1) {
                if (i >= 1) sum += sh(L_MU0, -1, -1);
                if (i < g.nx) sum += sh(L_MU0, 0, -1);
            }
            if (j < g.ny) {
                if (i >= 1) sum += sh(L_MU0, -1, 0);
                if (i < g.nx) sum += mu_c;
            }
            const double mue = sum / (double)(((i >= 1) + (i < g.nx)) * ((j >= 1) + (j < g.ny)));
            maxwell(mue, c.gdts_inv, ma, mb);
            txy = ma * cc.sxy + mb * c.gbg_half;
        }
        if (exz && lv >= 1 && lv < g.nz) {
            const double mue = 0.25 * (sh(L_MU0, -1, 0) + mu_c + sh(L_MU1, -1, 0) + mu_n);
            const double e = 0.5 * ((vx_n - vx_c) * c.dzi + (vz_n - sh(L_VZ1, -1, 0)) * c.dxi);
            maxwell(mue, c.gdts_inv, ma, mb);
            txz_n = ma * qn.sxz + mb * e;
        }
        if (eyz && lv >= 1 && lv < g.nz) {
            const double mue = 0.25 * (sh(L_MU0, 0, -1) + mu_c + sh(L_MU1, 0, -1) + mu_n);
            const double e = 0.5 * ((vy_n - vy_c) * c.dzi + (vz_n - sh(L_VZ1, 0, -1)) * c.dyi);
            maxwell(mue, c.gdts_inv, ma, mb);
            tyz_n = ma * qn.syz + mb * e;
        }
        // neighbour velocities for the normal strain rates, taken before the
        // barrier (the next step's staging overwrites them)
        const double vx_e = sh(L_VX, 1, 0), vy_n1 = sh(L_VY, 0, 1);
        const int bn = lv & 1, bc = pz & 1;
        sh(L_TXY, 0, 0) = txy;
        sh(L_TXZ + bn, 0, 0) = txz_n;
        sh(L_TYZ + bn, 0, 0) = tyz_n;
        __syncthreads();

        OSet out{};
        if (live && outc) {
            const KRef& r = *coefficients();
            const double s = exp(cc.lp);
            const double phi = 1.0 - s;
            const double rr = quot(phi, r.phi0);
            out.kc = (r.k0field ? cc.k0 : r.kmuf0) * rr * rr * rr;
            const double R = (cc.pf > cc.pt) ? quot(1.0, r.R0) : 1.0;
            const double eta_new = r.eta0 * cc.mn * quot(r.phi0, phi) * R;
            out.eta = r.first ? eta_new : exp(r.r_eta * log(eta_new) + (1.0 - r.r_eta) * log(cc.eta));

            // normal stresses at the cell
            maxwell(mu_c, c.gdts_inv, ma, mb);
            const double dxv = (vx_e - vx_c) * c.dxi;
            const double dyv = (vy_n1 - vy_c) * c.dyi;
            const double dzv = (vz_n - vz_c) * c.dzi;
            const double d3 = (dxv + dyv + dzv) * c.third;
            const double txx = ma * cc.sxx + mb * (dxv - d3);
            const double tyy = ma * cc.syy + mb * (dyv - d3);
            const double tzz = ma * cc.szz + mb * (dzv - d3);
            // edge stresses averaged to the cell
            const double axy = 0.25 * (txy + sh(L_TXY, 1, 0) + sh(L_TXY, 0, 1) + sh(L_TXY, 1, 1));
            const double axz = 0.25 * (txz_c + sh(L_TXZ + bc, 1, 0) + txz_n + sh(L_TXZ + bn, 1, 0));
            const double ayz = 0.25 * (tyz_c + sh(L_TYZ + bc, 0, 1) + tyz_n + sh(L_TYZ + bn, 0, 1));
            const double tii = sqrt(0.5 * (txx * txx + tyy * tyy + tzz * tzz) + axy * axy + axz * axz + ayz * ayz);

            double mn_new = r.mu0;
            if (r.powerlaw) {
                const double t = tii * r.tau0_inv;
                const double tp = (r.n_pow == 3.0) ? t * t : pow(t, r.n_pow - 1.0);
                mn_new = quot(r.mu0, 1.0 + tp);
            }
            if (r.dpcap) {
                const double tyl = fmax(r.coh_cos + (cc.pt - cc.pf) * r.sin_f, r.tau_y_min);
                // the viscosity that puts the present strain rate on the
                // yield surface, where it is below the viscous one
                if (tii > 0.0) mn_new = fmin(mn_new, quot(cc.mn * tyl, tii));
            }
            out.mn = r.first ? mn_new : exp(r.r_mu * log(mn_new) + (1.0 - r.r_mu) * log(cc.mn));
        }
        store(fields(), pz, live, out);

        mu_c = fresh(mu_n); vx_c = fresh(vx_n); vy_c = fresh(vy_n); vz_c = fresh(vz_n);
        txz_c = txz_n;
        tyz_c = tyz_n;
    };

    QSet qa, qb;
    CSet ca, cb;
    {
        // the level below the first cells; as many (empty) stores as a step
        // ends with, so that the first step waits as every other does
        const int p0 = at.kz0 - 1;
        KAux* const p = fields();
        load_q(p, p0, qb);
        load_q(p, p0 + 1, qa);
        load_c(p, p0, ca);
        store(p, p0, false, OSet{});
        mu_c = qb.mu; vx_c = qb.vx; vy_c = qb.vy; vz_c = qb.vz;
    }
    for (int pz = at.kz0 - 1; pz < at.kz1; pz += 2) {
        step(pz, qa, qb, ca, cb);
        if (pz + 1 >= at.kz1) break;
        step(pz + 1, qb, qa, cb, ca);
    }
}

// The stress-history divergence folded into face fields, after a refresh:
// mu_s = Mn phi0 cmu at the cells, then on every face owned by a tile cell
// (the x-, y- and z-faces at its low side) Fo = div(a So), with a = xi/(1+xi)
// at the cells and, for the shear components, at the edges from the mean of
// the four cells' mu_s; boundary faces carry zero.  Same tiling and march as
// the refresh: per plane the new mu_s and the normal components a So are
// staged in LDS, each edge's a_e So_e is formed once (xy edges of the plane,
// xz/yz edges of the level above; the level below is carried over).
template <int W, int H, bool STREAM>
__global__ __launch_bounds__(W * H, sweep_waves(W * H)) void k_fo_tiled(RefreshArgs args) {
    enum { L_MU0, L_MU1, L_ASX, L_ASY, L_EXY, L_EXZ, L_EYZ = L_EXZ + 2, NPL = L_EYZ + 2 };
    constexpr int WH = W * H, ONCE = STREAM ? NONTEMPORAL : 0;
    __shared__ double lds[NPL * WH + 2 * (W + 1)];
    const Geom& g = args.g;
    const Coef& c = args.c;
    const double mu_scale = args.r.cmu, phi0 = args.r.phi0;
    const Place<W, H> at(g);
    const int tx = at.tx, ty = at.ty, i = at.i, j = at.j;

    const bool ci = i >= 0 && i < g.nx, cj = j >= 0 && j < g.ny;
    const bool edge = tx >= 1 && ty >= 1;
    const bool tcol = tx >= 1 && tx <= W - 2, trow = ty >= 1 && ty <= H - 2;
    const bool outc = ci && cj && tcol && trow;
    const bool exy = edge && i >= 1 && i < g.nx && j >= 1 && j < g.ny;
    const bool exz = edge && i >= 1 && i < g.nx && cj;
    const bool eyz = edge && j >= 1 && j < g.ny && ci;
    // boundary xy edges carry a history under the background shear of eq (32)
    const bool bxy = edge && c.gbg_half != 0.0 && !exy && i >= 0 && i <= g.nx && j >= 0 && j <= g.ny;
    const u32 o_cell = ci && cj ? at.off : OFF_NONE;
    const u32 o_xy = exy || bxy ? at.off : OFF_NONE;
    const u32 o_xz = exz ? at.off : OFF_NONE;
    const u32 o_yz = eyz ? at.off : OFF_NONE;
    const u32 o_out = outc ? at.off : OFF_NONE;
    // boundary faces at i = nx and j = ny belong to no cell: the thread on
    // them (in exactly one block) writes their zero
    const u32 o_fx = outc || (trow && i == g.nx && cj) ? at.off : OFF_NONE;
    const u32 o_fy = outc || (tcol && ty >= 1 && j == g.ny && ci) ? at.off : OFF_NONE;

    // plane/level k along the own column: Mn, szz (cells), sxz, syz (levels)
    struct QSet { double mn, szz, sxz, syz; };
    // plane k: sxx, syy (cells), sxy (xy edges)
    struct CSet { double sxx, syy, sxy; };
    auto load_q = [&](KAux* p, int k, QSet& v) {
        const int64_t o = (int64_t)k * g.S + at.tile0;
        const u32 nb = k >= 0 && k < g.nz ? at.bytes : 0u;
        v.mn = ldp(p->mn + o, nb, o_cell);
        v.szz = ldp(p->szz + o, nb, o_out);
        v.sxz = ldp(p->sxz + o, nb, o_xz);
        v.syz = ldp(p->syz + o, nb, o_yz);
    };
    auto load_c = [&](KAux* p, int k, CSet& v) {
        const int64_t o = (int64_t)k * g.S + at.tile0;
        const u32 nb = k >= at.kz0 && k < at.kz1 ? at.bytes : 0u;
        v.sxx = ldp(p->sxx + o, nb, o_cell);
        v.syy = ldp(p->syy + o, nb, o_cell);
        v.sxy = ldp(p->sxy + o, nb, o_xy);
    };
    struct OSet { double mus, fx, fy, fz; };
    auto store = [&](KAux* p, int k, bool live, const OSet& v) {
        const int64_t o = (int64_t)k * g.S + at.tile0;
        const u32 nb = live ? at.bytes : 0u;
        stp<ONCE>(p->mus + o, nb, o_out, v.mus);
        stp<ONCE>(p->fox + o, nb, o_fx, v.fx);
        stp<ONCE>(p->foy + o, nb, o_fy, v.fy);
        stp<ONCE>(p->foz + o, nb, o_out, v.fz);
    };
    double* const me = lds + (W + 1) + ty * W + tx;
    auto sh = [&](int pl, int dx, int dy) -> double& { return me[pl * WH + dy * W + dx]; };
    auto mus_of = [&](double mn) { return mn * phi0 * mu_scale; };

    double mu_c, szz_c;                // own column, plane pz
    double exz_c = 0.0, eyz_c = 0.0;   // a_e So of the xz/yz edges of level pz
    double asz_p = 0.0;                // a szz of plane pz - 1

    auto step = [&](int pz, const QSet& qn, QSet& qnn, const CSet& cc, CSet& cn) __attribute__((always_inline)) {
        const bool live = pz >= at.kz0;
        KAux* const p = fields();
        load_q(p, pz + 2, qnn);

        const double mu_n = mus_of(qn.mn);
        const double a_c = maxwell_a(mu_c, c.gdts_inv);
        const double asx = a_c * cc.sxx, asy = a_c * cc.syy, asz = a_c * szz_c;
        sh(L_MU0, 0, 0) = mu_c;
        sh(L_MU1, 0, 0) = mu_n;
        sh(L_ASX, 0, 0) = asx;
        sh(L_ASY, 0, 0) = asy;
        __syncthreads();
        load_c(fields(), pz + 1, cn);

        const int lv = pz + 1;
        double e_xy = 0.0, e_xz = 0.0, e_yz = 0.0;
        if (live && exy) {
            const double mue = 0.25 * (sh(L_MU0, -1, -1) + sh(L_MU0, 0, -1) + sh(L_MU0, -1, 0) + mu_c);
            e_xy = maxwell_a(mue, c.gdts_inv) * cc.sxy;
        } else if (live && bxy) {
            double sum = 0.0;   // viscosity averaged over the cells inside
            if (j >= 1) {
                if (i >= 1) sum += sh(L_MU0, -1, -1);
                if (i < g.nx) sum += sh(L_MU0, 0, -1);
            }
            if (j < g.ny) {
                if (i >= 1) sum += sh(L_MU0, -1, 0);
                if (i < g.nx) sum += mu_c;
            }
            const double mue = sum / (double)(((i >= 1) + (i < g.nx)) * ((j >= 1) + (j < g.ny)));
            e_xy = maxwell_a(mue, c.gdts_inv) * cc.sxy;
        }
        if (exz && lv >= 1 && lv < g.nz) {
            const double mue = 0.25 * (sh(L_MU0, -1, 0) + mu_c + sh(L_MU1, -1, 0) + mu_n);
            e_xz = maxwell_a(mue, c.gdts_inv) * qn.sxz;
        }
        if (eyz && lv >= 1 && lv < g.nz) {
            const double mue = 0.25 * (sh(L_MU0, 0, -1) + mu_c + sh(L_MU1, 0, -1) + mu_n);
            e_yz = maxwell_a(mue, c.gdts_inv) * qn.syz;
        }
        // west and south neighbours' a So, taken before the barrier (the next
        // step's staging overwrites them)
        const double asx_w = sh(L_ASX, -1, 0), asy_s = sh(L_ASY, 0, -1);
        const int bn = lv & 1, bc = pz & 1;
        sh(L_EXY, 0, 0) = e_xy;
        sh(L_EXZ + bn, 0, 0) = e_xz;
        sh(L_EYZ + bn, 0, 0) = e_yz;
        __syncthreads();

        OSet out{};
        if (live && outc) {
            out.mus = mu_c;
            if (i >= 1) out.fx = (asx - asx_w) * c.dxi + (sh(L_EXY, 0, 1) - e_xy) * c.dyi + (e_xz - exz_c) * c.dzi;
            if (j >= 1) out.fy = (sh(L_EXY, 1, 0) - e_xy) * c.dxi + (asy - asy_s) * c.dyi + (e_yz - eyz_c) * c.dzi;
            if (pz >= 1)
                out.fz = (sh(L_EXZ + bc, 1, 0) - exz_c) * c.dxi + (sh(L_EYZ + bc, 0, 1) - eyz_c) * c.dyi +
                         (asz - asz_p) * c.dzi;
        }
        KAux* const pe = fields();
        store(pe, pz, live, out);
        if (pz == g.nz - 1) stp(pe->foz + (int64_t)g.nz * g.S + at.tile0, at.bytes, o_out, 0.0);

        mu_c = mu_n;
        szz_c = fresh(qn.szz);
        exz_c = e_xz;
        eyz_c = e_yz;
        asz_p = asz;
    };

    QSet qa, qb;
    CSet ca, cb;
    {
        const int p0 = at.kz0 - 1;
        KAux* const p = fields();
        load_q(p, p0, qb);
        load_q(p, p0 + 1, qa);
        load_c(p, p0, ca);
        store(p, p0, false, OSet{});
        mu_c = mus_of(qb.mn);
        szz_c = qb.szz;
    }
    for (int pz = at.kz0 - 1; pz < at.kz1; pz += 2) {
        step(pz, qa, qb, ca, cb);
        if (pz + 1 >= at.kz1) break;
        step(pz + 1, qb, qa, cb, ca);
    }
}

template <int W, int H, bool STREAM>
hipError_t launch_tile(bool fo, const TileShape& t, const RefreshArgs& a, hipStream_t s) {
    if (!rows_fit(a.g, H, sizeof(double))) return hipErrorInvalidValue;
    const dim3 grid((unsigned)sweep_blocks(a.g, t)), block(W * H);
    if (fo)
        hipLaunchKernelGGL((k_fo_tiled<W, H, STREAM>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_refresh_tiled<W, H, STREAM>), grid, block, 0, s, a);
    return hipGetLastError();
}

// The tile of the grid's plain FP64 sweeps.
hipError_t launch(bool fo, const Geom& g, const TileShape& t, const Coef& c, const RefreshCoef& r, const AuxPtrs& p,
                  hipStream_t s) {
    RefreshArgs a{g, c, r, p};
    a.g.kz = t.kz;
    switch (t.w * 100 + t.h) {
        case 6610: return t.stream ? launch_tile<66, 10, true>(fo, t, a, s) : launch_tile<66, 10, false>(fo, t, a, s);
        case 6606: return launch_tile<66, 6, false>(fo, t, a, s);
        case 3414: return launch_tile<34, 14, false>(fo, t, a, s);
        case 3406: return launch_tile<34, 6, false>(fo, t, a, s);
        case 3404: return launch_tile<34, 4, false>(fo, t, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fo_tiled(const Geom& g, const TileShape& t, const Coef& c, const RefreshCoef& r, const AuxPtrs& a,
                           hipStream_t s) {
    return launch(true, g, t, c, r, a, s);
}

hipError_t launch_refresh_tiled(const Geom& g, const TileShape& t, const Coef& c, const RefreshCoef& r, const AuxPtrs& a,
                                hipStream_t s) {
    return launch(false, g, t, c, r, a, s);
}

}  // namespace ptk
