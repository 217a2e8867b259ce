// Fused pseudo-transient sweep for gfx950.
//
// One launch performs a whole PT iteration (thesis article 1, section 2.2):
// total-pressure update (eq (17)), Darcy flux and fluid-pressure update
// (eqs (18), (20)), visco-elastic stresses (eq (21)), damped momentum update
// (eq (19)) and the porosity update in log space (eq (22)), all from the
// iteration-k state (Jacobi), with the boundary conditions of eqs (33)-(34).
//
// Modes of the same sweep:
//   THESIS  FP64, porosity updated every iteration (thesis schedule);
//   LINEAR  FP64, porosity frozen (one linear system of a Picard stage);
//   RESID   FP64, no update: writes the residuals f, r_Pt, r_Pf of the present
//           state (physical stress, current Pt) in FP32 for defect correction;
//   CORR    FP32 sweep on the correction system A(c) d = -r of a Picard stage:
//           the same iteration applied to x + d, with the FP64 residual of x as
//           right-hand side (no old values, no buoyancy, no history term).
//
// Work decomposition.  A W x H block owns a column of (W-2) x (H-2) cells
// plus a one-cell halo ring and marches upward through a chunk of g.kz planes.
// Per plane the block
//   1. stages the plane's velocities, fluid pressure, permeability, solid
//      fraction and shear viscosity in LDS (values of plane p+1 that the
//      column needs again next plane stay in registers: a z register queue);
//   2. computes cell quantities (div V, Pt', stresses) on the cells and the
//      low halo, shear stresses on edges, and Pf', ln(1-phi)' on the tile;
//   3. after one more barrier, updates the three face velocities of every
//      tile cell.
// The next plane's loads are issued one step ahead, in groups over the step.
// Stresses and Darcy fluxes never touch HBM; the iterated fields are written
// once.
//
// What bounds it: HBM on large grids (the 24 streams of a thesis sweep, at
// the rate that many concurrent streams reach), one wave's chain of dependent
// instructions through a plane step on small ones.  Both suffer from what
// keeps a step from overlapping the next one's memory traffic and from every
// instruction that is not arithmetic, so:
//   - loads and stores go through buffer descriptors whose range check
//     replaces the edges' branches and selects (see ldp); the number of
//     memory operations of a step is the same for every wave, so a step waits
//     for exactly its own plane's loads and never for its predecessor's
//     stores (before, every step ended with all of them drained);
//   - two steps per loop round on alternating register sets, so that no loaded
//     value is copied before it is needed;
//   - field pointers come from the argument segment at each step, constants
//     combined on the host, divisions without operand rescaling, one
//     pseudo-step quotient per cell: 355 vector instructions per plane step of
//     the linear sweep instead of 640.
// Measured at 511^3 (before all of this -> now): thesis sweep 6.18 -> 4.76 ms
// (5.7 TB/s of its 24 streams; a copy reaches 6.0), with norms 8.69 -> 6.49,
// linear 5.67 -> 4.37, residual 6.49 -> 3.78, FP32 correction 2.66 -> 2.22; at
// 32^3, mostly by its tile (sweep_shape, pt_internal.h), thesis 27.1 -> 7.7 us.
//
// Damped velocity update of the FP64 sweeps (eq (19) with the script's
// damping): R' = f/rho_i + d R, V' = V + dtau_V R'.  Between checks the
// sweep does not store R: with dtau_V unchanged since the last iteration,
// d R = d (V - V_prev) / dtau_V, and V_prev is the other copy of V (the one
// this sweep overwrites), so V' = V + dtau_V f/rho_i + d (V - V_prev) needs
// no R stream (three fewer of 27).  The first sweep after the pseudo steps
// change (a refresh) reads the stored R instead (c.rform); sweeps that end a
// check interval store R' = (V' - V)/dtau_V (c.rwrite), so that it is there
// when the next refresh comes.  The FP32 correction sweeps do the same with
// the damped residual of the correction.
#include "plane.h"
#include "pt_internal.h"

// The sweeps are many kernels: the build compiles this source three times,
// side by side, each time one part of the launchers at the end.
#ifdef SWEEP_PART
#define SWEEP_HAS(part) (SWEEP_PART == (part))
#else
#define SWEEP_HAS(part) 1
#endif

// Multiply-adds are fused where an expression of the source has one, not
// where the optimiser finds one: every variant and tile of the sweep rounds
// alike, so results do not depend on the tiling.
#pragma clang fp contract(on)

namespace ptk {

namespace {

// LDS planes of a block, each W x H values: inputs of plane p (L_VZ1, L_MU1:
// of plane p + 1), then what the face updates read.  A margin of one row and
// one value on either side lets every thread read its neighbours' places;
// what a thread at the rim of the block reads there is never used.
enum LdsPlane { L_VX, L_VY, L_VZ1, L_PF, L_KC, L_MU, L_MU1, L_PTN, L_TXX, L_TYY, L_TXY, L_TXZ, L_TYZ = L_TXZ + 2,
                L_CORE = L_TYZ + 2 };   // then, where used: the velocity pseudo step and the solid fraction of two
                                        // planes, tau_zz, the norms' W plane

// Constants in the working precision of the sweep, combined on the host (the
// scalar unit has no floating point: a product formed in the kernel would
// occupy vector registers).
template <typename T>
struct CT {
    T dxi, dyi, dzi, third;
    T hxx, hyy, buoy;                     // -1/(2 dx^2), -1/(2 dy^2); Darcy buoyancy
    T dtaupt_c, bdt, alpha, bda;          // beta_d/dt, alpha, alpha beta_d/dt
    T dtaupf_c, ab, bdab;                 // alpha/B, (alpha/B) beta_d/dt
    T gdts, gdts4, beta_n;                // 1/(G dtS), a quarter of it
    T rho_i_inv, dtauv_c, dampx, dampy, dampz;
    T rhofg, rhosg, rhobg;
    T hdx, hdy, hdz, bpt, dt;             // 1/(2 dx) ..., beta_phi/dt
    T gbg_half;
    explicit CT(const Coef& c)
        : dxi(T(c.dxi)), dyi(T(c.dyi)), dzi(T(c.dzi)), third(T(c.third)), hxx(T(-0.5 * c.dxi * c.dxi)),
          hyy(T(-0.5 * c.dyi * c.dyi)), buoy(T(c.buoy)), dtaupt_c(T(c.dtaupt_c)),
          bdt(T(c.beta_d * c.dti)), alpha(T(c.alpha)), bda(T(c.beta_d * c.alpha * c.dti)), dtaupf_c(T(c.dtaupf_c)),
          ab(T(c.ab)), bdab(T(c.beta_d * c.ab * c.dti)), gdts(T(c.gdts_inv)), gdts4(T(0.25 * c.gdts_inv)),
          beta_n(T(c.beta_n)), rho_i_inv(T(c.rho_i_inv)), dtauv_c(T(c.dtauv_c)), dampx(T(c.dampx)),
          dampy(T(c.dampy)), dampz(T(c.dampz)), rhofg(T(c.rhofg)), rhosg(T(c.rhosg)), rhobg(T(c.rhobg)),
          hdx(T(0.5 * c.dxi)), hdy(T(0.5 * c.dyi)), hdz(T(0.5 * c.dzi)), bpt(T(c.beta_phi * c.dti)), dt(T(c.dt)),
          gbg_half(T(c.gbg_half)) {}
};

// Kernel arguments as one block, so that they can be read again from the
// argument segment where they are used (see the sweep).
template <typename T>
struct SweepArgs {
    Geom g;
    CT<T> c;
    SweepPtrs<T> p;
};

// Damping memory of a sweep variant: the previous velocity iterate (in the
// rx..rz inputs), the stored damped residual, or none (damping factor 0).
// RM_FROZEN, mechanics off: V, R and Pt keep their values, whatever the forces
// (a variant of its own: zero pseudo steps let a non-finite force in, and a
// flag in the others made a multigrid stage at 127^3 1.6 % slower, a linear
// solve at 40^3 0.5 %).
constexpr int RM_VPREV = 0, RM_STORED = 1, RM_NONE = 2, RM_FROZEN = 3;

// One face's damped velocity update (see the header): returns V', sets the
// damped residual R' in r.  q: the stored R or V_prev.
template <int RM, typename T, typename C>
__device__ __forceinline__ T damped_update(const C& c, T v_c, T q, T f, T damp, T dtv, T& r) {
    if constexpr (RM == RM_FROZEN) {
        r = q;
        return v_c;
    } else if constexpr (RM == RM_STORED) {
        r = f * c.rho_i_inv + damp * q;
        return v_c + dtv * r;
    } else if constexpr (RM == RM_NONE) {
        r = f * c.rho_i_inv;
        return v_c + dtv * r;
    }
    const T v = v_c + dtv * (f * c.rho_i_inv) + damp * (v_c - q);
    r = quot(v - v_c, dtv);
    return v;
}

// RM: where the damping memory is; RW: store the damped residual R'.  W x H:
// the block's threads.  BGS: the background shear of eq (32) is on.  STREAM:
// the fields outgrow the last-level cache.
template <typename T, int MODE, bool NORMS, int RM, bool RW, int W, int H, bool BGS, bool STREAM>
__global__ __launch_bounds__(W * H, sweep_waves(W * H, NORMS && sizeof(T) == 8)) void k_sweep(SweepArgs<T> args) {
    static_assert(W * H <= 1024, "a block holds at most 1024 threads");
    constexpr bool UPD_LP = (MODE == MD_THESIS);
    constexpr bool RESID = (MODE == MD_RESID);
    constexpr bool CORR = (MODE == MD_CORR);
    constexpr bool WNORM = NORMS || RESID;
    constexpr bool RREAD = !RESID && RM != RM_NONE && (RM != RM_FROZEN || RW);
    constexpr bool GATED = (MODE == MD_LINEAR || CORR) && RM != RM_NONE;   // the sweeps of solves
    constexpr int L_DTV = L_CORE, L_S = L_DTV + (RESID ? 0 : 2), L_TZZ = L_S + (UPD_LP ? 2 : 0), L_W = L_TZZ + (UPD_LP ? 1 : 0), NPL = L_W + (NORMS ? 1 : 0);
    constexpr int WH = W * H;
    __shared__ T lds[NPL * WH + 2 * (W + 1)];
    const Geom& g = args.g;
    const CT<T>& c = args.c;
    const T zero = T(0), one = T(1), two = T(2), quarter = T(0.25);

    const int gx = (g.nx + W - 3) / (W - 2);
    const int gy = (g.ny + H - 3) / (H - 2);
    const int64_t total = (int64_t)gridDim.x;
    const int64_t Tt = xcd_tile(blockIdx.x, total);
    const int bx = (int)(Tt % gx);
    const int by = (int)((Tt / gx) % gy);
    const int bz = (int)(Tt / ((int64_t)gx * gy));

    int tx, ty;
    tile_thread<W, H>(tx, ty);
    const int i = bx * (W - 2) - 1 + tx;
    const int j = by * (H - 2) - 1 + ty;
    const int kz0 = bz * g.kz;
    const int kz1 = min(g.nz, kz0 + g.kz);

    const bool ci = (i >= 0) && (i < g.nx);
    const bool cj = (j >= 0) && (j < g.ny);
    const bool cell = ci && cj;
    const bool outc = cell && tx >= 1 && tx <= W - 2 && ty >= 1 && ty <= H - 2;
    const bool cellq = cell && tx <= W - 2 && ty <= H - 2;
    // waves without a row of the tile skip what only tile cells need
    const bool tile_wave = __builtin_amdgcn_ballot_w64(tx >= 1 && tx <= W - 2 && ty >= 1 && ty <= H - 2) != 0;
    const bool e_xy = i >= 1 && i < g.nx && j >= 1 && j < g.ny;   // interior edges of this column
    const bool e_xz = i >= 1 && i < g.nx && cj;
    const bool e_yz = j >= 1 && j < g.ny && ci;

    // Byte offsets in the tile's rows, OFF_NONE where the column has no such value
    // or the thread no use for it (halo columns would otherwise fetch
    // tile-only fields from HBM a second time).  Pf and k take the nearest
    // cell's value outside the domain: the gradient, so the Darcy flux,
    // through the wall comes out as zero and the largest neighbouring k is
    // the same.
    const u32 sz = (u32)sizeof(T);
    const int row0 = max(by * (H - 2) - 1, 0), rows = min(by * (H - 2) - 1 + H - 1, g.ny) - row0 + 1;
    const int64_t tile0 = (int64_t)row0 * g.P;
    const u32 col = (u32)(j - row0) * (u32)g.P + (u32)i;
    const u32 o_near = ((u32)(min(max(j, 0), g.ny - 1) - row0) * (u32)g.P + (u32)min(max(i, 0), g.nx - 1)) * sz;
    const u32 o_cell = cell ? col * sz : OFF_NONE;
    const u32 o_vx = ((i >= 0) && (i <= g.nx) && cj) ? col * sz : OFF_NONE;
    const u32 o_vy = (ci && (j >= 0) && (j <= g.ny)) ? col * sz : OFF_NONE;
    const u32 o_q = cellq ? col * sz : OFF_NONE;
    const u32 o_out = outc ? col * sz : OFF_NONE;
    const u32 so = RESID ? (u32)sizeof(float) : sz;              // stored values
    const u32 o_sx = (outc && i >= 1) ? col * so : OFF_NONE;
    const u32 o_sy = (outc && j >= 1) ? col * so : OFF_NONE;
    const u32 o_sc = outc ? col * so : OFF_NONE;
    const u32 tile_bytes = (u32)rows * (u32)g.P * sz;
    const u32 tile_store = (u32)rows * (u32)g.P * so;

    // The field pointers are read from the argument segment at every plane
    // step (scalar loads that hit the scalar cache): kept in registers they
    // and the constants exceed the scalar file, and the compiler parks them
    // in vector lanes (measured: 148 of 640 vector instructions per plane
    // step were lane reads).  The empty asm keeps the loads in the loop.
    using KPtrs = const __attribute__((address_space(4))) SweepPtrs<T>;
    KPtrs* const kargs = (KPtrs*)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() +
                                  offsetof(SweepArgs<T>, p));
    auto ptrs = [&]() {
        KPtrs* q = kargs;
        asm volatile("" : "+s"(q));
        return q;
    };

    // queue set of a plane (own column): needed at planes p-1..p+1
    struct QSet { T vx, vy, vz, pf, kc, lp, mu; };
    // cell set of a plane: needed for the cell quantities of plane p
    struct CSet { T pt, pto, pfo, eta; };
    // face set of a plane: needed when its faces and its porosity are updated
    struct FSet { T lpo, rx, ry, rz, fox, foy, foz; };
    auto load_q = [&](KPtrs* p, int k, QSet& q) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = (k >= 0 && k < g.nz) ? tile_bytes : 0u;
        const u32 nbz = (k >= 0 && k <= g.nz) ? tile_bytes : 0u;
        q.vx = ldp(p->vx + o, nb, o_vx);
        q.vy = ldp(p->vy + o, nb, o_vy);
        q.vz = ldp(p->vz + o, nbz, o_cell);
        q.pf = ldp(p->pf + o, nb, o_near);
    };
    auto load_q2 = [&](KPtrs* p, int k, QSet& q) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = (k >= 0 && k < g.nz) ? tile_bytes : 0u;
        q.kc = ldp(p->kc + o, nb, o_near);
        q.mu = ldp(p->mus + o, nb, o_cell);
        if constexpr (CORR) q.lp = zero;
        else q.lp = ldp(p->lp + o, nb, o_cell);
    };
    auto load_c = [&](KPtrs* p, int k, CSet& cs) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = (k >= 0 && k < g.nz) ? tile_bytes : 0u;
        cs.pt = ldp(p->pt + o, nb, o_q);
        cs.pto = ldp(p->pto + o, nb, o_q);
        cs.pfo = ldp(p->pfo + o, nb, o_q);
        cs.eta = ldp(p->eta + o, nb, o_q);
    };
    // Where the fields outgrow the last-level cache, what a launch reads once
    // (the tile-only fields) and what it writes bypass the caches, which
    // leaves them to the halo data that neighbouring tiles read again
    // (measured, none -> loads and stores: 511^3 thesis 5.30 -> 4.92 ms,
    // linear 4.96 -> 4.85, FP32 correction 2.52 -> 2.34; 255^3 661 -> 639,
    // 635 -> 616, 302 -> 282 us); where they fit, the next launch finds them
    // there (110^3 thesis 58.0 us without, 64.4 with).
    constexpr int ONCE = STREAM ? NONTEMPORAL : 0;
    auto load_f = [&](KPtrs* p, int k, FSet& f) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = (k >= kz0 && k < kz1) ? tile_bytes : 0u;
        if constexpr (UPD_LP) f.lpo = ldp<ONCE>(p->lpo + o, nb, o_out);
        else f.lpo = zero;
        if constexpr (RREAD) {
            f.rx = ldp<ONCE>(p->rx + o, nb, o_out);
            f.ry = ldp<ONCE>(p->ry + o, nb, o_out);
            f.rz = ldp<ONCE>(p->rz + o, nb, o_out);
        } else {
            f.rx = f.ry = f.rz = zero;
        }
        f.fox = ldp<ONCE>(p->fox + o, nb, o_out);
        f.foy = ldp<ONCE>(p->foy + o, nb, o_out);
        f.foz = ldp<ONCE>(p->foz + o, nb, o_out);
    };
    // outputs of a plane
    struct OSet { T vx, vy, vz, rx, ry, rz, pt, pf, lp; };
    auto store = [&](KPtrs* p, int k, bool live, const OSet& s) {
        const int64_t o = (int64_t)k * g.S + tile0;
        const u32 nb = live ? tile_store : 0u;
        const u32 nbz = (live && k >= 1) ? tile_store : 0u;
        if constexpr (RESID) {
            stp(p->res_fx + o, nb, o_sx, float(s.vx));
            stp(p->res_fy + o, nb, o_sy, float(s.vy));
            stp(p->res_fz + o, nbz, o_sc, float(s.vz));
            stp(p->res_rpt + o, nb, o_sc, float(s.pt));
            stp(p->res_rpf + o, nb, o_sc, float(s.pf));
        } else {
            stp<ONCE>(p->vx_o + o, nb, o_sx, s.vx);
            stp<ONCE>(p->vy_o + o, nb, o_sy, s.vy);
            stp<ONCE>(p->vz_o + o, nbz, o_sc, s.vz);
            if constexpr (RW) {
                stp<ONCE>(p->rx_o + o, nb, o_sx, s.rx);
                stp<ONCE>(p->ry_o + o, nb, o_sy, s.ry);
                stp<ONCE>(p->rz_o + o, nbz, o_sc, s.rz);
            }
            stp<ONCE>(p->pt_o + o, nb, o_sc, s.pt);
            stp<ONCE>(p->pf_o + o, nb, o_sc, s.pf);
            if constexpr (UPD_LP) stp<ONCE>(p->lp_o + o, nb, o_sc, s.lp);
        }
    };
    auto weight = [&](T s) -> T { return c.rhofg * (one - s) + c.rhosg * s; };
    auto solid = [&](T lp) -> T { return CORR ? one : T(exp(lp)); };

    T* const me = lds + (W + 1) + ty * W + tx;   // own place in a plane
    auto sh = [&](int pl, int dx, int dy) -> T& { return me[pl * WH + dy * W + dx]; };

    // register queue (own column): _p = plane p-1, _c = plane p, _n = plane p+1
    T vx_c, vy_c, vz_c, pf_c, kc_c, s_c, mu_c, lp_c;
    T tzz_r = zero, rg_p = zero, w_p = zero, txz_c = zero, tyz_c = zero;
    // of the level below plane p: Darcy flux, larger k and advection of the two cells
    T qz_c = zero, kz_c = zero, az_c = zero;
    T nm[NNORM];
#pragma unroll
    for (int q = 0; q < NNORM; ++q) nm[q] = zero;

    FSet ff;   // face set of plane p, loaded at the end of the step before

    // One plane step: plane pz + 1 of the queue is in qn, the cell set of
    // plane pz in cc (both loaded one step ahead), the queue's loads of the
    // next step go to qnn.  The loads are issued in four groups over the step
    // (the queue's before and after the first barrier, the cell set's before
    // the second, the face set's at the end): issued together at its start
    // they hold the waves up until the memory pipeline has taken them
    // (measured, together -> spread: linear sweep without damping 127^3 72.7 ->
    // 58.3 us, 300x255x201 555 -> 490 us; thesis 173x131x97 104 -> 97 us,
    // 255x255x510 1255 -> 1203 us, 511^3 4.76 -> 4.71 ms; FP32 95^3 17.6 ->
    // 16.7 us).
    auto step = [&](int pz, const QSet& qn, QSet& qnn, CSet& cc) __attribute__((always_inline)) {
        const bool plc = pz >= 0;                // plane pz is a real plane
        const bool pln = pz + 1 < g.nz;          // plane pz+1 is a real plane
        const bool live = pz >= kz0;             // outputs of this plane belong to the block
        const int bn = (pz + 1) & 1, bc = pz & 1;
        KPtrs* const p = ptrs();

        // prefetch what the next step needs
        load_q(p, pz + 2, qnn);

        const T vx_n = qn.vx, vy_n = qn.vy, vz_n = qn.vz, pf_n = qn.pf, kc_n = qn.kc;
        const T lp_n = qn.lp, mu_n = qn.mu;
        const T s_n = solid(lp_n);
        const T pt = cc.pt, pto = cc.pto, pfo = cc.pfo, eta = cc.eta;

        sh(L_VX, 0, 0) = vx_c;
        sh(L_VY, 0, 0) = vy_c;
        sh(L_VZ1, 0, 0) = vz_n;
        sh(L_PF, 0, 0) = pf_c;
        sh(L_KC, 0, 0) = kc_c;
        if constexpr (UPD_LP) sh(L_S + bc, 0, 0) = s_c;
        sh(L_MU, 0, 0) = mu_c;
        sh(L_MU1, 0, 0) = mu_n;
        __syncthreads();
        load_q2(ptrs(), pz + 2, qnn);

        // Cells outside the domain compute values from zeros that nothing
        // reads but the faces on the walls, which are not stored.
        // ---- cell quantities: div V, Pt' (eq (17)), stresses (eq (21)) ----
        T ptn, txx, tyy, tzz, rg = zero, w = zero, chi, rpt_k, txy, txz_n, tyz_n;
        T pfn = zero, lpn = zero, rpf_k = zero;
        auto cell_part = [&]() __attribute__((always_inline)) {
            const T dxv = (sh(L_VX, 1, 0) - vx_c) * c.dxi;
            const T dyv = (sh(L_VY, 0, 1) - vy_c) * c.dyi;
            const T dzv = (vz_n - vz_c) * c.dzi;
            const T divv = dxv + dyv + dzv;
            const T dtp = c.dtaupt_c * mu_c;
            // r_Pt of iteration k: the numerical-compressibility term of the
            // stresses takes it before the pressure update
            if constexpr (CORR) {
                // d Pt' = [d Pt - dtau (div dV + r_Pt(x) - beta_d alpha dPf/dt - dPf chi)]
                //         / (1 + dtau (beta_d/dt + chi)); chi is a stored field here
                chi = eta;
                ptn = quot(pt - dtp * (divv + pto - c.bda * pf_c - pf_c * chi), one + dtp * (c.bdt + chi));
                rpt_k = pto + divv + c.bdt * (pt - c.alpha * pf_c) + (pt - pf_c) * chi;
            } else {
                chi = quot(one, eta * s_c);
                if constexpr (RESID || RM == RM_FROZEN)
                    ptn = pt;
                else
                    ptn = quot(pt - dtp * (divv - c.bdt * (pto + c.alpha * (pf_c - pfo)) - pf_c * chi),
                               one + dtp * (c.bdt + chi));
                rpt_k = divv + c.bdt * ((pt - pto) - c.alpha * (pf_c - pfo)) + (pt - pf_c) * chi;
                if constexpr (!UPD_LP) rg = weight(s_c);
            }
            const T b = quot(two * mu_c, one + mu_c * c.gdts);
            const T d3 = divv * c.third;
            const T comp = RESID ? zero : c.beta_n * rpt_k;
            txx = b * ((dxv - d3) + comp);
            tyy = b * ((dyv - d3) + comp);
            tzz = b * ((dzv - d3) + comp);
            if (NORMS) w = b * comp - ptn + pt;
        };

        // ---- Darcy flux and fluid pressure (eqs (18), (20)); porosity (eq (22)) ----
        T qz_n = zero, kz_n = zero, az_n = zero;
        auto fluid_part = [&]() __attribute__((always_inline)) {
            const T kw = sh(L_KC, -1, 0), ke = sh(L_KC, 1, 0);
            const T ks = sh(L_KC, 0, -1), kn = sh(L_KC, 0, 1);
            // (fluxes of the x and y faces without their factors -1/(2 dx), -1/(2 dy);
            // products rounded before they are subtracted, so that equal
            // fluxes cancel exactly: the sign of Pf - Pt in a quiet medium
            // switches the bulk viscosity)
            T qx, qy;
            {
#pragma clang fp contract(off)
                qx = (kc_c + ke) * (sh(L_PF, 1, 0) - pf_c) - (kw + kc_c) * (pf_c - sh(L_PF, -1, 0));
                qy = (kc_c + kn) * (sh(L_PF, 0, 1) - pf_c) - (ks + kc_c) * (pf_c - sh(L_PF, 0, -1));
                // the flux through the level above, zero through the walls
                const T hz = (plc && pln) ? T(-0.5) : zero;
                qz_n = hz * (kc_c + kc_n) * ((pf_n - pf_c) * c.dzi + (CORR ? zero : c.buoy));
            }
            const T divq = c.hxx * qx + c.hyy * qy + (qz_n - qz_c) * c.dzi;
            // largest permeability of the cell and its face neighbours
            kz_n = max1(kc_c, kc_n);
            const T kl = max1(max1(max1(kw, ke), max1(ks, kn)), max1(kz_c, kz_n));
            const T dtf = quot_field(c.dtaupf_c, kl);
            if constexpr (CORR) {
                pfn = quot(pf_c - dtf * (divq + pfo - c.bda * pt - pt * chi), one + dtf * (c.bdab + chi));
                if (WNORM) rpf_k = pfo + divq + c.bdt * (c.ab * pf_c - c.alpha * pt) + (pf_c - pt) * chi;
            } else if constexpr (RESID) {
                pfn = pf_c;
                rpf_k = divq + c.bdt * (c.ab * (pf_c - pfo) - c.alpha * (pt - pto)) + (pf_c - pt) * chi;
            } else {
                pfn = quot(pf_c - dtf * (divq - c.bdt * (c.ab * pfo + c.alpha * (pt - pto)) - pt * chi),
                           one + dtf * (c.bdab + chi));
                if (WNORM) rpf_k = divq + c.bdt * (c.ab * (pf_c - pfo) - c.alpha * (pt - pto)) + (pf_c - pt) * chi;
            }
            if constexpr (UPD_LP) {
                az_n = vz_n * (s_n - s_c);
                const T adv = c.hdx * (vx_c * (s_c - sh(L_S + bc, -1, 0)) + sh(L_VX, 1, 0) * (sh(L_S + bc, 1, 0) - s_c)) +
                              c.hdy * (vy_c * (s_c - sh(L_S + bc, 0, -1)) + sh(L_VY, 0, 1) * (sh(L_S + bc, 0, 1) - s_c)) +
                              c.hdz * (az_c + az_n);
                const T dphidt = c.bpt * ((pfn - pfo) - (ptn - pto)) + quot(pfn - ptn, eta) + adv;
                lpn = ff.lpo - c.dt * dphidt;
            }
        };

        // ---- shear stresses on the xy-edges of plane pz and the xz/yz-edges of level pz+1 ----
        // (half the Maxwell coefficient 2 mu/(1 + xi) on an edge, from the sum
        // of its four cells' viscosities; the strain rates without their 1/2)
        auto edge_mu = [&](T sum) -> T { return quot(quarter * sum, one + sum * c.gdts4); };
        auto edge_part = [&]() __attribute__((always_inline)) {
            const T mu_w = sh(L_MU, -1, 0), mu_s = sh(L_MU, 0, -1);
            const T sxy = sh(L_MU, -1, -1) + mu_s + mu_w + mu_c;
            T exy = (vx_c - sh(L_VX, 0, -1)) * c.dyi + (vy_c - sh(L_VY, -1, 0)) * c.dxi;
            if constexpr (BGS) exy += two * c.gbg_half;   // background shear (eq (32))
            txy = edge_mu(sxy) * exy;
            txy = (e_xy && plc) ? txy : zero;
            if constexpr (BGS) {
                if (!e_xy && plc && i >= 0 && i <= g.nx && j >= 0 && j <= g.ny) {
                    // boundary edge: the perturbation slips freely, the background
                    // strain rate remains; viscosity averaged over the cells inside
                    // (the staged values outside the domain are zero)
                    const T cnt = T(((i >= 1) + (i < g.nx)) * ((j >= 1) + (j < g.ny)));
                    const T mue = quot(sxy, cnt);
                    txy = quot(two * mue, one + mue * c.gdts) * c.gbg_half;
                }
            }
            const bool lev = plc && pln;
            const T exz = (vx_n - vx_c) * c.dzi + (vz_n - sh(L_VZ1, -1, 0)) * c.dxi;
            txz_n = edge_mu(mu_w + mu_c + sh(L_MU1, -1, 0) + mu_n) * exz;
            txz_n = (e_xz && lev) ? txz_n : zero;
            const T eyz = (vy_n - vy_c) * c.dzi + (vz_n - sh(L_VZ1, 0, -1)) * c.dyi;
            tyz_n = edge_mu(mu_s + mu_c + sh(L_MU1, 0, -1) + mu_n) * eyz;
            tyz_n = (e_yz && lev) ? tyz_n : zero;
        };
        if (tile_wave) {
            // In the thesis sweeps the scheduler keeps the parts apart:
            // interleaved, they need more registers than eleven waves have
            // (the order is the one whose live values fit).
            cell_part();
            if constexpr (UPD_LP && BGS) {
                __builtin_amdgcn_sched_barrier(0);
                edge_part();
                __builtin_amdgcn_sched_barrier(0);
                fluid_part();
            } else {
                if constexpr (UPD_LP) __builtin_amdgcn_sched_barrier(0);
                fluid_part();
                if constexpr (UPD_LP) __builtin_amdgcn_sched_barrier(0);
                edge_part();
            }
        } else {
            cell_part();
            edge_part();
        }
        const T ptn_p = sh(L_PTN, 0, 0);   // plane p-1 (not used on the lowest plane)
        T tzz_p = tzz_r;
        if constexpr (UPD_LP) {
            tzz_p = sh(L_TZZ, 0, 0);
            sh(L_TZZ, 0, 0) = tzz;
        }
        sh(L_PTN, 0, 0) = ptn;
        // the velocity pseudo step of the cell; a face takes the smaller of its
        // cells' (the one of the larger viscosity): one quotient per cell
        // where each face took its own, in two planes by parity, so that the
        // thesis sweeps spill no register (511^3 4.85 -> 4.76 ms)
        if constexpr (!RESID && RM != RM_FROZEN) sh(L_DTV + bc, 0, 0) = quot_field(c.dtauv_c, mu_c);
        sh(L_TXX, 0, 0) = txx;
        sh(L_TYY, 0, 0) = tyy;
        sh(L_TXY, 0, 0) = txy;
        if constexpr (NORMS) sh(L_W, 0, 0) = w;
        sh(L_TXZ + bn, 0, 0) = txz_n;
        sh(L_TYZ + bn, 0, 0) = tyz_n;
        load_c(ptrs(), pz + 1, cc);
        __syncthreads();

        // ---- momentum (eq (19)) and damped velocity update on the tile ----
        OSet out{};
        if (tile_wave) {
            const T rx = ff.rx, ry = ff.ry, rz = ff.rz;
            const T fx = (txx - sh(L_TXX, -1, 0)) * c.dxi + (sh(L_TXY, 0, 1) - txy) * c.dyi +
                         (txz_n - txz_c) * c.dzi - (ptn - sh(L_PTN, -1, 0)) * c.dxi + ff.fox;
            const T fy = (sh(L_TXY, 1, 0) - txy) * c.dxi + (tyy - sh(L_TYY, 0, -1)) * c.dyi +
                         (tyz_n - tyz_c) * c.dzi - (ptn - sh(L_PTN, 0, -1)) * c.dyi + ff.foy;
            const T fs = (sh(L_TXZ + bc, 1, 0) - txz_c) * c.dxi + (sh(L_TYZ + bc, 0, 1) - tyz_c) * c.dyi +
                         (tzz - tzz_p) * c.dzi - (ptn - ptn_p) * c.dzi;
            T fz;
            if constexpr (CORR) {
                fz = fs + ff.foz;
            } else {
                // (the thesis sweep keeps plane p-1's solid fraction and tau_zz
                // in LDS: it has no register to spare for them)
                if constexpr (UPD_LP) fz = fs - (T(0.5) * (weight(sh(L_S + bn, 0, 0)) + weight(s_c)) - c.rhobg) + ff.foz;
                else fz = fs - (T(0.5) * (rg_p + rg) - c.rhobg) + ff.foz;
            }
            if constexpr (RESID) {
                out.vx = fx;
                out.vy = fy;
                out.vz = fz;
                out.pt = rpt_k;
                out.pf = rpf_k;
            } else {
                const T dtv = sh(L_DTV + bc, 0, 0);
                out.vx = damped_update<RM>(c, vx_c, rx, fx, c.dampx, min1(dtv, sh(L_DTV + bc, -1, 0)), out.rx);
                out.vy = damped_update<RM>(c, vy_c, ry, fy, c.dampy, min1(dtv, sh(L_DTV + bc, 0, -1)), out.ry);
                out.vz = damped_update<RM>(c, vz_c, rz, fz, c.dampz, min1(dtv, sh(L_DTV + bn, 0, 0)), out.rz);
                out.pt = ptn;
                out.pf = pfn;
                out.lp = lpn;
            }
            if constexpr (WNORM) {
                if (outc && live) {
                    const bool inx = i >= 1, iny = j >= 1, inz = pz >= 1;
                    if constexpr (RESID) {
                        if (inx) nm[0] = nanmax(nm[0], T(fabs(fx)));
                        if (iny) nm[0] = nanmax(nm[0], T(fabs(fy)));
                        if (inz) nm[0] = nanmax(nm[0], T(fabs(fz)));
                    } else {
                        if (inx) {
                            nm[0] = nanmax(nm[0], T(fabs(fx - (w - sh(L_W, -1, 0)) * c.dxi)));
                            nm[7] = nanmax(nm[7], T(fabs(out.vx - vx_c)));
                        }
                        if (iny) {
                            nm[0] = nanmax(nm[0], T(fabs(fy - (w - sh(L_W, 0, -1)) * c.dyi)));
                            nm[7] = nanmax(nm[7], T(fabs(out.vy - vy_c)));
                        }
                        if (inz) {
                            nm[0] = nanmax(nm[0], T(fabs(fz - (w - w_p) * c.dzi)));
                            nm[6] = nanmax(nm[6], T(fabs(out.vz - vz_c)));
                            nm[7] = nanmax(nm[7], T(fabs(out.vz - vz_c)));
                        }
                    }
                    // phi' outside (0, 1): ln(1-phi)' not in (-inf, 0); checked
                    // with the norms
                    if (UPD_LP && !(lpn < zero && lpn > T(-1.0e300))) *p->domain = 1.0;
                    nm[1] = nanmax(nm[1], T(fabs(rpt_k)));
                    nm[2] = nanmax(nm[2], T(fabs(rpf_k)));
                    if (UPD_LP) nm[3] = nanmax(nm[3], T(fabs(lpn - lp_c)));
                    nm[4] = nanmax(nm[4], T(fabs(ptn - pt)));
                    nm[5] = nanmax(nm[5], T(fabs(pfn - pf_c)));
                }
            }
        }
        KPtrs* const pe = ptrs();
        store(pe, pz, live, out);
        load_f(pe, pz + 1, ff);

        // advance the register queue
        vx_c = fresh(vx_n); vy_c = fresh(vy_n); vz_c = fresh(vz_n);
        pf_c = fresh(pf_n);
        kc_c = fresh(kc_n);
        s_c = s_n;
        if constexpr (!UPD_LP) rg_p = rg;
        mu_c = fresh(mu_n);
        if constexpr (NORMS && UPD_LP) lp_c = fresh(lp_n);
        if constexpr (!UPD_LP) tzz_r = tzz;
        w_p = w;
        txz_c = txz_n; tyz_c = tyz_n;
        qz_c = qz_n; kz_c = kz_n; az_c = az_n;
    };

    // Two steps per round, the sets loaded ahead alternating between two
    // register sets: no copy of a set still being loaded makes the wave wait
    // for it at the end of a step.
    QSet qa, qb;
    CSet cs;
    {
        const int p0 = kz0 - 1;
        KPtrs* const p = ptrs();
        load_q(p, p0, qb);
        load_q2(p, p0, qb);
        load_q(p, p0 + 1, qa);
        load_q2(p, p0 + 1, qa);
        load_c(p, p0, cs);
        // as many (empty) stores as a step ends with, so that the first
        // step waits for its loads as every other does
        store(p, p0, false, OSet{});
        load_f(p, p0, ff);
        if constexpr (GATED) {
            // behind a closed gate the block ends here; its first loads are
            // under way while the gate's value comes
            const auto* gate = (const __attribute__((address_space(4))) double*)p->gate;
            asm volatile("" ::: "memory");
            if (gate && *gate != 0.0) return;
        }
        vx_c = qb.vx; vy_c = qb.vy; vz_c = qb.vz; pf_c = qb.pf; kc_c = qb.kc; lp_c = qb.lp; mu_c = qb.mu;
        s_c = solid(lp_c);
    }
    for (int pz = kz0 - 1; pz < kz1; pz += 2) {
        step(pz, qa, qb, cs);
        if (pz + 1 >= kz1) break;
        step(pz + 1, qb, qa, cs);
    }

    if constexpr (WNORM) {
        // Block maximum: wave64 butterfly in each of the waves of whole tile
        // rows (the halo wave holds no tile cell and contributes nothing),
        // then across these waves through LDS.
        constexpr int NW = (W - 2) * H / 64;
        static_assert((W - 2) * H % 64 == 0, "whole waves of tile columns");
        __shared__ double red[NW][NNORM];
        const int L = threadIdx.x;
        const int wave = L >> 6, lane = L & 63;
        if (wave < NW) {
#pragma unroll
            for (int q = 0; q < NNORM; ++q) {
                T v = nm[q];
                for (int off = 32; off >= 1; off >>= 1) v = nanmax(v, T(__shfl_xor(v, off, 64)));
                nm[q] = v;
            }
            if (lane == 0) {
#pragma unroll
                for (int q = 0; q < NNORM; ++q) red[wave][q] = double(nm[q]);
            }
        }
        __syncthreads();
        if (L < NNORM) {
            double v = 0.0;
            for (int wv = 0; wv < NW; ++wv) v = nanmax(v, red[wv][L]);
            args.p.partials[(int64_t)blockIdx.x * NNORM + L] = v;
        }
    }
}

// The eight maxima over the blocks' partial ones, one block: thread t takes
// norm t mod 8 of every 128th block, so that a wave reads whole lines.
constexpr int RT = 1024;
__device__ __forceinline__ double reduce_max(const double* __restrict__ part, int64_t nb) {
    __shared__ double red[RT / 64][NNORM];
    double m = 0.0;
    const int64_t n = nb * NNORM;
    for (int64_t t = threadIdx.x; t < n; t += RT) m = nanmax(m, part[t]);
    for (int off = 32; off >= NNORM; off >>= 1) m = nanmax(m, __shfl_xor(m, off, 64));
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < NNORM) red[wave][lane] = m;
    __syncthreads();
    double v = 0.0;
    if (threadIdx.x < NNORM)
        for (int w = 0; w < RT / 64; ++w) v = nanmax(v, red[w][threadIdx.x]);
    return v;   // of thread q < NNORM: norm q
}

__global__ __launch_bounds__(RT) void k_reduce_max(const double* __restrict__ part, int64_t nb,
                                                   double* __restrict__ out) {
    const double v = reduce_max(part, nb);
    if (threadIdx.x < NNORM) out[threadIdx.x] = v;
}

// A check of a solve (see CheckRule).  The host waits for the number, which
// is written after the rest, not for a copy and the stream; without a slot it
// copies the norms, the domain flag and the gate, which follow each other.
__global__ __launch_bounds__(RT) void k_check(const double* __restrict__ part, int64_t nb, double* __restrict__ out,
                                              const double* __restrict__ domain, double* __restrict__ gate, CheckRule r,
                                              double* __restrict__ slot, double number) {
    if (gate[0] != 0.0) return;
    const double v = reduce_max(part, nb);
    if (threadIdx.x >= 64) return;
    double n[NNORM];
    bool finite = true;
    for (int q = 0; q < NNORM; ++q) {
        n[q] = __shfl(v, q, 64);
        finite = finite && isfinite(n[q]);
    }
    if (threadIdx.x != 0) return;
    auto rho = [&](double gv, double gp) {
        double x = 0.0;
        if (gv > 0.0) x = fmax(x, n[0] / gv);
        if (gp > 0.0) x = fmax(x, fmax(n[1], n[2]) / gp);
        return x;
    };
    const double flag = *domain;
    const double now = rho(r.ref_v, r.ref_p);
    bool stop = !finite || flag != 0.0 || now <= r.tol || rho(r.ref_v2, r.ref_p2) <= r.tol2;
    if (!stop && r.stall > 0) {
        const double best = r.first ? INFINITY : gate[1];
        if (now < 0.99 * best) {
            gate[1] = now;
            gate[2] = 0.0;
        } else {
            const double since = (r.first ? 0.0 : gate[2]) + 1.0;
            gate[2] = since;
            stop = since >= (double)r.stall;
        }
    }
    if (stop) gate[0] = 1.0;
    for (int q = 0; q < NNORM; ++q) out[q] = n[q];
    if (!slot) return;
    for (int q = 0; q < NNORM; ++q) slot[q] = n[q];
    slot[NNORM] = flag;
    slot[NNORM + 1] = stop ? 1.0 : 0.0;
    __hip_atomic_store(slot + NNORM + 2, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace

namespace {

template <typename T, int MODE, bool NORMS, int RM, bool RW, int W, int H, bool STREAM>
hipError_t launch_tile(const Geom& g, const TileShape& t, const Coef& c, const SweepPtrs<T>& p, hipStream_t s) {
    if (!rows_fit(g, H, sizeof(T))) return hipErrorInvalidValue;
    SweepArgs<T> a{g, CT<T>(c), p};
    a.g.kz = t.kz;
    const dim3 grid((unsigned)sweep_blocks(g, t)), block(W * H);
    // the correction system has no background term (it is in its right-hand side)
    if (MODE != MD_CORR && c.gbg_half != 0.0)
        hipLaunchKernelGGL((k_sweep<T, MODE, NORMS, RM, RW, W, H, MODE != MD_CORR, STREAM>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_sweep<T, MODE, NORMS, RM, RW, W, H, false, STREAM>), grid, block, 0, s, a);
    return hipGetLastError();
}

// One sweep variant on the tile chosen for it (the tiles of sweep_shapes).
template <typename T, int MODE, bool NORMS, int RM, bool RW>
hipError_t launch_sweep(const Geom& g, const Tiling& tl, const Coef& c, const SweepPtrs<T>& p, hipStream_t s) {
    constexpr SweepKind kind = sizeof(T) == 8 ? (NORMS ? SK_NORM64 : SK_F64) : (NORMS ? SK_NORM32 : SK_F32);
    const TileShape& t = tl.shape[kind];
    const int wh = t.w * 100 + t.h;
    // (the sweeps with norms and the residual sweep, whose results are read
    // next, measured the same either way; grids past the cache take the lower
    // tiles only where their rows are too wide for these)
    if constexpr (!NORMS && MODE != MD_RESID)
        if (t.stream) {
            if constexpr (sizeof(T) == 4)
                if (wh == 6614) return launch_tile<T, MODE, NORMS, RM, RW, 66, 14, true>(g, t, c, p, s);
            if (wh == 6610) return launch_tile<T, MODE, NORMS, RM, RW, 66, 10, true>(g, t, c, p, s);
            if (wh == 3414) return launch_tile<T, MODE, NORMS, RM, RW, 34, 14, true>(g, t, c, p, s);
        }
    if constexpr (NORMS) {
        if (wh == 6607) return launch_tile<T, MODE, NORMS, RM, RW, 66, 7, false>(g, t, c, p, s);
    } else {
        if constexpr (sizeof(T) == 4)
            if (wh == 6614) return launch_tile<T, MODE, NORMS, RM, RW, 66, 14, false>(g, t, c, p, s);
        if (wh == 6610) return launch_tile<T, MODE, NORMS, RM, RW, 66, 10, false>(g, t, c, p, s);
        if (wh == 6606) return launch_tile<T, MODE, NORMS, RM, RW, 66, 6, false>(g, t, c, p, s);
    }
    if (wh == 3414) return launch_tile<T, MODE, NORMS, RM, RW, 34, 14, false>(g, t, c, p, s);
    if (wh == 3406) return launch_tile<T, MODE, NORMS, RM, RW, 34, 6, false>(g, t, c, p, s);
    if constexpr (NORMS || sizeof(T) == 8)
        if (wh == 3404) return launch_tile<T, MODE, NORMS, RM, RW, 34, 4, false>(g, t, c, p, s);
    return hipErrorInvalidValue;
}

// The sweeps of one mode, by where the damping memory is and whether R' is
// stored (the combinations the drivers use: R' is always stored with norms).
template <typename T, int MODE>
hipError_t launch_mode(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<T>& p, int norms,
                       hipStream_t s) {
    if constexpr (MODE != MD_CORR)
        if (c.mech_off) {   // (R' = R is stored: it has moved to its other copy)
            if (norms) return launch_sweep<T, MODE, true, RM_FROZEN, true>(g, t, c, p, s);
            return launch_sweep<T, MODE, false, RM_FROZEN, true>(g, t, c, p, s);
        }
    if (norms) {
        if (c.rform) return launch_sweep<T, MODE, true, RM_STORED, true>(g, t, c, p, s);
        return launch_sweep<T, MODE, true, RM_VPREV, true>(g, t, c, p, s);
    }
    if (c.rwrite) {
        if constexpr (MODE != MD_THESIS)
            if (c.rform) return launch_sweep<T, MODE, false, RM_STORED, true>(g, t, c, p, s);
        if constexpr (MODE == MD_CORR) return launch_sweep<T, MODE, false, RM_VPREV, true>(g, t, c, p, s);
        return hipErrorInvalidValue;
    }
    if (c.rform) return launch_sweep<T, MODE, false, RM_STORED, false>(g, t, c, p, s);
    return launch_sweep<T, MODE, false, RM_VPREV, false>(g, t, c, p, s);
}

}  // namespace

// One PT iteration's sweep of the thesis schedule, and of a linear stage.
hipError_t launch_thesis(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int norms,
                         hipStream_t s);
hipError_t launch_linear(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int norms,
                         hipStream_t s);

#if SWEEP_HAS(0)
hipError_t launch_thesis(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int norms,
                         hipStream_t s) {
    return launch_mode<double, MD_THESIS>(g, t, c, p, norms, s);
}

hipError_t launch_reduce_max(const double* partials, int64_t nblocks, double* out8, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_max, dim3(1), dim3(RT), 0, s, partials, nblocks, out8);
    return hipGetLastError();
}

hipError_t launch_check(const double* partials, int64_t nblocks, double* out8, const double* domain, double* gate,
                        const CheckRule& r, double* slot, double number, hipStream_t s) {
    hipLaunchKernelGGL(k_check, dim3(1), dim3(RT), 0, s, partials, nblocks, out8, domain, gate, r, slot, number);
    return hipGetLastError();
}
#endif

#if SWEEP_HAS(1)
hipError_t launch_linear(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int norms,
                         hipStream_t s) {
    if (c.undamped) {
        if (c.mech_off) return launch_sweep<double, MD_LINEAR, false, RM_FROZEN, false>(g, t, c, p, s);
        return launch_sweep<double, MD_LINEAR, false, RM_NONE, false>(g, t, c, p, s);
    }
    return launch_mode<double, MD_LINEAR>(g, t, c, p, norms, s);
}
#endif

#if SWEEP_HAS(2)
hipError_t launch_iteration(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int mode,
                            int norms, hipStream_t s) {
    switch (mode) {
        case MD_THESIS: return launch_thesis(g, t, c, p, norms, s);
        case MD_LINEAR: return launch_linear(g, t, c, p, norms, s);
        case MD_RESID: return launch_sweep<double, MD_RESID, false, RM_NONE, false>(g, t, c, p, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_correction(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<float>& p, int norms,
                             hipStream_t s) {
    return launch_mode<float, MD_CORR>(g, t, c, p, norms, s);
}

hipError_t launch_correction64(const Geom& g, const Tiling& t, const Coef& c, const SweepPtrs<double>& p, int norms,
                               hipStream_t s) {
    if (norms) return launch_sweep<double, MD_CORR, true, RM_STORED, true>(g, t, c, p, s);
    return launch_sweep<double, MD_CORR, false, RM_STORED, true>(g, t, c, p, s);
}
#endif

}  // namespace ptk
