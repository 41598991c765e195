// Per-node arithmetic of the D2Q9 step and the arguments of its kernels, shared by the row marches
// (step2d.hip) and the tile kernels (tile2d.hip): eqs. 16-18 at a boundary node, the collision, and
// the chemical-potential model's constants.
#pragma once

#include "kernels_common.h"

namespace mcb {
namespace {

template <class S, class C>
struct Args2 {
    const S* fa;                 // post-collision populations of time t, SoA [9][N]
    S* fb;                       // post-collision populations of time t+1
    const int32_t* tag;          // >0: (boundary index << 8) | link bits; 0 fluid; -1 solid; -2-w wall w
    const C* rin;                // boundary records of time t, REC2 per boundary node
    C* rout;                     // boundary records of time t+1
    const C* la;                 // link coefficients, Q2_LINKS per boundary node (NO_LINK: none)
    const C* fac;                // eq. 15 factor per wall node: phi / weight of its fluid neighbours
    int32_t* flags;
    uint32_t n_bnodes, n_wall;
    int nx, ny, H, nsx, nblocks;
    C tau_inv, G, rho_ref;
    C kF, k18;                   // boundary scheme: weight of the forcing term, of eq. 18 (0 or 1)
    C s_e, s_eps, s_q;           // rates of the multiple-relaxation-time collision (eq. 3)
    C gx, gy;                    // body acceleration: F = F_nonideal + rho g, so du = F / rho gains g
    Eos<C> eos;
};

// D2Q9 weights
template <class C>
__device__ inline C w9(int i) {
    return i == 0 ? C(4.0 / 9.0) : (i < 5 ? C(1.0 / 9.0) : C(1.0 / 36.0));
}

__device__ constexpr int kOpp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
__device__ constexpr int kEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int kEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// e.(x, y) for a lattice vector of components 0 and +-1, folded when the components are constants
// (a product with 0 cannot be dropped under IEEE rules)
template <class C>
__device__ __forceinline__ C edot(int ex, int ey, C x, C y) {
    const C tx = ex > 0 ? x : -x, ty = ey > 0 ? y : -y;
    return ex == 0 ? ty : (ey == 0 ? tx : tx + ty);
}

// Eqs. 16-18 at a boundary node (bnd) from its record of time t (rec) and link coefficients (ca):
// replaces the populations pulled from solid neighbours by f_in and corrects the rest population;
// returns the correction and, in res, what rounding f_0 + correction to the compute type dropped.
// Lanes that are not boundary nodes keep f and return zeros.  Directions in which no lane of the wave has a link are
// skipped.  kF and k18 select the scheme: 1 and 1 the present one, 0 and 0 linear interpolation
// bounce-back (no forcing term, no eq. 18), 0 and 1 the same with eq. 18; halfway bounce-back is
// a = 1 on every link.
template <class S, class C>
__device__ __forceinline__ C apply_links(bool bnd, const C (&rec)[RF2 + 8], const C (&ca)[Q2_LINKS], C (&f)[9], C kF,
                                         C k18, C& res) {
    const C rho = rec[0] * kF, dux = rec[1], duy = rec[2], sx = rec[3], sy = rec[4], duu = rec[5];
    const C* fo = rec + RF2 - 1;  // own post-collision populations 1 .. 8
    // each slot opp(j) is replaced at most once, and never one that a later eq. 16 link reads (its
    // x2 = x - e_j is fluid, while a replaced slot was pulled from a solid node)
    double ds = 0.0;
#pragma unroll
    for (int j = 1; j < 9; ++j) {
        const C a = ca[j - 1];
        const bool lk = bnd && a < C(1.5);
        if (__builtin_amdgcn_ballot_w64(lk)) {
            const C c1 = a < C(0) ? -a : a, c2 = C(1) - c1;
            // eq. 13 term of direction j: w rho [3 e.du + 4.5 (e.du)(e.s) - 1.5 du.s]
            const C ed = edot<C>(kEx[j], kEy[j], dux, duy);
            const C es = edot<C>(kEx[j], kEy[j], sx, sy);
            const C Fj = w9<C>(j) * rho * (C(3) * ed + C(4.5) * ed * es - duu);
            C o = a < C(0) ? fo[kOpp[j]] : f[j];
            o = c2 != C(0) ? o : C(0);
            // rounded to the storage format, as the value would be stored; eq. 18 takes it so
            const C fin = Buf<S>::round(c1 * fo[j] + c2 * (o + Fj));
            ds += lk ? double(fo[j]) - double(fin) : 0.0;
            f[kOpp[j]] = lk ? fin : f[kOpp[j]];
        }
    }
    ds *= double(k18);
    const double f0 = double(f[0]) + ds;
    f[0] = C(f0);
    res = C(f0 - double(f[0]));
    return C(ds);
}

// Collision of one node (eq. 4, or eqs. 1-4 when MRT; eq. 13 forcing, eq. 14 equilibrium) from its
// pulled populations fA (stored format: shifted by w_i rho_ref), their sum rs_acc and the force
// (Fx, Fy) without the body force.  Writes the post-collision populations rounded to the storage
// format, f_0 taking the rounding so that the node keeps its mass exactly, and the forcing terms
// the boundary record carries.  coll = false (lanes that collide nothing) keeps the arithmetic finite.
template <class S, class C, bool MRT>
__device__ __forceinline__ void collide9(const Args2<S, C>& a, bool coll, const C (&fA)[9], MassAcc<S, C> rs_acc, C Fx, C Fy,
                                         C (&out)[9], C& rho, C& dux, C& duy, C& sx2, C& sy2, C& duu15) {
    const C rs = C(rs_acc);
    rho = rs + a.rho_ref;
    const C irho = rcp(coll ? rho : C(1));
    const C jx = fA[1] - fA[3] + fA[5] - fA[6] - fA[7] + fA[8];
    const C jy = fA[2] - fA[4] + fA[5] + fA[6] - fA[7] - fA[8];
    const C ux = jx * irho, uy = jy * irho;
    dux = Fx * irho + a.gx;
    duy = Fy * irho + a.gy;
    const C ti = a.tau_inv, omc = C(1) - ti;
    // per direction: out_i = f_i (1 - 1/tau) + w_i [rs/tau + rho (sym_i +- anti_i)] with
    //   sym  = (4.5 (e.u)^2 - 1.5 u^2) / tau + 4.5 (e.du)(e.(2u + du)) - 1.5 du.(2u + du)
    //   anti = 3 (e.u / tau + e.du)
    // (eq. 14 equilibrium, eq. 13 forcing term, eq. 4 with S = I / tau)
    const C uu15 = C(1.5) * (ux * ux + uy * uy);
    sx2 = C(2) * ux + dux;
    sy2 = C(2) * uy + duy;
    duu15 = C(1.5) * (dux * sx2 + duy * sy2);
    const C c0 = -(ti * uu15 + duu15);
    const C trs = ti * rs;
    auto pair = [&](int ip, int im, C w, C eu, C ed, C es) {
        const C sym = ti * C(4.5) * eu * eu + C(4.5) * ed * es + c0;
        const C anti = C(3) * (ti * eu + ed);
        const C base = w * (trs + rho * sym);
        const C wra = w * rho * anti;
        out[ip] = fA[ip] * omc + base + wra;
        out[im] = fA[im] * omc + base - wra;
    };
    if constexpr (!MRT) {
        pair(1, 3, C(1.0 / 9.0), ux, dux, sx2);
        pair(2, 4, C(1.0 / 9.0), uy, duy, sy2);
        pair(5, 7, C(1.0 / 36.0), ux + uy, dux + duy, sx2 + sy2);
        pair(6, 8, C(1.0 / 36.0), uy - ux, duy - dux, sy2 - sx2);
    } else {
        // eqs. 1-4 with the moment matrix of eq. 2: the six non-conserved moments of the stored
        // populations (the shift w_i rho_ref has moments rho_ref, -2 rho_ref, rho_ref, 0, ...,
        // folded in through rs), relaxed at the eq. 3 rates toward the Sec. 2.1 equilibria
        // (q^eq = -j); M^-1 = M^T diag(1/9, 1/36, 1/36, 1/6, 1/12, 1/6, 1/12, 1/4, 1/4)
        const C s14 = fA[1] + fA[2] + fA[3] + fA[4], s58 = fA[5] + fA[6] + fA[7] + fA[8];
        const C jj = rho * (ux * ux + uy * uy);
        const C de = a.s_e * (C(-4) * fA[0] - s14 + C(2) * s58 + C(2) * rs - C(3) * jj) * C(1.0 / 36.0);
        const C dp = a.s_eps * (C(4) * fA[0] - C(2) * s14 + s58 - rs + C(3) * jj) * C(1.0 / 36.0);
        const C dx = a.s_q * (C(-2) * (fA[1] - fA[3]) + (fA[5] - fA[6] - fA[7] + fA[8]) + jx) * C(1.0 / 12.0);
        const C dy = a.s_q * (C(-2) * (fA[2] - fA[4]) + (fA[5] + fA[6] - fA[7] - fA[8]) + jy) * C(1.0 / 12.0);
        const C dxx = ti * (fA[1] - fA[2] + fA[3] - fA[4] - rho * (ux * ux - uy * uy)) * C(0.25);
        const C dxy = ti * (fA[5] - fA[6] + fA[7] - fA[8] - rho * ux * uy) * C(0.25);
        // out = f - M^-1 S (m - m_eq) + F_i, F_i the eq. 13 term, by opposite pairs
        auto mpair = [&](int ip, int im, C w, C ed, C es, C sym, C anti) {
            const C wr = w * rho;
            const C fs = wr * (C(4.5) * ed * es - duu15) + sym;
            const C fa = wr * C(3) * ed + anti;
            out[ip] = fA[ip] + fs + fa;
            out[im] = fA[im] + fs - fa;
        };
        const C e1 = de + C(2) * dp, e2 = C(2) * de + dp;
        mpair(1, 3, C(1.0 / 9.0), dux, sx2, e1 - dxx, C(2) * dx);
        mpair(2, 4, C(1.0 / 9.0), duy, sy2, e1 + dxx, C(2) * dy);
        mpair(5, 7, C(1.0 / 36.0), dux + duy, sx2 + sy2, -(e2 + dxy), -(dx + dy));
        mpair(6, 8, C(1.0 / 36.0), duy - dux, sy2 - sx2, -(e2 - dxy), -(dy - dx));
    }
    // collision conserves mass (the equilibrium and the forcing term of eq. 13 have zero net
    // mass): set f_0 to the density minus the other eight outputs as stored, so the rounding of
    // the lattice weights and of the storage format cannot bias the total mass
    MassAcc<S, C> rest = 0;
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        out[i] = Buf<S>::round(out[i]);
        rest += MassAcc<S, C>(out[i]);
    }
    out[0] = C(rs_acc - rest);
}

template <class S, class C>
struct ArgsCP {
    Args2<S, C> a;
    C* rho;                 // density of the step: fluid nodes and solid layers 1-2
    C* mu;                  // chemical potential of the step: fluid nodes and solid layers 1-2
    const int8_t* layer;    // 0 fluid, 1 wall node, 2 second solid layer, 3 deeper
    const double* mus;      // assigned chemical potential per wall node
    int nt;                 // populations stored non-temporally
    C k2, kappa;            // eq. 12: k^2 and kappa
    C RT, b, c_log, aal;    // eq. 11: R T, b, a alpha / (2 sqrt 2 b), a alpha
};

// fourth-order central differences along an axis from the values at offsets -2 .. +2
template <class C>
__device__ __forceinline__ C cd1(C m2, C m1, C p1, C p2) {
    return (C(8) * (p1 - m1) - (p2 - m2)) * C(1.0 / 12.0);
}
template <class C>
__device__ __forceinline__ C cd2(C m2, C m1, C c, C p1, C p2) {
    return (C(16) * (p1 + m1) - (p2 + m2) - C(30) * c) * C(1.0 / 12.0);
}

__device__ __forceinline__ int wrapm(int v, int n) {
    const int r = v % n;
    return r < 0 ? r + n : r;
}

// the arguments of a pseudopotential step from fcur / rcur to fnext / rnext (the launch shape H, nsx,
// nblocks is left to the launcher)
template <class S, class C>
Args2<S, C> step_args(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext) {
    Args2<S, C> a;
    a.fa = static_cast<const S*>(fcur);
    a.fb = static_cast<S*>(fnext);
    a.tag = reinterpret_cast<const int32_t*>(c->lat + c->L.tag);
    a.rin = static_cast<const C*>(rcur);
    a.rout = static_cast<C*>(rnext);
    a.la = reinterpret_cast<const C*>(c->lk + c->L.lk_a);
    a.fac = reinterpret_cast<const C*>(c->lk + c->L.wl_fac);
    a.flags = reinterpret_cast<int32_t*>(c->lat + c->L.flags);
    a.n_bnodes = uint32_t(c->n_bnodes > 0 ? c->n_bnodes : 0);
    a.n_wall = uint32_t(c->n_wall > 0 ? c->n_wall : 0);
    a.nx = c->p.nx;
    a.ny = c->p.ny;
    a.H = a.nsx = a.nblocks = 0;
    a.tau_inv = C(1.0 / c->p.tau);
    a.G = C(c->p.G);
    a.rho_ref = c->p.precision == MCB_F64 ? C(0) : C(c->p.rho_ref);
    a.kF = c->p.bc_mode == MCB_BC_PRESENT ? C(1) : C(0);
    a.k18 = c->p.bc_mode == MCB_BC_IBC ? C(0) : C(1);
    a.s_e = C(c->p.s_e);
    a.s_eps = C(c->p.s_eps);
    a.s_q = C(c->p.s_q);
    a.gx = C(c->p.gravity[0]);
    a.gy = C(c->p.gravity[1]);
    a.eos.RT = C(c->p.eos_R * c->p.eos_T);
    a.eos.a = C(c->p.eos_a);
    a.eos.b4 = C(c->p.eos_b / 4.0);
    a.eos.two_over_G = C(2.0 / c->p.G);
    return a;
}

// the arguments of the chemical-potential kernels for one step from fcur / rcur to fnext / rnext
template <class S, class C>
ArgsCP<S, C> cp_args(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext) {
    ArgsCP<S, C> p;
    p.a = step_args<S, C>(c, fcur, rcur, fnext, rnext);
    p.a.fac = nullptr;  // no eq. 15 factors and no pseudopotential in this model
    p.a.G = C(0);
    p.a.eos = Eos<C>{};
    p.nt = 0;
    p.rho = reinterpret_cast<C*>(c->lat + c->L.cp_rho);
    p.mu = reinterpret_cast<C*>(c->lat + c->L.cp_mu);
    p.layer = reinterpret_cast<const int8_t*>(c->lat + c->L.cp_layer);
    p.mus = reinterpret_cast<const double*>(c->lk + c->L.wl_phi);
    const double T = c->p.eos_T, Tc = pr_tc(c->p.eos_a, c->p.eos_b, c->p.eos_R);
    const double om = c->p.pr_omega, mm = 0.37464 + 1.54226 * om - 0.26992 * om * om;
    const double sa = 1.0 + mm * (1.0 - std::sqrt(T / Tc));
    const double aal = c->p.eos_a * sa * sa;
    p.k2 = C(c->p.cp_k * c->p.cp_k);
    p.kappa = C(c->p.cp_kappa);
    p.RT = C(c->p.eos_R * T);
    p.b = C(c->p.eos_b);
    p.c_log = C(aal / (2.0 * std::sqrt(2.0) * c->p.eos_b));
    p.aal = C(aal);
    return p;
}

}  // namespace
}  // namespace mcb
