// Transposed D3Q19 step (the map and its transposes are written out in adjoint.hip) in six launches, four
// over the lattice and two over the list of wall nodes, one lane per node throughout:
//   k_adj3_pre      density, momentum, psi and psi' of time t + 1 from the state of time t
//   k_adj3_wall     psi, psi' and the eq. 15 average of the wall nodes
//   k_adj3_collide  transposed collision: lambda(t + 1) -> pbar; H = -G psi Fbar, and the node's own
//                   part of the transposed force
//   k_adj3_wall_T   transposed force and psi at the wall nodes: dphi, and what eq. 15 hands back
//   k_adj3_rho_T    the same at the fluid nodes, plus what the walls hand back: the density adjoint;
//                   boundary nodes fold the part of eq. 16 that goes to a neighbour into pbar
//   k_adj3_stream   transposed streaming and the node's own links -> lambda(t), lambda_R(t)
//
// What bounds it: each kernel is one or two round trips of independent loads, and the planes of lambda
// and pbar (19 doubles each, read and written once) carry nearly all of the bytes.  The collision's
// transpose needs only rho and rho u of the pre-collision state, so its populations are never stored; a
// wall or neighbour value is gathered as the one product that is used (H, not F, psi and a tag); the
// links of a boundary node are read as vectors, all at once, where a branch per direction waits for one
// load after another; and the neighbour's eq. 16 term is added where its node's values are at hand, so
// the streaming pass looks at no neighbour's tag, mask or coefficient.
//
// A reverse step at 60 x 57 x 52 FP32 storage against one pass per map with every intermediate stored: 86 ->
// 52 us (pre 8, walls 5.5 each, collision 11.5-14, rho_T 9.3, stream 12.5); a gradient of 24 steps there
// 4.30 -> 2.52 ms, at 20 x 21 x 22 FP64 3.39 -> 1.73 ms, at 200 x 180 x 150 FP64 100 -> 67 ms, where the
// collision moves 4.5 TB/s and the streaming 4.4.  Each XCD on a contiguous eighth of the lattice: the
// same up to 128^3, 4 % slower at 200 x 180 x 150.
#include "adjoint_dev.h"
#include "step3d_node.h"

namespace mcb {
namespace {

constexpr int NT = 256;

struct Adj3 {
    AdjDev A;
    const int32_t* wl_node;
    int64_t n_wall;
    AdjWork w;
};

// neighbours x + e_i as node numbers
__device__ __forceinline__ void nbr3(const AdjDev& A, const Node3& q, uint32_t (&x)[19]) {
    neighbours<char>(q, A.g.nx, A.g.ny, A.g.nz, x);
}
// sum of w_i v_i e_i over the directions 1..18, w the weights of the force stencil
__device__ __forceinline__ void stencil3(const double (&v)[19], double (&s)[3]) {
    const double exy1 = v[7] - v[8], exy2 = v[9] - v[10], exz1 = v[11] - v[12], exz2 = v[13] - v[14];
    const double eyz1 = v[15] - v[16], eyz2 = v[17] - v[18];
    constexpr double wa = 1.0 / 6.0, we = 1.0 / 12.0;
    s[0] = wa * (v[1] - v[2]) + we * (exy1 + exy2 + exz1 + exz2);
    s[1] = wa * (v[3] - v[4]) + we * (exy1 - exy2 + eyz1 + eyz2);
    s[2] = wa * (v[5] - v[6]) + we * (exz1 - exz2 + eyz1 - eyz2);
}
// sum of f_i e_i
__device__ __forceinline__ void momentum(const double (&f)[19], double (&j)[3]) {
    j[0] = (f[1] - f[2]) + (f[7] - f[8]) + (f[9] - f[10]) + (f[11] - f[12]) + (f[13] - f[14]);
    j[1] = (f[3] - f[4]) + (f[7] - f[8]) - (f[9] - f[10]) + (f[15] - f[16]) + (f[17] - f[18]);
    j[2] = (f[5] - f[6]) + (f[11] - f[12]) - (f[13] - f[14]) + (f[15] - f[16]) - (f[17] - f[18]);
}
// sum over k of w_k e_k . H(x - e_k), w the weights of the force stencil; nb: the neighbours x + e_i
__device__ __forceinline__ double gather_H(const AdjDev& A, const double* __restrict__ H, const uint32_t (&nb)[19]) {
    const int64_t N = A.g.N;
    double t[19];
#pragma unroll
    for (int k = 1; k < 19; ++k) {
        const uint32_t o = nb[opp<1>(k)] * 8u;
        const double hx = kEx3[k] ? ldo(H, o) : 0.0, hy = kEy3[k] ? ldo(H + N, o) : 0.0, hz = kEz3[k] ? ldo(H + 2 * N, o) : 0.0;
        t[k] = edot3<double>(kEx3[k], kEy3[k], kEz3[k], hx, hy, hz);
    }
    double a = 0.0, e = 0.0;
#pragma unroll
    for (int k = 1; k < 7; ++k) a += t[k];
#pragma unroll
    for (int k = 7; k < 19; ++k) e += t[k];
    return (1.0 / 6.0) * a + (1.0 / 12.0) * e;
}
// link coefficients of a boundary node (NO_LINK: none); zeros on other lanes
template <class RC>
__device__ __forceinline__ void coefs(const RC* la, uint32_t n_bnodes, int tg, double (&a)[18]) {
    RC c[18];
    ld_vec(make_res(la, uint64_t(n_bnodes) * Q3_LINKS * sizeof(RC)),
           tg > 0 ? uint32_t(tg - 1) * uint32_t(Q3_LINKS * sizeof(RC)) : OOB, c);
#pragma unroll
    for (int j = 0; j < 18; ++j) a[j] = double(c[j]);
}

// PULL = false: p = f^eq(rho0, 0), the first collision's input
template <class S, class RC, bool PULL>
__global__ __launch_bounds__(NT) void k_adj3_pre(Adj3 p, const S* __restrict__ gt, const RC* __restrict__ la,
                                                 const RC* __restrict__ rec) {
    const AdjDev& A = p.A;
    const int64_t N = A.g.N;
    const Node3 q = node3<NT>(A.g.nx, A.g.ny, A.g.nz);
    const int tg = ldo(A.tag, q.node * 4u);
    double r = 0.0, j[3] = {0, 0, 0};
    if (PULL) {
        uint32_t nb[19];
        nbr3(A, q, nb);
        double f[19];  // as stored (less w rho_ref, which drops out of the links and the momentum)
#pragma unroll
        for (int i = 0; i < 19; ++i)
            f[i] = kMixed<S> && i == 0 ? double(ldo(reinterpret_cast<const float*>(gt), q.node * 4u))
                                       : double(ldo(gt + plane_off<S>(i, N), nb[opp<1>(i)] * uint32_t(sizeof(S))));
        if (__any(tg > 0)) {
            // eqs. 16-18.  The forcing terms are those of the stored state, in FP64: an FP64 record holds them;
            // with an FP32 one density and momentum come from the node's own populations and only the
            // force from the record (F = rho du; the collision left j + F)
            RC h[RF3 + 18];
            double a[18];
            ld_vec(make_res(rec, uint64_t(p.A.nb) * REC3 * sizeof(RC)),
                   tg > 0 ? uint32_t(tg - 1) * uint32_t(REC3 * sizeof(RC)) : OOB, h);
            coefs(la, p.A.nb, tg, a);
            double kr = A.kF * double(h[0]), dx = double(h[1]), dy = double(h[2]), dz = double(h[3]);
            double sx = double(h[4]), sy = double(h[5]), sz = double(h[6]), duu = double(h[7]);
            if constexpr (sizeof(RC) == 4) {
                double own[19], ro = A.rho_ref, m[3];
                own[0] = f[0];
#pragma unroll
                for (int i = 1; i < 19; ++i) own[i] = double(h[RF3 + i - 1]);
#pragma unroll
                for (int i = 0; i < 19; ++i) ro += own[i];
                momentum(own, m);
                const double ir = 1.0 / ro, Fx = double(h[0]) * dx, Fy = double(h[0]) * dy, Fz = double(h[0]) * dz;
                kr = A.kF * ro;
                dx = Fx * ir;
                dy = Fy * ir;
                dz = Fz * ir;
                sx = 2.0 * (m[0] - Fx) * ir + dx;
                sy = 2.0 * (m[1] - Fy) * ir + dy;
                sz = 2.0 * (m[2] - Fz) * ir + dz;
                duu = 1.5 * (dx * sx + dy * sy + dz * sz);
            }
            double dm = 0.0;
            // a slot that a link replaces is never one that an eq. 16 link reads
#pragma unroll
            for (int i = 1; i < 19; ++i) {
                const bool lk = tg > 0 && a[i - 1] < 1.5;
                const double c1 = fabs(a[i - 1]), c2 = 1.0 - c1;
                const double ed = edot3<double>(kEx3[i], kEy3[i], kEz3[i], dx, dy, dz);
                const double es = edot3<double>(kEx3[i], kEy3[i], kEz3[i], sx, sy, sz);
                const double F = wgt<double>(1, i) * kr * (3.0 * ed + 4.5 * ed * es - duu);
                const double fj = double(h[RF3 + i - 1]);
                const double o = c2 != 0.0 ? (a[i - 1] < 0.0 ? double(h[RF3 + opp<1>(i) - 1]) : f[i]) : 0.0;
                const double B = c1 * fj + c2 * (o + F);
                f[opp<1>(i)] = lk ? B : f[opp<1>(i)];
                dm += lk ? fj - B : 0.0;
            }
            f[0] += A.k18 * dm;
        }
        r = A.rho_ref;
#pragma unroll
        for (int i = 0; i < 19; ++i) r += f[i];
        momentum(f, j);
    } else {
        r = ldo(p.w.rho0, q.node * 8u);
    }
    if (!q.on) return;
    double s = 0.0, ds = 0.0;
    if (tg >= 0) psi_d(A, r, &s, &ds);
    const uint32_t o = q.node * 8u;
    sto(p.w.rho, o, tg >= 0 ? r : 0.0);  // the walls' averages read 0 on solid nodes
    sto(p.w.psi, o, s);
    if (tg < 0) return;
    sto(p.w.dpsi, o, ds);
#pragma unroll
    for (int k = 0; k < 3; ++k) sto(p.w.mom + k * N, o, j[k]);
}

// one lane per wall node; rave, den and psi' are kept per wall node, psi per node
__device__ __forceinline__ Node3 wall_node(const Adj3& p, int64_t w) {
    const uint32_t x = uint32_t(p.wl_node[w]), nx = uint32_t(p.A.g.nx), nxy = nx * uint32_t(p.A.g.ny);
    const uint32_t z = x / nxy, y = (x - z * nxy) / nx;
    return {x, true, int(x - z * nxy - y * nx), int(y), int(z)};
}
__global__ __launch_bounds__(NT) void k_adj3_wall(Adj3 p) {
    const AdjDev& A = p.A;
    const int64_t w = int64_t(blockIdx.x) * NT + threadIdx.x;
    if (w >= p.n_wall) return;
    const Node3 q = wall_node(p, w);
    uint32_t nb[19];
    nbr3(A, q, nb);
    double v[19];
    int tg[19];
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        v[i] = ldo(p.w.rho, nb[i] * 8u);
        tg[i] = ldo(A.tag, nb[i] * 4u);
    }
    double num = 0.0, den = 0.0, s = 0.0, ds = 0.0;
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        num += wgt<double>(1, i) * v[i];
        den += tg[i] >= 0 ? wgt<double>(1, i) : 0.0;
    }
    const double ra = num / den;
    psi_d(A, A.phi[w] * ra, &s, &ds);
    sto(p.w.psi, q.node * 8u, s);
    sto(p.w.dpsi, q.node * 8u, ds);
    p.w.rave[w] = ra;
    p.w.den[w] = den;
}

__global__ __launch_bounds__(NT, 2) void k_adj3_collide(Adj3 p, const double* __restrict__ lam1, const double* __restrict__ lamR1) {
    const AdjDev& A = p.A;
    const int64_t N = A.g.N;
    const Node3 q = node3<NT>(A.g.nx, A.g.ny, A.g.nz);
    const uint32_t x = q.node * 8u;
    const int tg = ldo(A.tag, q.node * 4u);
    uint32_t nb[19];
    nbr3(A, q, nb);
    double lam[19], ps[19], j[3], F[3];
#pragma unroll
    for (int i = 0; i < 19; ++i) lam[i] = ldo(lam1 + i * N, x);
#pragma unroll
    for (int i = 0; i < 19; ++i) ps[i] = ldo(p.w.psi, nb[i] * 8u);
    const double r = ldo(p.w.rho, x);
#pragma unroll
    for (int k = 0; k < 3; ++k) j[k] = ldo(p.w.mom + k * N, x);
    double s3[3];
    stencil3(ps, s3);
    const double gp = -A.G * ps[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) F[k] = gp * s3[k] + r * A.grav[k];
    if (!q.on) return;
    if (tg < 0) {
        // the transposed stencil reads 0 on solid nodes
#pragma unroll
        for (int k = 0; k < 3; ++k) sto(p.w.Fbar + k * N, x, 0.0);
        return;
    }
    double rr[18];  // adjoint of the forcing term on each link (0 without a link)
#pragma unroll
    for (int i = 0; i < 18; ++i) rr[i] = 0.0;
    if (tg > 0) {
        const uint32_t mk = ldo(A.nmask, q.node * 4u);
        const double* lr = lamR1 + size_t(tg - 1) * Q3_LINKS;
        double v[18];
#pragma unroll
        for (int i = 0; i < 18; ++i) v[i] = lr[i];
#pragma unroll
        for (int i = 0; i < 18; ++i) rr[i] = ((mk >> i) & 1u) ? v[i] : 0.0;
    }
    const double m1[3] = {j[0] + F[0], j[1] + F[1], j[2] + F[2]};
    const double mm0 = j[0] * j[0] + j[1] * j[1] + j[2] * j[2];
    const double mm1 = m1[0] * m1[0] + m1[1] * m1[1] + m1[2] * m1[2];
    const double ir = 1.0 / r, ir2 = ir * ir, om = 1.0 - 1.0 / A.tau;
    // al = lambda + R-bar: adjoint of E_i(rho, j + F); be = -(1 - 1/tau) lambda - R-bar: of E_i(rho, j); both
    // with the weight w_i.  Opposite directions share (e.m)^2 and have opposite e.m, so each pair enters by
    // its sum and difference.
    double sa = wgt<double>(1, 0) * lam[0], sb = -wgt<double>(1, 0) * om * lam[0], qa = 0.0;
    double d1[3] = {0, 0, 0}, d0[3] = {0, 0, 0};
    auto eadd = [](int i, double v, double (&acc)[3]) {
        if (kEx3[i] != 0) acc[0] += kEx3[i] > 0 ? v : -v;
        if (kEy3[i] != 0) acc[1] += kEy3[i] > 0 ? v : -v;
        if (kEz3[i] != 0) acc[2] += kEz3[i] > 0 ? v : -v;
    };
#pragma unroll
    for (int i = 1; i < 19; i += 2) {
        const double w = wgt<double>(1, i);
        const double lp = lam[i] + lam[i + 1], lm = lam[i] - lam[i + 1], rp = rr[i - 1] + rr[i], rm = rr[i - 1] - rr[i];
        const double ap = w * (lp + rp), am = w * (lm + rm), bp = -w * (om * lp + rp), bm = -w * (om * lm + rm);
        const double em0 = edot3<double>(kEx3[i], kEy3[i], kEz3[i], j[0], j[1], j[2]);
        const double em1 = edot3<double>(kEx3[i], kEy3[i], kEz3[i], m1[0], m1[1], m1[2]);
        const double c1 = ap * em1, c0 = bp * em0;
        sa += ap;
        sb += bp;
        qa += c1 * em1 + c0 * em0;
        eadd(i, 3.0 * am + 9.0 * ir * c1, d1);
        eadd(i, 3.0 * bm + 9.0 * ir * c0, d0);
    }
    // d E / d rho and d E / d m at (rho, m), summed
    double rb = sa + sb + 1.5 * ir2 * (sa * mm1 + sb * mm0) - 4.5 * ir2 * qa;
    double jb[3], own = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double Fb = d1[k] - 3.0 * ir * sa * m1[k];
        jb[k] = Fb + d0[k] - 3.0 * ir * sb * j[k];
        rb += Fb * A.grav[k];  // the body force depends on rho: F = ... + rho g
        own -= A.G * Fb * s3[k];
        sto(p.w.Fbar + k * N, x, gp * Fb);
    }
    sto(p.w.own, x, own);
    sto(p.w.pbar, x, om * lam[0] + rb);
#pragma unroll
    for (int i = 1; i < 19; i += 2) {
        const double e = edot3<double>(kEx3[i], kEy3[i], kEz3[i], jb[0], jb[1], jb[2]);
        sto(p.w.pbar + i * N, x, om * lam[i] + rb + e);
        sto(p.w.pbar + (i + 1) * N, x, om * lam[i + 1] + rb - e);
    }
}

// rho_w-bar = psi'(rho_w) psibar; dphi += rho_w-bar rho_ave; to the fluid neighbours rho_w-bar phi / den
__global__ __launch_bounds__(NT) void k_adj3_wall_T(Adj3 p) {
    const AdjDev& A = p.A;
    const int64_t w = int64_t(blockIdx.x) * NT + threadIdx.x;
    if (w >= p.n_wall) return;
    const Node3 q = wall_node(p, w);
    uint32_t nb[19];
    nbr3(A, q, nb);
    const double dp = ldo(p.w.dpsi, q.node * 8u), ra = p.w.rave[w], den = p.w.den[w], ph = A.phi[w], d = p.w.dphi[w];
    const double rwb = dp * gather_H(A, p.w.Fbar, nb);
    p.w.dphi[w] = d + rwb * ra;
    sto(p.w.qbar, q.node * 8u, rwb * ph / den);
}

// The density adjoint rbar of every population of a fluid node (rho = sum_i p_i).  At a boundary node,
// then: a link (x, i) of eq. 16 uses o = f_i(x - e_i), which x also pulls in direction i, so the node adds
// c2 Bbar_i(x) to its pbar_i (no other link of x reads that one: x - e_i is fluid).
template <class RC>
__global__ __launch_bounds__(NT) void k_adj3_rho_T(Adj3 p, const RC* __restrict__ la) {
    const AdjDev& A = p.A;
    const int64_t N = A.g.N;
    const Node3 q = node3<NT>(A.g.nx, A.g.ny, A.g.nz);
    const uint32_t x = q.node * 8u;
    const int tg = ldo(A.tag, q.node * 4u);
    uint32_t nb[19];
    nbr3(A, q, nb);
    const double own = ldo(p.w.own, x), dp = ldo(p.w.dpsi, x);
    double r = dp * (own + gather_H(A, p.w.Fbar, nb));
    if (!q.on || tg < 0) return;
    if (tg > 0) {
        const uint32_t mk = ldo(A.nmask, q.node * 4u);
        double a[18], qb[19], pb[19];
#pragma unroll
        for (int i = 1; i < 19; ++i) qb[i] = ldo(p.w.qbar, nb[i] * 8u);
#pragma unroll
        for (int i = 1; i < 19; ++i) r += ((mk >> (i - 1)) & 1u) ? wgt<double>(1, i) * qb[i] : 0.0;
        __builtin_amdgcn_sched_barrier(0);  // (106 and 125 registers instead of 135 and 158)
        coefs(la, p.A.nb, tg, a);
#pragma unroll
        for (int i = 0; i < 19; ++i) pb[i] = ldo(p.w.pbar + i * N, x);
        const double z = A.k18 * (pb[0] + r);
#pragma unroll
        for (int i = 1; i < 19; ++i)
            if (a[i - 1] >= 0.0 && a[i - 1] < 1.0) sto(p.w.pbar + i * N, x, pb[i] + (1.0 - a[i - 1]) * (pb[opp<1>(i)] + r - z));
    }
    sto(p.w.rbar, x, r);
}

template <class RC>
__global__ __launch_bounds__(NT) void k_adj3_stream(Adj3 p, const RC* __restrict__ la, double* __restrict__ lam0,
                                                    double* __restrict__ lamR0) {
    const AdjDev& A = p.A;
    const int64_t N = A.g.N;
    const Node3 q = node3<NT>(A.g.nx, A.g.ny, A.g.nz);
    const uint32_t x = q.node * 8u;
    const int tg = ldo(A.tag, q.node * 4u);
    uint32_t nb[19];
    nbr3(A, q, nb);
    double acc[19], rb[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) acc[i] = ldo(p.w.pbar + i * N, nb[i] * 8u);
#pragma unroll
    for (int i = 0; i < 19; ++i) rb[i] = ldo(p.w.rbar, nb[i] * 8u);
    if (!q.on || tg < 0) return;  // lambda is read on fluid nodes only
#pragma unroll
    for (int i = 0; i < 19; ++i) acc[i] += rb[i];
    if (tg > 0) {
        double a[18], pb[19];
        coefs(la, p.A.nb, tg, a);
        pb[0] = acc[0];
#pragma unroll
        for (int i = 1; i < 19; ++i) pb[i] = ldo(p.w.pbar + i * N, x) + rb[0];
        const double z = A.k18 * acc[0];  // eq. 18 carries the adjoint of p_0 (if applied)
#pragma unroll
        for (int i = 1; i < 19; ++i) {
            const int io = opp<1>(i);
            if (a[i - 1] < 1.5) {
                const double c1 = fabs(a[i - 1]), Bb = pb[io] - z;
                acc[i] = c1 * Bb + z;
                lamR0[size_t(tg - 1) * Q3_LINKS + (i - 1)] = A.kF * (1.0 - c1) * Bb;
            }
        }
        // eq. 17 of the link (x, opp i): o = f_i(x)
#pragma unroll
        for (int i = 1; i < 19; ++i) {
            const double ao = a[opp<1>(i) - 1];
            acc[i] += ao < 0.0 ? (1.0 + ao) * (pb[i] - z) : 0.0;
        }
    }
#pragma unroll
    for (int i = 0; i < 19; ++i) sto(lam0 + i * N, x, acc[i]);
}

template <class S, class RC>
hipError_t adj3_t(mcb_ctx* c, const AdjWork& w, const void* gt, const void* rec, int pull, const double* lam1,
                  const double* lamR1, double* lam0, double* lamR0) {
    Adj3 p;
    p.A = make_dev(c);
    p.wl_node = reinterpret_cast<const int32_t*>(c->lk + c->L.wl_node);
    p.n_wall = c->n_wall > 0 ? c->n_wall : 0;
    p.w = w;
    const RC* la = reinterpret_cast<const RC*>(c->lk + c->L.lk_a);
    const dim3 G(unsigned((c->g.N + NT - 1) / NT)), W(unsigned((p.n_wall + NT - 1) / NT)), B(NT);
    hipLaunchKernelGGL((pull ? k_adj3_pre<S, RC, true> : k_adj3_pre<S, RC, false>), G, B, 0, c->stream, p,
                       static_cast<const S*>(gt), la, static_cast<const RC*>(rec));
    if (p.n_wall > 0) hipLaunchKernelGGL(k_adj3_wall, W, B, 0, c->stream, p);
    hipLaunchKernelGGL(k_adj3_collide, G, B, 0, c->stream, p, lam1, lamR1);
    if (p.n_wall > 0) hipLaunchKernelGGL(k_adj3_wall_T, W, B, 0, c->stream, p);
    if (pull) {
        hipLaunchKernelGGL((k_adj3_rho_T<RC>), G, B, 0, c->stream, p, la);
        hipLaunchKernelGGL((k_adj3_stream<RC>), G, B, 0, c->stream, p, la, lam0, lamR0);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t adj_step3d(mcb_ctx* c, const AdjWork& w, const void* gt, const void* rec, int pull, const double* lam1,
                      const double* lamR1, double* lam0, double* lamR0) {
    switch (c->p.precision) {
        case MCB_F64: return adj3_t<double, double>(c, w, gt, rec, pull, lam1, lamR1, lam0, lamR0);
        case MCB_F32S: return adj3_t<float, float>(c, w, gt, rec, pull, lam1, lamR1, lam0, lamR0);
        default: return adj3_t<__half, float>(c, w, gt, rec, pull, lam1, lamR1, lam0, lamR0);
    }
}

}  // namespace mcb
