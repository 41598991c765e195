// Transposed D2Q9 step in two tile kernels (the map and its transposes are written out in adjoint.hip).
//
// Why tiles.  One pass per transpose writes and reads every intermediate (p, rho, psi, pbar twice, F,
// rhobar, qbar) through memory: about 900 bytes per node and six launches of 5 to 17 us each at 512^2
// (eleven with the chemical-potential model), where the arrays live in the memory-side cache and each
// launch is bound by one round trip per dependent load.  Here the intermediates of a tile stay in LDS
// and registers, and only pbar, Fbar and the fields they belong to go from the first kernel to the
// second.  A reverse step at 512^2 FP32 storage: 65 -> 25 us (14.3 the first kernel, 4.2 TB/s of what it
// reads and writes, 10.6 the second); at 301 x 203 FP64 in the chemical-potential model 77 -> 20 us.
// Tiles of 32 x 16 instead of 32 x 8 for the pseudopotential kernels measured the same (15.6 and 14.3
// us); lambda loaded before the links instead of after spills 96 bytes a lane (22.7 us).
//
// The grid of a middle-sized box is one round, so a kernel lasts as long as its slowest wave, one with
// boundary nodes: the links take their coefficients, records and adjoints as whole vectors, one
// round trip after the tag (a load per link, each behind its branch: 15.3 and 13.8 us), and the eq. 16
// share of a neighbour is added to pbar by the first kernel, at its own node.
#include "adjoint_dev.h"

namespace mcb {
namespace {

__device__ constexpr int kEx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
__device__ constexpr int kEy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};

// e.(x, y) for a lattice vector, folded when its components are constants (a product with 0 cannot be
// dropped under IEEE rules), and acc += e v per component
__device__ __forceinline__ double edot(int i, double x, double y) {
    const double tx = kEx[i] > 0 ? x : -x, ty = kEy[i] > 0 ? y : -y;
    return kEx[i] == 0 ? ty : (kEy[i] == 0 ? tx : tx + ty);
}
__device__ __forceinline__ void eadd(int i, double v, double (&acc)[2]) {
    if (kEx[i] != 0) acc[0] += kEx[i] > 0 ? v : -v;
    if (kEy[i] != 0) acc[1] += kEy[i] > 0 ? v : -v;
}

// the tile of a workgroup, consecutive tiles on the same XCD
struct Tile {
    int x0, y0;
};
template <int TX, int TY>
__device__ __forceinline__ Tile tile_of(int nsx) {
    const int nb = gridDim.x, bid = blockIdx.x, per = nb >> 3, rem = nb & 7, xcd = bid & 7, k8 = bid >> 3;
    const int l = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k8;
    return {(l % nsx) * TX, (l / nsx) * TY};
}

// populations arriving at node (cx, cy) of a state (eq. 5, from x - e_i), as stored: less w rho_ref, which drops
// out of the links and the momentum
template <class S>
__device__ __forceinline__ void pops(const AdjDev& A, const S* __restrict__ g, int cx, int cy, double (&f)[9]) {
    const int nx = A.g.nx, ny = A.g.ny;
    const uint32_t xo[3] = {uint32_t(cx == nx - 1 ? 0 : cx + 1), uint32_t(cx), uint32_t(cx == 0 ? nx - 1 : cx - 1)};
    const uint32_t yo[3] = {uint32_t(cy == ny - 1 ? 0 : cy + 1) * uint32_t(nx), uint32_t(cy) * uint32_t(nx),
                            uint32_t(cy == 0 ? ny - 1 : cy - 1) * uint32_t(nx)};
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const uint32_t x = xo[kEx[i] + 1] + yo[kEy[i] + 1];
        if (kMixed<S> && i == 0)
            f[i] = double(ldo(reinterpret_cast<const float*>(g), x * 4u));  // FP16 storage: in FP32
        else
            f[i] = double(ldo(g + plane_off<S>(i, A.g.N), x * uint32_t(sizeof(S))));
    }
}

// link coefficients of a boundary node (NO_LINK: none)
template <class RC>
__device__ __forceinline__ void coefs(const AdjDev& A, const RC* __restrict__ la, int tg, RC (&a)[Q2_LINKS]) {
    ld_vec(make_res(la, uint64_t(A.nb) * Q2_LINKS * sizeof(RC)), uint32_t(tg >> 8) * uint32_t(Q2_LINKS * sizeof(RC)), a);
}

// Links of a boundary node (tag tg > 0) on its pulled populations v (v[0] its own): v becomes the pre-collision
// populations (eqs. 16-18).  The forcing terms are those of the stored state, in FP64: an FP64 record holds them;
// with an FP32 one density and momentum come from the node's own populations and only the force from
// the record (F = rho du; the collision left j + F).
template <class RC>
__device__ __forceinline__ void links_on(const AdjDev& A, const RC* __restrict__ la, const RC* __restrict__ rec, int tg,
                                         double (&v)[9]) {
    RC h[RF2 + 8], a[Q2_LINKS];
    ld_vec(make_res(rec, uint64_t(A.nb) * REC2 * sizeof(RC)), uint32_t(tg >> 8) * uint32_t(REC2 * sizeof(RC)), h);
    coefs(A, la, tg, a);
    double kr = A.kF * double(h[0]), dx = double(h[1]), dy = double(h[2]), sx = double(h[3]), sy = double(h[4]);
    double duu = double(h[5]);
    if constexpr (sizeof(RC) == 4) {
        double r = A.rho_ref + v[0], m[2] = {0, 0};
#pragma unroll
        for (int j = 1; j < 9; ++j) {
            r += double(h[RF2 + j - 1]);
            eadd(j, double(h[RF2 + j - 1]), m);
        }
        const double ir = 1.0 / r, Fx = double(h[0]) * dx, Fy = double(h[0]) * dy;
        kr = A.kF * r;
        dx = Fx * ir;
        dy = Fy * ir;
        sx = 2.0 * (m[0] - Fx) * ir + dx;
        sy = 2.0 * (m[1] - Fy) * ir + dy;
        duu = 1.5 * (dx * sx + dy * sy);
    }
    double dm = 0.0;
    // a slot that a link replaces is never one that an eq. 16 link reads (its x2 = x - e_j is fluid)
#pragma unroll
    for (int j = 1; j < 9; ++j) {
        const bool lk = (tg >> (j - 1)) & 1;
        const double aj = double(a[j - 1]), c1 = fabs(aj), c2 = 1.0 - c1, fj = double(h[RF2 + j - 1]);
        const double ed = edot(j, dx, dy), es = edot(j, sx, sy);
        const double F = wgt<double>(0, j) * kr * (3.0 * ed + 4.5 * ed * es - duu);
        const double o = c2 != 0.0 ? (aj < 0.0 ? double(h[RF2 + opp<0>(j) - 1]) : v[j]) : 0.0;
        const double B = c1 * fj + c2 * (o + F);
        v[opp<0>(j)] = lk ? B : v[opp<0>(j)];
        dm += lk ? fj - B : 0.0;
    }
    v[0] += A.k18 * dm;
}

__device__ __forceinline__ double sum9(const AdjDev& A, const double (&v)[9]) {
    double r = A.rho_ref;
#pragma unroll
    for (int i = 0; i < 9; ++i) r += v[i];
    return r;
}

// density of node (cx, cy) after the pull
template <class S, class RC>
__device__ __forceinline__ double density(const AdjDev& A, const S* __restrict__ g, const RC* __restrict__ la,
                                          const RC* __restrict__ rec, int tg, int cx, int cy) {
    double w[9];
    pops<S>(A, g, cx, cy, w);
    if (tg > 0) {
        if (A.k18 != 0.0) {
            // where eq. 18 applies, the node's own population on each link takes the place of f_in (its slot
            // was pulled from a solid node and holds 0)
            constexpr int B = int(RF2 * sizeof(RC)) & ~15, K = B / int(sizeof(RC));
            RC h[RF2 + 8 - K];
            ld_vec(make_res(rec, uint64_t(A.nb) * REC2 * sizeof(RC)), uint32_t(tg >> 8) * uint32_t(REC2 * sizeof(RC)) + B, h);
#pragma unroll
            for (int j = 1; j < 9; ++j) w[0] += ((tg >> (j - 1)) & 1) ? double(h[RF2 - K + j - 1]) : 0.0;
        } else {
            links_on<RC>(A, la, rec, tg, w);
        }
    }
    return sum9(A, w);
}

// Transposed collision of a fluid node (tag tg) with density r, momentum j and force F: from
// lam = lambda(t + 1) and the adjoints lamR1 of its links' forcing terms, the adjoint pb of p through
// the direct and the (rho, j) dependences, and Fb of F.  A link (x, i) of eq. 16 uses o = f_i(x - e_i), which x
// also pulls in direction i, so pb_i takes c2 Bbar_i(x) here, less its density part (no other link of x reads
// that pb_i: x - e_i is fluid).
template <class RC>
__device__ __forceinline__ void collide_T9(const AdjDev& A, const RC* __restrict__ la, double r, const double (&j)[2],
                                           const double (&F)[2], const double (&lam)[9], int tg,
                                           const double* __restrict__ lamR1, double (&pb)[9], double (&Fb)[2]) {
    double rr[Q2_LINKS];  // adjoint of the forcing term on each link (0 without a link)
    RC a[Q2_LINKS];
#pragma unroll
    for (int i = 0; i < Q2_LINKS; ++i) {
        rr[i] = 0.0;
        a[i] = RC(NO_LINK);
    }
    if (tg > 0) {
        ld_vec(make_res(lamR1, uint64_t(A.nb) * Q2_LINKS * 8u), uint32_t(tg >> 8) * (Q2_LINKS * 8u), rr);
        coefs(A, la, tg, a);
#pragma unroll
        for (int i = 0; i < Q2_LINKS; ++i) rr[i] = ((tg >> i) & 1) ? rr[i] : 0.0;
    }
    // lt = (I - K)^T lambda: the adjoint of the direct dependence on p
    double lt[9];
    if (A.mrt) {
        double mu[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            double v = 0.0;
#pragma unroll
            for (int i = 0; i < 9; ++i)
                if (kM2[k][i] != 0) v += kM2[k][i] * lam[i];
            mu[k] = A.msc[k] * v;
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            double v = 0.0;
#pragma unroll
            for (int k = 0; k < 9; ++k)
                if (kM2[k][i] != 0) v += kM2[k][i] * mu[k];
            lt[i] = lam[i] - v;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) lt[i] = lam[i] * (1.0 - 1.0 / A.tau);
    }
    const double m1[2] = {j[0] + F[0], j[1] + F[1]};
    const double mm0 = j[0] * j[0] + j[1] * j[1], mm1 = m1[0] * m1[0] + m1[1] * m1[1];
    const double ir = 1.0 / r, ir2 = ir * ir;
    // al: adjoint of E_i(rho, j + F); be: of E_i(rho, j), (K - I)^T lambda (both with the weight w_i).
    // Opposite directions share (e.m)^2 and have opposite e.m, so each pair enters by its sum and
    // difference.
    double sa = 0.0, sb = 0.0, qa = 0.0, d1[2] = {0, 0}, d0[2] = {0, 0};
    sa = wgt<double>(0, 0) * lam[0];
    sb = -wgt<double>(0, 0) * lt[0];
    constexpr int pairs[4] = {1, 2, 5, 6};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int i = pairs[p], o = opp<0>(i);
        const double w = wgt<double>(0, i), ri = rr[i - 1], ro = rr[o - 1];
        const double ai = lam[i] + ri, ao = lam[o] + ro, bi = lt[i] + ri, bo = lt[o] + ro;
        const double ap = w * (ai + ao), am = w * (ai - ao), bp = -w * (bi + bo), bm = -w * (bi - bo);
        const double em0 = edot(i, j[0], j[1]), em1 = edot(i, m1[0], m1[1]);
        const double c1 = ap * em1, c0 = bp * em0;
        sa += ap;
        sb += bp;
        qa += c1 * em1 + c0 * em0;
        eadd(i, 3.0 * am + 9.0 * ir * c1, d1);
        eadd(i, 3.0 * bm + 9.0 * ir * c0, d0);
    }
    // d E / d rho and d E / d m at (rho, m), summed
    double rb = sa + sb + 1.5 * ir2 * (sa * mm1 + sb * mm0) - 4.5 * ir2 * qa;
    double jb[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        Fb[k] = d1[k] - 3.0 * ir * sa * m1[k];
        jb[k] = Fb[k] + d0[k] - 3.0 * ir * sb * j[k];
    }
    // the body force depends on rho: F = ... + rho g
    rb += Fb[0] * A.grav[0] + Fb[1] * A.grav[1];
#pragma unroll
    for (int i = 0; i < 9; ++i) pb[i] = lt[i] + rb + (i == 0 ? 0.0 : edot(i, jb[0], jb[1]));
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const double c2 = a[i - 1] >= RC(0) && a[i - 1] < RC(1) ? 1.0 - double(a[i - 1]) : 0.0;
        pb[i] += c2 * (pb[opp<0>(i)] - A.k18 * pb[0]);
    }
}

// Transposed streaming, links and eq. 18 at a fluid node (tag tg): lambda(t) and lambda_R(t) from pbar of its
// neighbours x + e_i in direction i (pxi; pxi[0] its own), without the density adjoint, which rb holds
// around the node (row stride rs); tag_at(i): the tag of x + e_i.
template <class RC, class TagAt>
__device__ __forceinline__ void stream_T9(const AdjDev& A, const RC* __restrict__ la, const double* __restrict__ pbar, int tg,
                                          uint32_t y, const double (&pxi)[9], const double* rb, int rs, TagAt tag_at,
                                          double* __restrict__ lam0, double* __restrict__ lamR0) {
    const int64_t N = A.g.N;
    double acc[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) acc[i] = pxi[i] + rb[kEy[i] * rs + kEx[i]];
    const __amdgpu_buffer_rsrc_t rla = make_res(la, uint64_t(A.nb) * Q2_LINKS * sizeof(RC));
    if (A.k18 == 0.0) {
        // without eq. 18 the density part of a neighbour's c2 Bbar_i is left (see collide_T9)
        RC ax[9];
        bool lk[9];
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const int tx = tag_at(i);
            lk[i] = tx > 0 && ((tx >> (i - 1)) & 1);
            ax[i] = Buf<RC>::ld(rla, lk[i] ? (uint32_t(tx >> 8) * Q2_LINKS + uint32_t(i - 1)) * uint32_t(sizeof(RC)) : OOB);
        }
#pragma unroll
        for (int i = 1; i < 9; ++i)
            acc[i] += lk[i] && ax[i] >= RC(0) && ax[i] < RC(1) ? (1.0 - double(ax[i])) * rb[kEy[i] * rs + kEx[i]] : 0.0;
    }
    if (tg > 0) {
        RC a[Q2_LINKS];
        double pby[9], lr[Q2_LINKS];
        coefs(A, la, tg, a);
#pragma unroll
        for (int i = 1; i < 9; ++i) pby[i] = ldo(pbar + i * N, y * 8u) + rb[0];
        const double pz = A.k18 * acc[0];  // eq. 18 carries the adjoint of p_0 (if applied)
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const bool lk = (tg >> (i - 1)) & 1;
            const double c1 = fabs(double(a[i - 1])), Bb = pby[opp<0>(i)] - pz;
            acc[i] = lk ? c1 * Bb + pz : acc[i];
            lr[i - 1] = lk ? A.kF * (1.0 - c1) * Bb : 0.0;
        }
        // eq. 17 of the link (x, opp i): o = f_i(x)
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const double ao = double(a[opp<0>(i) - 1]);
            acc[i] += ao < 0.0 ? (1.0 + ao) * (pby[i] - pz) : 0.0;
        }
        st_vec(make_res(lamR0, uint64_t(A.nb) * Q2_LINKS * 8u), uint32_t(tg >> 8) * (Q2_LINKS * 8u), lr);
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) sto(lam0 + i * N, y * 8u, acc[i]);
}

// the columns and rows around a node: index e + 1
__device__ __forceinline__ void around(int cx, int cy, int nx, int ny, uint32_t (&xo)[3], uint32_t (&yo)[3]) {
    xo[0] = uint32_t(cx == 0 ? nx - 1 : cx - 1);
    xo[1] = uint32_t(cx);
    xo[2] = uint32_t(cx == nx - 1 ? 0 : cx + 1);
    yo[0] = uint32_t(cy == 0 ? ny - 1 : cy - 1) * uint32_t(nx);
    yo[1] = uint32_t(cy) * uint32_t(nx);
    yo[2] = uint32_t(cy == ny - 1 ? 0 : cy + 1) * uint32_t(nx);
}

// ---- first kernel: pre-collision state of time t + 1 from the stored state of time t, then the
// transposed collision.  Phase 1: populations and density of the own nodes, densities of the ring two
// nodes wide, to LDS.  Phase 2: psi and its derivative on the tile and the nodes around it (wall nodes
// by eq. 15).  Phase 3: lambda(t + 1) -> pbar (without the density terms) and Fbar of the own nodes.
// PULL = false: the first collision, p = f^eq(rho0, 0).
// OWN lanes own the tile's nodes; lanes past them, where there are any, take the ring.
template <class S, class RC, int TX, int OWN, int NT, bool PULL>
__global__ __launch_bounds__(NT, 4) void k_adj2_collide(AdjDev A, int nsx, const S* __restrict__ gt, const RC* __restrict__ la,
                                                        const RC* __restrict__ rec, const double* __restrict__ rho0,
                                                        const double* __restrict__ lam1, const double* __restrict__ lamR1,
                                                        double* __restrict__ pbar, double* __restrict__ Fbar,
                                                        double* __restrict__ psi, double* __restrict__ dpsi,
                                                        double* __restrict__ rave, double* __restrict__ den) {
    constexpr int TY = OWN / TX, RX = TX + 4, RY = TY + 4, NRING = RX * RY - TX * TY, PX = TX + 2, PY = TY + 2, NP = PX * PY;
    __shared__ double s_rho[RY * RX], s_psi[NP];
    __shared__ int s_tag[RY * RX];
    const Tile T = tile_of<TX, TY>(nsx);
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = A.g.nx, ny = A.g.ny;
    const int64_t N = A.g.N;
    auto node = [&](int rx, int ry, int& cx, int& cy) {
        cx = image(T.x0 - 2 + rx, nx);
        cy = image(T.y0 - 2 + ry, ny);
        return uint32_t(cy) * uint32_t(nx) + uint32_t(cx);
    };
    // ---- 1
    constexpr bool SPLIT = OWN < NT;
    static_assert(OWN % 64 == 0 && NRING <= (SPLIT ? NT - OWN : NT), "one ring node per lane");
    const bool mine = !SPLIT || t < OWN;  // uniform in a wave
    bool own = false;
    uint32_t x = 0;
    int tg = -1;
    double v[9], lv[9], r = 0.0;
    int cx, cy;
    if (mine) {
        x = node(lx + 2, ly + 2, cx, cy);
        own = T.x0 + lx < nx && T.y0 + ly < ny;
        tg = ldo(A.tag, x * 4u);
        if (PULL) {
            pops<S>(A, gt, cx, cy, v);
        } else {
            const double d = rho0[x] - A.rho_ref;
#pragma unroll
            for (int i = 0; i < 9; ++i) v[i] = wgt<double>(0, i) * d;
        }
    }
    if (!SPLIT || !mine) {
        // the ring; lanes past its last entry repeat it
        int rx, ry, gx, gy;
        ring_at<TX, TY, 2>(min(SPLIT ? t - OWN : t, NRING - 1), rx, ry);
        const uint32_t xr = node(rx, ry, gx, gy);
        const int tr = ldo(A.tag, xr * 4u);
        const double rr = PULL ? density<S, RC>(A, gt, la, rec, tr, gx, gy) : rho0[xr];
        s_rho[ry * RX + rx] = rr;
        s_tag[ry * RX + rx] = tr;
    }
    if (mine) {
        if (PULL && tg > 0) links_on<RC>(A, la, rec, tg, v);
        // (here, so that they arrive during phase 2 without holding registers through the links)
#pragma unroll
        for (int i = 0; i < 9; ++i) lv[i] = ldo(lam1 + i * N, x * 8u);
        r = sum9(A, v);
        s_rho[(ly + 2) * RX + lx + 2] = r;
        s_tag[(ly + 2) * RX + lx + 2] = tg;
    }
    __syncthreads();
    // ---- 2
#pragma unroll
    for (int h = 0; h < (NP + NT - 1) / NT; ++h) {
        const int e = t + h * NT, px = e % PX, py = e / PX, c = (py + 1) * RX + px + 1;
        if (e >= NP) break;
        const int g = s_tag[c];
        double s = 0.0, ds = 0.0, num = 0.0, dn = 0.0, ra = 0.0;
        if (g <= -2) {
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int o = c + kEy[i] * RX + kEx[i];
                const bool fl = s_tag[o] >= 0;
                num += fl ? wgt<double>(0, i) * s_rho[o] : 0.0;
                dn += fl ? wgt<double>(0, i) : 0.0;
            }
            ra = num / dn;
        }
        if (g != -1) psi_d(A, g >= 0 ? s_rho[c] : A.phi[-g - 2] * ra, &s, &ds);
        s_psi[e] = s;
        if (px >= 1 && px <= TX && py >= 1 && py <= TY && T.x0 + px - 1 < nx && T.y0 + py - 1 < ny) {
            const uint32_t y = uint32_t(T.y0 + py - 1) * uint32_t(nx) + uint32_t(T.x0 + px - 1);
            sto(psi, y * 8u, s);
            sto(dpsi, y * 8u, ds);
            if (g <= -2) {
                sto(rave, y * 8u, ra);
                sto(den, y * 8u, dn);
            }
        }
    }
    __syncthreads();
    // ---- 3
    if (!own || tg < 0) return;
    double jm[2] = {0, 0}, S2[2] = {0, 0};
    const double* P = s_psi + (ly + 1) * PX + lx + 1;
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        eadd(i, v[i], jm);
        eadd(i, wforce(0, i) * P[kEy[i] * PX + kEx[i]], S2);
    }
    const double gp = -A.G * P[0];
    const double F[2] = {gp * S2[0] + r * A.grav[0], gp * S2[1] + r * A.grav[1]};
    double pb[9], Fb[2];
    collide_T9(A, la, r, jm, F, lv, tg, lamR1, pb, Fb);
#pragma unroll
    for (int i = 0; i < 9; ++i) sto(pbar + i * N, x * 8u, pb[i]);
    sto(Fbar, x * 8u, Fb[0]);
    sto(Fbar + N, x * 8u, Fb[1]);
}

// ---- second kernel: the transposed force stencil and psi, density sum, streaming and links.
// Phase 1: Fbar (zero off the fluid), psi and tags of the tile and three nodes around it, to LDS.
// Phase 2: psibar -> rhobar of the fluid nodes next to or in the tile, and of the wall nodes up to two
// nodes out their density adjoint per unit eq. 15 weight (and dphi of the own ones).  Phase 3: the
// density adjoint of the tile and the nodes around it.  Phase 4 (STREAM): lambda(t) and lambda_R(t).
template <class RC, int TX, int OWN, int NT, bool STREAM>
__global__ __launch_bounds__(NT, 4) void k_adj2_stream(AdjDev A, int nsx, const RC* __restrict__ la,
                                                       const double* __restrict__ psi, const double* __restrict__ dpsi,
                                                       const double* __restrict__ rave, const double* __restrict__ den,
                                                       const double* __restrict__ Fbar, const double* __restrict__ pbar,
                                                       double* __restrict__ dphi, double* __restrict__ lam0,
                                                       double* __restrict__ lamR0) {
    constexpr int TY = OWN / TX, RX = TX + 6, RY = TY + 6, NR = RX * RY, QX = TX + 4, QY = TY + 4, NQ = QX * QY;
    constexpr int PX = TX + 2, PY = TY + 2, NP = PX * PY;
    __shared__ double s_psi[NR], s_fx[NR], s_fy[NR], s_q[NQ], s_rb[NQ];
    __shared__ int s_tag[NR];
    const Tile T = tile_of<TX, TY>(nsx);
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = A.g.nx, ny = A.g.ny;
    const int64_t N = A.g.N;
    // ---- 1 (every load that depends on no other is issued here)
    constexpr int NRL = (NR + NT - 1) / NT, NQL = (NQ + NT - 1) / NT;
    int gr[NRL];
    double fx[NRL], fy[NRL], ps[NRL], dp[NQL], pxi[9];
#pragma unroll
    for (int h = 0; h < NRL; ++h) {
        const int e = min(t + h * NT, NR - 1);
        const uint32_t x = uint32_t(image(T.y0 - 3 + e / RX, ny)) * uint32_t(nx) + uint32_t(image(T.x0 - 3 + e % RX, nx));
        gr[h] = ldo(A.tag, x * 4u);
        fx[h] = ldo(Fbar, x * 8u);
        fy[h] = ldo(Fbar + N, x * 8u);
        ps[h] = ldo(psi, x * 8u);
    }
    uint32_t yq[NQL];
#pragma unroll
    for (int h = 0; h < NQL; ++h) {
        const int e = min(t + h * NT, NQ - 1);
        yq[h] = uint32_t(image(T.y0 - 2 + e / QX, ny)) * uint32_t(nx) + uint32_t(image(T.x0 - 2 + e % QX, nx));
        dp[h] = ldo(dpsi, yq[h] * 8u);
    }
    const bool own = (OWN == NT || t < OWN) && T.x0 + lx < nx && T.y0 + ly < ny;
    const int cx = image(T.x0 + lx, nx), cy = image(T.y0 + ly, ny);
    uint32_t xo[3], yo[3];
    around(cx, cy, nx, ny, xo, yo);
    if (STREAM && (OWN == NT || t < OWN)) {
#pragma unroll
        for (int i = 0; i < 9; ++i) pxi[i] = ldo(pbar + i * N, (xo[kEx[i] + 1] + yo[kEy[i] + 1]) * 8u);
    }
#pragma unroll
    for (int h = 0; h < NRL; ++h) {
        const int e = min(t + h * NT, NR - 1);
        s_tag[e] = gr[h];
        s_psi[e] = ps[h];
        s_fx[e] = gr[h] >= 0 ? fx[h] : 0.0;
        s_fy[e] = gr[h] >= 0 ? fy[h] : 0.0;
    }
    __syncthreads();
    // ---- 2
#pragma unroll
    for (int h = 0; h < NQL; ++h) {
        const int e = t + h * NT, qx = e % QX, qy = e / QX, c = (qy + 1) * RX + qx + 1;
        if (e >= NQ) break;
        const int g = s_tag[c];
        double qb = 0.0, rb = 0.0;
        const bool inner = qx >= 1 && qx < QX - 1 && qy >= 1 && qy < QY - 1;
        if (g <= -2 || (g >= 0 && inner)) {
            const uint32_t y = yq[h];
            double pb = 0.0, S2[2] = {0, 0};
            // the neighbours x = y - e_k whose force uses psi(y), and the node's own force -G psi(y) S(y)
#pragma unroll
            for (int k = 1; k < 9; ++k) {
                const int o = c - kEy[k] * RX - kEx[k], n = c + kEy[k] * RX + kEx[k];
                pb -= A.G * s_psi[o] * wforce(0, k) * edot(k, s_fx[o], s_fy[o]);
                eadd(k, wforce(0, k) * s_psi[n], S2);
            }
            pb -= A.G * (s_fx[c] * S2[0] + s_fy[c] * S2[1]);
            if (g >= 0) {
                rb = dp[h] * pb;
            } else {
                const double rwb = dp[h] * pb;
                qb = rwb * A.phi[-g - 2] / ldo(den, y * 8u);
                if (qx >= 2 && qx < TX + 2 && qy >= 2 && qy < TY + 2 && T.x0 + qx - 2 < nx && T.y0 + qy - 2 < ny)
                    dphi[-g - 2] += rwb * ldo(rave, y * 8u);
            }
        }
        s_q[e] = qb;
        s_rb[e] = rb;
    }
    if (!STREAM) return;
    __syncthreads();
    // ---- 3 (rhobar of a node is read by its own lane alone)
#pragma unroll
    for (int h = 0; h < (NP + NT - 1) / NT; ++h) {
        const int e = t + h * NT, c = (e / PX + 1) * QX + e % PX + 1;
        if (e >= NP) break;
        double rb = s_rb[c];
#pragma unroll
        for (int k = 1; k < 9; ++k) rb += wgt<double>(0, k) * s_q[c - kEy[k] * QX - kEx[k]];
        s_rb[c] = rb;
    }
    // ---- 4
    __syncthreads();
    if (!own) return;
    const int c3 = (ly + 3) * RX + lx + 3, c2 = (ly + 2) * QX + lx + 2;
    const int tg = s_tag[c3];
    if (tg < 0) return;  // lambda is read on fluid nodes only
    stream_T9(A, la, pbar, tg, xo[1] + yo[1], pxi, s_rb + c2, QX, [&](int i) { return s_tag[c3 + kEy[i] * RX + kEx[i]]; }, lam0,
              lamR0);
}

// ================================================================ chemical-potential model
// The same two kernels with that model's fields between the density and the force: the solid layers' densities (eq. 15), mu (eq. 12) and F (eq. 9) of the recomputed state, and
// their transposes.  Fourth-order central differences: d/dx v = sum_m c_m v(x + m), m = -2..2,
// c = (1, -8, 0, 8, -1) / 12; d2/dx2 v = sum_m d_m v(x + m), d = (-1, 16, -30, 16, -1) / 12.
__device__ constexpr double cdc(int m) { return m == -2 ? 1.0 / 12.0 : m == -1 ? -8.0 / 12.0 : m == 1 ? 8.0 / 12.0 : m == 2 ? -1.0 / 12.0 : 0.0; }
__device__ constexpr double cdd(int m) { return (m == -2 || m == 2) ? -1.0 / 12.0 : (m == -1 || m == 1) ? 16.0 / 12.0 : -30.0 / 12.0; }

// sum of c_m v(m st) over the offsets of an axis of stride st
__device__ __forceinline__ double diff1(const double* v, int st) {
    return (8.0 * (v[st] - v[-st]) - (v[2 * st] - v[-2 * st])) * (1.0 / 12.0);
}

// mu_PR of eq. 11 (without the gradient term) and its derivative
__device__ __forceinline__ double pr_mu0(const AdjDev& A, double r) {
    const double br = A.pb * r, s2 = 1.4142135623730951, iq = 1.0 / (1.0 - br);
    return A.pRT * log(r * iq) - A.pclog * log((s2 - 1.0 + br) / (s2 + 1.0 - br)) + A.pRT * iq -
           A.paal * r / (1.0 + 2.0 * br - br * br);
}
__device__ __forceinline__ double pr_dmu0(const AdjDev& A, double r) {
    const double br = A.pb * r, iq = 1.0 / (1.0 - br), iD = 1.0 / (1.0 + 2.0 * br - br * br);
    return A.pRT * iq * (1.0 / r + A.pb * iq) - A.paal * iD * (1.0 + (1.0 + br * br) * iD);
}

// the weights of eq. 15 around entry c (row stride st): sum of w_i over the neighbours of layer l, and of
// w_i val(neighbour) over them
template <class Val>
__device__ __forceinline__ void around_layer(const int8_t* lay, int c, int st, int l, Val val, double& num, double& den) {
    num = den = 0.0;
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const int o = c + kEy[i] * st + kEx[i];
        if (lay[o] == l) {
            num += wgt<double>(0, i) * val(o);
            den += wgt<double>(0, i);
        }
    }
}

// ---- first kernel: as k_adj2_collide, with the fields of a ring of six nodes (as the forward tiles).
// rho and mu of every node go to the second kernel.
template <class S, class RC, int TX, int OWN, int NT, bool PULL>
__global__ __launch_bounds__(NT, 4) void k_adj2cp_collide(AdjDev A, int nsx, const S* __restrict__ gt, const RC* __restrict__ la,
                                                           const RC* __restrict__ rec, const double* __restrict__ rho0,
                                                           const double* __restrict__ lam1, const double* __restrict__ lamR1,
                                                           double* __restrict__ pbar, double* __restrict__ Fbar,
                                                           double* __restrict__ rho, double* __restrict__ mu) {
    constexpr int TY = OWN / TX, HC = 6, RX = TX + 2 * HC, RY = TY + 2 * HC, NR = RX * RY, NRING = NR - TX * TY;
    constexpr int MX = TX + 4, MY = TY + 4, NM = MX * MY;
    __shared__ double s_rho[NR], s_mu[NM];
    __shared__ int s_tag[NR];
    __shared__ int8_t s_lay[NR];
    const Tile T = tile_of<TX, TY>(nsx);
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = A.g.nx, ny = A.g.ny;
    const int64_t N = A.g.N;
    auto node = [&](int rx, int ry, int& cx, int& cy) {
        cx = image(T.x0 - HC + rx, nx);
        cy = image(T.y0 - HC + ry, ny);
        return uint32_t(cy) * uint32_t(nx) + uint32_t(cx);
    };
    // ---- 1: densities, layers and tags
    bool solid = false;
    const bool mine = OWN == NT || t < OWN;  // uniform in a wave
    for (int k = OWN == NT ? t : (t >= OWN ? t - OWN : t + NT - OWN); k < NRING; k += NT) {
        int rx, ry, gx, gy;
        ring_at<TX, TY, HC>(k, rx, ry);
        const uint32_t x = node(rx, ry, gx, gy);
        const int g = ldo(A.tag, x * 4u);
        const int8_t l = ldo(A.layer, x);
        const double r = PULL ? density<S, RC>(A, gt, la, rec, g, gx, gy) : rho0[x];
        s_rho[ry * RX + rx] = l == 0 ? r : 0.0;
        s_tag[ry * RX + rx] = g;
        s_lay[ry * RX + rx] = l;
        solid = solid || l == 1 || l == 2;
    }
    uint32_t x = 0;
    bool own = false;
    int tg = -1;
    const int c0 = (ly + HC) * RX + lx + HC;
    double v[9], lv[9], r = 0.0;
    if (mine) {
        int cx, cy;
        x = node(lx + HC, ly + HC, cx, cy);
        own = T.x0 + lx < nx && T.y0 + ly < ny;
        tg = ldo(A.tag, x * 4u);
        const int8_t lay = ldo(A.layer, x);
        if (PULL) {
            pops<S>(A, gt, cx, cy, v);
            if (tg > 0) links_on<RC>(A, la, rec, tg, v);
        } else {
#pragma unroll
            for (int i = 0; i < 9; ++i) v[i] = wgt<double>(0, i) * (rho0[x] - A.rho_ref);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) lv[i] = ldo(lam1 + i * N, x * 8u);
        r = sum9(A, v);
        s_rho[c0] = lay == 0 ? r : 0.0;
        s_tag[c0] = tg;
        s_lay[c0] = lay;
        solid = solid || lay == 1 || lay == 2;
    }
    // ---- 2, 3: the solid layers
    if (__syncthreads_or(solid)) {
#pragma unroll 1
        for (int l = 1; l <= 2; ++l) {
            for (int e = t; e < NR; e += NT) {
                const int ex = e % RX, ey = e / RX;
                if (ex >= l && ex < RX - l && ey >= l && ey < RY - l && s_lay[e] == l) {
                    double num, den;
                    around_layer(s_lay, e, RX, l - 1, [&](int o) { return s_rho[o]; }, num, den);
                    s_rho[e] = num / den;
                }
            }
            __syncthreads();
        }
    }
    // ---- 4: mu
    for (int j = t; j < NM; j += NT) {
        const int e = (j / MX + HC - 2) * RX + j % MX + HC - 2;
        const int l = s_lay[e];
        double m = 0.0;
        if (l == 0) {
            const double rc = s_rho[e];
            const double lap = (16.0 * (s_rho[e + 1] + s_rho[e - 1]) - (s_rho[e + 2] + s_rho[e - 2]) - 30.0 * rc) * (1.0 / 12.0) +
                               (16.0 * (s_rho[e + RX] + s_rho[e - RX]) - (s_rho[e + 2 * RX] + s_rho[e - 2 * RX]) - 30.0 * rc) *
                                   (1.0 / 12.0);
            m = A.k2 * pr_mu0(A, rc) - A.kappa * lap;
        } else if (l == 1) {
            m = A.phi[-s_tag[e] - 2];
        } else if (l == 2) {
            double num, den;
            around_layer(s_lay, e, RX, 1, [&](int o) { return A.phi[-s_tag[o] - 2]; }, num, den);
            m = num / den;
        }
        s_mu[j] = m;
    }
    __syncthreads();
    // ---- 5
    if (!own) return;
    const double* R = s_rho + c0;
    const double* U = s_mu + (ly + 2) * MX + lx + 2;
    sto(rho, x * 8u, R[0]);
    sto(mu, x * 8u, U[0]);
    if (tg < 0) return;
    double jm[2] = {0, 0};
#pragma unroll
    for (int i = 1; i < 9; ++i) eadd(i, v[i], jm);
    const double F[2] = {-r * diff1(U, 1) + diff1(R, 1) * (1.0 / 3.0) + r * A.grav[0],
                         -r * diff1(U, MX) + diff1(R, RX) * (1.0 / 3.0) + r * A.grav[1]};
    double pb[9], Fb[2];
    collide_T9(A, la, r, jm, F, lv, tg, lamR1, pb, Fb);
#pragma unroll
    for (int i = 0; i < 9; ++i) sto(pbar + i * N, x * 8u, pb[i]);
    sto(Fbar, x * 8u, Fb[0]);
    sto(Fbar + N, x * 8u, Fb[1]);
}

// ---- second kernel.  Phase 1: Fbar (zero off the fluid), rho, layers, tags seven nodes around the tile, mu
// five.  Phase 2: mubar five nodes around (F = -rho grad mu + ... : the fluid nodes whose force reads
// it).  Phase 3: dphi of the own wall nodes (their own mubar and the second layer's, which is their
// weighted mean), and rhobar three nodes around (from F, and from mu: the Peng-Robinson slope and the
// transposed Laplacian).  Phase 4: the second layer's rhobar onto the first, and that per unit eq. 15
// weight of its fluid neighbours, two nodes around.  Phase 5: the density adjoint of the fluid nodes
// next to or in the tile.  Phase 6: transposed streaming.
template <class RC, int TX, int OWN, int NT, bool STREAM>
__global__ __launch_bounds__(NT, 4) void k_adj2cp_stream(AdjDev A, int nsx, const RC* __restrict__ la,
                                                          const double* __restrict__ rho, const double* __restrict__ mu,
                                                          const double* __restrict__ Fbar, const double* __restrict__ pbar,
                                                          double* __restrict__ dphi, double* __restrict__ lam0,
                                                          double* __restrict__ lamR0) {
    constexpr int TY = OWN / TX, H = 7, RX = TX + 2 * H, RY = TY + 2 * H, NR = RX * RY;
    __shared__ double s_f[2][NR], s_r[NR], s_u[NR], s_ub[NR], s_rb[NR];
    __shared__ int s_tag[NR];
    __shared__ int8_t s_lay[NR];
    const Tile T = tile_of<TX, TY>(nsx);
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = A.g.nx, ny = A.g.ny;
    const int64_t N = A.g.N;
    // ---- 1
    for (int e = t; e < NR; e += NT) {
        const uint32_t x = uint32_t(image(T.y0 - H + e / RX, ny)) * uint32_t(nx) + uint32_t(image(T.x0 - H + e % RX, nx));
        const int8_t l = ldo(A.layer, x);
        const double fx = ldo(Fbar, x * 8u), fy = ldo(Fbar + N, x * 8u);
        s_r[e] = ldo(rho, x * 8u);
        s_u[e] = ldo(mu, x * 8u);
        s_tag[e] = ldo(A.tag, x * 4u);
        s_lay[e] = l;
        s_f[0][e] = l == 0 ? fx : 0.0;
        s_f[1][e] = l == 0 ? fy : 0.0;
    }
    const bool mine = OWN == NT || t < OWN;  // uniform in a wave
    const bool own = mine && T.x0 + lx < nx && T.y0 + ly < ny;
    const int c0 = mine ? (ly + H) * RX + lx + H : 0;
    uint32_t xo[3], yo[3];
    around(image(T.x0 + lx, nx), image(T.y0 + ly, ny), nx, ny, xo, yo);
    double pxi[9];
    if (STREAM && mine) {
#pragma unroll
        for (int i = 0; i < 9; ++i) pxi[i] = ldo(pbar + i * N, (xo[kEx[i] + 1] + yo[kEy[i] + 1]) * 8u);
    }
    __syncthreads();
    // entries at most m nodes from the tile
    auto within = [&](int e, int m) {
        const int ex = e % RX, ey = e / RX;
        return ex >= H - m && ex < TX + H + m && ey >= H - m && ey < TY + H + m;
    };
    // ---- 2 (a node x = y - d e_k off the fluid has Fbar = 0)
    for (int e = t; e < NR; e += NT) {
        double ub = 0.0;
        if (within(e, 5) && s_lay[e] <= 2) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int st = k == 0 ? 1 : RX;
#pragma unroll
                for (int d = -2; d <= 2; ++d)
                    if (d != 0) ub -= s_f[k][e - d * st] * s_r[e - d * st] * cdc(d);
            }
        }
        s_ub[e] = ub;
    }
    __syncthreads();
    // ---- 3
    if (own && s_lay[c0] == 1) {
        double g = s_ub[c0];
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const int o = c0 + kEy[i] * RX + kEx[i];
            if (s_lay[o] == 2) {
                double num, den;
                around_layer(s_lay, o, RX, 1, [](int) { return 0.0; }, num, den);
                g += s_ub[o] * wgt<double>(0, i) / den;
            }
        }
        dphi[-s_tag[c0] - 2] += g;
    }
    if (!STREAM) return;
    for (int e = t; e < NR; e += NT) {
        const int l = s_lay[e];
        double rb = 0.0;
        if (within(e, 3) && l <= 2) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int st = k == 0 ? 1 : RX;
#pragma unroll
                for (int d = -2; d <= 2; ++d) {
                    const int o = e - d * st;
                    if (d != 0) rb += s_f[k][o] * (cdc(d) * (1.0 / 3.0));
                    if (s_lay[o] == 0) rb -= A.kappa * cdd(d) * s_ub[o];
                }
                if (l == 0) rb -= s_f[k][e] * diff1(s_u + e, st);
            }
            if (l == 0) rb += s_ub[e] * A.k2 * pr_dmu0(A, s_r[e]);
        }
        s_rb[e] = rb;
    }
    __syncthreads();
    // ---- 4 (into s_ub, which nothing reads any more)
    for (int e = t; e < NR; e += NT) {
        double q = 0.0;
        if (within(e, 2) && s_lay[e] == 1) {
            q = s_rb[e];
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int o = e + kEy[i] * RX + kEx[i];
                if (s_lay[o] == 2) {
                    double num, den;
                    around_layer(s_lay, o, RX, 1, [](int) { return 0.0; }, num, den);
                    q += s_rb[o] * wgt<double>(0, i) / den;
                }
            }
            double num, den;
            around_layer(s_lay, e, RX, 0, [](int) { return 0.0; }, num, den);
            q /= den;
        }
        s_ub[e] = q;
    }
    __syncthreads();
    // ---- 5 (each entry is read by its own lane alone)
    for (int e = t; e < NR; e += NT) {
        if (within(e, 1) && s_lay[e] == 0) {
            double rb = s_rb[e];
#pragma unroll
            for (int k = 1; k < 9; ++k) rb += wgt<double>(0, k) * s_ub[e - kEy[k] * RX - kEx[k]];
            s_rb[e] = rb;
        }
    }
    __syncthreads();
    // ---- 6
    if (!own || s_tag[c0] < 0) return;  // lambda is read on fluid nodes only
    stream_T9(A, la, pbar, s_tag[c0], xo[1] + yo[1], pxi, s_rb + c0, RX, [&](int i) { return s_tag[c0 + kEy[i] * RX + kEx[i]]; },
              lam0, lamR0);
}

// the two kernels on tiles of TX x OWN / TX nodes, NT lanes a workgroup
struct Adj2 {
    mcb_ctx* c;
    const AdjWork& w;
    const void *gt, *rec;
    int pull;
    const double *lam1, *lamR1;
    double *lam0, *lamR0;
};
template <class S, class RC, int TX, int OWN, int NT, bool CP>
hipError_t launch2(const Adj2& p) {
    constexpr int TY = OWN / TX;
    mcb_ctx* c = p.c;
    const AdjWork& w = p.w;
    const AdjDev A = make_dev(c);
    const int nsx = (c->p.nx + TX - 1) / TX;
    const RC* la = reinterpret_cast<const RC*>(c->lk + c->L.lk_a);
    const dim3 grid(unsigned(nsx) * unsigned((c->p.ny + TY - 1) / TY)), blk(NT);
    if constexpr (CP) {
        hipLaunchKernelGGL((p.pull ? k_adj2cp_collide<S, RC, TX, OWN, NT, true> : k_adj2cp_collide<S, RC, TX, OWN, NT, false>), grid,
                           blk, 0, c->stream, A, nsx, static_cast<const S*>(p.gt), la, static_cast<const RC*>(p.rec), w.rho0,
                           p.lam1, p.lamR1, w.pbar, w.Fbar, w.rho, w.psi);
        hipLaunchKernelGGL((p.pull ? k_adj2cp_stream<RC, TX, OWN, NT, true> : k_adj2cp_stream<RC, TX, OWN, NT, false>), grid, blk, 0,
                           c->stream, A, nsx, la, w.rho, w.psi, w.Fbar, w.pbar, w.dphi, p.lam0, p.lamR0);
    } else {
        hipLaunchKernelGGL((p.pull ? k_adj2_collide<S, RC, TX, OWN, NT, true> : k_adj2_collide<S, RC, TX, OWN, NT, false>), grid, blk,
                           0, c->stream, A, nsx, static_cast<const S*>(p.gt), la, static_cast<const RC*>(p.rec), w.rho0, p.lam1,
                           p.lamR1, w.pbar, w.Fbar, w.psi, w.dpsi, w.rave, w.den);
        hipLaunchKernelGGL((p.pull ? k_adj2_stream<RC, TX, OWN, NT, true> : k_adj2_stream<RC, TX, OWN, NT, false>), grid, blk, 0,
                           c->stream, A, nsx, la, w.psi, w.dpsi, w.rave, w.den, w.Fbar, w.pbar, w.dphi, p.lam0, p.lamR0);
    }
    return hipGetLastError();
}

// The forward step's rules (tile2d.hip), for the same reason: a box whose tiles are all resident waits for the
// chain of one of them, which more lanes shorten.  Pseudopotential model (128 registers: two tiles of seven
// waves a compute unit): a gradient of 50 steps at 64 x 60 1.56 -> 1.28 ms, 200 x 190 1.62 -> 1.49,
// 256 x 250 1.86 -> 1.70, 350 x 360 1.81 -> 1.77; 512^2, four tiles a unit, 2.94 -> 3.06.  Chemical
// potential, against 32 x 16 tiles of 512 lanes: 64 x 60 2.80 -> 1.90 ms, 301 x 203 3.14 -> 2.58, 500 x 300
// 3.23 -> 2.98, 512 x 384 3.58 -> 3.27.
template <class S, class RC>
hipError_t adj2_t(const Adj2& p) {
    const mcb_ctx* c = p.c;
    auto tiles = [&](int tx, int ty) { return int64_t((c->p.nx + tx - 1) / tx) * ((c->p.ny + ty - 1) / ty); };
    auto fits = [&](int tx, int ty) { return tiles(tx, ty) <= c->n_cu; };
    if (c->p.model == MCB_MODEL_CHEMPOT) {
        if (fits(8, 8)) return launch2<S, RC, 8, 64, 448, true>(p);
        if (fits(16, 8)) return launch2<S, RC, 16, 128, 576, true>(p);
        if (fits(16, 16)) return launch2<S, RC, 16, 256, 768, true>(p);
        if (fits(32, 16)) return launch2<S, RC, 32, 512, 1024, true>(p);
        if (fits(32, 20)) return launch2<S, RC, 32, 640, 1024, true>(p);
        if (fits(32, 24)) return launch2<S, RC, 32, 768, 1024, true>(p);
        return launch2<S, RC, 32, 512, 512, true>(p);
    }
    if (tiles(8, 8) <= 3 * c->n_cu) return launch2<S, RC, 8, 64, 192, false>(p);
    if (tiles(32, 8) <= 2 * c->n_cu) return launch2<S, RC, 32, 256, 448, false>(p);
    return launch2<S, RC, 32, 256, 256, false>(p);
}

}  // namespace

hipError_t adj_step2d(mcb_ctx* c, const AdjWork& w, const void* gt, const void* rec, int pull, const double* lam1,
                      const double* lamR1, double* lam0, double* lamR0) {
    const Adj2 p{c, w, gt, rec, pull, lam1, lamR1, lam0, lamR0};
    switch (c->p.precision) {
        case MCB_F64: return adj2_t<double, double>(p);
        case MCB_F32S: return adj2_t<float, float>(p);
        default: return adj2_t<__half, float>(p);
    }
}

}  // namespace mcb
