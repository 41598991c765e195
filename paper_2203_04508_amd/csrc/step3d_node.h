// Per-node arithmetic of the D3Q19 step and the arguments of its kernels, shared by the plane march
// (step3d.hip) and the flat kernels (flat3d.hip).
#pragma once

#include "kernels_common.h"

namespace mcb {
namespace {

// D3Q19: rest, the six axis vectors, the twelve edge vectors; opposite pairs side by side
__device__ constexpr int kEx3[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
__device__ constexpr int kEy3[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
__device__ constexpr int kEz3[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};

// D3Q19 weights
template <class C>
__device__ inline C w19(int i) {
    return i == 0 ? C(1.0 / 3.0) : (i < 7 ? C(1.0 / 18.0) : C(1.0 / 36.0));
}

__device__ inline int zinc(int z, int nz) { return z == nz - 1 ? 0 : z + 1; }
__device__ inline int zdec(int z, int nz) { return z == 0 ? nz - 1 : z - 1; }
__device__ inline int wrapn(int a, int n) { return ((a % n) + n) % n; }

// e.(x, y, z) for a lattice vector of components 0 and +-1, folded when the components are
// constants (a product with 0 cannot be dropped under IEEE rules)
template <class C>
__device__ __forceinline__ C edot3(int ex, int ey, int ez, C x, C y, C z) {
    const C tx = ex > 0 ? x : -x, ty = ey > 0 ? y : -y, tz = ez > 0 ? z : -z;
    const C a = ex == 0 ? ty : (ey == 0 ? tx : tx + ty);  // D3Q19: at most two components are set
    return ez == 0 ? a : ((ex == 0 && ey == 0) ? tz : a + tz);
}

// One lane per node, NT consecutive nodes of the lattice per workgroup: the node of a lane (one scalar
// division per workgroup; lanes past the last node repeat node 0) and the byte offsets of its
// neighbours x + e_i in an array of T.
struct Node3 {
    uint32_t node;
    bool on;
    int x, y, z;
};
template <int NT>
__device__ __forceinline__ Node3 node3(int nx, int ny, int nz) {
    const uint32_t n0 = uint32_t(blockIdx.x) * NT, t = threadIdx.x;
    const uint32_t nxy = uint32_t(nx) * uint32_t(ny), N = nxy * uint32_t(nz);
    Node3 r;
    const uint32_t z0 = n0 / nxy, y0 = (n0 - z0 * nxy) / uint32_t(nx);
    r.node = n0 + t;
    r.on = r.node < N;
    r.x = int(n0 - z0 * nxy - y0 * uint32_t(nx) + t);
    r.y = int(y0);
    r.z = int(z0);
    while (r.x >= nx) {
        r.x -= nx;
        ++r.y;
    }
    while (r.y >= ny) {
        r.y -= ny;
        ++r.z;
    }
    if (!r.on) r.node = 0, r.x = r.y = r.z = 0;
    return r;
}
template <class T>
__device__ __forceinline__ void neighbours(const Node3& p, int nx, int ny, int nz, uint32_t (&off)[19]) {
    constexpr uint32_t s = sizeof(T);
    const uint32_t row = uint32_t(nx) * s, pl = row * uint32_t(ny), o = p.node * s;
    const uint32_t xo[3] = {p.x == 0 ? row - s : 0u - s, 0u, p.x == nx - 1 ? s - row : s};
    const uint32_t yo[3] = {o + (p.y == 0 ? pl - row : 0u - row), o, o + (p.y == ny - 1 ? row - pl : row)};
    const uint32_t zo[3] = {p.z == 0 ? pl * uint32_t(nz - 1) : 0u - pl, 0u, p.z == nz - 1 ? 0u - pl * uint32_t(nz - 1) : pl};
#pragma unroll
    for (int i = 0; i < 19; ++i) off[i] = yo[kEy3[i] + 1] + xo[kEx3[i] + 1] + zo[kEz3[i] + 1];
}
__device__ constexpr int opp3(int i) { return i == 0 ? 0 : ((i & 1) ? i + 1 : i - 1); }

template <class S, class C>
struct Args3 {
    const S* fa;                 // post-collision populations of time t, SoA [19][N]
    S* fb;                       // post-collision populations of time t+1
    const int32_t* tag;          // >0: boundary index + 1; 0 fluid; -1 solid; -2-w wall w
    const uint32_t* nmask;       // link bits of each boundary node (bit j-1: x + e_j solid)
    const C* rho;                // density pass output (rho; -eq. 15 factor at wall nodes; 0 solid)
    const C* rin;                // boundary records of time t, REC3 per boundary node
    C* rout;                     // boundary records of time t+1
    const C* la;                 // link coefficients, Q3_LINKS per boundary node (NO_LINK: none)
    int32_t* flags;
    uint32_t n_bnodes;
    int nx, ny, nz, D, ntx, nty, nblocks;
    C tau_inv, G, rho_ref;
    C kF, k18;                   // boundary scheme: weights of the forcing term and of eq. 18
    C gx, gy, gz;                // body acceleration: F = F_nonideal + rho g, so du = F / rho gains g
    Eos<C> eos;
};

// Eqs. 16-18 at a boundary node (bnd) from its record of time t (rec: forcing terms and the
// populations 1..18) and link coefficients (ca): replaces the populations pulled from solid
// neighbours by f_in (see the two-dimensional kernel for the three cases) and corrects the rest
// population; returns the correction and, in res, what rounding f_0 + correction to the compute type
// dropped.  Lanes that are not boundary nodes keep f and return zeros;
// directions in which no lane of the wave has a link are skipped.  LOAD: rec and ca are loaded
// here, from rin at byte offset roff and la at aoff, in two halves, each just before its directions
// (keeps the FP64 kernel within its registers).  kF = 0 drops the forcing term (MIBC); halfway
// bounce-back is a = 1 on every link; k18 = 0 drops eq. 18 (IBC).
template <class S, class C, bool LOAD>
__device__ __forceinline__ C apply_links3(bool bnd, C (&rec)[RF3 + 18], C (&ca)[18], C (&f)[19], __amdgpu_buffer_rsrc_t rin,
                                          uint32_t roff, __amdgpu_buffer_rsrc_t la, uint32_t aoff, C kF, C k18, C& res) {
    constexpr int H1 = RF3 + 8, A1 = 8;  // first half: forcing terms, f~_1..f~_8; directions 1..8
    if (LOAD) {
        C h[H1], g[A1];
        ld_vec(rin, roff, h);
        ld_vec(la, aoff, g);
#pragma unroll
        for (int i = 0; i < H1; ++i) rec[i] = h[i];
#pragma unroll
        for (int i = 0; i < A1; ++i) ca[i] = g[i];
    }
    const C rho = rec[0] * kF, dux = rec[1], duy = rec[2], duz = rec[3];
    const C sx = rec[4], sy = rec[5], sz = rec[6], duu = rec[7];
    // each slot opp(j) is replaced at most once, and never one that a later eq. 16 link reads (its
    // x2 = x - e_j is fluid, while a replaced slot was pulled from a solid node)
    double ds = 0.0;
    auto link = [&](int j) {
        const C a = ca[j - 1];
        const bool lk = bnd && a < C(1.5);
        if (__builtin_amdgcn_ballot_w64(lk)) {
            const C c1 = a < C(0) ? -a : a, c2 = C(1) - c1;
            // eq. 13 term of direction j
            const C ed = edot3<C>(kEx3[j], kEy3[j], kEz3[j], dux, duy, duz);
            const C es = edot3<C>(kEx3[j], kEy3[j], kEz3[j], sx, sy, sz);
            const C Fj = w19<C>(j) * rho * (C(3) * ed + C(4.5) * ed * es - duu);
            const int jo = (j & 1) ? j + 1 : j - 1;  // opposite direction
            C o = a < C(0) ? rec[RF3 + jo - 1] : f[j];
            o = c2 != C(0) ? o : C(0);
            const C fin = Buf<S>::round(c1 * rec[RF3 + j - 1] + c2 * (o + Fj));
            ds += lk ? double(rec[RF3 + j - 1]) - double(fin) : 0.0;
            f[jo] = lk ? fin : f[jo];
        }
    };
#pragma unroll
    for (int j = 1; j <= A1; ++j) link(j);
    if (LOAD) {
        __builtin_amdgcn_sched_barrier(0);
        C h[RF3 + 18 - H1], g[18 - A1];
        ld_vec(rin, roff + uint32_t(H1 * sizeof(C)), h);
        ld_vec(la, aoff + uint32_t(A1 * sizeof(C)), g);
#pragma unroll
        for (int i = 0; i < RF3 + 18 - H1; ++i) rec[H1 + i] = h[i];
#pragma unroll
        for (int i = 0; i < 18 - A1; ++i) ca[A1 + i] = g[i];
    }
#pragma unroll
    for (int j = A1 + 1; j < 19; ++j) link(j);
    ds *= double(k18);
    const double f0 = double(f[0]) + ds;
    f[0] = C(f0);
    res = C(f0 - double(f[0]));
    return C(ds);
}

// the arguments of a step from fcur / rcur to fnext / rnext (the launch shape and rho are left to the launcher)
template <class S, class C>
Args3<S, C> args3(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext) {
    Args3<S, C> a;
    a.fa = static_cast<const S*>(fcur);
    a.fb = static_cast<S*>(fnext);
    a.tag = reinterpret_cast<const int32_t*>(c->lat + c->L.tag);
    a.nmask = reinterpret_cast<const uint32_t*>(c->lat + c->L.nmask);
    a.rho = nullptr;
    a.rin = static_cast<const C*>(rcur);
    a.rout = static_cast<C*>(rnext);
    a.la = reinterpret_cast<const C*>(c->lk + c->L.lk_a);
    a.flags = reinterpret_cast<int32_t*>(c->lat + c->L.flags);
    a.n_bnodes = uint32_t(c->n_bnodes > 0 ? c->n_bnodes : 0);
    a.nx = c->p.nx;
    a.ny = c->p.ny;
    a.nz = c->p.nz;
    a.D = a.ntx = a.nty = a.nblocks = 0;
    a.tau_inv = C(1.0 / c->p.tau);
    a.G = C(c->p.G);
    a.rho_ref = c->p.precision == MCB_F64 ? C(0) : C(c->p.rho_ref);
    a.kF = c->p.bc_mode == MCB_BC_PRESENT ? C(1) : C(0);
    a.k18 = c->p.bc_mode == MCB_BC_IBC ? C(0) : C(1);
    a.gx = C(c->p.gravity[0]);
    a.gy = C(c->p.gravity[1]);
    a.gz = C(c->p.gravity[2]);
    a.eos.RT = C(c->p.eos_R * c->p.eos_T);
    a.eos.a = C(c->p.eos_a);
    a.eos.b4 = C(c->p.eos_b / 4.0);
    a.eos.two_over_G = C(2.0 / c->p.G);
    return a;
}

}  // namespace
}  // namespace mcb
