// Device data and helpers of the reverse mode, shared by the loss kernels (adjoint.hip), the D2Q9 tile
// kernels (adjoint2d.hip) and the D3Q19 kernels (adjoint3d.hip).
#pragma once

#include "kernels_common.h"

namespace mcb {
namespace {

template <class C>
__device__ inline C wgt(int L, int i) {
    if (L == 0) return i == 0 ? C(4.0 / 9.0) : (i < 5 ? C(1.0 / 9.0) : C(1.0 / 36.0));
    return i == 0 ? C(1.0 / 3.0) : (i < 7 ? C(1.0 / 18.0) : C(1.0 / 36.0));
}
// interaction-force stencil weights, sum_i w^_i e_i e_i^T = I
__device__ inline double wforce(int L, int i) {
    if (L == 0) return i < 5 ? 1.0 / 3.0 : 1.0 / 12.0;
    return i < 7 ? 1.0 / 6.0 : 1.0 / 12.0;
}

// opposite direction, a compile-time constant inside unrolled loops (D2Q9 pairs 1-3, 2-4, 5-7, 6-8;
// D3Q19 pairs 2k-1, 2k)
template <int L>
__host__ __device__ constexpr int opp(int i) {
    return L == 0 ? (i == 0 ? 0 : (i < 5 ? (i + 1) % 4 + 1 : (i - 3) % 4 + 5)) : (i == 0 ? 0 : ((i & 1) ? i + 1 : i - 1));
}
static_assert(opp<0>(1) == 3 && opp<0>(2) == 4 && opp<0>(3) == 1 && opp<0>(4) == 2 && opp<0>(5) == 7 &&
                  opp<0>(6) == 8 && opp<0>(7) == 5 && opp<0>(8) == 6 && opp<0>(0) == 0,
              "D2Q9 opposites");
static_assert(opp<1>(1) == 2 && opp<1>(2) == 1 && opp<1>(17) == 18 && opp<1>(18) == 17 && opp<1>(0) == 0,
              "D3Q19 opposites");

struct AdjDev {
    GridDev g;
    int L;                       // 0: D2Q9, 1: D3Q19
    const int32_t* tag;          // node tags (see the step kernels)
    const uint32_t* nmask;       // 3-D link bits
    const double* phi;           // wettability factor per wall node
    uint32_t nb;                 // boundary nodes
    double tau, G, two_over_G, RT, a, b4, rho_ref;
    double kF, k18;              // boundary scheme: weights of the forcing term and of eq. 18
    double grav[3];              // body acceleration
    int mrt;                     // 1: K = M^-1 S M with msc[k] = s_k / |row k of M|^2 (D2Q9)
    double msc[9];
    // chemical-potential model (D2Q9): solid layers, eq. 12 and the Peng-Robinson potential
    int cp;
    const int8_t* layer;
    double k2, kappa, pRT, pb, pclog, paal;
};

// D2Q9 moment matrix of eq. 2 (rows rho, e, epsilon, j_x, q_x, j_y, q_y, p_xx, p_xy); its rows are
// orthogonal, so M^-1 = M^T diag(1 / |row k|^2)
__device__ constexpr int kM2[9][9] = {{1, 1, 1, 1, 1, 1, 1, 1, 1},     {-4, -1, -1, -1, -1, 2, 2, 2, 2},
                                      {4, -2, -2, -2, -2, 1, 1, 1, 1},  {0, 1, 0, -1, 0, 1, -1, -1, 1},
                                      {0, -2, 0, 2, 0, 1, -1, -1, 1},   {0, 0, 1, 0, -1, 1, 1, -1, -1},
                                      {0, 0, -2, 0, 2, 1, 1, -1, -1},   {0, 1, -1, 1, -1, 0, 0, 0, 0},
                                      {0, 0, 0, 0, 0, 1, -1, 1, -1}};

// link bits (bit j-1: x + e_j solid) of a fluid node
__device__ inline uint32_t link_bits(const AdjDev& A, int64_t x, int tg) {
    if (tg <= 0) return 0u;
    return A.L == 0 ? uint32_t(tg) & 0xFFu : A.nmask[x];
}

// psi(rho) = sqrt(2 (p - rho/3) / G), p the Carnahan-Starling pressure, and d psi / d rho
__device__ inline void psi_d(const AdjDev& A, double rho, double* psi, double* dpsi) {
    const double eta = rho * A.b4, i1 = 1.0 / (1.0 - eta), i3 = i1 * i1 * i1;
    const double h = (1.0 + eta + eta * eta - eta * eta * eta) * i3;
    const double dh = (1.0 + 2.0 * eta - 3.0 * eta * eta) * i3 + 3.0 * h * i1;
    const double p = rho * A.RT * h - A.a * rho * rho;
    const double dp = A.RT * (h + eta * dh) - 2.0 * A.a * rho;
    const double arg = (p - rho * (1.0 / 3.0)) * A.two_over_G;
    const double s = arg > 0.0 ? sqrt(arg) : 0.0;
    *psi = s;
    *dpsi = s > 0.0 ? (dp - 1.0 / 3.0) / (A.G * s) : 0.0;
}

template <class S>
__device__ inline double ldf(const S* g, const AdjDev& A, int i, int64_t x) {
    return double(ldp<S, float>(g, i, A.g.N, x)) + wgt<double>(A.L, i) * A.rho_ref;
}
template <>
__device__ inline double ldf<double>(const double* g, const AdjDev& A, int i, int64_t x) {
    return g[i * A.g.N + x] + wgt<double>(A.L, i) * A.rho_ref;
}

// the value at a byte offset below 4 GiB from a uniform base (the address is a scalar base and a 32-bit
// lane offset; an array of one double per node stays below 4 GiB, since a population lattice does)
template <class T>
__device__ __forceinline__ T ldo(const T* base, uint32_t off) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}
template <class T>
__device__ __forceinline__ void sto(T* base, uint32_t off, T v) {
    *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + off) = v;
}

AdjDev make_dev(const mcb_ctx* c) {
    AdjDev A;
    A.g = c->g;
    A.L = c->g.dim == 2 ? 0 : 1;
    A.tag = reinterpret_cast<const int32_t*>(c->lat + c->L.tag);
    A.nmask = reinterpret_cast<const uint32_t*>(c->lat + c->L.nmask);
    A.phi = reinterpret_cast<const double*>(c->lk + c->L.wl_phi);
    A.nb = uint32_t(c->n_bnodes > 0 ? c->n_bnodes : 0);
    A.tau = c->p.tau;
    A.G = c->p.G;
    A.two_over_G = 2.0 / c->p.G;
    A.RT = c->p.eos_R * c->p.eos_T;
    A.a = c->p.eos_a;
    A.b4 = c->p.eos_b / 4.0;
    A.rho_ref = c->p.precision == MCB_F64 ? 0.0 : c->p.rho_ref;
    A.kF = c->p.bc_mode == MCB_BC_PRESENT ? 1.0 : 0.0;
    A.k18 = c->p.bc_mode == MCB_BC_IBC ? 0.0 : 1.0;
    for (int k = 0; k < 3; ++k) A.grav[k] = c->p.gravity[k];
    A.mrt = c->p.collision == MCB_COLL_MRT ? 1 : 0;
    const double sn = 1.0 / c->p.tau;
    const double rate[9] = {1.0, c->p.s_e, c->p.s_eps, 1.0, c->p.s_q, 1.0, c->p.s_q, sn, sn};
    const double norm[9] = {9.0, 36.0, 36.0, 6.0, 12.0, 6.0, 12.0, 4.0, 4.0};
    for (int k = 0; k < 9; ++k) A.msc[k] = rate[k] / norm[k];
    A.cp = c->p.model == MCB_MODEL_CHEMPOT ? 1 : 0;
    A.layer = reinterpret_cast<const int8_t*>(c->lat + c->L.cp_layer);
    A.k2 = c->p.cp_k * c->p.cp_k;
    A.kappa = c->p.cp_kappa;
    A.pRT = c->p.eos_R * c->p.eos_T;
    A.pb = c->p.eos_b;
    A.paal = A.cp ? pr_aalpha(c->p.eos_a, c->p.eos_b, c->p.eos_R, c->p.eos_T, c->p.pr_omega) : 0.0;
    A.pclog = A.paal / (2.0 * std::sqrt(2.0) * c->p.eos_b);
    return A;
}

}  // namespace
}  // namespace mcb
