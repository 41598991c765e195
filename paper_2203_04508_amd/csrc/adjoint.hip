// Reverse mode of the step: the hand-written discrete adjoint of the map from the post-collision
// state of time t to that of time t+1, and of the first collision from the equilibrium start.
// Together with checkpointed recomputation of the forward states (api layer) it gives the exact
// gradient (to rounding) of a loss of the final state with respect to the wettability of every wall
// node: the factor phi (pseudopotential model) or the assigned chemical potential (chemical-potential
// model).
//
// State.  The forward step reads, besides the populations g(t), the forcing term F_j(x, t) of
// eq. 13 on every fluid-solid link (eqs. 16-17 use it one step later), so the state is the pair
// (g, R) with R the per-link forcing terms; its adjoint is (lambda, lambda_R).  The step keeps
// the forcing terms of each boundary node in its boundary record (rho and du = F / rho among them);
// the reverse sweep takes F = rho du from the record of each state and recomputes R from F and the
// node's own populations.
//
// Forward step, per fluid node x (f = g + w rho_ref in the shifted storages):
//   streaming, eq. 5:     p_i(x) = f_i(x - e_i)                           (x - e_i fluid)
//   link (x, j), i = opp j: p_i(x) = B_j = c1 f_j(x) + c2 o + c3 R_j(x)     (eqs. 16-17)
//        eq. 16: c1 = 2q, c2 = c3 = 1 - 2q, o = f_j(x - e_j); bounce-back: c1 = 1, c2 = c3 = 0;
//        eq. 17: c1 = 1/(2q), c2 = c3 = 1 - 1/(2q), o = f_opp(j)(x)
//   eq. 18:               p_0(x) += sum_links (f_j(x) - B_j)
//   the comparison schemes weight the forcing term R by kF and the eq. 18 sum by k18 (0 or 1)
//   collision, with E_i(rho, m) = w_i (rho + 3 e_i.m + (4.5 (e_i.m)^2 - 1.5 m.m) / rho), the
//   equilibrium of eq. 14 written with the momentum m = rho u, and K = M^-1 S M (eqs. 1-4; BGK:
//   K = I / tau):
//        g' = (I - K) p + (K - I) E(rho, j) + E(rho, j + F),   R'_i = E_i(rho, j + F) - E_i(rho, j)
//   (the MRT equilibria are M E(rho, j)), rho = sum p, j = sum p e, F = -G psi(x) sum_k w^_k
//   psi(x + e_k) e_k + rho g, psi = psi(rho) on fluid nodes and psi(phi_s rho_ave(s)) on wall
//   nodes s, rho_ave the eq. 15 weighted mean of the fluid neighbours' densities.
// The kernels apply the transposes of these maps in reverse order; every scatter of the
// forward map becomes a gather, so each output is written by exactly one thread and the result is
// deterministic.  adjoint2d.hip holds them for D2Q9 (two tile kernels for each of the two models),
// adjoint3d.hip for D3Q19; this file holds the losses.
#include "adjoint_dev.h"

namespace mcb {
namespace {

// ---- loss of the final state: deterministic two-pass reduction, then its gradient
__device__ inline double wave_sum(double v) {
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

template <class S>
__device__ inline double node_rho(const AdjDev& A, const S* g, int64_t x) {
    double r = 0.0;
    for (int i = 0; i < A.g.Q; ++i) r += ldf<S>(g, A, i, x);
    return r;
}

__device__ inline double link_len(int L, int j) {
    const int n2 = c_ex[L][j] * c_ex[L][j] + c_ey[L][j] * c_ey[L][j] + c_ez[L][j] * c_ez[L][j];
    return n2 == 1 ? 1.0 : (n2 == 2 ? 1.4142135623730951 : 1.7320508075688772);
}

template <class S>
__global__ __launch_bounds__(256) void k_loss_partial(AdjDev A, const S* __restrict__ g, int kind, double p0, double p1,
                                                      double* __restrict__ part) {
    double a = 0.0, b = 0.0;
    for (int64_t x = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; x < A.g.N; x += int64_t(gridDim.x) * blockDim.x) {
        const int tg = A.tag[x];
        if (tg < 0) continue;
        const double r = node_rho<S>(A, g, x);
        if (kind == 0) {
            a += double(x % A.g.nx) * (r - p0);
            b += r - p0;
        } else if (kind == 1) {
            const uint32_t m = link_bits(A, x, tg);
            for (int j = 1; j < A.g.Q; ++j)
                if ((m >> (j - 1)) & 1u) a += link_len(A.L, j) * 0.5 * (1.0 + tanh((r - p0) / p1));
        } else {
            a += r;
        }
    }
    __shared__ double sa[4], sb[4];
    a = wave_sum(a);
    b = wave_sum(b);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sa[w] = a;
        sb[w] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        part[blockIdx.x] = sa[0] + sa[1] + sa[2] + sa[3];
        part[gridDim.x + blockIdx.x] = sb[0] + sb[1] + sb[2] + sb[3];
    }
}

__global__ __launch_bounds__(256) void k_loss_final(const double* __restrict__ part, int n, double* __restrict__ out) {
    __shared__ double sa[4], sb[4];
    double a = 0.0, b = 0.0;
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        a += part[k];
        b += part[n + k];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sa[w] = a;
        sb[w] = b;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        out[0] = sa[0] + sa[1] + sa[2] + sa[3];
        out[1] = sb[0] + sb[1] + sb[2] + sb[3];
    }
}

// lambda(T) = dloss * d loss / d g(T) (every population of a node enters through its density);
// lambda_R(T) = 0.  sums = {a, b} of the reduction (kind 0: loss = a / b).
template <class S>
__global__ void k_loss_grad(AdjDev A, const S* __restrict__ g, int kind, double p0, double p1, const double* __restrict__ sums,
                            double dloss, double* __restrict__ lam) {
    const int64_t N = A.g.N;
    for (int64_t x = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; x < N; x += int64_t(gridDim.x) * blockDim.x) {
        const int tg = A.tag[x];
        double d = 0.0;
        if (tg >= 0) {
            if (kind == 0) {
                d = (double(x % A.g.nx) - sums[0] / sums[1]) / sums[1];
            } else if (kind == 1) {
                const double th = tanh((node_rho<S>(A, g, x) - p0) / p1);
                const uint32_t m = link_bits(A, x, tg);
                for (int j = 1; j < A.g.Q; ++j)
                    if ((m >> (j - 1)) & 1u) d += link_len(A.L, j) * 0.5 * (1.0 - th * th) / p1;
            } else {
                d = 1.0;
            }
        }
        for (int i = 0; i < A.g.Q; ++i) lam[i * N + x] = dloss * d;
    }
}

inline unsigned grid_for(int64_t n) {
    int64_t b = (n + 255) / 256;
    if (b > 8192) b = 8192;
    return unsigned(b < 1 ? 1 : b);
}

template <class S>
hipError_t adj_loss_t(mcb_ctx* c, const AdjWork& w, const void* g, int kind, const double* prm, double dloss, double* lam) {
    const AdjDev A = make_dev(c);
    hipLaunchKernelGGL((k_loss_partial<S>), dim3(MON_BLOCKS), dim3(256), 0, c->stream, A, static_cast<const S*>(g), kind, prm[0],
                       prm[1], w.part);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, c->stream, w.part, MON_BLOCKS, w.sums);
    if (lam)
        hipLaunchKernelGGL((k_loss_grad<S>), dim3(grid_for(c->g.N)), dim3(256), 0, c->stream, A, static_cast<const S*>(g), kind,
                           prm[0], prm[1], w.sums, dloss, lam);
    return hipGetLastError();
}

}  // namespace

hipError_t adj_step(mcb_ctx* c, const AdjWork& w, const void* gt, const void* rec, int pull, const double* lam1,
                    const double* lamR1, double* lam0, double* lamR0) {
    return c->g.dim == 2 ? adj_step2d(c, w, gt, rec, pull, lam1, lamR1, lam0, lamR0)
                         : adj_step3d(c, w, gt, rec, pull, lam1, lamR1, lam0, lamR0);
}

hipError_t adj_loss(mcb_ctx* c, const AdjWork& w, const void* g, int kind, const double* prm, double dloss, double* lam) {
    switch (c->p.precision) {
        case MCB_F64: return adj_loss_t<double>(c, w, g, kind, prm, dloss, lam);
        case MCB_F32S: return adj_loss_t<float>(c, w, g, kind, prm, dloss, lam);
        default: return adj_loss_t<__half>(c, w, g, kind, prm, dloss, lam);
    }
}

}  // namespace mcb
