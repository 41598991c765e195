// D3Q19 step, FP64 and FP32 storage, in three kernels without LDS, barriers or marches: the density and
// psi of every node (k_rho3f), psi of the wall nodes from their list (k_psi3w, eq. 15), and the
// collision (k_collide3f), which reads psi of the eighteen neighbours through the caches.  One lane per
// node, consecutive nodes of the lattice whatever the row length.
//
// Why.  The plane march that FP16 storage keeps (step3d.hip) recomputes psi of a 34 x 10 region per
// 32 x 8 tile and marches along z, which ties its speed to the iteration count, leaves ragged boxes with
// part-empty tiles and small ones with a handful of waves.  Storing psi costs one value written and,
// through the caches, about one read per node (of 19 + 19 populations), and makes every node independent:
// the collision runs at the rate of its streams.  Time per step against the march: 32^3 FP32 27 -> 13.5
// us, 97 x 75 x 130 FP64 156 -> 99, 180 x 190 x 170 FP32 513 -> 313, 256^3 FP32 904 -> 860 (the density
// pass 287 us, 5.0 TB/s; the collision 571 us, 4.8 TB/s; the walls 19 us; a plain D3Q19 pull of the same
// lattice reaches 5.5-5.8 TB/s), 256^3 FP64 1831 -> 1775.
//
// Measured and not taken: each XCD on a contiguous eighth of the lattice (256^3 FP32 878-910 us);
// registers bounded to six and eight waves per SIMD instead of five (spills: 910 and 1075 us).
#include "step3d_node.h"

namespace mcb {
namespace {

constexpr int NT = 256;

template <class S, class C>
struct Flat3 {
    Args3<S, C> a;
    C* rho;            // density of boundary nodes, 0 on solid ones (not written elsewhere)
    C* psi;            // pseudopotential of fluid and wall nodes, 0 on other solid ones
    const C* fac;      // eq. 15 factor per wall node
    const int32_t* wl_node;
    int64_t n_wall;
};

template <class S, class C, bool PULL, bool IBC>
__global__ __launch_bounds__(NT) void k_rho3f(Flat3<S, C> p) {
    const Args3<S, C>& a = p.a;
    constexpr uint32_t s = sizeof(S);
    const uint32_t N = uint32_t(a.nx) * uint32_t(a.ny) * uint32_t(a.nz), ns = N * s;
    const __amdgpu_buffer_rsrc_t fa = make_res(a.fa, uint64_t(19) * ns);
    const Node3 q = node3<NT>(a.nx, a.ny, a.nz);
    const int tg = a.tag[q.node];
    uint32_t off[19];
    neighbours<S>(q, a.nx, a.ny, a.nz, off);
    C f[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) f[i] = Buf<S>::ld(fa, off[PULL ? opp3(i) : 0], uint32_t(i) * ns);
    C rs = C(0);
#pragma unroll
    for (int i = 0; i < 19; ++i) rs += f[i];
    if (PULL && tg > 0) {
        const C* rec = a.rin + size_t(tg - 1) * REC3;
        if (!IBC) {
            // boundary node: its own f~_j(x, t) on each link (the slot pulled from the solid node holds 0)
            rs += rec[RF3 + 18];
        } else {
            // IBC (no forcing term, no eq. 18): the f_in of each link j, which replaces the zero
            // pulled into slot opp(j) -- eq. 16 from the value pulled from x2 into slot j, eq. 17
            // from the node's own opposite population
            const C* ca = a.la + size_t(tg - 1) * Q3_LINKS;
#pragma unroll
            for (int j = 1; j < 19; ++j) {
                const C c = ca[j - 1];
                const C c1 = c < C(0) ? -c : c, c2 = C(1) - c1;
                C o = c < C(0) ? rec[RF3 + opp3(j) - 1] : f[j];
                o = c2 != C(0) ? o : C(0);
                rs += c < C(1.5) ? Buf<S>::round(c1 * rec[RF3 + j - 1] + c2 * o) : C(0);
            }
        }
    }
    if (!q.on) return;
    bool bad = false;
    const C r = tg >= 0 ? rs + a.rho_ref : C(0);
    // the wall nodes' psi reads the density of boundary nodes and of solid ones only
    if (tg != 0) p.rho[q.node] = r;
    p.psi[q.node] = tg >= 0 ? psi_val(r, a.eos, &bad) : C(0);
    raise_domain(bad, a.flags);
}

template <class S, class C>
__global__ __launch_bounds__(NT) void k_psi3w(Flat3<S, C> p) {
    const Args3<S, C>& a = p.a;
    const int64_t w = int64_t(blockIdx.x) * NT + threadIdx.x;
    if (w >= p.n_wall) return;
    const uint32_t x = uint32_t(p.wl_node[w]), nx = uint32_t(a.nx), nxy = nx * uint32_t(a.ny);
    Node3 q;
    q.node = x;
    q.on = true;
    q.z = int(x / nxy);
    q.y = int((x - uint32_t(q.z) * nxy) / nx);
    q.x = int(x - uint32_t(q.z) * nxy - uint32_t(q.y) * nx);
    uint32_t off[19];
    neighbours<C>(q, a.nx, a.ny, a.nz, off);
    const __amdgpu_buffer_rsrc_t rr = make_res(p.rho, uint64_t(nxy) * a.nz * sizeof(C));
    C v[19];
#pragma unroll
    for (int i = 1; i < 19; ++i) v[i] = Buf<C>::ld(rr, off[i]);
    C num = C(0);
#pragma unroll
    for (int i = 1; i < 19; ++i) num += w19<C>(i) * v[i];
    bool bad = false;
    p.psi[x] = psi_val(p.fac[w] * num, a.eos, &bad);
    raise_domain(bad, a.flags);
}

template <class S, class C, bool PULL>
__global__ __launch_bounds__(NT, sizeof(C) == 8 ? 2 : 4) void k_collide3f(Flat3<S, C> p) {
    const Args3<S, C>& a = p.a;
    constexpr uint32_t s = sizeof(S), sc = sizeof(C);
    static_assert(s == sc, "one set of neighbour offsets serves populations and psi");
    const uint32_t N = uint32_t(a.nx) * uint32_t(a.ny) * uint32_t(a.nz), ns = N * s;
    const __amdgpu_buffer_rsrc_t fa = make_res(a.fa, uint64_t(19) * ns), fb = make_res(a.fb, uint64_t(19) * ns);
    const __amdgpu_buffer_rsrc_t rpsi = make_res(p.psi, uint64_t(N) * sc);
    const __amdgpu_buffer_rsrc_t rin = make_res(a.rin, uint64_t(a.n_bnodes) * REC3 * sc);
    const __amdgpu_buffer_rsrc_t rout = make_res(a.rout, uint64_t(a.n_bnodes) * REC3 * sc);
    const __amdgpu_buffer_rsrc_t rla = make_res(a.la, uint64_t(a.n_bnodes) * Q3_LINKS * sc);
    const Node3 q = node3<NT>(a.nx, a.ny, a.nz);
    const int tg = a.tag[q.node];
    uint32_t off[19];
    neighbours<S>(q, a.nx, a.ny, a.nz, off);
    C f[19], ps[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) f[i] = Buf<S>::ld(fa, off[PULL ? opp3(i) : 0], uint32_t(i) * ns);
#pragma unroll
    for (int i = 0; i < 19; ++i) ps[i] = Buf<C>::ld(rpsi, off[i]);
    const bool coll = q.on && tg >= 0;
    C ds = C(0), er = C(0);
    if (PULL && __any(tg > 0)) {
        const uint32_t bi = uint32_t(tg - 1);
        C rec[RF3 + 18], ca[18];
        ds = apply_links3<S, C, true>(tg > 0, rec, ca, f, rin, tg > 0 ? bi * (REC3 * sc) : OOB, rla,
                                      tg > 0 ? bi * (Q3_LINKS * sc) : OOB, a.kF, a.k18, er);
    }
    // the node's density at t+1 from its pulled values; the collision hands all of it back, with f_0
    // taking the rounding
    MassAcc<S, C> rs_acc = MassAcc<S, C>(er);
#pragma unroll
    for (int i = 0; i < 19; ++i) rs_acc += MassAcc<S, C>(f[i]);
    const C rs = C(rs_acc);
    // F = -G psi(x) sum_i w^_i psi(x + e_i) e_i, w^ = 1/6 (axes), 1/12 (edges)
    const C gp = -a.G * ps[0];
    const C exy1 = ps[7] - ps[8], exy2 = ps[9] - ps[10], exz1 = ps[11] - ps[12], exz2 = ps[13] - ps[14];
    const C eyz1 = ps[15] - ps[16], eyz2 = ps[17] - ps[18];
    const C Fx = gp * (C(1.0 / 6.0) * (ps[1] - ps[2]) + C(1.0 / 12.0) * (exy1 + exy2 + exz1 + exz2));
    const C Fy = gp * (C(1.0 / 6.0) * (ps[3] - ps[4]) + C(1.0 / 12.0) * (exy1 - exy2 + eyz1 + eyz2));
    const C Fz = gp * (C(1.0 / 6.0) * (ps[5] - ps[6]) + C(1.0 / 12.0) * (exz1 - exz2 + eyz1 - eyz2));
    const C rho = rs + a.rho_ref;
    const C irho = rcp(coll ? rho : C(1));
    const C jx = (f[1] - f[2]) + (f[7] - f[8]) + (f[9] - f[10]) + (f[11] - f[12]) + (f[13] - f[14]);
    const C jy = (f[3] - f[4]) + (f[7] - f[8]) - (f[9] - f[10]) + (f[15] - f[16]) + (f[17] - f[18]);
    const C jz = (f[5] - f[6]) + (f[11] - f[12]) - (f[13] - f[14]) + (f[15] - f[16]) - (f[17] - f[18]);
    const C ux = jx * irho, uy = jy * irho, uz = jz * irho;
    const C dux = Fx * irho + a.gx, duy = Fy * irho + a.gy, duz = Fz * irho + a.gz;
    const C ti = a.tau_inv, omc = C(1) - ti;
    // per direction: out_i = f_i (1 - 1/tau) + w_i [rs/tau + rho (sym_i +- anti_i)] with
    //   sym  = (4.5 (e.u)^2 - 1.5 u^2) / tau + 4.5 (e.du)(e.(2u + du)) - 1.5 du.(2u + du)
    //   anti = 3 (e.u / tau + e.du)
    // (eq. 14 equilibrium, eq. 13 forcing term, eq. 4 with S = I / tau)
    const C uu15 = C(1.5) * (ux * ux + uy * uy + uz * uz);
    const C sx2 = C(2) * ux + dux, sy2 = C(2) * uy + duy, sz2 = C(2) * uz + duz;
    const C duu15 = C(1.5) * (dux * sx2 + duy * sy2 + duz * sz2);
    const C c0 = -(ti * uu15 + duu15);
    const C trs = ti * rs;
    C out[19];
    auto pair = [&](int ip, int im, C w, C eu, C ed, C es) {
        const C sym = ti * C(4.5) * eu * eu + C(4.5) * ed * es + c0;
        const C anti = C(3) * (ti * eu + ed);
        const C base = w * (trs + rho * sym);
        const C wra = w * rho * anti;
        out[ip] = f[ip] * omc + base + wra;
        out[im] = f[im] * omc + base - wra;
    };
    constexpr C wa = C(1.0 / 18.0), we = C(1.0 / 36.0);
    pair(1, 2, wa, ux, dux, sx2);
    pair(3, 4, wa, uy, duy, sy2);
    pair(5, 6, wa, uz, duz, sz2);
    pair(7, 8, we, ux + uy, dux + duy, sx2 + sy2);
    pair(9, 10, we, ux - uy, dux - duy, sx2 - sy2);
    pair(11, 12, we, ux + uz, dux + duz, sx2 + sz2);
    pair(13, 14, we, ux - uz, dux - duz, sx2 - sz2);
    pair(15, 16, we, uy + uz, duy + duz, sy2 + sz2);
    pair(17, 18, we, uy - uz, duy - duz, sy2 - sz2);
    // the collision conserves mass: f_0 is the density minus the other outputs as stored
    MassAcc<S, C> rest = 0;
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        out[i] = Buf<S>::round(out[i]);
        rest += MassAcc<S, C>(out[i]);
    }
    out[0] = C(rs_acc - rest);
    // solid nodes store zeros (the density pass and the links read 0 from them)
    const uint32_t xst = q.on ? q.node * s : OOB;
#pragma unroll
    for (int i = 0; i < 19; ++i) Buf<S>::st_nt(fb, sat_add(xst, uint32_t(i) * ns), coll ? out[i] : C(0));
    // boundary record of time t+1
    if (__any(coll && tg > 0)) {
        const uint32_t mk = tg > 0 ? a.nmask[q.node] : 0u;
        C rv[REC3];
        rv[0] = rho;
        rv[1] = dux;
        rv[2] = duy;
        rv[3] = duz;
        rv[4] = sx2;
        rv[5] = sy2;
        rv[6] = sz2;
        rv[7] = duu15;
#pragma unroll
        for (int i = 1; i < 19; ++i) rv[RF3 + i - 1] = out[i];  // rounded to the storage format above
        // the node's own populations on its links, for the density pass of the next step
        C sl = C(0);
#pragma unroll
        for (int j = 1; j < 19; ++j) sl += ((mk >> (j - 1)) & 1u) ? out[j] : C(0);
        rv[RF3 + 18] = sl;
        rv[RF3 + 19] = ds;
        st_vec(rout, (coll && tg > 0) ? uint32_t(tg - 1) * (REC3 * sc) : OOB, rv);
    }
}

template <class S, class C>
hipError_t flat_t(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    Flat3<S, C> p;
    p.a = args3<S, C>(c, fcur, rcur, fnext, rnext);
    p.rho = reinterpret_cast<C*>(c->lat + c->L.rho3);
    p.psi = reinterpret_cast<C*>(c->lat + c->L.scratch);  // free between the calls that stage host data in it
    p.fac = reinterpret_cast<const C*>(c->lk + c->L.wl_fac);
    p.wl_node = reinterpret_cast<const int32_t*>(c->lk + c->L.wl_node);
    p.n_wall = c->n_wall > 0 ? c->n_wall : 0;
    const bool ibc = c->p.bc_mode == MCB_BC_IBC;
    const dim3 grid(unsigned((c->g.N + NT - 1) / NT)), blk(NT);
    hipLaunchKernelGGL((!pull ? k_rho3f<S, C, false, false> : (ibc ? k_rho3f<S, C, true, true> : k_rho3f<S, C, true, false>)),
                       grid, blk, 0, c->stream, p);
    if (p.n_wall > 0)
        hipLaunchKernelGGL((k_psi3w<S, C>), dim3(unsigned((p.n_wall + NT - 1) / NT)), blk, 0, c->stream, p);
    hipLaunchKernelGGL((pull ? k_collide3f<S, C, true> : k_collide3f<S, C, false>), grid, blk, 0, c->stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t flat3d(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    return c->p.precision == MCB_F64 ? flat_t<double, double>(c, fcur, rcur, fnext, rnext, pull)
                                     : flat_t<float, float>(c, fcur, rcur, fnext, rnext, pull);
}

}  // namespace mcb
