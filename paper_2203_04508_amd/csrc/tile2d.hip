// D2Q9 step of small and middle-sized lattices: one workgroup computes one tile of the new state
// (the same per-node arithmetic as the row marches of step2d.hip, which large lattices take).
#include "step2d_node.h"

namespace mcb {
namespace {

// Offset, in a population plane, of the node that population i of node (cx, cy) is pulled from, from
// the three columns and three rows around it.
template <class S>
struct Around {
    uint32_t x[3], y[3];  // byte offsets of columns x + 1, x, x - 1 and of rows y + 1, y, y - 1: index e + 1
};

template <class S>
__device__ __forceinline__ Around<S> around(int cx, int cy, int nx, int ny) {
    constexpr uint32_t s = sizeof(S);
    const uint32_t row = uint32_t(nx) * s;
    return {{uint32_t(cx == nx - 1 ? 0 : cx + 1) * s, uint32_t(cx) * s, uint32_t(cx == 0 ? nx - 1 : cx - 1) * s},
            {uint32_t(cy == ny - 1 ? 0 : cy + 1) * row, uint32_t(cy) * row, uint32_t(cy == 0 ? ny - 1 : cy - 1) * row}};
}

// Issue the loads of the nine populations arriving at a node (eq. 5; PULL = false: its own).
template <class S, class C, bool PULL>
__device__ __forceinline__ void pull_at(__amdgpu_buffer_rsrc_t fa, uint32_t ns, const Around<S>& A, C (&f)[9]) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const uint32_t o = PULL ? A.x[kEx[i] + 1] + A.y[kEy[i] + 1] : A.x[1] + A.y[1];
        if (kMixed<S> && i == 0)
            f[0] = Buf<float>::ld(fa, o * 2u);  // FP16 storage: the rest population in FP32
        else
            f[i] = Buf<S>::ld(fa, o, uint32_t(i + (kMixed<S> ? 1 : 0)) * ns);
    }
}

// periodic image of a coordinate v >= -2 (m >= 3; one subtraction unless the box is smaller than a tile)
__device__ __forceinline__ int image(int v, int m) {
    v = v < 0 ? v + m : v;
    while (v >= m) v -= m;
    return v;
}

// ---------------------------------------------------------------- pseudopotential model
// A workgroup of NT lanes owns a tile of TX x TY nodes, TY = RPL NT / TX; lane t owns column t % TX
// of rows t / TX + r NT / TX.  Three phases, two barriers:
//   1  every lane pulls its own nodes and up to NRL nodes of the ring two nodes wide around the tile
//      (psi of the ring next to the tile needs, through the wall nodes, the density two nodes out),
//      applies eqs. 16-18 to its own, and puts the densities of the (TX + 4) x (TY + 4) region in LDS: a wall
//      node's entry is minus its eq. 15 factor, any other solid node's is zero;
//   2  psi of the (TX + 2) x (TY + 2) region, wall nodes from the entries around them (eq. 15);
//   3  force, collision, store and boundary record of the own nodes, whose populations stayed in
//      registers.
// Why tiles here: a march gives a workgroup one row at a time, a serial chain of about 2 us per row on
// a box that leaves most of the chip idle; a tile runs its whole chain once (one round of loads,
// then the loads that depend on the tags, and two barriers).  Time per step, one-wave row march against
// tiles: 64^2 FP64 24.5 -> 5.3 us, 512^2 FP32 20.3 -> 8.6, 1024^2 FP32 32.6 -> 20.8 (3.6 TB/s of populations),
// FP64 61.6 -> 35.6 (4.3 TB/s), 1531 x 1021 FP64 81 -> 49.  About 16 rounds of 550 vector instructions
// per SIMD make up two thirds of the 1024^2 FP32 time.
// Every node past the box's edge is its periodic image, so partial tiles need no cases of their own:
// they only do not store.
// WPE: waves per SIMD the registers are bounded to.
template <class S, class C, int TX, int NT, int RPL, int WPE, bool PULL, bool MRT>
__global__ __launch_bounds__(NT, WPE) void k_tile2d(Args2<S, C> a) {
    constexpr int LY = NT / TX, TY = LY * RPL;
    constexpr int RX = TX + 4, RY = TY + 4, PX = TX + 2, PY = TY + 2;
    constexpr int NRING = RX * RY - TX * TY, NRL = (NRING + NT - 1) / NT;
    constexpr int NP = PX * PY, NPL = (NP + NT - 1) / NT;
    constexpr uint32_t s = sizeof(S), sc = sizeof(C), P0 = kMixed<S> ? 1 : 0;
    __shared__ C s_rho[RY * RX];
    __shared__ C s_psi[PY * PX];
    // XCD-aware order: consecutive tiles go to the same XCD (one L2)
    const int bid = blockIdx.x;
    const int per = a.nblocks >> 3, rem = a.nblocks & 7;
    const int xcd = bid & 7, k8 = bid >> 3;
    const int logical = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k8;
    const int x0 = (logical % a.nsx) * TX, y0 = (logical / a.nsx) * TY;
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = a.nx, ny = a.ny;
    const uint32_t n = uint32_t(nx) * uint32_t(ny), ns = n * s;
    const __amdgpu_buffer_rsrc_t rfa = make_res(a.fa, uint64_t(9 + P0) * ns);
    const __amdgpu_buffer_rsrc_t rfb = make_res(a.fb, uint64_t(9 + P0) * ns);
    const __amdgpu_buffer_rsrc_t rtag = make_res(a.tag, uint64_t(n) * 4);
    const __amdgpu_buffer_rsrc_t rin = make_res(a.rin, uint64_t(a.n_bnodes) * REC2 * sc);
    const __amdgpu_buffer_rsrc_t rout = make_res(a.rout, uint64_t(a.n_bnodes) * REC2 * sc);
    const __amdgpu_buffer_rsrc_t rla = make_res(a.la, uint64_t(a.n_bnodes) * Q2_LINKS * sc);
    const __amdgpu_buffer_rsrc_t rfac = make_res(a.fac, uint64_t(a.n_wall) * sc);
    // the density of a boundary node where eq. 18 applies: f_in enters its sum once and is subtracted
    // once from f_0, which leaves the node's own populations on its links; its record holds their sum
    const bool link_sum = PULL && a.k18 != C(0);
    bool bad = false;

    // ---- 1: tags first, then the populations (the loads that depend on a tag follow both)
    int tg[RPL], tgr[NRL], pr[NRL];  // tags of the own and ring nodes, region entry of the ring nodes
    C f[RPL][9], fr[NRL][9];
    Around<S> own[RPL], rng[NRL];
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const int cx = image(x0 + lx, nx), cy = image(y0 + ly + r * LY, ny);
        own[r] = around<S>(cx, cy, nx, ny);
        tg[r] = ld_i32(rtag, (uint32_t(cy) * uint32_t(nx) + uint32_t(cx)) * 4u);
    }
#pragma unroll
    for (int h = 0; h < NRL; ++h) {
        // ring entries: two rows below, two above, then two columns on either side of each tile row;
        // lanes past the last entry repeat it
        const int j = min(t + h * NT, NRING - 1), q = j - 4 * RX;
        const int ry = j < 4 * RX ? (j < 2 * RX ? j / RX : TY + j / RX) : q / 4 + 2;
        const int rx = j < 4 * RX ? j % RX : ((q & 3) < 2 ? (q & 3) : TX + (q & 3));
        pr[h] = ry * RX + rx;
        const int cx = image(x0 - 2 + rx, nx), cy = image(y0 - 2 + ry, ny);
        rng[h] = around<S>(cx, cy, nx, ny);
        tgr[h] = ld_i32(rtag, (uint32_t(cy) * uint32_t(nx) + uint32_t(cx)) * 4u);
    }
#pragma unroll
    for (int r = 0; r < RPL; ++r) pull_at<S, C, PULL>(rfa, ns, own[r], f[r]);
#pragma unroll
    for (int h = 0; h < NRL; ++h) pull_at<S, C, PULL>(rfa, ns, rng[h], fr[h]);
    C ds[RPL], er[RPL];
    auto sum9 = [](const C (&v)[9]) {
        C sr = C(0);
#pragma unroll
        for (int i = 0; i < 9; ++i) sr += v[i];
        return sr;
    };
    // eqs. 16-18 on the pulled populations v of a boundary node (g > 0); returns its link sum
    auto links = [&](int g, C (&v)[9], C& d, C& e) {
        C rec[RF2 + 9], head[RF2 + 8], ca[Q2_LINKS];
        const uint32_t bi = uint32_t(g >> 8);
        ld_vec(rin, g > 0 ? bi * (REC2 * sc) : OOB, rec);
        ld_vec(rla, g > 0 ? bi * (Q2_LINKS * sc) : OOB, ca);
#pragma unroll
        for (int i = 0; i < RF2 + 8; ++i) head[i] = rec[i];
        d = apply_links<S, C>(g > 0, head, ca, v, a.kF, a.k18, e);
        return rec[RF2 + 8];
    };
    auto put = [&](int at, int g, C sr) {
        const C fac = Buf<C>::ld(rfac, g <= -2 ? uint32_t(-g - 2) * sc : OOB);
        const C rho = sr + a.rho_ref;
        if (!(g >= 0 ? rho > C(0) : (g == -1 || fac > C(0)))) bad = true;  // the signs carry meaning below
        s_rho[at] = g >= 0 ? rho : (g == -1 ? C(0) : -fac);
    };
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        C sr = sum9(f[r]);
        ds[r] = er[r] = C(0);
        if (PULL && __any(tg[r] > 0)) {
            const C ls = links(tg[r], f[r], ds[r], er[r]);
            sr = link_sum ? sr + (tg[r] > 0 ? ls : C(0)) : sum9(f[r]);
        }
        put((ly + r * LY + 2) * RX + lx + 2, tg[r], sr);
    }
#pragma unroll
    for (int h = 0; h < NRL; ++h) {
        if (link_sum) {
            const C ls = Buf<C>::ld(rin, tgr[h] > 0 ? uint32_t(tgr[h] >> 8) * (REC2 * sc) + (RF2 + 8) * sc : OOB);
            put(pr[h], tgr[h], sum9(fr[h]) + ls);
        } else {
            C d, e;
            if (PULL && __any(tgr[h] > 0)) links(tgr[h], fr[h], d, e);
            put(pr[h], tgr[h], sum9(fr[h]));
        }
    }
    __syncthreads();

    // ---- 2: psi
#pragma unroll
    for (int h = 0; h < NPL; ++h) {
        const int j = t + h * NT;
        if (j < NP) {
            const int c = (j / PX + 1) * RX + j % PX + 1;
            const C rc = s_rho[c];
            C rn = rc;
            if (rc < C(0)) {
                // wall node: the weighted sum of its fluid neighbours' densities times the factor
                C num = C(0);
#pragma unroll
                for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
                    for (int dx = -1; dx <= 1; ++dx) {
                        if (dx == 0 && dy == 0) continue;
                        const C w = (dx == 0 || dy == 0) ? C(1.0 / 9.0) : C(1.0 / 36.0);
                        const C v = s_rho[c + dy * RX + dx];
                        num += w * (v > C(0) ? v : C(0));
                    }
                rn = -rc * num;
            }
            s_psi[j] = rc == C(0) ? C(0) : psi_val(rn, a.eos, &bad);
        }
    }
    __syncthreads();

    // ---- 3: force, collision, store
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        const bool out_node = x0 + lx < nx && y0 + ly + r * LY < ny;
        const bool coll = out_node && tg[r] >= 0;
        MassAcc<S, C> rs_acc = 0;
#pragma unroll
        for (int i = 0; i < 9; ++i) rs_acc += MassAcc<S, C>(f[r][i]);
        rs_acc += MassAcc<S, C>(er[r]);  // what rounding kept out of f_0 (apply_links)
        const C* P = s_psi + (ly + r * LY + 1) * PX + lx + 1;
        // F = -G psi(x) sum_i w^_i psi(x + e_i) e_i, w^ = 1/3 (axes), 1/12 (diagonals)
        const C gp = -a.G * P[0];
        const C Fx = gp * (C(1.0 / 3.0) * (P[1] - P[-1]) + C(1.0 / 12.0) * (P[PX + 1] - P[PX - 1] - P[-PX - 1] + P[-PX + 1]));
        const C Fy = gp * (C(1.0 / 3.0) * (P[PX] - P[-PX]) + C(1.0 / 12.0) * (P[PX + 1] + P[PX - 1] - P[-PX - 1] - P[-PX + 1]));
        C out[9];
        C rho, dux, duy, sx2, sy2, duu15;
        collide9<S, C, MRT>(a, coll, f[r], rs_acc, Fx, Fy, out, rho, dux, duy, sx2, sy2, duu15);
        // solid nodes store zeros (the pull replaces what it takes from them)
        const uint32_t xst = out_node ? own[r].x[1] + own[r].y[1] : OOB;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (kMixed<S> && i == 0)
                Buf<float>::st(rfb, xst == OOB ? OOB : xst * 2u, coll ? out[0] : C(0));
            else
                Buf<S>::st(rfb, sat_add(xst, uint32_t(i + P0) * ns), coll ? out[i] : C(0));
        }
        if (__any(coll && tg[r] > 0)) {
            C rv[REC2];
            rv[0] = rho;
            rv[1] = dux;
            rv[2] = duy;
            rv[3] = sx2;
            rv[4] = sy2;
            rv[5] = duu15;
#pragma unroll
            for (int i = 1; i < 9; ++i) rv[RF2 + i - 1] = out[i];  // rounded to the storage format
            C sl = C(0);  // the populations on the node's links (tag bits 0 .. 7)
#pragma unroll
            for (int j = 0; j < 8; ++j) sl += ((tg[r] >> j) & 1) ? out[j + 1] : C(0);
            rv[RF2 + 8] = sl;
            rv[RF2 + 9] = ds[r];
            st_vec(rout, (coll && tg[r] > 0) ? uint32_t(tg[r] >> 8) * (REC2 * sc) : OOB, rv);
        }
    }
    if (bad) atomicOr(&a.flags[FLAG_DOMAIN], 1);
}

template <class S, class C, int TX, int NT, int RPL, int WPE>
hipError_t launch_tile(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    constexpr int TY = NT / TX * RPL;
    Args2<S, C> a = step_args<S, C>(c, fcur, rcur, fnext, rnext);
    a.nsx = (a.nx + TX - 1) / TX;
    a.nblocks = a.nsx * ((a.ny + TY - 1) / TY);
    const bool mrt = c->p.collision == MCB_COLL_MRT;
    const auto k = pull ? (mrt ? k_tile2d<S, C, TX, NT, RPL, WPE, true, true> : k_tile2d<S, C, TX, NT, RPL, WPE, true, false>)
                        : (mrt ? k_tile2d<S, C, TX, NT, RPL, WPE, false, true> : k_tile2d<S, C, TX, NT, RPL, WPE, false, false>);
    hipLaunchKernelGGL(k, dim3(unsigned(a.nblocks)), dim3(NT), 0, c->stream, a);
    return hipGetLastError();
}

// 32 x 8 tiles: one node and at most one ring node per lane, so that FP32 arithmetic fits 64 VGPRs (eight
// waves per SIMD) and FP64 128 (four).  Wider tiles pull less ring (64 x 8 one pull in 2.2, 32 x 16 one
// in 2.4, against one in 1.7) but run fewer waves or spill: 1024^2 FP32 21.6 us with 32 x 16 and 22.7 with
// 64 x 16 against 20.8, FP64 38 and 44 against 35.6.  A box of fewer such tiles than half the
// compute units takes 16 x 8 tiles of two waves, which spread it over twice as many units (64^2
// FP64 5.3 us a step against 5.9, 128 x 160 5.6 against 6.2; at 256^2, one tile a unit, 7.1 against 6.7).
template <class S, class C>
hipError_t tile_t(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    constexpr int WPE = sizeof(C) == 8 ? 4 : 8;
    const int64_t tiles = int64_t((c->p.nx + 31) / 32) * ((c->p.ny + 7) / 8);
    if (2 * tiles < c->n_cu) return launch_tile<S, C, 16, 128, 1, WPE>(c, fcur, rcur, fnext, rnext, pull);
    return launch_tile<S, C, 32, 256, 1, WPE>(c, fcur, rcur, fnext, rnext, pull);
}

}  // namespace

hipError_t tile2d(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    switch (c->p.precision) {
        case MCB_F64: return tile_t<double, double>(c, fcur, rcur, fnext, rnext, pull);
        case MCB_F32S: return tile_t<float, float>(c, fcur, rcur, fnext, rnext, pull);
        default: return tile_t<__half, float>(c, fcur, rcur, fnext, rnext, pull);
    }
}

}  // namespace mcb
