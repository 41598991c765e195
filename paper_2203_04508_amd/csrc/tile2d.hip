// D2Q9 step in tiles, FP64 and FP32 storage: one workgroup computes one tile of the new state (the same
// per-node arithmetic as the row marches of step2d.hip).  Small and middle-sized lattices of the
// pseudopotential model, all of the chemical-potential model's.
#include "step2d_node.h"

namespace mcb {
namespace {

// a buffer of at most BUF_MAX bytes: mcb_create keeps a population lattice below it (the chemical-potential
// model comes here up to that), mcb_build_links the boundary records
__device__ __forceinline__ __amdgpu_buffer_rsrc_t res32(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, int(bytes), 0x00020000);
}

// Issue the loads of the nine populations arriving at node (cx, cy) (eq. 5, from x - e_i; PULL = false:
// its own).  INNER: the node and its neighbours lie inside the box, so one lane offset serves all nine
// and the rest of each address is uniform; otherwise the neighbours are wrapped one by one.
template <class S, class C, bool PULL, bool INNER>
__device__ __forceinline__ void pull_at(__amdgpu_buffer_rsrc_t fa, int cx, int cy, int nx, int ny, C (&f)[9]) {
    constexpr uint32_t s = sizeof(S);
    const uint32_t row = uint32_t(nx) * s, ns = row * uint32_t(ny);
    const uint32_t o = uint32_t(cy) * row + uint32_t(cx) * s;
    uint32_t xo[3], yo[3];  // columns x + 1, x, x - 1 and rows y + 1, y, y - 1: index e + 1
    if (PULL && !INNER) {
        xo[0] = uint32_t(cx == nx - 1 ? 0 : cx + 1) * s;
        xo[1] = uint32_t(cx) * s;
        xo[2] = uint32_t(cx == 0 ? nx - 1 : cx - 1) * s;
        yo[0] = uint32_t(cy == ny - 1 ? 0 : cy + 1) * row;
        yo[1] = uint32_t(cy) * row;
        yo[2] = uint32_t(cy == 0 ? ny - 1 : cy - 1) * row;
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if (PULL && !INNER)
            f[i] = Buf<S>::ld(fa, xo[kEx[i] + 1] + yo[kEy[i] + 1], uint32_t(i) * ns);
        else
            f[i] = Buf<S>::ld(fa, o, uint32_t(i) * ns - (PULL ? uint32_t(kEy[i]) * row + uint32_t(kEx[i]) * s : 0u));
    }
}

// The new state of a node (offset xst in a population plane, or OOB: not stored): its populations, zeros
// on solid nodes (the pull replaces what it takes from them), and a boundary node's record.  nt (uniform):
// the populations with non-temporal stores.
template <class S, class C>
__device__ __forceinline__ void store_node(bool nt, __amdgpu_buffer_rsrc_t fb, __amdgpu_buffer_rsrc_t rout, uint32_t ns,
                                           uint32_t xst, bool coll, int tg, const C (&out)[9], C rho, C dux, C duy, C sx2, C sy2, C duu15,
                                           C ds) {
    constexpr uint32_t sc = sizeof(C);
    if (nt) {
#pragma unroll
        for (int i = 0; i < 9; ++i) Buf<S>::st_nt(fb, sat_add(xst, uint32_t(i) * ns), coll ? out[i] : C(0));
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) Buf<S>::st(fb, sat_add(xst, uint32_t(i) * ns), coll ? out[i] : C(0));
    }
    if (__any(coll && tg > 0)) {
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
        for (int j = 0; j < 8; ++j) sl += ((tg >> j) & 1) ? out[j + 1] : C(0);
        rv[RF2 + 8] = sl;
        rv[RF2 + 9] = ds;
        st_vec(rout, (coll && tg > 0) ? uint32_t(tg >> 8) * (REC2 * sc) : OOB, rv);
    }
}

// ---------------------------------------------------------------- pseudopotential model
// A workgroup owns a tile of TX x TY nodes, TY = OWN / TX; lane t < OWN owns column t % TX of row t / TX.
// Three phases, two barriers:
//   1  every node of the tile and of the ring two nodes wide around it is pulled by one lane (psi of the
//      ring next to the tile needs, through the wall nodes, the density two nodes out); eqs. 16-18 are
//      applied to the tile's own, and the densities of the (TX + 4) x (TY + 4) region go to LDS, zero on
//      solid nodes; the place of psi holds what it takes: a wall node's eq. 15 factor, zero on other solid
//      nodes, -1 on fluid ones.  Lanes past the own ones pull the ring (OWN < NT), or the own lanes pull
//      a node of it too (OWN = NT);
//   2  psi of the (TX + 2) x (TY + 2) region, wall nodes from the entries around them (eq. 15);
//   3  force, collision, store and boundary record of the own nodes, whose populations stayed in
//      registers.
// Why tiles here: a march gives a workgroup one row at a time, a serial chain of about 2 us per row on
// a box that leaves most of the chip idle; a tile runs its whole chain once (one round of loads,
// then the loads that depend on the tags, and two barriers).  Time per step, one-wave row march against
// tiles: 64^2 FP64 24.5 -> 4.1 us, 512^2 FP32 20.3 -> 8.0, 1024^2 FP32 32.6 -> 19.2 (3.9 TB/s of populations),
// FP64 61.6 -> 32 (4.7 TB/s), 1531 x 1021 FP64 83 -> 47.  At 1024^2 FP32 the SIMDs issue vector
// instructions in 72 % of their cycles, at six waves each.
// Every node past the box's edge is its periodic image, so partial tiles need no cases of their own:
// they only do not store.
// WPE: waves per SIMD the registers are bounded to.
template <class S, class C, int TX, int NT, int OWN, int WPE, bool PULL, bool MRT>
__global__ __launch_bounds__(NT, WPE) void k_tile2d(Args2<S, C> a) {
    constexpr int TY = OWN / TX;
    constexpr int RX = TX + 4, RY = TY + 4, PX = TX + 2, PY = TY + 2, NRING = RX * RY - TX * TY;
    constexpr bool SPLIT = OWN < NT;  // the lanes past the own ones pull the ring
    static_assert(OWN % 64 == 0 && NRING <= (SPLIT ? NT - OWN : NT), "one ring node per lane");
    constexpr int NP = PX * PY, NPL = (NP + NT - 1) / NT;
    constexpr uint32_t s = sizeof(S), sc = sizeof(C);
    __shared__ C s_rho[RY * RX];
    __shared__ C s_psi[RY * RX];
    // XCD-aware order: consecutive tiles go to the same XCD (one L2)
    const int bid = blockIdx.x;
    const int per = a.nblocks >> 3, rem = a.nblocks & 7;
    const int xcd = bid & 7, k8 = bid >> 3;
    const int logical = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k8;
    const int x0 = (logical % a.nsx) * TX, y0 = (logical / a.nsx) * TY;
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = a.nx, ny = a.ny;
    const bool mine = !SPLIT || t < OWN;  // uniform in a wave
    const uint32_t n = uint32_t(nx) * uint32_t(ny), ns = n * s;
    const __amdgpu_buffer_rsrc_t rfa = res32(a.fa, 9u * ns), rfb = res32(a.fb, 9u * ns);
    const __amdgpu_buffer_rsrc_t rtag = res32(a.tag, n * 4u), rfac = res32(a.fac, a.n_wall * sc);
    const __amdgpu_buffer_rsrc_t rin = res32(a.rin, a.n_bnodes * (REC2 * sc)), rout = res32(a.rout, a.n_bnodes * (REC2 * sc));
    const __amdgpu_buffer_rsrc_t rla = res32(a.la, a.n_bnodes * (Q2_LINKS * sc));
    // the density of a boundary node where eq. 18 applies: f_in enters its sum once and is subtracted
    // once from f_0, which leaves the node's own populations on its links; its record holds their sum
    const bool link_sum = PULL && a.k18 != C(0);
    bool bad = false;

    // ---- 1: tags first, then the populations (the loads that depend on a tag follow both)
    constexpr int K = SPLIT ? 1 : 2;  // nodes a lane pulls: its own (or its ring) node, its ring node
    int tg[K], at[K];                 // their tags and region entries
    C f[K][9];
    // INNER: the region and the nodes around it lie inside the box (all but the tiles along its edges)
    auto load = [&](auto in) {
        constexpr bool INNER = decltype(in)::value;
        int cx[K], cy[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int rx = lx + 2, ry = ly + 2;
            // lanes past the ring's last entry repeat it
            if (k == 1 || !mine) ring_at<TX, TY, 2>(min(SPLIT ? t - OWN : t, NRING - 1), rx, ry);
            at[k] = ry * RX + rx;
            cx[k] = INNER ? x0 - 2 + rx : image(x0 - 2 + rx, nx);
            cy[k] = INNER ? y0 - 2 + ry : image(y0 - 2 + ry, ny);
            tg[k] = ld_i32(rtag, (uint32_t(cy[k]) * uint32_t(nx) + uint32_t(cx[k])) * 4u);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) pull_at<S, C, PULL, INNER>(rfa, cx[k], cy[k], nx, ny, f[k]);
    };
    if (x0 >= 3 && y0 >= 3 && x0 + TX + 3 <= nx && y0 + TY + 3 <= ny)
        load(std::true_type{});
    else
        load(std::false_type{});
    C ds = C(0), er = C(0);
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
    // what depends on the tags alone, before the links wait for their loads (1024^2 FP64 34.4 -> 31.9 us)
    C fac[K];
#pragma unroll
    for (int k = 0; k < K; ++k) fac[k] = Buf<C>::ld(rfac, tg[k] <= -2 ? uint32_t(-tg[k] - 2) * sc : OOB);
    constexpr int KR = K - 1;  // the ring node
    C ls_ring = C(0);
    if (link_sum && (!SPLIT || !mine))
        ls_ring = Buf<C>::ld(rin, tg[KR] > 0 ? uint32_t(tg[KR] >> 8) * (REC2 * sc) + (RF2 + 8) * sc : OOB);
    auto put = [&](int k, C sr) {
        const int g = tg[k];
        if (g <= -2 && !(fac[k] > C(0))) bad = true;  // its sign carries meaning below
        s_rho[at[k]] = g >= 0 ? sr + a.rho_ref : C(0);
        s_psi[at[k]] = g >= 0 ? C(-1) : fac[k];  // (0 on solid nodes that are no wall nodes)
    };
    if (mine) {
        C sr = sum9(f[0]);
        if (PULL && __any(tg[0] > 0)) {
            const C ls = links(tg[0], f[0], ds, er);
            sr = link_sum ? sr + (tg[0] > 0 ? ls : C(0)) : sum9(f[0]);
        }
        put(0, sr);
    }
    if (!SPLIT || !mine) {
        C d, e;
        if (PULL && !link_sum && __any(tg[KR] > 0)) links(tg[KR], f[KR], d, e);
        put(KR, sum9(f[KR]) + ls_ring);
    }
    __syncthreads();

    // ---- 2: psi
#pragma unroll
    for (int h = 0; h < NPL; ++h) {
        const int j = t + h * NT;
        if (j < NP) {
            const int c = (j / PX + 1) * RX + j % PX + 1;
            const C fw = s_psi[c];
            C rn = s_rho[c];
            if (fw > C(0)) {
                // wall node: the weighted sum of its fluid neighbours' densities times the factor
                C num = C(0);
#pragma unroll
                for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
                    for (int dx = -1; dx <= 1; ++dx) {
                        if (dx == 0 && dy == 0) continue;
                        const C w = (dx == 0 || dy == 0) ? C(1.0 / 9.0) : C(1.0 / 36.0);
                        num += w * s_rho[c + dy * RX + dx];
                    }
                rn = fw * num;
            }
            s_psi[c] = fw == C(0) ? C(0) : psi_val(rn, a.eos, &bad);
        }
    }
    __syncthreads();

    // ---- 3: force, collision, store
    if (mine) {
        const bool out_node = x0 + lx < nx && y0 + ly < ny;
        const bool coll = out_node && tg[0] >= 0;
        MassAcc<S, C> rs_acc = 0;
#pragma unroll
        for (int i = 0; i < 9; ++i) rs_acc += MassAcc<S, C>(f[0][i]);
        rs_acc += MassAcc<S, C>(er);  // what rounding kept out of f_0 (apply_links)
        const C* P = s_psi + (ly + 2) * RX + lx + 2;
        // F = -G psi(x) sum_i w^_i psi(x + e_i) e_i, w^ = 1/3 (axes), 1/12 (diagonals)
        const C gp = -a.G * P[0];
        const C Fx = gp * (C(1.0 / 3.0) * (P[1] - P[-1]) + C(1.0 / 12.0) * (P[RX + 1] - P[RX - 1] - P[-RX - 1] + P[-RX + 1]));
        const C Fy = gp * (C(1.0 / 3.0) * (P[RX] - P[-RX]) + C(1.0 / 12.0) * (P[RX + 1] + P[RX - 1] - P[-RX - 1] - P[-RX + 1]));
        C out[9];
        C rho, dux, duy, sx2, sy2, duu15;
        collide9<S, C, MRT>(a, coll, f[0], rs_acc, Fx, Fy, out, rho, dux, duy, sx2, sy2, duu15);
        const uint32_t x = uint32_t(y0 + ly) * uint32_t(nx) + uint32_t(x0 + lx);
        store_node<S, C>(false, rfb, rout, ns, out_node ? x * s : OOB, coll, tg[0], out, rho, dux, duy, sx2, sy2, duu15, ds);
    }
    raise_domain(bad, a.flags);
}

template <class S, class C, int TX, int NT, int OWN, int WPE>
hipError_t launch_tile(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    constexpr int TY = OWN / TX;
    Args2<S, C> a = step_args<S, C>(c, fcur, rcur, fnext, rnext);
    a.nsx = (a.nx + TX - 1) / TX;
    a.nblocks = a.nsx * ((a.ny + TY - 1) / TY);
    const bool mrt = c->p.collision == MCB_COLL_MRT;
    const auto k = pull ? (mrt ? k_tile2d<S, C, TX, NT, OWN, WPE, true, true> : k_tile2d<S, C, TX, NT, OWN, WPE, true, false>)
                        : (mrt ? k_tile2d<S, C, TX, NT, OWN, WPE, false, true> : k_tile2d<S, C, TX, NT, OWN, WPE, false, false>);
    hipLaunchKernelGGL(k, dim3(unsigned(a.nblocks)), dim3(NT), 0, c->stream, a);
    return hipGetLastError();
}

// Large boxes: 32 x 8 tiles whose lanes pull one node and at most one ring node each, so that FP32 arithmetic
// fits 64 VGPRs (eight waves per SIMD) and FP64 128 (four).  Wider tiles pull less ring (64 x 8 one pull in
// 2.2, 32 x 16 one in 2.4, against one in 1.7) but run fewer waves or spill: 1024^2 FP32 21.6 us with 32 x
// 16 and 22.7 with 64 x 16 against 20.8, FP64 38 and 44 against 35.6.
// Boxes whose tiles are all resident at once wait for one chain of loads and dependent arithmetic, which is
// shorter with lanes of their own for the ring: 256^2 FP64 7.0 -> 6.1 us a step, 400 x 300 8.5 -> 8.0, 512^2 FP32
// 8.8 -> 8.0 (seven waves a tile: FP64 keeps two tiles a compute unit, FP32 four; past that they lose,
// 512^2 FP64 12.4 -> 13.2, 724^2 FP32 12.7 -> 13.3).  Still smaller boxes take 8 x 8 tiles of three waves,
// spread over four times as many units: 64^2 FP64 5.3 -> 4.4 us, 128 x 160 5.4 -> 5.2, 200^2 6.4 -> 5.9
// (against 6.15 with 32 x 8 split; at 256^2, four tiles a unit, 6.3 against 6.1).
template <class S, class C>
hipError_t tile_t(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    auto tiles = [&](int tx, int ty) { return int64_t((c->p.nx + tx - 1) / tx) * ((c->p.ny + ty - 1) / ty); };
    if (tiles(8, 8) <= 3 * c->n_cu) return launch_tile<S, C, 8, 192, 64, 4>(c, fcur, rcur, fnext, rnext, pull);
    if (tiles(32, 8) <= (sizeof(C) == 8 ? 2 : 4) * c->n_cu)
        return launch_tile<S, C, 32, 448, 256, 4>(c, fcur, rcur, fnext, rnext, pull);
    return launch_tile<S, C, 32, 256, 256, sizeof(C) == 8 ? 4 : 8>(c, fcur, rcur, fnext, rnext, pull);
}

// ---------------------------------------------------------------- chemical-potential model
// The same with a wider reach.  The collision of a node needs mu and rho two nodes away on each axis
// (eq. 9), mu of a fluid node rho two nodes away (eq. 12), the second solid layer's density the first
// layer's around it, and the first layer's the fluid densities around it (eq. 15): densities up to
// six nodes away.  Five phases:
//   1  own nodes and the ring six nodes wide: pulled density and solid layer, to LDS.  Where eq. 18
//      applies, a boundary node's density is its pulled populations plus the link sum of its record;
//      without it (IBC) eqs. 16-17 run on the ring too;
//   2  the first solid layer's density, 3 the second's (skipped by tiles without solid nodes);
//   4  mu of the tile and two nodes around it (eq. 12; solid nodes take their assigned values);
//   5  force from both fields, eqs. 16-18 and the collision of the own nodes.
// Measured against a march (one row per iteration, five barriers a row) that this replaces: 500 x 300
// FP64 102 -> 11 us a step on a flat wall, 1024^2 FP32 on balls 144 -> 30, FP64 184 -> 55, 4096^2 FP32
// 483 -> 430, FP64 1048 -> 847.  At 4096^2 FP32 the SIMDs issue vector instructions in 71 % of their cycles.
// Lanes t < OWN own the tile's nodes; where OWN < NT, ring entries go to the lanes past them first.
template <class S, class C, int TX, int NT, int OWN, int RPL, int WPE, bool PULL, bool MRT>
__global__ __launch_bounds__(NT, WPE) void k_cptile(ArgsCP<S, C> p) {
    constexpr int HC = 6, LY = OWN / TX, TY = LY * RPL;
    constexpr int RX = TX + 2 * HC, RY = TY + 2 * HC, NR = RX * RY;
    constexpr int MX = TX + 4, MY = TY + 4, NM = MX * MY, NML = (NM + NT - 1) / NT;
    constexpr int NRING = NR - TX * TY, NRL = (NRING + NT - 1) / NT;
    static_assert(OWN == NT || (RPL == 1 && NRL == 1 && OWN % 64 == 0), "lanes past the own ones make ring entries only");
    constexpr uint32_t s = sizeof(S), sc = sizeof(C);
    const Args2<S, C>& a = p.a;
    __shared__ C s_rho[NR];
    __shared__ C s_mu[NM];
    __shared__ int8_t s_lay[NR];
    const int bid = blockIdx.x;
    const int per = a.nblocks >> 3, rem = a.nblocks & 7;
    const int xcd = bid & 7, k8 = bid >> 3;
    const int logical = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + k8;
    // consecutive tiles run along panels of a.H tile columns, so that the ring a tile shares with the one
    // above it is still in the XCD's L2 when that one reads it
    int pan = 0, rp = logical, pw = a.nsx;
    if (a.nsx > a.H) {
        const int per_pan = a.H * (a.nblocks / a.nsx);
        pan = logical / per_pan;
        rp = logical - pan * per_pan;
        pw = min(a.H, a.nsx - pan * a.H);
    }
    const int rq = rp / pw, x0 = (pan * a.H + rp - rq * pw) * TX, y0 = rq * TY;
    const int t = threadIdx.x, lx = t % TX, ly = t / TX, nx = a.nx, ny = a.ny;
    // whether the lane owns nodes, its first ring entry, and whether its wave has any
    const bool mine = OWN == NT || t < OWN;
    const int jr = OWN == NT ? t : (t >= OWN ? t - OWN : t + NT - OWN);
    const bool ring = OWN == NT || (jr & ~63) < NRING;
    const uint32_t n = uint32_t(nx) * uint32_t(ny), ns = n * s;
    const __amdgpu_buffer_rsrc_t rfa = res32(a.fa, 9u * ns), rfb = res32(a.fb, 9u * ns);
    const __amdgpu_buffer_rsrc_t rtag = res32(a.tag, n * 4u), rlay = res32(p.layer, n), rmu = res32(p.mu, n * sc);
    const __amdgpu_buffer_rsrc_t rin = res32(a.rin, a.n_bnodes * (REC2 * sc)), rout = res32(a.rout, a.n_bnodes * (REC2 * sc));
    const __amdgpu_buffer_rsrc_t rla = res32(a.la, a.n_bnodes * (Q2_LINKS * sc));
    const bool link_sum = PULL && a.k18 != C(0);
    bool bad = false, solid = false;

    // ---- 1
    int tg[RPL];
    C f[RPL][9], ds[RPL];
    // region entry of a node: layer l, density from the sum rs of its populations.  The lane keeps the
    // entries it makes, to serve their solid layers itself: entry | layer << 16, layer 3 where the
    // neighbours of a layer node do not all lie in the region (nothing reads those).
    int ent[RPL + NRL];
    if (OWN != NT)
#pragma unroll
        for (int k = 0; k < RPL + NRL; ++k) ent[k] = 3 << 16;
    auto put = [&](int k, int rx, int ry, int g, int l, MassAcc<S, C> rs) {
        const int at = ry * RX + rx;
        s_rho[at] = g >= 0 ? C(rs) + a.rho_ref : C(0);
        s_lay[at] = int8_t(l);
        const bool in = k < RPL || (rx >= l && rx < RX - l && ry >= l && ry < RY - l);
        ent[k] = at | ((in ? l : 3) << 16);
        solid = solid || l == 1 || l == 2;
    };
    auto sum9 = [](const C (&v)[9]) {
        MassAcc<S, C> rs = MassAcc<S, C>(0);
#pragma unroll
        for (int i = 0; i < 9; ++i) rs += MassAcc<S, C>(v[i]);
        return rs;
    };
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
    int lay[RPL];
    C mus[NML];  // the solid nodes' assigned potentials of the mu region (fluid nodes' entries are not used)
    auto load = [&](auto in) {
        constexpr bool INNER = decltype(in)::value;
        auto coord = [&](int rx, int ry, int& cx, int& cy) {
            cx = INNER ? x0 - HC + rx : image(x0 - HC + rx, nx);
            cy = INNER ? y0 - HC + ry : image(y0 - HC + ry, ny);
            return uint32_t(cy) * uint32_t(nx) + uint32_t(cx);
        };
        int cx[RPL + NRL], cy[RPL + NRL], tgr[NRL], layr[NRL], px[NRL], py[NRL];
#pragma unroll
        for (int k = 0; k < RPL + NRL; ++k) {
            int rx = lx + HC, ry = ly + k * LY + HC;
            if (k >= RPL) {
                ring_at<TX, TY, HC>(min(jr + (k - RPL) * NT, NRING - 1), rx, ry);
                px[k - RPL] = rx;
                py[k - RPL] = ry;
            }
            const uint32_t x = coord(rx, ry, cx[k], cy[k]);
            (k < RPL ? tg[k < RPL ? k : 0] : tgr[k < RPL ? 0 : k - RPL]) = ld_i32(rtag, x * 4u);
            (k < RPL ? lay[k < RPL ? k : 0] : layr[k < RPL ? 0 : k - RPL]) =
                int8_t(__builtin_amdgcn_raw_buffer_load_b8(rlay, x, 0, 0));
        }
#pragma unroll
        for (int h = 0; h < NML; ++h) {
            const int j = min(t + h * NT, NM - 1);
            int mx, my;
            mus[h] = Buf<C>::ld(rmu, coord(j % MX + HC - 2, j / MX + HC - 2, mx, my) * sc);
        }
#pragma unroll
        for (int r = 0; r < RPL; ++r)
            if (mine) pull_at<S, C, PULL, INNER>(rfa, cx[r], cy[r], nx, ny, f[r]);
#pragma unroll
        for (int h = 0; h < NRL; ++h) {
            if (!ring) break;
            C v[9], ls = C(0);
            pull_at<S, C, PULL, INNER>(rfa, cx[RPL + h], cy[RPL + h], nx, ny, v);
            if (link_sum) {
                ls = Buf<C>::ld(rin, tgr[h] > 0 ? uint32_t(tgr[h] >> 8) * (REC2 * sc) + (RF2 + 8) * sc : OOB);
            } else if (PULL && __any(tgr[h] > 0)) {
                C d;
                links(tgr[h], v, d, ls);
            }
            put(RPL + h, px[h], py[h], tgr[h], layr[h], sum9(v) + MassAcc<S, C>(ls));
        }
    };
    if (x0 > HC && y0 > HC && x0 + TX + HC + 1 <= nx && y0 + TY + HC + 1 <= ny)
        load(std::true_type{});
    else
        load(std::false_type{});
    MassAcc<S, C> rs[RPL];  // what the collision hands back: the sum after eqs. 16-18
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        if (!mine) break;
        ds[r] = C(0);
        rs[r] = sum9(f[r]);
        MassAcc<S, C> rd = rs[r];
        if (PULL && __any(tg[r] > 0)) {
            C er;
            const C ls = links(tg[r], f[r], ds[r], er);
            rs[r] = sum9(f[r]) + MassAcc<S, C>(er);
            rd = link_sum ? rd + MassAcc<S, C>(tg[r] > 0 ? ls : C(0)) : rs[r];
        }
        put(r, lx + HC, ly + r * LY + HC, tg[r], lay[r], rd);
    }
    // ---- 2, 3: the solid layers (eq. 15 over the layer above), where the tile's region holds any
    if (__syncthreads_or(solid)) {
#pragma unroll 1
        for (int l = 1; l <= 2; ++l) {
#pragma unroll
            for (int h = 0; h < RPL + NRL; ++h) {
                const int e = ent[h] & 0xFFFF;
                if ((ent[h] >> 16) == l) {
                    // every neighbour's layer and density first, then the selection
                    int nl[9];
                    C nr[9];
#pragma unroll
                    for (int i = 1; i < 9; ++i) {
                        nl[i] = s_lay[e + kEy[i] * RX + kEx[i]];
                        nr[i] = s_rho[e + kEy[i] * RX + kEx[i]];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    C num = C(0), den = C(0);
#pragma unroll
                    for (int i = 1; i < 9; ++i) {
                        num += nl[i] == l - 1 ? w9<C>(i) * nr[i] : C(0);
                        den += nl[i] == l - 1 ? w9<C>(i) : C(0);
                    }
                    s_rho[e] = num / den;
                }
            }
            __syncthreads();
        }
    }
    // ---- 4: chemical potential (eq. 12 with the Peng-Robinson mu of eq. 11)
    const C s2 = C(1.4142135623730951);
#pragma unroll
    for (int h = 0; h < NML; ++h) {
        const int j = t + h * NT;
        if (j < NM) {
            const int e = (j / MX + HC - 2) * RX + j % MX + HC - 2;
            C m = mus[h];
            if (s_lay[e] == 0) {
                const C rc = s_rho[e];
                const C br = p.b * rc;
                if (!(rc > C(0)) || !(br < C(1))) bad = true;
                const C rf = rc > C(0) && br < C(1) ? rc : C(1);  // a harmless stand-in past the domain
                const C brf = p.b * rf;
                const C iq = rcp(C(1) - brf);
                const C m0 = p.RT * log(rf * iq) - p.c_log * log((s2 - C(1) + brf) * rcp(s2 + C(1) - brf)) +
                             p.RT * iq - p.aal * rf * rcp(C(1) + C(2) * brf - brf * brf);
                C lap = C(0);
                lap += cd2(s_rho[e - 2], s_rho[e - 1], rc, s_rho[e + 1], s_rho[e + 2]);
                lap += cd2(s_rho[e - 2 * RX], s_rho[e - RX], rc, s_rho[e + RX], s_rho[e + 2 * RX]);
                m = p.k2 * m0 - p.kappa * lap;
            }
            s_mu[j] = m;
        }
    }
    __syncthreads();
    // ---- 5: force, collision, store
#pragma unroll
    for (int r = 0; r < RPL; ++r) {
        if (!mine) break;
        const bool out_node = x0 + lx < nx && y0 + ly + r * LY < ny;
        const bool coll = out_node && tg[r] >= 0;
        const C* R = s_rho + (ly + r * LY + HC) * RX + lx + HC;
        const C* U = s_mu + (ly + r * LY + 2) * MX + lx + 2;
        const C rr = R[0];
        const C Fx = -rr * cd1(U[-2], U[-1], U[1], U[2]) + cd1(R[-2], R[-1], R[1], R[2]) / C(3);
        const C Fy = -rr * cd1(U[-2 * MX], U[-MX], U[MX], U[2 * MX]) + cd1(R[-2 * RX], R[-RX], R[RX], R[2 * RX]) / C(3);
        C out[9];
        C rho, dux, duy, sx2, sy2, duu15;
        collide9<S, C, MRT>(a, coll, f[r], rs[r], coll ? Fx : C(0), coll ? Fy : C(0), out, rho, dux, duy, sx2, sy2, duu15);
        const uint32_t x = uint32_t(y0 + ly + r * LY) * uint32_t(nx) + uint32_t(x0 + lx);
        store_node<S, C>(p.nt, rfb, rout, ns, out_node ? x * s : OOB, coll, tg[r], out, rho, dux, duy, sx2, sy2,
                         duu15, ds[r]);
    }
    raise_domain(bad, a.flags);
}

template <class S, class C, int TX, int NT, int OWN, int RPL, int WPE>
hipError_t launch_cptile(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    constexpr int TY = OWN / TX * RPL;
    ArgsCP<S, C> p = cp_args<S, C>(c, fcur, rcur, fnext, rnext);
    p.a.nsx = (p.a.nx + TX - 1) / TX;
    // Panels of 16 tiles: 4096^2 FP32 482 -> 451 us (1.16 -> 0.94 GB read), FP64 948 -> 872; 8, 32 and 64
    // tiles 472, 458 and 478; no difference at 3000 x 2900.  Non-temporal stores once the lattices outgrow
    // the memory-side cache, where they keep the lattice being read in it: 4096^2 FP32 451 -> 435, FP64
    // 872 -> 847, 2560 x 2500 FP32 187 -> 179, FP64 1400 x 1300 (262 MB) 112 -> 105; below it they cost up
    // to a third (1800 x 1500 FP32 60 -> 82).  A tile row of FP32 is one cache line, written in two
    // parts where the rows of the lattice are not whole lines: there they are no gain (3000 x 2900
    // 260 -> 283, 3600 x 3500 364 -> 366, 2000 x 1850 112 -> 107).
    p.a.H = 16;
    const int64_t bytes = 2 * state_bytes(c->p.precision, 9, c->g.N);
    p.nt = bytes > (int64_t(1) << 28) && (sizeof(S) == 8 || (p.a.nx * int(sizeof(S))) % 128 == 0);
    p.a.nblocks = p.a.nsx * ((p.a.ny + TY - 1) / TY);
    const bool mrt = c->p.collision == MCB_COLL_MRT;
    const auto k = pull ? (mrt ? k_cptile<S, C, TX, NT, OWN, RPL, WPE, true, true> : k_cptile<S, C, TX, NT, OWN, RPL, WPE, true, false>)
                        : (mrt ? k_cptile<S, C, TX, NT, OWN, RPL, WPE, false, true> : k_cptile<S, C, TX, NT, OWN, RPL, WPE, false, false>);
    hipLaunchKernelGGL(k, dim3(unsigned(p.a.nblocks)), dim3(NT), 0, c->stream, p);
    return hipGetLastError();
}

// A box whose tiles fit one per compute unit waits for one tile's chain of dependent loads and arithmetic:
// the smallest tile that fits is taken, with lanes of their own for (nearly all of) its ring, which is three
// to five times the tile in the small ones and is worked off in one pass with the tile instead of after
// it.  FP64 on balls, against 32 x 16 tiles of 512 lanes: 64^2 13.0 -> 6.9 us a step, 128 x 160 14.7 -> 7.7,
// 301 x 203 13.7 -> 10.0, 400 x 250 14.3 -> 11.9, 500 x 300 19.5 -> 14.3 (flat wall 14.5 -> 11.3), 512 x 384
// 19.4 -> 15.3; 512^2, 24 rows a tile no longer one a unit, 20.5 -> 26.
// 32 x 32 tiles of two nodes a lane pull 0.9 ring nodes per node, 32 x 16 tiles of one node a lane 1.4, but
// run a shorter chain; the larger ones are taken once the box holds two of them per compute unit
// (1024^2 FP64 58 us against 62, 2048 x 1024 FP32 52 against 56, 4096^2 FP32 480 against 534; 512^2 FP64,
// one a unit, 24 against 21, 724^2 42 against 38; panels and streaming stores came after).  FP32 arithmetic
// fits 80 VGPRs, six waves per SIMD; FP64 is held to 128 (a 28-byte spill): unbounded, at three waves,
// 1024^2 took 78 us against 60.
template <class S, class C>
hipError_t cptile_t(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    constexpr int WPE = sizeof(C) == 8 ? 4 : 6;
    auto tiles = [&](int tx, int ty) { return int64_t((c->p.nx + tx - 1) / tx) * ((c->p.ny + ty - 1) / ty); };
    auto fits = [&](int tx, int ty) { return tiles(tx, ty) <= c->n_cu; };
    if (tiles(32, 32) >= 2 * c->n_cu) return launch_cptile<S, C, 32, 512, 512, 2, WPE>(c, fcur, rcur, fnext, rnext, pull);
    if (fits(8, 8)) return launch_cptile<S, C, 8, 448, 64, 1, 4>(c, fcur, rcur, fnext, rnext, pull);
    if (fits(16, 8)) return launch_cptile<S, C, 16, 576, 128, 1, 4>(c, fcur, rcur, fnext, rnext, pull);
    if (fits(16, 16)) return launch_cptile<S, C, 16, 768, 256, 1, 4>(c, fcur, rcur, fnext, rnext, pull);
    if (fits(32, 16)) return launch_cptile<S, C, 32, 1024, 512, 1, 4>(c, fcur, rcur, fnext, rnext, pull);
    if (fits(32, 20)) return launch_cptile<S, C, 32, 1024, 640, 1, 4>(c, fcur, rcur, fnext, rnext, pull);
    if (fits(32, 24)) return launch_cptile<S, C, 32, 1024, 768, 1, 4>(c, fcur, rcur, fnext, rnext, pull);
    return launch_cptile<S, C, 32, 512, 512, 1, WPE>(c, fcur, rcur, fnext, rnext, pull);
}

}  // namespace

// FP16 storage stays with the row marches (see step2d)
hipError_t tile2d(mcb_ctx* c, const void* fcur, const void* rcur, void* fnext, void* rnext, bool pull) {
    const bool f64 = c->p.precision == MCB_F64;
    if (c->p.model == MCB_MODEL_CHEMPOT)
        return f64 ? cptile_t<double, double>(c, fcur, rcur, fnext, rnext, pull)
                   : cptile_t<float, float>(c, fcur, rcur, fnext, rnext, pull);
    return f64 ? tile_t<double, double>(c, fcur, rcur, fnext, rnext, pull)
               : tile_t<float, float>(c, fcur, rcur, fnext, rnext, pull);
}

}  // namespace mcb
