"""The D2Q9 tile kernels (FP64 and FP32 boxes whose two lattices fit the memory-side cache; the
chemical-potential model at every size) at the edges of their tiles
(32 x 8 and, on boxes of few tiles, 8 x 8) and at boxes smaller than a tile, every storage type,
boundary scheme and collision; and the row march on either side of the switch between the two, and for FP16 storage throughout.
Against the FP64 oracle, with the per-step tolerances of the parity tests of each storage type
(a handful of roundings of the storage format per step)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32s": 3e-6, "f16s": 3e-3}
BC = {"present": 0, "ibc": 1, "mibc": 2, "hbbc": 3}


@pytest.fixture(scope="module")
def mcb():
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb as m

    m.load()
    return m


def run_case(mcb, dims, prec, bc, collision, radii, n_balls, steps=3):
    print(f"\n[case] {dims} {prec} {bc} {collision}", flush=True)
    rng = np.random.default_rng(dims[0] * 1000 + dims[1])
    dims3 = (*dims, 1)
    shapes = W.random_links_case(rng, dims3, 2, n_balls, *radii)
    rv, rl = W.MAXWELL[0.7]
    r0 = 0.3 * min(dims)
    drops = [((rng.uniform(0, dims[0]), rng.uniform(0, dims[1])), r0) for _ in range(2)]
    rho = W.drop_field(dims3, 2, drops, rv, rl, 4.0)
    T, g = 0.7 * W.CS_TC, (2e-6, -3e-6)
    P = oracle.make_params(2, *dims3, tau=0.9, T=T)
    sim, (solid, *_r) = oracle.sim_from_shapes(P, shapes)
    sim.set_bc_mode(BC[bc])
    sim.set_gravity(g)
    if collision == "mrt":
        sim.set_mrt()
    phi = rng.uniform(0.9, 1.1, sim.n_wall)
    sim.set_phi(phi)
    lat = mcb.Lattice(2, dims3, 0.9, T, precision=prec, rho_ref=0.0 if prec == "f64" else rv, bc_mode=bc,
                      collision=collision, gravity=g)
    lat.set_geometry(shapes)
    lat.set_wettability(phi)
    sim.init_eq(rho)
    lat.init_equilibrium(rho)
    fluid = solid == 0
    for k in range(1, steps + 1):
        sim.step(1)
        lat.step(1)
        a, b = lat.get_f()[:, fluid], sim.get_f()[:, fluid]
        e = np.abs(a - b).max() / np.abs(b).max()
        assert e < TOL[prec] * (k + 1), (k, e)
    lat.close()


EDGES = [((5, 40), (1.1, 1.6), 3), ((33, 6), (1.1, 1.8), 3), ((31, 7), (1.5, 2.4), 4), ((16, 8), (1.5, 2.4), 2),
         ((32, 8), (1.5, 2.4), 3), ((35, 17), (2.0, 4.0), 4), ((130, 100), (2.0, 8.0), 12), ((257, 130), (2.0, 9.0), 30)]


@pytest.mark.parametrize("prec", ["f64", "f32s", "f16s"])
@pytest.mark.parametrize("dims,radii,n", EDGES, ids=[f"{d[0]}x{d[1]}" for d, *_ in EDGES])
def test_tile_edges(mcb, dims, radii, n, prec):
    for k, bc in enumerate(BC):
        run_case(mcb, dims, prec, bc, "mrt" if k % 2 else "bgk", radii, n)


# just below and above the switch, ragged in both directions
@pytest.mark.parametrize("dims,prec", [((1287, 1289), "f64"), ((1293, 1291), "f64"), ((1825, 1820), "f32s"),
                                       ((1827, 1830), "f32s"), ((2449, 2443), "f16s"), ((2451, 2455), "f16s")],
                         ids=lambda v: f"{v[0]}x{v[1]}" if isinstance(v, tuple) else v)
def test_switch_to_the_march(mcb, dims, prec):
    run_case(mcb, dims, prec, "present", "bgk", (8.0, 24.0), 60, steps=2)


CP_EDGES = [(32, 16), (33, 17), (31, 33), (63, 15), (13, 70), (715, 730)]


@pytest.mark.parametrize("prec", ["f64", "f32s", "f16s"])
@pytest.mark.parametrize("dims", CP_EDGES, ids=lambda d: f"{d[0]}x{d[1]}")
def test_chempot_tile_edges(mcb, dims, prec):
    """Chemical-potential tiles: 8 x 8, and 32 x 32 on the last box (two of them per compute unit)."""
    print(f"\n[case] chempot {dims} {prec}", flush=True)
    rv, rl = W.PR_MAXWELL[0.80]
    T, T_cs = 0.80 * W.PR_TC, 0.7 * W.CS_TC
    dims3 = (*dims, 1)
    shapes = [W.band_y(-0.5, 3.4, 0)]
    if min(dims) >= 30:
        shapes.append(W.ball((0.48 * dims[0], 0.55 * dims[1]), 0.17 * min(dims) + 0.3, 1))
    shapes = np.array(shapes, np.int64)
    rho = W.drop_field(dims3, 2, [((0.3 * dims[0], 0.7 * dims[1]), 0.25 * min(dims))], rv, rl, W.CP_WIDTH)
    for k, bc in enumerate(BC):
        coll = "mrt" if k % 2 else "bgk"
        P = oracle.make_params(2, *dims3, tau=0.8, T=T_cs)
        sim, (solid, *_r) = oracle.sim_from_shapes(P, shapes)
        sim.set_chempot(T, k=W.CP_K, kappa=W.CP_KAPPA)
        sim.set_bc_mode(BC[bc])
        if coll == "mrt":
            sim.set_mrt()
        mu = W.CP_K ** 2 * W.MU_PR_COEX[0.80] * np.linspace(0.95, 1.05, sim.n_wall)
        sim.set_mu_wall(mu)
        lat = mcb.Lattice(2, dims3, 0.8, T, precision=prec, rho_ref=0.0 if prec == "f64" else rv, bc_mode=bc,
                          collision=coll, model="chempot", cp_k=W.CP_K, cp_kappa=W.CP_KAPPA)
        lat.set_geometry(shapes)
        lat.set_wettability(mu)
        sim.init_eq(rho)
        lat.init_equilibrium(rho)
        fluid = solid == 0
        for t in range(1, 4):
            sim.step(1)
            lat.step(1)
            a, b = lat.get_f()[:, fluid], sim.get_f()[:, fluid]
            e = np.abs(a - b).max() / np.abs(b).max()
            assert e < TOL[prec] * (t + 1), (bc, t, e)
        lat.close()


def test_vanishing_wall_factor_is_refused(mcb):
    """A wettability that underflows in the compute type makes the wall density zero: a domain error."""
    print("\n[case] vanishing wall factor", flush=True)
    wl = W.make("c0")
    lat = mcb.Lattice(2, wl.dims, wl.tau, wl.T, precision="f32s", rho_ref=wl.rho_v)
    lat.set_geometry(wl.shapes)
    lat.set_wettability(1e-60)
    with pytest.raises(mcb.MCBError):
        lat.init_equilibrium(wl.rho0())
    lat.close()
