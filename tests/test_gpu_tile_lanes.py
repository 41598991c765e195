"""D2Q9 tiles whose lanes past the own ones pull the ring: a box on either side of each line of the dispatch (by the
number of tiles against the compute units: 8 x 8 and 32 x 8 tiles of the pseudopotential model; 8 x 8, 16 x 8, 16 x 16
and 32 x 16, 20, 24 of the chemical-potential model), forward and reverse, ragged, walls round the periodic
boundary.  Against the FP64 oracle, with the per-step tolerances of the parity tests of each storage type; gradients
against its dual numbers with the tolerance of the other reverse-mode tests (1e-8 relative to the largest
directional derivative)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = {"f64": 1e-12, "f32s": 3e-6}
BC = {"present": 0, "ibc": 1, "mibc": 2, "hbbc": 3}
PSEUDO = [(8, 9), (221, 217), (229, 217), (500, 255), (517, 257), (1001, 257), (1030, 257)]
CHEMPOT = [(7, 9), (125, 127), (129, 130), (255, 125), (257, 127), (255, 250), (301, 255), (385, 300), (515, 300),
           (480, 355), (509, 381), (515, 385)]


@pytest.fixture(scope="module")
def mcb():
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb as m

    m.load()
    return m


@pytest.mark.parametrize("model,dims", [("pseudo", d) for d in PSEUDO] + [("chempot", d) for d in CHEMPOT],
                         ids=lambda v: v if isinstance(v, str) else f"{v[0]}x{v[1]}")
def test_dispatch_lines(mcb, model, dims):
    cp = model == "chempot"
    dims3 = (*dims, 1)
    rv, rl = W.PR_MAXWELL[0.80] if cp else W.MAXWELL[0.70]
    T_cs = 0.7 * W.CS_TC
    T = 0.80 * W.PR_TC if cp else T_cs
    rng = np.random.default_rng(dims[0] + 1000 * dims[1])
    lo = min(dims)
    shapes = [W.band_y(-0.5, 1.4, 0)]
    if lo >= 100:
        shapes += [W.ball((0.3, 0.5 * dims[1]), 0.09 * lo + 0.3, 1), W.ball((0.6 * dims[0], 0.98 * dims[1]), 0.13 * lo + 0.1, 2)]
    shapes = np.array(shapes, np.int64)
    rho0 = W.drop_field(dims3, 2, [((0.45 * dims[0], 0.55 * dims[1]), 0.25 * lo)], rv, rl, W.CP_WIDTH if cp else 4.0)
    for k, (bc, prec) in enumerate((("present", "f64"), ("ibc", "f32s"), ("mibc", "f64"))):
        coll = "mrt" if k % 2 else "bgk"
        print(f"\n[case] {model} {dims} {bc} {prec} {coll}", flush=True)
        P = oracle.make_params(2, *dims3, tau=0.9, T=T_cs)
        solid = oracle.classify(P, shapes)
        node, d, cls, q = oracle.links(P, shapes, solid)
        n = len(oracle.wall_nodes(P, solid))
        val = W.CP_K ** 2 * W.MU_PR_COEX[0.80] + rng.uniform(-0.01, 0.01, n) if cp else rng.uniform(0.9, 1.1, n)
        dirs = rng.standard_normal((4, n))
        sim, _ = oracle.sim_from_shapes(P, shapes)
        ds = oracle.DualSim(P, solid, node, d, q)
        for s in (sim, ds):
            if cp:
                s.set_chempot(T, k=W.CP_K, kappa=W.CP_KAPPA)
            s.set_bc_mode(BC[bc])
            s.set_gravity((1e-6, -2e-6))
            if coll == "mrt":
                s.set_mrt()
        if cp:
            sim.set_mu_wall(val)
            ds.set_phi(np.ones(n))
            ds.set_mu_wall(val, dirs)
        else:
            sim.set_phi(val)
            ds.set_phi(val, dirs)
        sim.init_eq(rho0)
        ds.init_eq(rho0)
        lat = mcb.Lattice(2, dims3, 0.9, T, precision=prec, rho_ref=0.0 if prec == "f64" else rv, bc_mode=bc, collision=coll,
                          gravity=(1e-6, -2e-6), **(dict(model="chempot", cp_k=W.CP_K, cp_kappa=W.CP_KAPPA) if cp else {}))
        lat.set_geometry(shapes)
        lat.set_wettability(val)
        lat.init_equilibrium(rho0)
        fluid = solid == 0
        for t in range(1, 3):
            sim.step(1)
            lat.step(1)
            a, b = lat.get_f()[:, fluid], sim.get_f()[:, fluid]
            e = np.abs(a - b).max() / np.abs(b).max()
            assert e < TOL[prec] * (t + 1), (bc, t, e)
        if prec == "f64":
            ds.step(3)
            L_o, dL_o = ds.loss(0, (rv, 1.0))
            assert abs(lat.adj_forward(rho0, 3, 2, 0, (rv, 1.0)) - L_o) <= 1e-12 * max(1.0, abs(L_o))
            dL_g = dirs @ lat.adj_backward(1.0)
            scale = np.abs(dL_o).max()
            assert scale > 0.0
            assert np.abs(dL_g - dL_o).max() <= 1e-8 * scale + 1e-14, (bc, dL_g, dL_o)
        lat.close()
