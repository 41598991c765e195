"""The transposed D2Q9 step's tile kernels on boxes that end inside, at and just past a tile of 8, 16 or 32
columns, with walls across tile edges and round the periodic boundary;
against the oracle's dual numbers, with the tolerance of the other reverse-mode tests (FP64 sums of a
few hundred terms of one sign each: 1e-8 relative to the largest directional derivative)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu
BC = {"present": 0, "ibc": 1, "mibc": 2, "hbbc": 3}


@pytest.fixture(scope="module")
def mcb():
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb as m

    m.load()
    return m


DIMS = [(20, 33), (31, 15), (32, 16), (33, 17), (65, 25), (97, 40)]


@pytest.mark.parametrize("model", ["pseudo", "chempot"])
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: f"{d[0]}x{d[1]}")
def test_reverse_step_tile_edges(mcb, dims, model):
    cp = model == "chempot"
    dims3 = (*dims, 1)
    rv, rl = W.PR_MAXWELL[0.80] if cp else W.MAXWELL[0.70]
    T = 0.80 * W.PR_TC if cp else 0.70 * W.CS_TC
    rng = np.random.default_rng(dims[0] + 100 * dims[1])
    # a slab across the lower boundary, a ball on it across a tile edge, another across the side
    shapes = [W.band_y(-1.5, 2.4, 0), W.ball((0.5 * dims[0], 2.4), 3.2, 1)]
    if dims[0] >= 60:
        shapes.append(W.ball((0.3, 0.6 * dims[1]), 3.1, 2))
    shapes = np.array(shapes, np.int64)
    rho0 = W.drop_field(dims3, 2, [((0.45 * dims[0], 0.6 * dims[1]), 0.25 * min(dims))], rv, rl, 6.0 if cp else 3.0)
    for k, bc in enumerate(BC):
        coll = "mrt" if k % 2 else "bgk"
        print(f"\n[case] reverse {model} {dims} {bc} {coll}", flush=True)
        g = (1e-6, -2e-6)
        P = oracle.make_params(2, *dims3, tau=0.8, T=0.05 if cp else T)
        solid = oracle.classify(P, shapes)
        node, d, cls, q = oracle.links(P, shapes, solid)
        n = len(oracle.wall_nodes(P, solid))
        val = W.CP_K ** 2 * W.MU_PR_COEX[0.80] + rng.uniform(-0.01, 0.01, n) if cp else rng.uniform(0.9, 1.1, n)
        dirs = rng.standard_normal((4, n))
        ds = oracle.DualSim(P, solid, node, d, q)
        if cp:
            ds.set_chempot(T, k=W.CP_K, kappa=W.CP_KAPPA)
            ds.set_phi(np.ones(n))
            ds.set_mu_wall(val, dirs)
        else:
            ds.set_phi(val, dirs)
        ds.set_bc_mode(BC[bc])
        ds.set_gravity(g)
        if coll == "mrt":
            ds.set_mrt()
        ds.init_eq(rho0)
        ds.step(7)
        lat = mcb.Lattice(2, dims3, 0.8, T, bc_mode=bc, collision=coll, gravity=g,
                          **(dict(model="chempot", cp_k=W.CP_K, cp_kappa=W.CP_KAPPA) if cp else {}))
        lat.set_geometry(shapes)
        lat.set_wettability(val)
        for kind, prm in ((0, (rv, 1.0)), (1, ((rv + rl) / 2, 0.1 * (rl - rv)))):
            L_o, dL_o = ds.loss(kind, prm)
            L_g = lat.adj_forward(rho0, 7, 3, kind, prm)
            assert abs(L_g - L_o) <= 1e-12 * max(1.0, abs(L_o))
            dL_g = dirs @ lat.adj_backward(1.0)
            scale = np.abs(dL_o).max()
            assert scale > 0.0
            assert np.abs(dL_g - dL_o).max() <= 1e-8 * scale + 1e-14, (bc, kind, dL_g, dL_o)
        lat.close()
