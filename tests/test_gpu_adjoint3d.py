"""The transposed D3Q19 step (one lane per node, 256 consecutive nodes per workgroup, wall nodes from their list) on
boxes of less than one workgroup, with rows shorter and longer than one and ragged ends, walls round the
periodic boundary and none at all, every boundary scheme and storage; against the oracle's dual numbers, with the
tolerance of the other reverse-mode tests for FP64 (sums of a few hundred terms of one sign each: 1e-8 relative to the
largest directional derivative).  FP32 and FP16 storage take the gradient of their own trajectory, so the same
quantity is the central difference of their losses only within the rounding of the state: they are held to the
FP64 gradient within the per-step tolerance of the storage type times the seven steps and a factor of 10
for the sharpness of the loss (its transition spans a tenth of the density difference)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu
BC = {"present": 0, "ibc": 1, "mibc": 2, "hbbc": 3}
TOL = {"f64": 1e-8, "f32s": 10 * 7 * 3e-6, "f16s": 10 * 7 * 3e-3}


@pytest.fixture(scope="module")
def mcb():
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb as m

    m.load()
    return m


@pytest.mark.parametrize("dims", [(8, 8, 8), (257, 6, 5), (7, 6, 6), (31, 33, 9)], ids=lambda d: "x".join(map(str, d)))
def test_reverse_step_edges(mcb, dims):
    rv, rl = W.MAXWELL[0.70]
    T = 0.70 * W.CS_TC
    rng = np.random.default_rng(sum(dims))
    r = 0.3 * min(dims)
    shapes = np.array([W.ball((0.2, 0.4 * dims[1], 0.5 * dims[2]), min(r, 4.3), 0),
                       W.ball((0.6 * dims[0], 0.9 * dims[1], 0.1 * dims[2]), 0.8 * min(r, 4.1), 1)], np.int64)
    rho0 = W.drop_field(dims, 3, [((0.45 * dims[0], 0.5 * dims[1], 0.5 * dims[2]), 0.25 * min(dims))], rv, rl, 4.0)
    g = (1e-6, -2e-6, 3e-6)
    for bc in BC:
        P = oracle.make_params(3, *dims, tau=0.9, T=T)
        solid = oracle.classify(P, shapes)
        node, d, cls, q = oracle.links(P, shapes, solid)
        n = len(oracle.wall_nodes(P, solid))
        val = rng.uniform(0.9, 1.1, n)
        dirs = rng.standard_normal((4, n))
        ds = oracle.DualSim(P, solid, node, d, q)
        ds.set_phi(val, dirs)
        ds.set_bc_mode(BC[bc])
        ds.set_gravity(g)
        ds.init_eq(rho0)
        ds.step(7)
        for prec in TOL:
            print(f"\n[case] reverse {dims} {bc} {prec}", flush=True)
            lat = mcb.Lattice(3, dims, 0.9, T, precision=prec, rho_ref=0.0 if prec == "f64" else rv, bc_mode=bc, gravity=g)
            lat.set_geometry(shapes)
            lat.set_wettability(val)
            for kind, prm in ((0, (rv, 1.0)), (1, ((rv + rl) / 2, 0.1 * (rl - rv)))):
                L_o, dL_o = ds.loss(kind, prm)
                L_g = lat.adj_forward(rho0, 7, 3, kind, prm)
                dL_g = dirs @ lat.adj_backward(1.0)
                scale = np.abs(dL_o).max()
                assert scale > 0.0
                if prec == "f64":
                    assert abs(L_g - L_o) <= 1e-12 * max(1.0, abs(L_o))
                assert np.abs(dL_g - dL_o).max() <= TOL[prec] * scale + 1e-14, (bc, prec, kind, dL_g, dL_o)
            lat.close()


def test_reverse_step_without_walls(mcb):
    rv, rl = W.MAXWELL[0.70]
    dims = (9, 8, 10)
    rho0 = W.drop_field(dims, 3, [((4.0, 4.0, 5.0), 2.5)], rv, rl, 3.0)
    lat = mcb.Lattice(3, dims, 0.9, 0.70 * W.CS_TC)
    lat.set_geometry(np.zeros((0, 8), np.int64))
    L = lat.adj_forward(rho0, 3, 2, 2, (0.0, 1.0))
    assert abs(L - rho0.sum()) <= 1e-12 * rho0.sum()
    assert lat.adj_backward(1.0).size == 0
    lat.close()
