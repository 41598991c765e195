"""The D3Q19 kernels of FP64 and FP32 storage (one lane per node, 256 consecutive nodes per workgroup) on boxes
of less than one workgroup, whole workgroups, rows shorter and longer than a workgroup and ragged ends, every
boundary scheme, walls round the periodic boundary; and FP16 storage's march on the same boxes.  Against
the FP64 oracle, with the per-step tolerances of the parity tests of each storage type."""
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


@pytest.mark.parametrize("prec", ["f64", "f32s", "f16s"])
@pytest.mark.parametrize("dims", [(8, 8, 8), (257, 6, 5), (7, 6, 6), (31, 33, 17), (64, 40, 9)],
                         ids=lambda d: "x".join(map(str, d)))
def test_flat_kernels_edges(mcb, dims, prec):
    rv, rl = W.MAXWELL[0.7]
    rng = np.random.default_rng(sum(dims))
    r = 0.3 * min(dims)
    shapes = np.array([W.ball((0.2, 0.4 * dims[1], 0.5 * dims[2]), min(r, 5.3), 0),
                       W.ball((0.6 * dims[0], 0.9 * dims[1], 0.1 * dims[2]), 0.8 * min(r, 4.1), 1)], np.int64)
    rho = W.drop_field(dims, 3, [((0.45 * dims[0], 0.5 * dims[1], 0.5 * dims[2]), 0.25 * min(dims))], rv, rl, 4.0)
    T, g = 0.7 * W.CS_TC, (1e-6, -2e-6, 3e-6)
    for bc in BC:
        print(f"\n[case] {dims} {prec} {bc}", flush=True)
        P = oracle.make_params(3, *dims, tau=0.9, T=T)
        sim, (solid, *_r) = oracle.sim_from_shapes(P, shapes)
        sim.set_bc_mode(BC[bc])
        sim.set_gravity(g)
        phi = rng.uniform(0.9, 1.1, sim.n_wall)
        sim.set_phi(phi)
        lat = mcb.Lattice(3, dims, 0.9, T, precision=prec, rho_ref=0.0 if prec == "f64" else rv, bc_mode=bc, gravity=g)
        lat.set_geometry(shapes)
        lat.set_wettability(phi)
        sim.init_eq(rho)
        lat.init_equilibrium(rho)
        fluid = solid == 0
        for k in range(1, 4):
            sim.step(1)
            lat.step(1)
            a, b = lat.get_f()[:, fluid], sim.get_f()[:, fluid]
            e = np.abs(a - b).max() / np.abs(b).max()
            assert e < TOL[prec] * (k + 1), (bc, k, e)
            lat.moments()  # stages fields in the scratch that holds psi during a step
        lat.close()
