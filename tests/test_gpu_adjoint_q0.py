"""A fluid node exactly on the wall (q = 0 on its link: eq. 16 with c1 = 0, c2 = 1) in the reverse mode, both lattices
and with and without eq. 18; against the oracle's dual numbers, with the tolerance of the other
reverse-mode tests (1e-8 relative to the largest directional derivative)."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu
BC = {"present": 0, "ibc": 1, "mibc": 2}


@pytest.mark.parametrize("bc", list(BC))
@pytest.mark.parametrize("dim", [2, 3])
def test_gradient_with_a_node_on_the_wall(dim, bc):
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb

    mcb.load()
    print(f"\n[case] node on the wall, {dim}-D {bc}", flush=True)
    dims = (20, 18, 1) if dim == 2 else (16, 12, 14)
    rv, rl = W.MAXWELL[0.70]
    T = 0.70 * W.CS_TC
    # whole-numbered centre and radius: the six (four) axis nodes lie on the sphere, on its outside
    c = (9.0, 6.0) if dim == 2 else (8.0, 5.0, 7.0)
    shapes = np.array([W.ball(c, 3.0, 0)], np.int64)
    rho0 = W.drop_field(dims, dim, [((4.0, 12.0) if dim == 2 else (4.0, 9.0, 7.0), 4.0)], rv, rl, 3.0)
    P = oracle.make_params(dim, *dims, tau=0.9, T=T)
    solid = oracle.classify(P, shapes)
    node, d, cls, q = oracle.links(P, shapes, solid)
    assert (np.asarray(q) == 0).any()
    n = len(oracle.wall_nodes(P, solid))
    rng = np.random.default_rng(3)
    val, dirs = rng.uniform(0.9, 1.1, n), rng.standard_normal((4, n))
    ds = oracle.DualSim(P, solid, node, d, q)
    ds.set_phi(val, dirs)
    ds.set_bc_mode(BC[bc])
    ds.init_eq(rho0)
    ds.step(5)
    lat = mcb.Lattice(dim, dims, 0.9, T, bc_mode=bc)
    lat.set_geometry(shapes)
    lat.set_wettability(val)
    L_o, dL_o = ds.loss(0, (rv, 1.0))
    L_g = lat.adj_forward(rho0, 5, 2, 0, (rv, 1.0))
    assert abs(L_g - L_o) <= 1e-12 * max(1.0, abs(L_o))
    dL_g = dirs @ lat.adj_backward(1.0)
    assert np.abs(dL_g - dL_o).max() <= 1e-8 * np.abs(dL_o).max() + 1e-14, (dL_g, dL_o)
    lat.close()
