"""The D2Q9 tiles on a state past psi's domain: the call reports MCB_EDOMAIN, psi is 0 on the fluid nodes of
non-positive density, and these enter the eq. 15 mean of the walls as they are, as in the row marches.  First
collision from rest against numpy in FP64 (psi 0 where eq. 15 or the node itself leaves the domain); bounds: the
per-step tolerances of the parity tests."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

pytestmark = pytest.mark.gpu
T = 0.70 * W.CS_TC
TOL = {"f64": 1e-12, "f32s": 3e-6}


def collision(dims, shapes, rho, phi):
    P = oracle.make_params(2, *dims, tau=0.9, T=T)
    solid = oracle.classify(P, shapes).reshape(dims[1], dims[0]) != 0
    walls = np.asarray(oracle.wall_nodes(P, oracle.classify(P, shapes)), np.int64)
    e = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
    w = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
    wf = [0] + [1 / 3] * 4 + [1 / 12] * 4
    at = lambda a, k: np.roll(a, (-e[k][1], -e[k][0]), (0, 1))  # a(x + e_k)
    r = np.where(solid, 0.0, rho.reshape(dims[1], dims[0]))
    num = sum(w[k] * at(r, k) for k in range(1, 9))
    den = sum(w[k] * at(~solid, k) for k in range(1, 9))
    full = r.copy().reshape(-1)
    full[walls] = phi * (num.reshape(-1)[walls] / den.reshape(-1)[walls])
    full = full.reshape(r.shape)
    pr = full * T * (1 + full + full ** 2 - full ** 3) / (1 - full) ** 3 - full ** 2
    psi = np.where(full > 0, np.sqrt(np.maximum(2 * (full / 3 - pr), 0.0)), 0.0)
    F = [psi * sum(wf[k] * e[k][a] * at(psi, k) for k in range(1, 9)) for a in (0, 1)]
    out = []
    for k in range(9):
        ef = e[k][0] * F[0] + e[k][1] * F[1]
        with np.errstate(all="ignore"):
            q = np.where(solid, 0.0, (4.5 * ef ** 2 - 1.5 * (F[0] ** 2 + F[1] ** 2)) / np.where(solid, 1.0, r))
        out.append(np.where(solid, 0.0, w[k] * (r + 3 * ef + q)))
    return np.stack(out).reshape(9, -1), walls, ~solid.reshape(-1)


@pytest.mark.parametrize("prec", list(TOL))
def test_non_positive_density(prec):
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb

    L = mcb.load()
    print(f"\n[case] non-positive density, {prec}", flush=True)
    dims = (45, 37, 1)
    shapes = np.array([W.band_y(-0.5, 1.4, 0), W.ball((22.3, 18.6), 4.2, 1)], np.int64)
    rv, rl = W.MAXWELL[0.70]
    rho = rv + 0.02 * np.random.default_rng(4).random(dims[0] * dims[1])
    # inside the fluid, beside the band and the ball, and at a corner of four tiles (rows 20 and 24 lie beside the ball)
    for x, y in ((8, 8), (30, 2), (22, 24), (31, 31), (0, 20)):
        rho[y * dims[0] + x] = -0.05
    lat = mcb.Lattice(2, dims, 0.9, T, precision=prec, rho_ref=0.0 if prec == "f64" else rv)
    lat.set_geometry(shapes)
    phi = np.random.default_rng(5).uniform(0.9, 1.1, lat.n_wall)
    lat.set_wettability(phi)
    with pytest.raises(mcb.MCBError) as err:
        lat.init_equilibrium(rho)
    assert err.value.code == mcb.MCB_EDOMAIN
    f = np.zeros((9, lat.N))
    assert L.mcb_get_f(lat.ctx, mcb._ptr(f)) == mcb.MCB_EDOMAIN
    want, walls, fluid = collision(dims, shapes, rho, phi)
    assert np.array_equal(walls, lat.wall_nodes())
    lat.close()
    e = np.abs(f - want)[:, fluid].max() / np.abs(want).max()
    assert e < TOL[prec], e
