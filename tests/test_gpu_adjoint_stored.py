"""The reverse mode of the shifted storages is the adjoint of the FP64 step linearised at the stored states: the eq. 13
terms of the links follow in FP64 from the node's stored populations and the force of its boundary record.  The
reference is one reverse sweep over two steps by torch's autograd in FP64 on the CPU, from the states that the library
stored.  FP16 storage tells a boundary record's velocity from that of the stored populations: with the former the
reference's gradient moves by 1.4e-6 (2-D) and 7e-7 (3-D) of its norm.  What the reference does not know is the record's
force in its FP32 digits; FP32 in place of FP64 in it moves the gradient by 1.5e-9.  Bound: 1e-7; FP64 storage, as a check
of the reference, 1e-8 as in the other reverse-mode tests."""
import numpy as np
import pytest

from oracle import oracle
from paper_2203_04508_amd import workloads as W

T = 0.70 * W.CS_TC
RV, RL = W.MAXWELL[0.70]
TAU = 0.8
TOL = {"f64": 1e-8, "f16s": 1e-7}


def case(dim):
    if dim == 2:
        dims, g = (18, 15, 1), (0.05, 0.0, 0.0)
        shapes = [W.band_y(-0.4, 1.7, 0), W.ball((8.3, 1.7), 2.9, 1)]
        drop = ((9.0, 9.0), 4.0)
    else:
        dims, g = (11, 10, 9), (0.2, 0.0, 0.0)
        shapes = [W.band_y(-0.4, 1.7, 0), W.ball((5.3, 1.7, 4.2), 2.4, 1)]
        drop = ((5.0, 6.0, 4.0), 3.0)
    return dims, g, np.array(shapes, np.int64), W.drop_field(dims, dim, [drop], RV, RL, 3.0)


class Reference:
    """One FP64 step and collision as torch functions of the populations (Q x N), the links' forcing terms (one per link)
    and phi (one per wall node)."""

    def __init__(self, dim, dims, g, shapes, single):
        import torch

        self.torch, self.nx, self.g = torch, dims[0], g
        P = oracle.make_params(dim, *dims, tau=TAU, T=T)
        self.e, self.w, _ = (np.asarray(a) for a in oracle.lattice(dim)[:3])
        e = self.e.reshape(len(self.w), -1)
        self.e = np.zeros((len(self.w), 3))
        self.e[:, : e.shape[1]] = e
        N = int(np.prod(dims))
        x = np.arange(N)
        c = np.stack([x % dims[0], x // dims[0] % dims[1], x // (dims[0] * dims[1])])
        at = lambda k: (lambda p: p[0] + dims[0] * (p[1] + dims[1] * p[2]))((c + k[:, None]) % np.array(dims)[:, None])
        self.nb = np.stack([at(k.astype(int)) for k in self.e])  # x + e_i
        self.opp = np.array([int(np.flatnonzero((self.e == -k).all(1))[0]) for k in self.e])
        self.src = self.nb[self.opp]                             # x - e_i
        self.solid = oracle.classify(P, shapes) != 0
        self.node, self.d, cls, q = (np.asarray(a, np.int64) for a in oracle.links(P, shapes, oracle.classify(P, shapes)))
        self.walls = np.asarray(oracle.wall_nodes(P, oracle.classify(P, shapes)), np.int64)
        q2 = q * (2.0 / 65536.0)
        c1 = np.where(cls == 0, q2, np.where(cls == 2, 1.0 / np.maximum(q2, 1e-300), 1.0))
        self.c1 = torch.tensor(c1.astype(np.float32).astype(np.float64) if single else c1)
        self.eq16 = torch.tensor(cls == 0)
        self.W, self.E = torch.tensor(self.w), torch.tensor(self.e)
        self.fluid = torch.tensor(~self.solid, dtype=torch.float64)
        # force stencil: sum of w^ e e = identity
        n2 = (self.e ** 2).sum(1)
        self.wf = torch.tensor(np.where(n2 == 0, 0, np.where(n2 == 1, 1 / 3 if dim == 2 else 1 / 6, 1 / 12)))

    def psi(self, r):
        eta = r  # b = 4: eta = b rho / 4
        p = r * T * (1 + eta + eta ** 2 - eta ** 3) / (1 - eta) ** 3 - r * r
        return (2.0 * (r / 3.0 - p)).sqrt()  # G = -1

    def force(self, rho, phi):
        t = self.torch
        num, den = 0.0, 0.0
        for i in range(1, len(self.w)):
            y = self.nb[i][self.walls]
            num = num + self.w[i] * (rho * self.fluid)[y]
            den = den + self.w[i] * self.fluid[y]
        r = t.where(self.fluid > 0, rho, t.full_like(rho, RV)).index_put((t.tensor(self.walls),), phi * num / den)
        has = self.fluid.index_put((t.tensor(self.walls),), t.ones(len(self.walls), dtype=t.float64))
        psi = self.psi(r) * has
        F = t.stack([psi * sum(self.wf[i] * self.e[i, k] * psi[self.nb[i]] for i in range(1, len(self.w))) for k in range(3)])
        return (F + rho * t.tensor(self.g, dtype=t.float64)[:, None]) * self.fluid

    def eq(self, rho, m):  # E_i(rho, m)
        r = self.torch.where(self.fluid > 0, rho, self.torch.ones_like(rho))
        em = self.E @ m
        return self.W[:, None] * (rho + 3 * em + (4.5 * em * em - 1.5 * (m * m).sum(0)) / r)

    def terms(self, rho, m, F):  # R of each link
        return (self.eq(rho, m + F) - self.eq(rho, m))[self.d, self.node]

    def collide(self, p, phi):
        rho, j = p.sum(0), self.E.T @ p
        F = self.force(rho, phi)
        return (p + (self.eq(rho, j) - p) / TAU + self.eq(rho, j + F) - self.eq(rho, j)) * self.fluid, self.terms(rho, j, F)

    def pull(self, g, R):
        t = self.torch
        i = t.arange(len(self.w))[:, None]
        p = g[i, t.tensor(self.src)]
        nd, d, o = t.tensor(self.node), t.tensor(self.d), t.tensor(self.opp[self.d])
        other = t.where(self.eq16, g[d, t.tensor(self.src[self.d, self.node])], g[o, nd])
        fin = self.c1 * g[d, nd] + (1 - self.c1) * (other + R)
        p = p.index_put((o, nd), fin)
        p0 = p[0].index_add(0, nd, g[d, nd] - fin)
        return t.cat([p0[None], p[1:]]) * self.fluid

    def stored_terms(self, g, phi):  # R from the stored populations and the record's force
        t = self.torch
        rho, j = g.sum(0), self.E.T @ g
        F = self.force(rho, phi)
        return self.terms(rho, j - F, F)

    def gradient(self, rho0, states, phi):
        """d COM_X / d phi from the states of times 0 .. n."""
        t = self.torch
        phi = t.tensor(phi)
        g = [t.tensor(s) for s in states]
        X = t.arange(g[0].shape[1]) % self.nx
        ex = (g[-1].sum(0) - RV) * self.fluid
        d = (X - (X * ex).sum() / ex.sum()) / ex.sum() * self.fluid
        lam, lamR, grad = d.expand(len(self.w), -1), t.zeros(len(self.node), dtype=t.float64), t.zeros_like(phi)
        for gt in g[-2::-1]:
            a, R, ph = gt.clone().requires_grad_(), self.stored_terms(gt, phi).requires_grad_(), phi.clone().requires_grad_()
            g1, R1 = self.collide(self.pull(a, R), ph)
            lam, lamR, gp = t.autograd.grad((lam * g1).sum() + (lamR * R1).sum(), (a, R, ph))
            grad = grad + gp
        ph = phi.clone().requires_grad_()
        g1, R1 = self.collide(self.W[:, None] * t.tensor(rho0.reshape(-1)) * self.fluid, ph)
        return (grad + t.autograd.grad((lam * g1).sum() + (lamR * R1).sum(), ph)[0]).numpy()


def test_reference_against_dual_numbers():
    """(on the CPU) the reference sweep over the oracle's FP64 states is the oracle's own derivative"""
    for dim in (2, 3):
        dims, g, shapes, rho0 = case(dim)
        P = oracle.make_params(dim, *dims, tau=TAU, T=T)
        solid = oracle.classify(P, shapes)
        node, d, _, q = oracle.links(P, shapes, solid)
        n = len(oracle.wall_nodes(P, solid))
        phi, dirs = np.random.default_rng(dim).uniform(0.95, 1.05, n), np.random.default_rng(9).standard_normal((4, n))
        sim, _ = oracle.sim_from_shapes(P, shapes)
        ds = oracle.DualSim(P, solid, node, d, q)
        for s in (sim, ds):
            s.set_gravity(g[:dim] if dim == 3 else g[:2])
        sim.set_phi(phi)
        ds.set_phi(phi, dirs)
        sim.init_eq(rho0)
        ds.init_eq(rho0)
        states = [sim.get_f()]
        for _ in range(2):
            sim.step(1)
            states.append(sim.get_f())
        ds.step(2)
        ref = Reference(dim, dims, g, shapes, False)
        _, dL = ds.loss(0, (RV, 1.0))
        e = np.abs(dirs @ ref.gradient(rho0, states, phi) - dL).max() / np.abs(dL).max()
        assert e < 1e-10, (dim, e)


@pytest.mark.gpu
@pytest.mark.parametrize("prec", list(TOL))
@pytest.mark.parametrize("dim", [2, 3])
def test_gradient_at_the_stored_states(dim, prec):
    import torch  # before the library: both use the HIP runtime that torch brings

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2203_04508_amd import mcb

    mcb.load()
    print(f"\n[case] gradient at the stored states, {dim}-D {prec}", flush=True)
    dims, g, shapes, rho0 = case(dim)
    lat = mcb.Lattice(dim, dims, TAU, T, precision=prec, rho_ref=0.0 if prec == "f64" else RV, gravity=g)
    lat.set_geometry(shapes)
    phi = np.random.default_rng(dim).uniform(0.95, 1.05, lat.n_wall)
    lat.set_wettability(phi)
    lat.init_equilibrium(rho0)
    states = [lat.get_f()]
    for _ in range(2):
        lat.step(1)
        states.append(lat.get_f())
    lat.adj_forward(rho0, 2, 2, 0, (RV, 1.0))
    grad = lat.adj_backward(1.0)
    lat.close()
    ref = Reference(dim, dims, g, shapes, prec != "f64")
    want = ref.gradient(rho0, states, phi)
    e = np.linalg.norm(grad - want) / np.linalg.norm(want)
    assert e < TOL[prec], e
