"""The temperature of the kappa(T) source, element by element, on cells far from equilibrium (radiation
temperatures spread lognormally by a factor e around the gas's), where Newton's first steps are long and
a short step after a long one says little about the next.

Tolerance 1e-13, relative per cell, on 110,592 cells a law: f's terms carry up to 2 K + 30 roundings
(1.7e-14 at K = 24) in either program, and for these laws every term of f' T has the sign of rho cv T
and the terms' magnitudes add up to at most four times it, so a root is fixed to 7e-14; the oracle ends
at a step of 1e-14 T.
"""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bP,bJ", [(-3.5, -3.5), (-2.0, -2.0), (1.0, 1.0), (-3.5, -2.0), (-3.3, -2.0)])
def test_root_far_from_equilibrium(bP, bJ):
    K, n = 24, 16
    p = inp.make_problem(0, n=n, K=K, steps=1)
    N = p.mesh.n_cells
    ph = inp.Physics(c_red=100.0, c_light=1000.0)
    dt = 1e-2
    mesh = rt.Mesh.from_inputs(p.mesh, p.state.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, dt, rt.F64)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")  # noqa: E731
    worst = 0.0
    for draw in range(27):
        rng = np.random.default_rng(draw)
        rho = np.exp(rng.normal(0.0, 0.5, N))
        Tg = rng.uniform(0.5, 2.0, N)
        v = rng.normal(0.0, 0.1, (N, 3))
        mom = rho[:, None] * v
        etot = rho * ph.cv * Tg + 0.5 * rho * np.sum(v * v, axis=1)
        Tr = Tg * np.exp(rng.normal(0.0, 1.0, N))
        I0 = ph.a_rad * Tr[:, None] ** 4 / (4.0 * np.pi) * rng.uniform(0.9, 1.1, (N, K))
        k0, ks = 10.0 ** rng.uniform(-1.0, 1.0, N), np.full(N, 0.1)
        I, m, e, T = d(I0), d(mom), d(etot), d(np.zeros(N))
        rt.source_implicit_kT(mesh, prm, ang, I, d(rho), m, e, d(k0), d(k0), d(ks), 1.0, bP, bJ, T)
        To = orc.source_kT(p.dirs, p.weights, ph, dt, I0, rho, mom, etot, k0, k0, ks, 1.0, bP, bJ)[3]
        worst = max(worst, float(np.max(np.abs(T.cpu().numpy() - To) / To)))
    print(bP, bJ, worst)
    mesh.free()
    assert worst < 1e-13
