"""Rounding of the power law kappa0 (T/T_ref)^b near T_ref.  Gas at rest without scattering and without
incoming radiation leaves every angle with I' = y kP B / (1 + y kJ), y = dt cbar rho, B = a T^4 / 4 pi, at the
temperature the source returns, so the law's error shows in the intensities; T_ref = 1 and powers of two
elsewhere keep other roundings few.

Tolerance: about 14 of at most half an eps each in y, B, the product and the quotient (7 eps), and 2 + |b ln x|
ulp of the law with |b ln x| < 1: 10 eps.  (x^20 by plain repeated squaring is up to 10 eps off, x^-20 up to 20.)
"""
import numpy as np
import pytest
import torch

from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("K", [24, 80])
@pytest.mark.parametrize("b", [20.0, -20.0, 19.5, -19.5, -3.5, -0.5, 0.5, 1.0, -1.0, 0.0, 7.5, -16.0, 16.0, -3.3])
def test_law_near_the_reference_temperature(b, K):
    p = inp.make_problem(0, n=12, K=K, steps=1)
    N = p.mesh.n_cells
    dt, c_red, c, cv = 2.0 ** -12, 4.0, 64.0, 2.0 ** 10
    rng = np.random.default_rng(8)
    Tg = np.exp(rng.uniform(-0.045, 0.045, N))
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")  # noqa: E731
    mesh = rt.Mesh.from_inputs(p.mesh, p.state.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(c_red, c, 1.0, cv, dt, rt.F64)
    one, zero = np.ones(N), np.zeros(N)
    I, T = d(np.zeros((N, K))), d(zero)
    rt.source_implicit_kT(mesh, prm, ang, I, d(one), d(np.zeros((N, 3))), d(cv * Tg), d(one), d(one), d(zero), 1.0, b, b, T)
    mesh.free()
    x = T.cpu().numpy().astype(np.longdouble)
    assert float(np.max(np.abs(np.log(x)))) < 0.05
    k = x ** np.longdouble(b)
    y = np.longdouble(dt * c_red)
    ref = (y * k * x ** 4 / (4.0 * np.longdouble("3.14159265358979323846"))) / (1.0 + y * k)
    err = float(np.max(np.abs(I.cpu().numpy() - ref[:, None]) / ref[:, None]))
    print(b, K, err / EPS)
    assert err < 10.0 * EPS
