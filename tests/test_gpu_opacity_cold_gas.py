"""kappa(T) on a gas whose total energy is below its kinetic energy: no temperature exists, and whatever the
law's exponents the cell comes back non-finite and rt_diagnostics counts it, as with any power of a
negative number; its neighbours are untouched by it.  Thermal energy zero is the same, except that rising
laws have no opacity there and leave the cell as it was."""
import numpy as np
import pytest
import torch

from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu


def _source(b, thermal, K, dtype):
    p = inp.make_problem(0, n=6, K=K, steps=1)
    st, ph, at = p.state, p.phys, 41
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")  # noqa: E731
    mom, etot = st.mom.copy(), st.etot.copy()
    mom[at] = 0.0
    etot[at] = thermal * st.rho[at] * ph.cv
    mesh = rt.Mesh.from_inputs(p.mesh, st.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, p.dt, dtype)
    I, m, e = d(st.I).to(rt.torch_dtype(dtype)), d(mom), d(etot)
    before = I.clone()
    rt.source_implicit_kT(mesh, prm, ang, I, d(st.rho), m, e, d(st.kP), d(st.kJ), d(st.ks), 1.0, b[0], b[1])
    counted = rt.diagnostics(mesh, prm, ang, I, d(st.vol), e, m, allow_nonfinite=True)[9]
    row, bad = I[at], ~torch.isfinite(I)
    bad[at] = False
    mesh.free()
    assert not bool(bad.any())
    return before[at], row, counted, K


LAWS = [(1.0, 1.0), (2.0, 2.0), (-2.0, -2.0), (-3.5, -3.5), (-3.3, -3.3), (0.0, 0.0), (2.0, -1.0), (0.0, 1.0)]


@pytest.mark.parametrize("b", LAWS)
@pytest.mark.parametrize("K", [24, 80])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_negative_thermal_energy_is_reported(dtype, K, b):
    _, row, counted, K = _source(b, -0.3, K, dtype)
    assert bool(torch.isnan(row).all())
    assert counted == K + 4  # the row, the gas energy and the three momenta


@pytest.mark.parametrize("b", LAWS)
def test_zero_thermal_energy(b):
    before, row, counted, K = _source(b, 0.0, 24, rt.F64)
    if min(b) > 0.0:
        assert bool(torch.isfinite(row).all()) and counted == 0
    else:
        assert bool(torch.isnan(row).all()) and counted == K + 4
