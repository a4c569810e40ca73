"""kappa(T) power laws on either side of the kernel's rule: whole and half-whole exponents are formed by
repeated multiplication, others by exp(b ln x).  Both against the oracle's pow, at exponents up to the
allowed +-20, in the paired (4 and 8 lanes, 12 angles per lane) and the general layouts.

Tolerance: the temperature root and the intensities follow the opacities with logarithmic sensitivities
of order one here (unique roots), and either power is within (|b| + |b ln x| + 3) ulp of x^b with
|ln x| < 1, so 64 ulp; sums over angles add up to K ulp: 1e-12 leaves a factor 20 in FP64.
"""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_helpers import rel_err
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bP,bJ", [(0.5, 0.5), (-0.5, 2.5), (7.5, -2.0), (20.0, 20.0), (-20.0, -19.5), (0.3, 0.3),
                                   (-3.5000001, -3.5), (1.0, 0.25)])
@pytest.mark.parametrize("K", [24, 37, 96, 120])
def test_power_rule_matches_oracle(K, bP, bJ):
    p = inp.make_problem(0, n=6, K=K if K in (24, 120) else 120, steps=1)
    st, ph = p.state, p.phys
    if K == 37:
        rng = np.random.default_rng(3)
        d = rng.normal(size=(K, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
    elif K == 96:  # antipodal pairs, 12 angles per lane
        rng = np.random.default_rng(4)
        d = rng.normal(size=(K // 2, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        d = np.concatenate([d, -d])
    else:
        d = p.dirs
    d = np.ascontiguousarray(d)
    w = np.full(K, 1.0 / K)
    I0 = np.ascontiguousarray(st.I[:, :K])
    mesh = rt.Mesh.from_inputs(p.mesh, st.mesh_vel, k_max=K)
    ang = rt.AngleSet(d, w)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, p.dt, rt.F64)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")
    I, mom, etot = t(I0), t(st.mom), t(st.etot)
    T = torch.zeros(p.mesh.n_cells, dtype=torch.float64, device="cuda")
    Tr = 1.1
    rt.source_implicit_kT(mesh, prm, ang, I, t(st.rho), mom, etot, t(st.kP), t(st.kJ), t(st.ks), Tr, bP, bJ, T)
    Io, mo, eo, To = orc.source_kT(d, w, ph, p.dt, I0, st.rho, st.mom, st.etot, st.kP, st.kJ, st.ks, Tr, bP, bJ)
    assert rel_err(T.cpu().numpy(), To) < 1e-12
    assert rel_err(I.cpu().numpy(), Io) < 1e-12
    assert rel_err(etot.cpu().numpy(), eo) < 1e-12
    assert rel_err(mom.cpu().numpy(), mo) < 1e-12
    mesh.free()
