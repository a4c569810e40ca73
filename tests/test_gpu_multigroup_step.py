"""Multigroup steps over the forms of the whole-step kernel: one group, an odd and an even number of
them, rows that wait in registers only or in LDS too, and more groups than LDS holds (the separate
launches), in paired and general lane layouts, against the oracle.

Tolerances: those of the same comparison at three groups, 1e-12 normwise in FP64 and 1e-5 on the
intensities in FP32.
"""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as orc
from gpu_helpers import rel_err
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt
from test_gpu_multigroup import TOL, _d, _mg_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,layout", [(24, "half"), (80, "adjacent"), (80, "half"), (37, "subset"), (120, "half")])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 16])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_step_mg_forms_match_oracle(dtype, G, K, layout):
    p, I, kP, kJ, ks, Wg = _mg_problem(120 if layout == "subset" else K, G, n=6)
    perm = np.arange(K) if layout != "adjacent" else inp.adjacent_pair_order(K)
    p, I = inp.with_angle_order(p, perm), np.ascontiguousarray(I[:, :, perm])
    if layout == "subset":
        p = dataclasses.replace(p, weights=np.full(K, 1.0 / K))
    st, ph = p.state, p.phys
    mesh = rt.Mesh.from_inputs(p.mesh, st.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, p.dt, dtype)
    td = rt.torch_dtype(dtype)
    Ia, Ib = _d(I).to(td), torch.full((G,) + st.I.shape, float("nan"), dtype=td, device="cuda")
    vol, mom, etot = _d(st.vol), _d(st.mom), _d(st.etot)
    T = torch.zeros(p.mesh.n_cells, dtype=torch.float64, device="cuda")
    om = orc.OracleMesh(p.mesh, st.mesh_vel)
    Io, vo, mo, eo = I.copy(), st.vol.copy(), st.mom.copy(), st.etot.copy()
    for _ in range(2):
        rt.step_mg(mesh, prm, ang, _d(Wg), Ia, Ib, vol, _d(st.rho), mom, etot, _d(kP), _d(kJ), _d(ks), T)
        Ia, Ib = Ib, Ia
        tr = [orc.step(om, p.dirs, p.weights, ph, p.dt, orc.OState(Io[j], vo, mo, eo), st.rho, kP[j], kJ[j], ks[j],
                       with_source=False)[0] for j in range(G)]
        vo = tr[0].vol
        Io, mo, eo, To = orc.source_mg(p.dirs, p.weights, Wg, ph, p.dt, np.stack([t.I for t in tr]), st.rho, mo, eo,
                                       kP, kJ, ks)
    assert rel_err(Ia.double().cpu().numpy(), Io) < TOL[dtype]
    assert rel_err(vol.cpu().numpy(), vo) < 1e-14
    if dtype == rt.F64:
        assert rel_err(T.cpu().numpy(), To) < 1e-12
        assert rel_err(etot.cpu().numpy(), eo) < 1e-12
        assert rel_err(mom.cpu().numpy(), mo) < 1e-12
    mesh.free()
