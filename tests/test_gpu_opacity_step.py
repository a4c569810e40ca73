"""Steps with kappa(T) in one kernel, over its lane layouts and both power forms, and on meshes whose
face records leave no room for it in LDS (transport and source launched apart), multigroup steps too.

Tolerances: those of the single-layout comparison, 1e-12 normwise in FP64 and 1e-5 on the intensities
in FP32 (rounding of the transported FP32 values).
"""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as orc
from gpu_helpers import rel_err
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt
from test_gpu_parity import _split_face_lattice_problem

pytestmark = pytest.mark.gpu

TOL = {rt.F64: 1e-12, rt.F32: 1e-5}


def _d(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def _check_kT(p, dtype, bP, bJ, steps=2):
    st, ph, K = p.state, p.phys, p.dirs.shape[0]
    mesh = rt.Mesh.from_inputs(p.mesh, st.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, p.dt, dtype)
    td = rt.torch_dtype(dtype)
    Ia, Ib = _d(st.I).to(td), torch.full(st.I.shape, float("nan"), dtype=td, device="cuda")
    vol, mom, etot = _d(st.vol), _d(st.mom), _d(st.etot)
    T = torch.zeros(p.mesh.n_cells, dtype=torch.float64, device="cuda")
    om = orc.OracleMesh(p.mesh, st.mesh_vel)
    so = orc.OState(st.I.copy(), st.vol.copy(), st.mom.copy(), st.etot.copy())
    for _ in range(steps):
        rt.step_kT(mesh, prm, ang, Ia, Ib, vol, _d(st.rho), mom, etot, _d(st.kP), _d(st.kJ), _d(st.ks), 1.1, bP, bJ, T)
        Ia, Ib = Ib, Ia
        tr = orc.step(om, p.dirs, p.weights, ph, p.dt, so, st.rho, st.kP, st.kJ, st.ks, with_source=False)[0]
        I, m, e, To = orc.source_kT(p.dirs, p.weights, ph, p.dt, tr.I, st.rho, so.mom, so.etot, st.kP, st.kJ, st.ks,
                                    1.1, bP, bJ)
        so = orc.OState(I, tr.vol, m, e)
    assert rel_err(Ia.double().cpu().numpy(), so.I) < TOL[dtype]
    assert rel_err(vol.cpu().numpy(), so.vol) < 1e-14
    if dtype == rt.F64:
        assert rel_err(T.cpu().numpy(), To) < 1e-12
        assert rel_err(etot.cpu().numpy(), so.etot) < 1e-12
        assert rel_err(mom.cpu().numpy(), so.mom) < 1e-12
    mesh.free()


@pytest.mark.parametrize("bP,bJ", [(-3.5, -3.5), (-3.3, -2.0)])
@pytest.mark.parametrize("K,layout", [(8, "half"), (24, "adjacent"), (48, "half"), (80, "adjacent"), (80, "half"),
                                      (120, "half"), (37, "subset"), (61, "subset"), (5, "subset")])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_step_kT_layouts_match_oracle(dtype, K, layout, bP, bJ):
    p = inp.make_problem(0, n=6, K=120 if layout == "subset" else K, steps=2)
    if layout == "adjacent":
        p = inp.with_angle_order(p, inp.adjacent_pair_order(K))
    elif layout == "subset":
        p = dataclasses.replace(inp.with_angle_order(p, np.arange(K)), weights=np.full(K, 1.0 / K))
    _check_kT(p, dtype, bP, bJ)


@pytest.mark.parametrize("K", [24, 80])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_step_kT_with_many_faces_matches_oracle(dtype, K):
    _check_kT(_split_face_lattice_problem(K, m=8), dtype, -3.5, -3.5, steps=1)


@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_step_mg_with_many_faces_equals_separate_calls(dtype, G):
    """The same update through transport_step per group and source_implicit_mg: sums in another order
    only, so 1e-13 in FP64 (16 faces or 100 angles of rounding, 1e-14) and 1e-6 in FP32."""
    p = _split_face_lattice_problem(48, m=8)
    st, ph, K, N = p.state, p.phys, 48, p.mesh.n_cells
    mesh = rt.Mesh.from_inputs(p.mesh, st.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, p.dt, dtype)
    td = rt.torch_dtype(dtype)
    scale = np.arange(1.0, G + 1)[:, None]
    I = _d(st.I[None] * scale[:, :, None]).to(td)
    k, ks, wg = _d(st.kP[None] * scale), _d(st.ks[None] * np.ones((G, 1))), _d(np.full(G, 1.0 / G))
    out = []
    for fused in (True, False):
        vol, mom, etot = _d(st.vol), _d(st.mom), _d(st.etot)
        T = torch.zeros(N, dtype=torch.float64, device="cuda")
        O = torch.full_like(I, float("nan"))
        if fused:
            rt.step_mg(mesh, prm, ang, wg, I, O, vol, _d(st.rho), mom, etot, k, k, ks, T)
        else:
            for j in range(G):
                v = vol.clone()
                rt.transport_step(mesh, prm, ang, I[j], O[j], v)
            vol = v
            rt.source_implicit_mg(mesh, prm, ang, wg, O, _d(st.rho), mom, etot, k, k, ks, T)
        out.append([x.double().cpu().numpy() for x in (O, vol, mom, etot, T)])
    for x, y in zip(*out):
        assert rel_err(x, y) < (1e-13 if dtype == rt.F64 else 1e-6)
    mesh.free()
