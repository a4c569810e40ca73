"""Multigroup and kappa(T) steps on a mesh whose face records alone outgrow half the LDS, so that no one-kernel
form has room and the transport and the source are launched apart, against the oracle.

The mesh is a cubic lattice whose faces at the slab x < n/2 are each cut in 75; that its records do not
fit is asserted from the face counts of 16 consecutive cells (the fewest a workgroup takes).

Tolerances: 1e-12 in FP64; in FP32 450 faces of rounding add up to at most 450 eps = 2.7e-5.
"""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_helpers import rel_err
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu

TOL = {rt.F64: 1e-12, rt.F32: 2.7e-5}
HALF_LDS = 81920


def _cut_lattice(n=6, cuts=(5, 15)):
    """Unjittered periodic n^3 lattice, every face with a cell of the slab on a side in cuts[0] x cuts[1] parts."""
    h = 1.0 / n
    x, y, z = (a.ravel(order="F") for a in np.meshgrid(*[np.arange(n)] * 3, indexing="ij"))
    site = np.stack([x, y, z], axis=1)
    gen = (site + 0.5) * h
    fc, fs, fa, fn, fcen = [], [], [], [], []
    for i in range(n ** 3):
        for ax in range(3):
            nb = site[i].copy()
            nb[ax] = (nb[ax] + 1) % n
            j = int(nb[0] + n * nb[1] + n * n * nb[2])
            e = np.eye(3)[ax]
            shift = (np.eye(3)[ax] * (site[i, ax] == n - 1)).astype(np.int8)
            a, b = cuts if min(site[i, 0], nb[0]) < n // 2 else (1, 1)
            t1, t2 = [t for t in range(3) if t != ax]
            for p in range(a * b):
                c = gen[i] + 0.5 * h * e
                c[t1] += ((p // b + 0.5) / a - 0.5) * h
                c[t2] += ((p % b + 0.5) / b - 0.5) * h
                fc.append((i, j))
                fs.append(shift)
                fa.append(h * h / (a * b))
                fn.append(e)
                fcen.append(c)
    return inp.Mesh(n=n, box=1.0, gen=gen, com=gen.copy(), vol=np.full(n ** 3, h ** 3), cell_lat=site.astype(np.int32),
                    face_cells=np.array(fc, np.int32), face_shift=np.array(fs, np.int8), face_area=np.array(fa),
                    face_normal=np.array(fn), face_centroid=np.array(fcen))


def _setup(K, dtype):
    mesh, ph = _cut_lattice(), inp.Physics()
    faces = np.bincount(mesh.face_cells.ravel(), minlength=mesh.n_cells)
    most = max(int(faces[c:c + 16].sum()) for c in range(0, mesh.n_cells, 16))
    assert most * (20 if dtype == rt.F32 else 36) > 1.05 * HALF_LDS
    st = inp.initial_state(mesh, K, inp.seed_streams(0), ph)
    dirs, w = inp.angle_set(K)
    dt = inp.courant_dt(mesh, ph.c_red)
    return mesh, st, ph, dirs, w, dt, orc.OracleMesh(mesh, st.mesh_vel)


def _d(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")


def _transported(om, dirs, w, ph, dt, I, st, k, ks):
    return orc.step(om, dirs, w, ph, dt, orc.OState(I.copy(), st.vol.copy(), st.mom.copy(), st.etot.copy()), st.rho, k,
                    k, ks, with_source=False)[0]


@pytest.mark.parametrize("b", [(-3.5, -3.5), (-3.3, -2.0)])
@pytest.mark.parametrize("K", [24, 80])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_opacity_step(dtype, K, b):
    m, st, ph, dirs, w, dt, om = _setup(K, dtype)
    mesh, ang = rt.Mesh.from_inputs(m, st.mesh_vel, k_max=K), rt.AngleSet(dirs, w)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, dt, dtype)
    I = _d(st.I).to(rt.torch_dtype(dtype))
    O = torch.full_like(I, float("nan"))
    vol, mom, etot, T = _d(st.vol), _d(st.mom), _d(st.etot), _d(np.zeros(m.n_cells))
    rt.step_kT(mesh, prm, ang, I, O, vol, _d(st.rho), mom, etot, _d(st.kP), _d(st.kP), _d(st.ks), 1.1, b[0], b[1], T)
    tr = _transported(om, dirs, w, ph, dt, I.double().cpu().numpy(), st, st.kP, st.ks)
    Io, mo, eo, To = orc.source_kT(dirs, w, ph, dt, tr.I, st.rho, st.mom, st.etot, st.kP, st.kP, st.ks, 1.1, b[0], b[1])
    assert rel_err(O.double().cpu().numpy(), Io) < TOL[dtype]
    assert rel_err(vol.cpu().numpy(), tr.vol) < 1e-14
    assert rel_err(T.cpu().numpy(), To) < TOL[dtype]
    if dtype == rt.F64:
        assert rel_err(etot.cpu().numpy(), eo) < 1e-12 and rel_err(mom.cpu().numpy(), mo) < 1e-12
    mesh.free()


@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("K", [24, 48])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_multigroup_step(dtype, K, G):
    m, st, ph, dirs, w, dt, om = _setup(K, dtype)
    mesh, ang = rt.Mesh.from_inputs(m, st.mesh_vel, k_max=K), rt.AngleSet(dirs, w)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, dt, dtype)
    scale = np.arange(1.0, G + 1)[:, None]
    I = _d(st.I[None] * scale[:, :, None]).to(rt.torch_dtype(dtype))
    k, ks, wg = st.kP[None] * scale, st.ks[None] * np.ones((G, 1)), np.full(G, 1.0 / G)
    O = torch.full_like(I, float("nan"))
    vol, mom, etot, T = _d(st.vol), _d(st.mom), _d(st.etot), _d(np.zeros(m.n_cells))
    rt.step_mg(mesh, prm, ang, _d(wg), I, O, vol, _d(st.rho), mom, etot, _d(k), _d(k), _d(ks), T)
    tr = [_transported(om, dirs, w, ph, dt, I[j].double().cpu().numpy(), st, k[j], ks[j]) for j in range(G)]
    Io, mo, eo, To = orc.source_mg(dirs, w, wg, ph, dt, np.stack([t.I for t in tr]), st.rho, st.mom, st.etot, k, k, ks)
    assert rel_err(O.double().cpu().numpy(), Io) < TOL[dtype]
    assert rel_err(vol.cpu().numpy(), tr[0].vol) < 1e-14
    assert rel_err(T.cpu().numpy(), To) < TOL[dtype]
    if dtype == rt.F64:
        assert rel_err(etot.cpu().numpy(), eo) < 1e-12 and rel_err(mom.cpu().numpy(), mo) < 1e-12
    mesh.free()
