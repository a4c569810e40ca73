"""Multigroup steps of sets with antipodal pairs whose rows do not fit in their paired layout, on both sides of
the mesh size from which they take separate launches instead of the general one-kernel form, against the
same update made call by call (each call is compared with the oracle elsewhere).

Tolerances: sums in another order only, 1e-13 in FP64 (about 100 roundings) and 1e-6 in FP32.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import rel_err
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32, 33])
@pytest.mark.parametrize("dtype,K,G", [(rt.F32, 80, 12), (rt.F64, 48, 10), (rt.F64, 80, 8), (rt.F32, 48, 16)])
def test_step_equals_separate_calls(dtype, K, G, n):
    p = inp.make_problem(0, n=n, K=K, steps=1)
    st, ph, N = p.state, p.phys, p.mesh.n_cells
    mesh = rt.Mesh.from_inputs(p.mesh, st.mesh_vel, k_max=K)
    ang = rt.AngleSet(p.dirs, p.weights)
    prm = rt.make_params(ph.c_red, ph.c_light, ph.a_rad, ph.cv, p.dt, dtype)
    d = lambda a: torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda")  # noqa: E731
    scale = torch.arange(1.0, G + 1, dtype=torch.float64, device="cuda")[:, None]
    I = (d(st.I)[None] * scale[:, :, None]).to(rt.torch_dtype(dtype)).contiguous()
    k, ks, wg = (d(st.kP)[None] * scale).contiguous(), (d(st.ks)[None] + 0.0 * scale).contiguous(), torch.full_like(scale[:, 0], 1.0 / G)
    out = []
    for whole in (True, False):
        vol, mom, etot = d(st.vol), d(st.mom), d(st.etot)
        T, O = torch.zeros(N, dtype=torch.float64, device="cuda"), torch.full_like(I, float("nan"))
        if whole:
            rt.step_mg(mesh, prm, ang, wg, I, O, vol, d(st.rho), mom, etot, k, k, ks, T)
        else:
            for j in range(G):
                v = vol.clone()
                rt.transport_step(mesh, prm, ang, I[j], O[j], v)
            vol = v
            rt.source_implicit_mg(mesh, prm, ang, wg, O, d(st.rho), mom, etot, k, k, ks, T)
        out.append([x.double().cpu().numpy() for x in (O, vol, mom, etot, T)])
    for x, y in zip(*out):
        assert rel_err(x, y) < (1e-13 if dtype == rt.F64 else 1e-6)
    mesh.free()
