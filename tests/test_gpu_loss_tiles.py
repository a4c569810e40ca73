"""The flux loss on both sides of its change of tiles (fewer or more than 256 workgroups of 64 cells: 16 or 32
cells each below, 64 above, the last one partly filled), with no, one, few and all faces weighted.

Tolerance: as for any order of a sum of n terms, 2 n eps times the sum of their magnitudes; a seed is one
rounding of its type and a few of FP64.
"""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_helpers import DeviceProblem
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
@pytest.mark.parametrize("n,K", [(25, 8), (25, 80), (26, 8), (26, 80)])
def test_loss_on_both_sides_of_the_tile_rule(dtype, n, K):
    dp = DeviceProblem(inp.make_problem(0, n=n, K=K, steps=1), dtype=dtype)
    m, c = dp.p.mesh, dp.p.phys.c_light
    F, I = m.n_faces, dp.I.double().cpu().numpy()
    rng = np.random.default_rng(6)
    one = np.zeros(F)
    one[F // 3] = 0.4
    for u in (np.zeros(F), one, np.where(rng.uniform(size=F) < 0.05, 1.0, 0.0), rng.uniform(-1.0, 1.0, F)):
        loss, seed = torch.full((1,), 3.0, dtype=torch.float64, device="cuda"), torch.ones_like(dp.I)
        rt.flux_loss(dp.mesh, dp.params, dp.angles, dp.I, torch.as_tensor(u, device="cuda"), loss, seed)
        ref, ref_seed = orc.flux_loss(dp.om, dp.p.dirs, dp.p.weights, c, I, u, want_seed=True)
        size = float(np.sum(np.abs(u) * m.face_area)) * 4.0 * np.pi * c * float(np.max(np.abs(I)))
        assert abs(float(loss) - ref) <= (2.0 * F * K + 16.0) * EPS * size
        eps = np.finfo(np.float32).eps if dtype == rt.F32 else EPS
        err = np.max(np.abs(seed.double().cpu().numpy() - (1.0 + ref_seed)))
        assert err <= (64.0 * EPS + eps) * (1.0 + np.max(np.abs(ref_seed)))
    dp.mesh.free()
