"""Loss and conservation totals where their tiling can go wrong: a last tile of 61, 24 or 25 of its 64
cells, both lane layouts, no weight at all, one weighted face and every face weighted,
and non-finite entries in the last cell.

Tolerances: a sum of n terms in any order differs from another order by at most 2 n eps times the sum of
the terms' magnitudes; each term carries a few roundings of its own (16 eps covers either side's).
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


def _problem(n, K, dtype):
    return DeviceProblem(inp.make_problem(0, n=n, K=K, steps=1), dtype=dtype)


@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
@pytest.mark.parametrize("n,K", [(5, 8), (5, 80), (6, 24), (9, 24)])
def test_loss_over_tiles(n, K, dtype):
    dp = _problem(n, K, dtype)
    F = dp.mesh.n_faces
    rng = np.random.default_rng(5)
    last = np.zeros(F)
    last[F - 1] = -0.7
    I = dp.I.double().cpu().numpy()
    for u in (np.zeros(F), last, rng.uniform(-1.0, 1.0, F)):
        loss = torch.full((1,), 3.0, dtype=torch.float64, device="cuda")
        seed = torch.ones_like(dp.I)
        rt.flux_loss(dp.mesh, dp.params, dp.angles, dp.I, torch.as_tensor(u, device="cuda"), loss, seed)
        other = torch.zeros_like(loss)
        rt.flux_loss_noalloc(dp.mesh, dp.params, dp.angles, dp.I, torch.as_tensor(u, device="cuda"), other)
        ref, ref_seed = orc.flux_loss(dp.om, dp.p.dirs, dp.p.weights, dp.p.phys.c_light, I, u, want_seed=True)
        # the sum of magnitudes: every face's largest possible term
        m = dp.p.mesh
        size = float(np.sum(np.abs(u) * m.face_area)) * 4.0 * np.pi * dp.p.phys.c_light * float(np.max(np.abs(I)))
        tol = (2.0 * F * K + 16.0) * EPS * size
        assert abs(float(loss) - ref) <= tol
        assert float(other) == float(loss)
        # the seed is added to, and rounded once to the intensities' type
        eps = np.finfo(np.float32).eps if dtype == rt.F32 else EPS
        got = seed.double().cpu().numpy()
        scale = 1.0 + np.max(np.abs(ref_seed))
        assert np.max(np.abs(got - (1.0 + ref_seed))) <= (64.0 * EPS + eps) * scale
        if not u.any():
            assert float(loss) == 0.0 and torch.equal(seed, torch.ones_like(seed))


@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
@pytest.mark.parametrize("n,K", [(5, 8), (6, 20), (5, 80), (7, 24)])
def test_totals_over_tiles(n, K, dtype):
    if K == 20:  # padded lanes: a set of no paired or level-symmetric layout
        rng = np.random.default_rng(1)
        p = inp.make_problem(0, n=n, K=24, steps=1)
        d = rng.normal(size=(K, 3))
        p.dirs = np.ascontiguousarray(d / np.linalg.norm(d, axis=1, keepdims=True))
        p.weights = np.full(K, 1.0 / K)
        p.state.I = np.ascontiguousarray(p.state.I[:, :K])
        dp = DeviceProblem(p, dtype=dtype)
    else:
        dp = _problem(n, K, dtype)
    st = dp.p.state
    I = dp.I.double().cpu().numpy()
    got = rt.diagnostics(dp.mesh, dp.params, dp.angles, dp.I, dp.vol, dp.etot, dp.mom)
    ref = orc.diagnostics(dp.p.dirs, dp.p.weights, dp.p.phys, I, st.vol, st.etot, st.mom)
    size = np.array(ref)
    rad = float(ref[1]) * dp.p.phys.c_red / dp.p.phys.c_light
    size[2:5] = np.sum(st.vol[:, None] * np.abs(st.mom), axis=0)
    size[5:8] = rad / dp.p.phys.c_red
    tol = (2.0 * I.size + 16.0) * EPS * np.abs(size)
    assert np.all(np.abs(got - ref)[:8] <= tol[:8])
    assert got[8] == I.min() and got[9] == 0
    # non-finite entries of the last cell, in its first and last angle and its gas state
    dp.I[-1, 0] = float("nan")
    dp.I[-1, K - 1] = float("inf")
    dp.mom[-1, 1] = float("-inf")
    got = rt.diagnostics(dp.mesh, dp.params, dp.angles, dp.I, dp.vol, dp.etot, dp.mom, allow_nonfinite=True)
    assert got[9] == 3
