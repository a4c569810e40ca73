"""Conservation totals of a state with one infinite intensity: the energy and the flux totals are infinite with
that intensity's sign and directions, not NaN, wherever the entry sits -- in the first or last cell (the
last one is also what the idle lanes of a last tile look at) and in angle 0 (which the idle slots of sets
that do not fill their lanes look at) -- and the minimum, the gas totals and the count stay what they are.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import DeviceProblem
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
@pytest.mark.parametrize("n,K", [(5, 8), (6, 24), (5, 37), (5, 80), (6, 90)])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_one_infinite_intensity(dtype, n, K, value):
    p = inp.make_problem(0, n=n, K=K if K in (8, 24, 80) else 120, steps=1)
    if K in (37, 90):
        rng = np.random.default_rng(2)
        d = rng.normal(size=(K, 3))
        p.dirs = np.ascontiguousarray(d / np.linalg.norm(d, axis=1, keepdims=True))
        p.weights = np.full(K, 1.0 / K)
        p.state.I = np.ascontiguousarray(p.state.I[:, :K])
    dp = DeviceProblem(p, dtype=dtype)
    totals = lambda I, **kw: rt.diagnostics(dp.mesh, dp.params, dp.angles, I, dp.vol, dp.etot, dp.mom, **kw)  # noqa: E731
    plain = totals(dp.I)
    for cell in (0, p.mesh.n_cells // 2, p.mesh.n_cells - 1):
        for k in (0, K - 1):
            I = dp.I.clone()
            I[cell, k] = value
            got = totals(I, allow_nonfinite=True)
            sign = np.sign(value) * np.concatenate([[1.0], np.sign(p.dirs[k])])
            assert np.array_equal(got[[1, 5, 6, 7]], sign * np.inf), (cell, k, got)
            assert np.array_equal(got[[0, 2, 3, 4]], plain[[0, 2, 3, 4]])
            assert got[8] == float(I.min()) and got[9] == 1
    dp.mesh.free()
