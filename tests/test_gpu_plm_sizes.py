"""PLM-VL2 steps at the sizes where stage 2 takes another form: the mesh is just above or below a size from
which it addresses its own rows past the caches (81,920 cells or 22 MB), or gathers fewer states of
a pair (workgroups per compute unit), and in every paired layout.

Two steps on faces that move at 0.3 of the reduced speed of light, where both directions of an antipodal pair
often enter through one face, against the oracle.  Tolerances: those of the same comparison on small
meshes, 1e-12 normwise in FP64 and 1e-5 on the intensities in FP32.
"""
import numpy as np
import pytest

from gpu_helpers import DeviceProblem, regime_problem, rel_err
from paper_2002_08377_amd import inputs as inp
from paper_2002_08377_amd import rt

pytestmark = pytest.mark.gpu


def _check(dtype, n, K, order):
    p = regime_problem("reduced_fast", index=1, n=n, K=K, steps=2)
    if order == "adjacent":
        p = inp.with_angle_order(p, inp.adjacent_pair_order(K))
    _compare(p, dtype)


def _compare(p, dtype):
    dp = DeviceProblem(p, dtype=dtype, scheme=rt.PLM_VL2)
    dp.run_gpu(p.steps)
    so, To = dp.run_oracle(p.steps, "plm_vl2")
    err = rel_err(dp.host(dp.I), so.I)
    print(dtype, p.mesh.n_cells, p.dirs.shape[0], err)
    assert err < (1e-12 if dtype == rt.F64 else 1e-5)
    if dtype == rt.F64:
        assert rel_err(dp.T.cpu().numpy(), To) < 1e-12
    dp.mesh.free()


@pytest.mark.parametrize("dtype,n,K", [(rt.F64, 43, 24), (rt.F64, 44, 24), (rt.F64, 39, 48), (rt.F64, 40, 48), (rt.F32, 43, 48), (rt.F32, 44, 48)])
def test_rows_past_the_caches(dtype, n, K):
    _check(dtype, n, K, "adjacent")


# Workgroups per compute unit (256 of them; 32 cells each, 64 at K = 8, 24 and 40) decide which states of a pair
# are gathered: at most one (FP32 also two below 8 angles per lane), more, and in FP32 more than ten.
@pytest.mark.parametrize("order", ["half", "adjacent"])
@pytest.mark.parametrize("dtype,n,K", [(rt.F32, 8, 24), (rt.F32, 32, 8), (rt.F32, 33, 8), (rt.F32, 33, 24), (rt.F32, 25, 48),
                                       (rt.F32, 26, 48), (rt.F32, 20, 80), (rt.F32, 21, 80), (rt.F32, 43, 80),
                                       (rt.F32, 44, 80), (rt.F64, 20, 80), (rt.F64, 21, 80)])
def test_gathered_states(dtype, n, K, order):
    _check(dtype, n, K, order)


def _pairs(K, order):
    """K angles in antipodal pairs, of any even K."""
    rng = np.random.default_rng(K)
    d = rng.normal(size=(K // 2, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    d = np.concatenate([d, -d])
    return np.ascontiguousarray(d[inp.adjacent_pair_order(K)] if order == "adjacent" else d)


@pytest.mark.parametrize("order", ["half", "adjacent"])
@pytest.mark.parametrize("n", [6, 29])
@pytest.mark.parametrize("K", [16, 32, 40, 64, 96])
@pytest.mark.parametrize("dtype", [rt.F64, rt.F32])
def test_gathered_states_of_other_sets(dtype, K, n, order):
    p = regime_problem("reduced_fast", index=1, n=n, K=120, steps=2)
    p.dirs, p.weights = _pairs(K, order), np.full(K, 1.0 / K)
    p.state.I = np.ascontiguousarray(p.state.I[:, :K])
    _compare(p, dtype)
