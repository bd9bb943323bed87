"""Rollouts of small models: every lane count and model count of the kernel, at the
edges of its rules, against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_POINTMASS2D, DYN_QUAD_HYBRID, OBS_SMOOTH

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu
F32, F64 = np.float32, np.float64


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


def _check(prob, model, dtype):
    dm = pi.DeviceModel(model)
    got = pi.rollout_cost(pi.DeviceProblem(prob), dm)
    folded = pi.rollout_cost(pi.DeviceProblem(prob), dm.fold())
    assert torch.equal(got, folded)
    ref = oracle.rollout_cost(prob, model)
    got = got.cpu().numpy().astype(np.float64)
    # the bounds that trajectory costs are held to, tightened tenfold for short horizons
    tol = 1e-11 if dtype == F64 else 1e-5
    assert np.all(np.abs(got.sum(1) - ref.sum(1)) <= tol * np.abs(ref.sum(1)).max())


# models per output: one, a row of 16 lanes and one more, two and one more, the
# limits of either type and one more
@pytest.mark.parametrize("L", [1, 3, 16, 17, 32, 33, 40, 41, 64, 65])
@pytest.mark.parametrize("dyn", [DYN_POINTMASS2D, DYN_QUAD_HYBRID])
@pytest.mark.parametrize("dtype", [F32, F64])
def test_model_counts(L, dyn, dtype):
    Ls = [L, 1] if dyn == DYN_POINTMASS2D else [1, L, max(1, L - 5)]
    # steps that end inside a chunk of draws, rows that end inside a wave
    for K, T, M, n_obs, kind in ((1, 1, 1, 0, 0), (5, 17, 0, 1, 0), (33, 35, 3, 6, OBS_SMOOTH)):
        prob, model = synth.tiny_problem(91 + L, dyn=dyn, L=Ls, R=2, K=K, T=T, M=M, dtype=dtype, n_obs=n_obs,
                                         obs_kind=kind)
        _check(prob, model, dtype)


# either side of the sub-rollout counts at which the lanes per sub-rollout change
@pytest.mark.parametrize("dtype,L,n", [(F32, 16, 24576), (F32, 20, 12288), (F32, 36, 6144), (F32, 50, 4096),
                                       (F64, 16, 12288), (F64, 20, 12288), (F64, 36, 2048),
                                       (F64, 36, 8191), (F64, 50, 32768)])
@pytest.mark.parametrize("past", [0, 1])
def test_lane_counts(dtype, L, n, past):
    for dyn, Ls in ((DYN_POINTMASS2D, [L, 3]), (DYN_QUAD_HYBRID, [2, L, 7])):
        prob, model = synth.tiny_problem(92, dyn=dyn, L=Ls, R=2, K=n + past, T=5, M=1, dtype=dtype, n_obs=2,
                                         obs_kind=OBS_SMOOTH)
        _check(prob, model, dtype)


@pytest.mark.parametrize("dtype", [F32, F64])
@pytest.mark.parametrize("n", [60, 13000])
def test_control_terms(dtype, n):
    prob, model = synth.tiny_problem(93, dyn=DYN_QUAD_HYBRID, L=[15, 15, 24], R=2, K=n, T=9, M=2, dtype=dtype, n_obs=3)
    prob.ctrl_cost = 1
    _check(prob, model, dtype)


def test_library_choice_and_explicit_launches():
    prob, model = synth.tiny_problem(94, dyn=DYN_QUAD_HYBRID, L=[15, 15, 24], R=2, K=64, T=5, M=1, dtype=F32)
    dm = pi.DeviceModel(model)
    assert pi.rollout_describe(pi.DeviceProblem(prob), dm)["variant"] == "direct"
    for kw in (dict(variant=pi.PI_VARIANT_MFMA), dict(tile_samples=16), dict(tile_waves=4), dict(tile_split=1)):
        assert pi.rollout_describe(pi.DeviceProblem(prob, **kw), dm)["variant"] == "mfma"
