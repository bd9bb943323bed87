"""Predictions from a model as given, without a fold: either side of the rule, lanes
left over, models past a wave's lanes, loadings of their own, far inputs."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_POINTMASS2D, DYN_QUAD_HYBRID

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("dyn,L,N", [(DYN_POINTMASS2D, [1, 3], 1), (DYN_POINTMASS2D, [16, 64], 1024),
                                     (DYN_POINTMASS2D, [16, 64], 1025), (DYN_POINTMASS2D, [65, 9], 33),
                                     (DYN_QUAD_HYBRID, [512, 1, 70], 7), (DYN_QUAD_HYBRID, [513, 1, 70], 7),
                                     (DYN_QUAD_HYBRID, [15, 15, 24], 682), (DYN_POINTMASS2D, [100, 100], 5000),
                                     (DYN_POINTMASS2D, [100, 100], 5001)])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("loadings", [False, True])
def test_unfolded_predictions(dyn, L, N, dtype, loadings):
    _, model = synth.tiny_problem(41, dyn=dyn, L=L, R=3, K=4, T=3, M=1, dtype=dtype)
    if loadings:
        model.proj_p = (np.random.default_rng(2).normal(0, 0.5, model.proj_u.shape)).astype(dtype)
    dm = pi.DeviceModel(model)
    for spread in (1.0, 30.0):
        Z = np.random.default_rng(3).uniform(-spread, spread, (N, model.d)).astype(dtype)
        mu, var = pi.lwpr_predict(dm, torch.from_numpy(Z).cuda())
        rmu, rvar = oracle.lwpr_predict(model, Z)[:2]
        # the bounds of predictions; far inputs of the folded float32 form carry
        # exponents of 1e4 rounded to 1e-3, so only the unfolded ones are held there
        raw = max(L) <= 512 and N * len(L) * -(-max(L) // 64) <= 2048
        tol = 1e-10 if dtype == np.float64 else 1e-5
        if spread == 1.0 or raw or dtype == np.float64:
            assert np.linalg.norm(mu.cpu().numpy() - rmu) <= tol * np.linalg.norm(rmu)
            assert np.linalg.norm(var.cpu().numpy() - rvar) <= tol * np.linalg.norm(rvar)
