"""The 64-row shared tile on four waves (two waves to a row group, which take the model
tiles in turn) at the edges of its pipeline: few, odd and single model tiles, outputs
that end inside a stage, rows past the last rollout."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_QUAD12, OBS_SMOOTH

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu
BF3, HF2 = 3, 4


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


# 6, 7, 8, 11 and 17 model tiles
@pytest.mark.parametrize("L", [1, [17, 1, 16, 3, 1, 2], [16, 33, 1, 1, 5, 16], [20, 17, 33, 16, 1, 40],
                               [16, 48, 47, 65, 30, 49]])
@pytest.mark.parametrize("spw", [33, 64])
@pytest.mark.parametrize("variant", [BF3, HF2])
def test_edges(variant, spw, L):
    for K, M, scale in ((1, 1, 1.0), (65, 1, 1.0), (50, 3, 1.0), (70, 1, 3000.0)):
        prob, model = synth.tiny_problem(71, dyn=DYN_QUAD12, L=L, R=3, K=K, T=7, M=M, dtype=np.float32,
                                         n_obs=5, obs_kind=OBS_SMOOTH)
        model.metric[::3] *= np.float32(scale)   # past 2^14: fp16 models with scales
        dp = pi.DeviceProblem(prob, variant=variant, tile_samples=spw, tile_waves=4, tile_split=1)
        got = pi.rollout_cost(dp, pi.DeviceModel(model)).cpu().numpy().astype(np.float64)
        ref = oracle.rollout_cost(prob, model)
        # the 1e-4 that trajectory costs are held to, tightened tenfold for seven steps
        assert np.all(np.abs(got.sum(1) - ref.sum(1)) <= 1e-5 * np.abs(ref.sum(1))), (K, M, scale)
