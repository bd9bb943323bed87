"""The pieces forms' shared-tile launch at the edges of its tile pipeline (few,
odd and single model tiles, rows past the last rollout), and the fp16 batch's
choice of tile at its threshold."""
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


# 6, 7, 8 and 11 model tiles: stages of two tiles, an odd last one, outputs that
# end inside a stage, fewer stages than the ring holds
@pytest.mark.parametrize("L", [1, [17, 1, 16, 3, 1, 2], [16, 33, 1, 1, 5, 16], [20, 17, 33, 16, 1, 40]])
@pytest.mark.parametrize("variant,waves", [(BF3, 4), (BF3, 8), (HF2, 4), (HF2, 8)])
def test_shared_tile_edges(variant, waves, L):
    for K, M in ((1, 1), (129, 1), (50, 3)):
        prob, model = synth.tiny_problem(71, dyn=DYN_QUAD12, L=L, R=3, K=K, T=7, M=M, dtype=np.float32,
                                         n_obs=5, obs_kind=OBS_SMOOTH)
        dp = pi.DeviceProblem(prob, variant=variant, tile_samples=128, tile_waves=waves, tile_split=1)
        got = pi.rollout_cost(dp, pi.DeviceModel(model)).cpu().numpy().astype(np.float64)
        ref = oracle.rollout_cost(prob, model)
        # seven float32 steps: well inside the 1e-4 that trajectory costs are held to
        assert np.all(np.abs(got.sum(1) - ref.sum(1)) <= 1e-5 * np.abs(ref.sum(1))), (K, M)


# the fp16 batch that leaves its tiles to the library: 16 rows below 16384
# rollouts, 128 from there on, each bitwise the plain launch of that tile
@pytest.mark.parametrize("K,spw", [(8191, 16), (8192, 128)])
def test_batch_default_tile_threshold(K, spw):
    prob, model = synth.tiny_problem(72, dyn=DYN_QUAD12, L=5, R=2, K=K, T=3, M=1, dtype=np.float32, n_obs=3)
    dm = pi.DeviceModel(model).fold()
    mk = lambda **kw: pi.DeviceProblem(prob, variant=HF2, tile_split=1, tile_waves=4, **kw)
    br = pi.BatchedRollout([mk(), mk()], [dm, dm])
    plain = pi.rollout_cost(mk(tile_samples=spw), dm)
    for c in br.run():
        assert torch.equal(c, plain)
