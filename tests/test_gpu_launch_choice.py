"""The launches that the library picks, either side of each of its limits."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_POINTMASS2D, DYN_QUAD12, DYN_QUAD_HYBRID, OBS_SMOOTH

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


def _problem(K, L, dyn=DYN_QUAD12, T=3, **kw):
    prob, model = synth.tiny_problem(74, dyn=dyn, L=L, R=2, K=K, T=T, M=1, dtype=np.float32, n_obs=2,
                                     obs_kind=OBS_SMOOTH)
    return prob, model, pi.DeviceProblem(prob, **kw), pi.DeviceModel(model)


def _parity(prob, model, dp, dm):
    got = pi.rollout_cost(dp, dm).cpu().numpy().astype(np.float64)
    ref = oracle.rollout_cost(prob, model)
    # three float32 steps: well inside the 1e-4 that trajectory costs are held to
    assert np.all(np.abs(got.sum(1) - ref.sum(1)) <= 1e-5 * np.abs(ref.sum(1)))


# pairs of workgroups: up to half the compute units' tiles, and for many local models
# of the small dynamics up to all of them (128 and 255 tiles of 16 on 256 units)
@pytest.mark.parametrize("dyn,L,K,split", [
    (DYN_QUAD_HYBRID, [590, 600, 590], 2048, 2), (DYN_QUAD_HYBRID, [590, 600, 590], 2049, 2),
    (DYN_QUAD_HYBRID, [590, 600, 590], 4080, 2), (DYN_QUAD_HYBRID, [590, 600, 590], 4081, 1),
    (DYN_QUAD_HYBRID, [400, 400, 400], 2048, 2), (DYN_QUAD_HYBRID, [400, 400, 400], 2049, 1),
    (DYN_POINTMASS2D, [900, 892], 4080, 2), (DYN_POINTMASS2D, [700, 700], 2049, 1)])
def test_pairs_of_the_small_dynamics(dyn, L, K, split):
    prob, model, dp, dm = _problem(K, L, dyn)
    assert pi.rollout_describe(dp, dm)["tile_split"] == split
    _parity(prob, model, dp, dm)


# tiles of the pieces forms left to the library: few local models (6 x 16 and fewer: 6
# model tiles) and many rollouts take the large tiles too.  Parity where the oracle is quick
@pytest.mark.parametrize("variant,waves,L,K,spw", [
    (0, 0, 5, 2049, 16), (0, 0, 5, 16000, 16), (0, 0, 5, 32768, 128),
    (3, 0, 5, 8000, 16), (3, 0, 5, 20000, 128), (3, 0, 5, 32768, 128), (3, 8, 5, 32768, 128), (3, 8, 5, 65536, 128),
    (3, 4, 5, 65536, 128), (4, 0, 5, 8000, 16), (4, 0, 5, 16000, 64), (4, 0, 5, 49152, 128), (4, 8, 5, 33000, 128),
    (4, 4, 5, 50000, 128), (4, 0, 61, 4000, 16), (4, 0, 61, 65536, 128), (0, 0, 256, 2048, 16), (0, 0, 256, 2049, 16),
    (0, 0, 256, 6000, 32), (0, 0, 256, 16384, 64), (3, 0, 256, 6000, 32), (3, 0, 256, 16384, 64),
    (3, 0, 256, 32768, 128), (4, 0, 256, 4096, 16), (4, 0, 256, 6000, 32), (4, 0, 256, 14000, 64),
    (4, 0, 256, 20000, 128), (4, 4, 256, 20000, 128), (4, 4, 192, 17000, 128), (4, 8, 256, 6000, 16),
    (4, 8, 256, 20000, 128)])
def test_tiles_of_the_pieces(variant, waves, L, K, spw):
    prob, model, dp, dm = _problem(K, L, variant=variant, tile_waves=waves)
    d = pi.rollout_describe(dp, dm)
    assert d["tile_samples"] == spw
    if variant == 0:
        assert d["variant"] == ("mfma" if K <= 2048 else "mfma-bf16x3")
    if L < 16:
        _parity(prob, model, dp, dm)


# waves of 16-row tiles, at most one workgroup to a unit: eight, but four for the pieces
# forms without pairs, except with very few or very many model tiles
@pytest.mark.parametrize("variant,L,K,split,waves", [
    (2, 5, 4096, 1, 8), (2, 256, 4096, 1, 8), (2, 256, 1024, 2, 8), (3, 5, 2100, 1, 8), (3, 20, 2100, 1, 4),
    (3, 256, 2100, 1, 4), (3, 256, 1024, 2, 8), (4, 5, 2100, 1, 8), (4, 20, 2100, 1, 4), (4, 256, 4096, 1, 4),
    (4, 256, 1024, 2, 8), (4, 1024, 2100, 1, 8), (0, 256, 2100, 1, 4)])
def test_waves(variant, L, K, split, waves):
    prob, model, dp, dm = _problem(K, L, variant=variant)
    d = pi.rollout_describe(dp, dm)
    assert (d["tile_samples"], d["tile_split"], d["tile_waves"]) == (16, split, waves)
    if L < 64:
        _parity(prob, model, dp, dm)
