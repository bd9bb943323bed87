"""Predictions of d = 16 models left to the library (bf16 pieces: a coarse pass
for the anchors, then the full one) at the edges of its tiles and row splits,
for inputs near and far from the models."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_QUAD12

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


def _check(model, Z, tol=1e-5):
    mean, var = pi.lwpr_predict(pi.DeviceModel(model), torch.from_numpy(Z).cuda())
    om, ov = oracle.lwpr_predict(model, Z)
    for g, o in ((mean, om), (var, ov)):
        g = g.cpu().numpy().astype(np.float64)
        # the normwise 1e-5 that predictions are held to
        assert np.all(np.abs(g - o).max(0) <= tol * np.abs(o).max(0))


# 16- and 32-row tiles, their last rows, one input
@pytest.mark.parametrize("N", [1, 15, 17, 4097, 8192, 8193])
@pytest.mark.parametrize("L", [[17, 1, 16, 3, 1, 2], [130, 96, 250, 33, 177, 301]])
def test_prediction_row_edges(N, L):
    _, model = synth.tiny_problem(81, dyn=DYN_QUAD12, L=L, R=3, dtype=np.float32)
    Z = np.random.default_rng(N).uniform(-1, 1, (N, 16)).astype(np.float32)
    _check(model, Z)


# whole passes of 128-row workgroups, and a remainder in each other tile
@pytest.mark.parametrize("N", [32768, 32768 + 33, 2 * 32768 + 5000, 65536 - 1])
def test_prediction_shared_tile_rows(N):
    _, model = synth.tiny_problem(82, dyn=DYN_QUAD12, L=[5, 1, 9, 17, 2, 3], R=2, dtype=np.float32)
    Z = np.random.default_rng(N).uniform(-1, 1, (N, 16)).astype(np.float32)
    rows = np.r_[0:40, 32700:32768, N - 40:N]
    mean, var = pi.lwpr_predict(pi.DeviceModel(model), torch.from_numpy(Z).cuda())
    om, ov = oracle.lwpr_predict(model, Z[rows])
    for g, o in ((mean, om), (var, ov)):
        g = g.cpu().numpy().astype(np.float64)[rows]
        assert np.all(np.abs(g - o).max(0) <= 1e-5 * np.abs(o).max(0))


# inputs so far out that the coarse pass misses the activations by hundreds of
# units and the predictions by whole standard deviations (further passes).  One
# local model per output, so that the moments stay well conditioned: its
# prediction, 18 products summed in float32, and its sigma^2
@pytest.mark.parametrize("N", [50, 32768 + 20])
def test_prediction_far_inputs(N):
    _, model = synth.tiny_problem(84, dyn=DYN_QUAD12, L=1, R=3, dtype=np.float32)
    Z = (np.random.default_rng(6).uniform(-1, 1, (N, 16)) * 60.0).astype(np.float32)
    Z[::2] /= 60.0
    _check(model, Z)


# more outputs than the shared tile holds
def test_prediction_eight_outputs():
    rng = np.random.Generator(np.random.PCG64(7))
    model = synth.make_lwpr(rng, 16, [9, 17, 5, 33, 2, 16, 7, 1], 2).astype(np.float32)
    _check(model, rng.uniform(-1, 1, (33000, 16)).astype(np.float32))
