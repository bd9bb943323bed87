"""fp16 pieces of outputs whose models do not fill their last tile: the padded slots
need no scale beside ordinary models, and have no weight however far out a row is."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_QUAD12, OBS_SMOOTH

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu
HF2 = pi.PI_VARIANT_MFMA_F16X2


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


def _problem(L, K=70, T=5, **kw):
    return synth.tiny_problem(76, dyn=DYN_QUAD12, L=L, R=2, K=K, T=T, M=1, dtype=np.float32, n_obs=3,
                              obs_kind=OBS_SMOOTH, **kw)


# a fold ends with 64 floats per tile of 16 models, the 49th 1 where none carries a scale
def _plain_tiles(model):
    dm = pi.DeviceModel(model).fold()
    n = sum((int(b) - int(a) + 15) // 16 for a, b in zip(model.L_off[:-1], model.L_off[1:]))
    return dm.folded[-256 * n:].view(torch.float32).reshape(n, 64)[:, 48].cpu().numpy() == 1.0


def test_padded_tiles_carry_no_scales():
    _, model = _problem([1, 3, 17, 16, 5, 33])
    assert _plain_tiles(model).all()
    # a metric past 2^13 in the last, padded tile (alpha D_aa = 0.72 D_aa), and one in a full tile
    model.metric[model.L_off[-1] - 1, 2, 2] = 1.5e4
    model.metric[model.L_off[3], 2, 2] = 1.5e4
    assert list(_plain_tiles(model)) == [True] * 8 + [False]


# rows near, far (activations of -1e4 and less) and past the row scales' 2^14, with
# narrow models up to the limit of the unscaled range
@pytest.mark.parametrize("out", [0.0, 90.0, 400.0])
@pytest.mark.parametrize("narrow", [1.0, 1000.0])
@pytest.mark.parametrize("kw", [dict(tile_samples=16, tile_split=1), dict(tile_samples=16, tile_split=2),
                                dict(tile_samples=32), dict(tile_samples=64, tile_waves=4),
                                dict(tile_samples=128, tile_waves=4), dict(tile_samples=128, tile_waves=8)])
def test_padded_slots_have_no_weight(kw, narrow, out):
    prob, model = _problem([1, 3, 17, 2, 5, 9])
    prob.x0[:3] += np.float32(out)
    model.centre[:, :3] += np.float32(out and out - 60.0)
    model.metric *= np.float32(narrow)
    got = pi.rollout_cost(pi.DeviceProblem(prob, variant=HF2, **kw), pi.DeviceModel(model)).cpu().numpy()
    f32 = pi.rollout_cost(pi.DeviceProblem(prob, variant=pi.PI_VARIANT_MFMA), pi.DeviceModel(model)).cpu().numpy()
    ref = oracle.rollout_cost(prob, model)
    S, Sf, So = (a.astype(np.float64).sum(1) for a in (got, f32, ref))
    # as near as the float32 products, or the 1e-4 that trajectory costs are held to
    assert np.abs(S - So).max() <= max(1e-4 * np.abs(So).max(), 2 * np.abs(Sf - So).max())
