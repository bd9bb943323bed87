"""The float32 adjoint's recomputed segments repeat the forward's states: with steps
far below an ulp of the state the trajectory lives in the carried rounding errors,
and a cost about the start makes the gradient one of single ulps."""
import numpy as np
import pytest

import synth
from synth import DYN_POINTMASS2D, DYN_QUAD12

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("ckpt", [1, 7, 0])
@pytest.mark.parametrize("dyn,kw", [(DYN_POINTMASS2D, {}), (DYN_QUAD12, {}),
                                    (DYN_QUAD12, dict(variant=pi.PI_VARIANT_MFMA_F16X2))])
def test_segments_keep_the_carried_errors(dyn, kw, ckpt):
    T, npos = 64, 2 if dyn == DYN_POINTMASS2D else 3
    prob, model = synth.tiny_problem(62, dyn=dyn, L=7, R=2, K=20, T=T, M=0, dtype=np.float32, n_obs=0)
    prob.dt = float(np.float32(1e-8))                # a sixth of an ulp of 0.75 per step of speed 1
    prob.x0[:npos], prob.x0[npos:2 * npos] = 0.75, 1.0
    prob.goal[:npos], prob.w_pos[:] = 0.75, 1e6      # |x - goal| is at most eleven ulps
    prob.w_ang = prob.w_vel = 0.0
    dp, dm = pi.DeviceProblem(prob, **kw), pi.DeviceModel(model)
    whole = pi.rollout_adjoint(dp, dm, ckpt_every=T)   # one segment: the forward itself is traced
    got = pi.rollout_adjoint(dp, dm, ckpt_every=ckpt)
    assert got[0].item() == whole[0].item()
    # a lost carry is a whole ulp of these eleven, about every sixth step; the
    # accelerations differ by float32 rounding only
    for g, w in zip(got[1:], whole[1:]):
        assert w.abs().max() > 0 and (g - w).abs().max() <= 1e-4 * w.abs().max()
