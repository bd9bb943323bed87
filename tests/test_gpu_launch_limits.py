"""Sizes whose work does not fit one thread per item of a launch (2^32 threads)."""
import numpy as np
import pytest

import synth
from synth import DYN_POINTMASS2D

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    kept = dict(pi._ws.buf)
    yield
    torch.cuda.synchronize()
    pi._ws.buf.clear()       # the large workspaces go back, the others stay
    pi._ws.buf.update(kept)
    torch.cuda.empty_cache()


def _problem(dtype, K, T):
    prob, model = synth.tiny_problem(95, dyn=DYN_POINTMASS2D, L=2, R=1, K=K, T=T, M=0, dtype=dtype, n_obs=0)
    return prob, model


# float64 rollouts of a small model past 2^30: one step each, checked at both ends
# from the draws and the prediction entry point
def test_more_rollouts_than_a_quarter_of_the_threads():
    K = (1 << 30) + 70
    prob, model = _problem(np.float64, K, 1)
    prob.w_vel = 1.0
    dp, dm = pi.DeviceProblem(prob), pi.DeviceModel(model)
    cost = pi.rollout_cost(dp, dm)
    for k0 in (0, K - 70):
        eps = pi.noise(dp, pi.PI_TAG_CTRL, k0, 70)[:, 0]
        x0 = dp.x0.expand(70, 4)
        acc, _ = pi.lwpr_predict(dm, torch.cat([x0, dp.u_nom[0] + eps], 1))
        p, v = x0[:, :2] + prob.dt * x0[:, 2:], x0[:, 2:] + prob.dt * acc
        goal, w = (torch.as_tensor(np.asarray(a[:2]), device="cuda") for a in (prob.goal, prob.w_pos))
        ref = prob.dt * ((w * (p - goal) ** 2).sum(1) + (v ** 2).sum(1))
        assert (cost[k0:k0 + 70, 0] - ref).abs().max() <= 1e-12 * ref.abs().max()


# updates with 2^24 steps and more (a block per step), and with 2^29 rollouts and more
# (eight threads each).  One rollout is free and the others' weights vanish: the plan
# moves by that rollout's draws
@pytest.mark.parametrize("K,T", [(3, (1 << 24) + 16), ((1 << 29) + 40, 9)])
def test_more_steps_or_rollouts_than_blocks(K, T):
    prob, _ = _problem(np.float32, K, 4)
    prob.T, prob.u_nom = T, np.zeros((T, 2), np.float32)
    dp = pi.DeviceProblem(prob)
    cost = torch.full((K, T), 2000.0, device="cuda")
    cost[K - 1] = 0.0
    eps = pi.noise(dp, pi.PI_TAG_CTRL, K - 1, 1)[0]
    u, _ = pi.update(dp, cost)
    assert torch.equal(u, eps) and int(dp.iter) == 1
