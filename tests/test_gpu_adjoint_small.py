"""The float32 adjoint where its parameter pass is cut finely: few rollouts, one
record chunk and many, models of few and several tile groups, indicator and
smooth obstacles, against float64."""
import numpy as np
import pytest

import synth
from synth import DYN_POINTMASS2D, DYN_QUAD12, OBS_SMOOTH

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


# records per segment below one chunk's 64, between the rules, and past them; 2047
# and 2049 rollouts: 8- and 4-wave forwards; a sample count that ends inside a tile
@pytest.mark.parametrize("K,M,T,ckpt,L", [(1, 1, 3, 0, 5), (17, 1, 9, 2, 40), (50, 3, 12, 5, 90), (2047, 1, 4, 2, 9),
                                          (2049, 0, 4, 3, 30), (4097, 1, 3, 0, 9)])
@pytest.mark.parametrize("dyn,kind,n_obs", [(DYN_QUAD12, OBS_SMOOTH, 35), (DYN_QUAD12, 0, 3),
                                            (DYN_POINTMASS2D, OBS_SMOOTH, 2)])
def test_small_adjoints(K, M, T, ckpt, L, dyn, kind, n_obs):
    prob, model = synth.tiny_problem(61, dyn=dyn, L=L, R=2, K=K, T=T, M=M, dtype=np.float32, n_obs=n_obs,
                                     obs_kind=kind)
    got = pi.rollout_adjoint(pi.DeviceProblem(prob), pi.DeviceModel(model), ckpt_every=ckpt)
    ref = pi.rollout_adjoint(pi.DeviceProblem(prob, dtype=torch.float64), pi.DeviceModel(model, dtype=torch.float64),
                             ckpt_every=ckpt)
    for g, r in zip(got, ref):   # the 1e-4 that float32 gradients are held to
        assert (g.double() - r).norm() <= 1e-4 * r.norm()
