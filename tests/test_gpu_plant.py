"""The plant step and plan shift in one block (up to eight model chunks over the
outputs) and in two kernels, with plans shorter and longer than a block."""
import numpy as np
import pytest

import oracle
import synth
from synth import DYN_POINTMASS2D, DYN_QUAD12, DYN_QUAD_HYBRID

torch = pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("dyn,L", [(DYN_POINTMASS2D, [1, 3]), (DYN_POINTMASS2D, [64, 256]), (DYN_POINTMASS2D, [257, 9]),
                                   (DYN_QUAD_HYBRID, [15, 128, 24]), (DYN_QUAD_HYBRID, [129, 15, 24]),
                                   (DYN_QUAD12, [64, 2, 33, 1, 64, 10]), (DYN_QUAD12, [65, 2, 33, 1, 64, 10])])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("T", [1, 2, 129, 700])
def test_plant_forms(dyn, L, dtype, T):
    prob, model = synth.tiny_problem(51, dyn=dyn, L=L, R=2, K=4, T=T, dtype=dtype)
    dp, dm = pi.DeviceProblem(prob), pi.DeviceModel(model)
    dp.iter.fill_(3)
    pi.rh_shift(dp, dm)
    ox, ou = oracle.rh_shift(prob, model, prob.x0, prob.u_nom, 3)
    assert np.array_equal(dp.u_nom.cpu().numpy(), ou.astype(dtype))
    tol = 1e-12 if dtype == np.float64 else 1e-6     # as for the existing shift
    assert np.max(np.abs(dp.x0.cpu().numpy() - ox)) <= tol * max(1.0, np.abs(ox).max())
