"""The update's two forms -- every wave summing its rows itself, and cost-to-go at
segment boundaries -- at the edges of tiles, chunks, segments and blocks, with
unaligned costs, both weightings, chunks of infinite costs and chunks far apart."""
import numpy as np
import pytest

import oracle
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


# rows summed by the waves: one rollout, a tile and one more, one segment at many
# rollouts, the last step count and size of the rule; boundaries and one step per
# wave; tiles and steps grouped from the first size on; T of whole and ragged
# segments, rows that are not 16-byte multiples, more than 64 segments of 8 steps
@pytest.mark.parametrize("K,T", [(1, 1), (65, 3), (200001, 1), (30000, 8), (4864, 40), (1, 41), (4800, 41),
                                 (30000, 9), (4865, 40), (641, 516), (6500, 39), (33, 513), (256, 1030)])
@pytest.mark.parametrize("dyn,dtype", [(DYN_QUAD12, np.float32), (DYN_QUAD12, np.float64),
                                       (DYN_POINTMASS2D, np.float32), (DYN_POINTMASS2D, np.float64)])
@pytest.mark.parametrize("weighting", [0, 1])
def test_update_forms(K, T, dyn, dtype, weighting):
    prob, _ = synth.tiny_problem(81, dyn=dyn, K=K, T=T, dtype=dtype)
    prob.weighting, prob.lam = weighting, 0.3
    rng = np.random.default_rng(K + T)
    base = rng.uniform(0.0, 1.0, (K, T)).astype(dtype)
    far = base.copy()
    far[: K // 2] += dtype(50)           # chunks whose minima lie far apart
    inf = base.copy()
    inf[: min(300, K - 1), T - 1] = np.inf   # a whole chunk without a finite cost-to-go
    # float32: draws within 1e-6 of float64, the rest in double; float64: sums
    # of up to 1e3 steps, rounded to 2e-13, over lambda
    tol = 1e-11 if dtype == np.float64 else 2e-6
    for cost in (base, far, inf):
        for off in (0, 1):               # the second time not 16-byte aligned
            buf = torch.empty(K * T + off, dtype=torch.from_numpy(base).dtype, device="cuda")
            c = buf[off:].view(K, T)
            c.copy_(torch.from_numpy(cost))
            dp = pi.DeviceProblem(prob)
            dp.iter.fill_(2)
            got = pi.update(dp, c)[0].cpu().numpy()
            ref = oracle.update(prob, cost, it=2)
            ref = ref[0] if isinstance(ref, tuple) else ref
            assert int(dp.iter.item()) == 3
            assert np.max(np.abs(got - ref)) <= tol * max(1.0, np.abs(ref).max()), off
