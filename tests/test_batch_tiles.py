"""Which tiles a batch of problems may mix (host side of the batched calls: the
workspace query validates and lays out without a device)."""
import ctypes as C

import numpy as np
import pytest

import synth
from synth import DYN_QUAD12

pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")
AUTO, BF3, HF2 = 0, 3, 4


def _accepted(K, problems, waves):
    prob, model = synth.tiny_problem(73, dyn=DYN_QUAD12, L=3, R=2, K=K, T=2, M=1, dtype=np.float32, n_obs=0)
    dm = pi.DeviceModel(model, device="cpu")
    ps = [pi.DeviceProblem(prob, device="cpu", variant=v, tile_samples=t) for v, t in problems]
    ps[0].tile_waves = waves
    n = len(ps)
    sz = pi.load().pi_batched_workspace_bytes(n, (pi.pi_problem * n)(*[p.struct() for p in ps]),
                                              (pi.pi_lwpr * n)(*[dm.struct()] * n))
    return sz != C.c_size_t(-1).value


# whether a batch is taken does not depend on how many rollouts it has, though the
# tile that the library picks does (16 rows below 16384 rollouts in all, 128 from there)
@pytest.mark.parametrize("K", [100, 8191, 8192, 20000])
@pytest.mark.parametrize("problems,waves,ok", [
    ([(HF2, 24), (HF2, 0)], 8, True),     # 24 rows on 8 waves: only as shared tiles, beside a 128-row default
    ([(HF2, 0), (HF2, 24)], 8, True),
    ([(HF2, 32), (HF2, 0)], 4, True),
    ([(HF2, 24), (HF2, 16)], 8, False),
    ([(HF2, 0), (HF2, 0)], 8, True),
    ([(HF2, 16), (HF2, 0)], 8, True),
    ([(HF2, 40), (HF2, 0)], 8, True),
    ([(BF3, 24), (HF2, 0)], 8, True),
    ([(BF3, 24), (BF3, 0)], 8, False),
    ([(AUTO, 0), (HF2, 0)], 4, False),    # float32 products take no 128-row tile
    ([(AUTO, 0), (AUTO, 0)], 8, True),
])
def test_accepted_mixes(K, problems, waves, ok):
    assert _accepted(K, problems, waves) == ok
