"""Scratch of pieces-form rollouts whose tile is left to the library (host side: the
workspace query needs no device): no pair-exchange slots for problems that fill the
device, whichever tile the models' number makes the cheapest, so that the
allocation-free entry point takes them."""
import numpy as np
import pytest

import synth
from synth import DYN_QUAD12

pytest.importorskip("torch")
pi = pytest.importorskip("paper_1503_00330_amd")


def _need(K, L, **kw):
    prob, model = synth.tiny_problem(75, dyn=DYN_QUAD12, L=L, R=2, K=K, T=2, M=1, dtype=np.float32, n_obs=0)
    dp, dm = pi.DeviceProblem(prob, device="cpu", **kw), pi.DeviceModel(model, device="cpu")
    return pi.workspace_bytes(pi.PI_OP_ROLLOUT, dp, dm)


@pytest.mark.parametrize("variant", [3, 4])
@pytest.mark.parametrize("waves", [0, 4, 8])
@pytest.mark.parametrize("L", [3, 16, 20, 60])
@pytest.mark.parametrize("K", [32768, 32769, 65536])
def test_no_slots_past_the_pairs(K, L, waves, variant):
    kw = dict(variant=variant, tile_waves=waves)
    assert _need(K, L, **kw) == _need(K, L, **kw, tile_split=1) <= 32 << 20


@pytest.mark.parametrize("variant", [2, 3, 4])
@pytest.mark.parametrize("K", [100, 2048, 4096])
def test_slots_where_pairs_may_be(K, variant):
    assert _need(K, 3, variant=variant) > _need(K, 3, variant=variant, tile_split=1)
