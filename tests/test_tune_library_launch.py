"""The tuner beside the launches that the library picks by itself (their tiles are not
all candidates), and cache entries of other launch sets.  Timings are given, not
measured."""
import json
from types import SimpleNamespace

import pytest

pi = pytest.importorskip("paper_1503_00330_amd")
torch = pytest.importorskip("torch")
from paper_1503_00330_amd import tune


@pytest.fixture
def prob(monkeypatch):
    p = SimpleNamespace(dyn=pi.PI_DYN_QUAD12, dtype=torch.float32, K=4, M=1, T=2, variant=0, tile_samples=0,
                        tile_waves=0, tile_split=0, device="cpu")
    monkeypatch.setattr(tune, "_arch", lambda: "gfx950")
    monkeypatch.setattr(pi, "rollout_describe", lambda p, m: {"variant": "mfma"})
    monkeypatch.setattr(pi, "rollout_cost", lambda p, m, out: None)
    return p


MODEL = SimpleNamespace(d=16, n_out=6, R=2, L_off=[0, 3, 6, 9, 12, 15, 18])


def _times(monkeypatch, prob, table, default):
    monkeypatch.setattr(tune, "_time", lambda fn, reps: table.get(tune._launch(prob), default))


@pytest.mark.parametrize("table,best", [({(0, 0, 0, 4): 1.0, (0, 0, 0, 0): 1.5}, (0, 0, 0, 4)),
                                        ({(0, 0, 0, 0): 1.0}, (0, 0, 0, 0)),
                                        ({(128, 8, 1, 4): 1.0, (0, 0, 0, 4): 1.1}, (128, 8, 1, 4))])
def test_ensure_keeps_the_fastest_launch(tmp_path, monkeypatch, prob, table, best):
    _times(monkeypatch, prob, table, 2.0)
    path = str(tmp_path / "t.json")
    assert tune.ensure(prob, MODEL, path=path) == best
    assert list(tune.load_cache(path).values()) == [list(best)]
    # a second problem of the shape takes it from the cache, with nothing timed
    monkeypatch.setattr(tune, "_time", None)
    again = SimpleNamespace(**{k: v for k, v in vars(prob).items() if not k.startswith("_")})
    again.variant = again.tile_samples = again.tile_waves = again.tile_split = 0
    assert tune.ensure(again, MODEL, path=path) == best


def test_a_named_variant_stays(tmp_path, monkeypatch, prob):
    prob.variant = 3
    _times(monkeypatch, prob, {(0, 0, 0, 4): 1.0, (0, 0, 0, 3): 1.5}, 2.0)
    assert tune.ensure(prob, MODEL, path=str(tmp_path / "t.json")) == (0, 0, 0, 3)


def test_entries_of_other_launch_sets_are_tuned_again(tmp_path, monkeypatch, prob):
    path = str(tmp_path / "t.json")
    key = tune.key_for(prob, MODEL)
    monkeypatch.setattr(tune, "LAUNCH_SET", tune.LAUNCH_SET - 1)
    assert tune.key_for(prob, MODEL) != key
    tune.save_cache({tune.key_for(prob, MODEL): [16, 4, 1, 4]}, path)
    monkeypatch.undo()
    monkeypatch.setattr(tune, "_arch", lambda: "gfx950")
    assert not tune.apply(prob, MODEL, path=path)


def test_library_entries_in_the_cache(tmp_path):
    p = str(tmp_path / "t.json")
    with open(p, "w") as f:
        json.dump({"a": [0, 0, 0, 4], "b": [0, 0, 0, 0], "c": [0, 0, 1, 4], "d": [0, 4, 0, 4], "e": [0, 0, 0, 1]}, f)
    assert tune.load_cache(p) == {"a": [0, 0, 0, 4], "b": [0, 0, 0, 0]}


def test_batches_try_the_64_row_tile():
    assert (64, 4, 3) in tune.BATCH_CANDIDATES and (64, 4, 4) in tune.BATCH_CANDIDATES
    assert not any(c[0] == 64 and (c[1] == 8 or c[2] == 2) for c in tune.BATCH_CANDIDATES)
