"""bench.py's ensemble rates count the bytes that the launches move: a plain
ensemble takes two steps to a pass over its state, a learned one one."""
import types

import pytest

import bench


class _Ensemble:
    nodes = 10 ** 9

    def __init__(self, boxes, q, precision):
        pass

    def fallback_count(self):
        return 0

    init = set_mlp = tune = step = close = lambda self, *a: None


@pytest.mark.parametrize("two_step,per_pass", [(None, 2), ("0", 1)])
def test_ensemble_rates(two_step, per_pass, monkeypatch):
    if two_step is None:
        monkeypatch.delenv("LBM_TWO_STEP", raising=False)
    else:
        monkeypatch.setenv("LBM_TWO_STEP", two_step)
    clock = iter(range(100))
    monkeypatch.setattr(bench.time, "perf_counter", lambda: float(next(clock)))
    inputs = types.SimpleNamespace(ensemble_boxes=lambda: [(8, 1e-3, 1)], omega_from_nu=lambda nu: 1.9,
                                   random_phase_field=lambda n, u, seed: (None, None))
    torch = types.SimpleNamespace(cuda=types.SimpleNamespace(synchronize=lambda: None))
    steps = 20  # in one second
    out = bench.time_ensemble(types.SimpleNamespace(Ensemble=_Ensemble), inputs, torch, steps, 4, object())
    for name, q, passes in (("q19", 19, steps / per_pass), ("q19_learned", 19, steps), ("q27", 27, steps / per_pass)):
        assert out[name]["mlups"] == pytest.approx(1e9 * steps / 1e6, abs=0.05)
        moved = 1e9 * 2 * q * 4 * passes / 1e9  # in and out once a pass
        assert out[name]["achieved_GBs"] == pytest.approx(moved, abs=0.06)
        assert out[name]["algo_bytes_per_node"] * out[name]["steps_per_pass"] == 2 * q * 4
