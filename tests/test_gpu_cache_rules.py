"""The default's accesses and plane order by the state's size (ordinary ones
where the last-level cache holds the state or rows share 128-byte lines, single
steps upwards and downwards in turn) against streaming accesses in one
direction (cache_policy 1): neither enters the arithmetic, so the populations
agree bit for bit.  Sizes on both sides of each bound of the rule, odd step
counts, rows of whole lines and ragged ones."""
import numpy as np
import pytest

from paper_2010_01628_amd import inputs
from paper_2010_01628_amd import lbm as L

pytestmark = pytest.mark.gpu


def _flow(size, steps, two_step, monkeypatch, learned=False, **kw):
    monkeypatch.setenv("LBM_TWO_STEP", two_step)
    rho, u, _ = inputs.random_lattice_fields(*size, seed=3, umax=0.05, fmax=1e-3)
    lat = L.Lattice(L.make_params(*size, omega=1.7, **kw))
    lat.init(rho, u)
    if learned:
        theta = (0.02 * np.random.default_rng(1).standard_normal(1737)).astype(np.float32)
        net = L.Mlp(theta, np.ones(11))
        lat.attach_mlp(net)
    for n in steps:
        lat.step(n)
    f = lat.get_populations()
    lat.close()
    return f


@pytest.mark.parametrize("streaming", ["ab", "aa"])
@pytest.mark.parametrize("size,precision", [
    ((96, 90, 80), "fp32"),    # one buffer 52 MB
    ((96, 57, 57), "fp32"),    # one buffer just below 24 MB
    ((97, 61, 63), "fp64"),    # one buffer 57 MB, ragged rows
    ((128, 90, 60), "fp16"),   # one buffer 26 MB
    ((160, 140, 160), "fp32"), # two buffers 545 MB, one in place 272 MB
    ((170, 150, 141), "fp16"), # ragged, two buffers 273 MB
])
def test_flow(size, precision, streaming, monkeypatch):
    import torch

    for kw in ({}, {"walls_y": True}):
        for two in ("0", "1"):
            runs = [_flow(size, (3, 2), two, monkeypatch, precision=precision, streaming=streaming, cache_policy=c, **kw)
                    for c in (0, 1)]
            assert torch.isfinite(runs[0]).all()
            assert torch.equal(runs[0], runs[1]), (size, precision, streaming, two, kw)


@pytest.mark.parametrize("streaming", ["ab", "aa"])
@pytest.mark.parametrize("precision", ["fp32", "fp16"])
def test_learned(precision, streaming, monkeypatch):
    import torch

    for size in ((128, 90, 60), (97, 91, 83)):
        runs = [_flow(size, (3,), "0", monkeypatch, learned=True, precision=precision, streaming=streaming, cache_policy=c)
                for c in (0, 1)]
        assert torch.equal(runs[0], runs[1]), (size, precision, streaming)


@pytest.mark.parametrize("size", [(64, 40, 33), (64, 64, 50), (96, 128, 96)])
def test_magnetic(size):
    import torch

    rho, u, b = inputs.random_lattice_fields(*size, seed=4, umax=0.02, fmax=0.02)
    runs = []
    for c in (0, 1):
        lat = L.Lattice(L.make_params(*size, omega=1.25, walls_y=True, cache_policy=c,
                                      magnetic=dict(eta=0.1, b_wall=(0.0, 0.01, 0.0))))
        lat.init_magnetic(rho, u, b)
        lat.step(3)
        runs.append((lat.get_populations(), *lat.magnetic_fields()))
        lat.close()
    for x, y in zip(*runs):
        assert torch.equal(x, y), size


@pytest.mark.parametrize("size,precision,kw", [
    ((128, 128, 128), "fp32", {}),                    # 319 MB, staged rows of whole lines
    ((128, 128, 128), "fp32", {"walls_y": True}),     # direct reads
    ((144, 144, 140), "fp32", {}),                    # 441 MB, ragged rows
    ((144, 144, 140), "fp32", {"walls_y": True}),
    ((96, 96, 104), "fp64", {}),                      # 291 MB
    ((128, 100, 100), "fp32", {"q": 27}),             # 276 MB
    ((128, 100, 100), "fp32", {"moments": "raw", "q": 27}),
    ((128, 160, 140), "fp32", {}),                    # 436 MB
    ((128, 160, 160), "fp32", {}),                    # 498 MB: beyond the rule, always upwards
])
def test_two_buffers_in_turn(size, precision, kw, monkeypatch):
    """A-B single steps upwards and downwards in turn: two buffers that hold
    256 MiB to 480 MB."""
    import torch

    runs = [_flow(size, (3, 2), "0", monkeypatch, precision=precision, cache_policy=c, **kw) for c in (0, 1)]
    assert torch.isfinite(runs[0]).all()
    assert torch.equal(runs[0], runs[1])


@pytest.mark.parametrize("size,walls", [((128, 128, 128), False), ((128, 128, 128), True), ((144, 144, 140), False)])
def test_two_buffers_in_turn_learned(size, walls, monkeypatch):
    import torch

    runs = [_flow(size, (3, 2), "0", monkeypatch, learned=True, precision="fp32", cache_policy=c, walls_y=walls) for c in (0, 1)]
    assert torch.isfinite(runs[0]).all()
    assert torch.equal(runs[0], runs[1])
