"""Two steps per pass over memory (lbm_step with n >= 2, A-B; LBM_TWO_STEP=1
takes it wherever it is possible) against the single-step kernels
(LBM_TWO_STEP=0): the same arithmetic in the same order at every node, so the
populations agree bit for bit.  The default takes blocks of whole rows on
lattices small enough for one work-group per compute unit.  Sizes at the edges
of the tiles: rows and columns one tile spans whole (no halo), ones it just
does not, ragged last tiles, one to three z planes."""
import os

import numpy as np
import pytest

from paper_2010_01628_amd import inputs
from paper_2010_01628_amd import lbm as L

pytestmark = pytest.mark.gpu

SIZES = [(16, 12, 10), (32, 16, 8), (33, 17, 5), (70, 41, 9), (1, 3, 2), (2, 1, 1), (130, 9, 3), (23, 300, 4), (512, 2, 3),
         (513, 2, 3), (1100, 5, 2), (64, 64, 64), (16, 16, 16), (32, 32, 32), (100, 20, 10), (1, 1, 1), (5, 2, 1)]


def _run(n, size, two_step, seed=5, **kw):
    import torch

    nx, ny, nz = size
    rho, u, F = inputs.random_lattice_fields(nx, ny, nz, seed=seed, umax=0.05, fmax=1e-3)
    Ft = torch.from_numpy(F).cuda()
    force = kw.pop("force_kind", "field")
    if force == "field":
        kw.update(force_mode=L.LBM_FORCE_FIELD, force_field_ptr=Ft.data_ptr())
    elif force == "uniform":
        kw.update(force_mode=L.LBM_FORCE_UNIFORM, force=(1e-4, -2e-4, 3e-4))
    elif force == "kolmogorov":
        kw.update(force_mode=L.LBM_FORCE_KOLMOGOROV, kolmogorov_amp=1e-4)
    saved = os.environ.get("LBM_TWO_STEP")
    if two_step is None:
        os.environ.pop("LBM_TWO_STEP", None)
    else:
        os.environ["LBM_TWO_STEP"] = two_step
    try:
        lat = L.Lattice(L.make_params(nx, ny, nz, omega=1.7, **kw), force_field=Ft)
    finally:
        if saved is None:
            os.environ.pop("LBM_TWO_STEP", None)
        else:
            os.environ["LBM_TWO_STEP"] = saved
    lat.init(rho, u)
    lat.step(n)
    f = lat.get_populations()
    assert lat.step_count == n
    lat.close()
    return f


def _same(n, size, **kw):
    import torch

    a = _run(n, size, "0", **kw)
    assert torch.isfinite(a).all()
    for mode in ("1", None):  # sweeps; the default (blocks on small lattices)
        b = _run(n, size, mode, **kw)
        assert torch.equal(a, b), (mode, float((a - b).abs().max()))


@pytest.mark.parametrize("size", SIZES)
@pytest.mark.parametrize("walls", [False, True])
def test_sizes(size, walls):
    if walls and size[1] < 2:
        pytest.skip("walls need ny >= 2")
    _same(5, size, precision="fp32", walls_y=walls)


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("kw", [dict(), dict(walls_y=True), dict(moments="raw"), dict(moments="raw", walls_y=True),
                                dict(omega_bulk=1.2, omega_hi=[0.9, 1.1, 1.2, 0.8, 1.3, 1.0, 0.7, 1.4, 1.05]),
                                dict(omega_bulk=1.2, walls_y=True)])
@pytest.mark.parametrize("force", ["none", "uniform", "kolmogorov"])
def test_storage_and_collisions(precision, kw, force):
    _same(4, (37, 19, 11), precision=precision, force_kind=force, **kw)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("moments", ["central", "raw"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("size", [(37, 19, 11), (32, 24, 3), (16, 16, 16)])
def test_d3q27(precision, moments, walls, size):
    _same(5, size, precision=precision, q=27, moments=moments, walls_y=walls)


def test_stochastic_rounding():
    _same(6, (37, 19, 11), precision="bf16", rounding="stochastic", seed=3)


def test_checks_between_pairs():
    """check_every falls on odd steps too: the state there is a whole step's."""
    _same(7, (33, 17, 9), precision="fp32", check_every=3)


@pytest.mark.parametrize("size", [(33, 17, 5), (64, 30, 7)])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("mode", ["1", None])
def test_against_oracle(size, walls, mode):
    import oracle

    nx, ny, nz = size
    rho, u, F = inputs.random_lattice_fields(nx, ny, nz, seed=5, umax=0.05, fmax=1e-3)
    f = _run(6, size, mode, precision="fp64", walls_y=walls).cpu().numpy()
    ref = oracle.run(oracle.init(rho, u), 6, oracle.K(1.7), F=F, walls_y=walls)
    # FP64 against the oracle's dense solve: summation order only
    assert np.abs(f - ref).max() < 1e-13


@pytest.mark.parametrize("q", [19, 27])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("steps,chunk", [(5, "0"), (21, "6"), (35, "16")])
def test_ensemble(q, precision, steps, chunk, monkeypatch):
    """Uneven boxes, with and without captured launches, odd step counts: bit
    for bit the single-step ensemble's."""
    boxes = [(2, 1.2), (7, 1.9), (33, 1.7), (16, 1.5), (70, 1.95), (7, 1.1)]
    monkeypatch.setenv("LBM_ENSEMBLE_GRAPH_STEPS", chunk)

    def run(two):
        monkeypatch.setenv("LBM_TWO_STEP", two)
        ens = L.Ensemble(boxes, q=q, precision=precision)
        for b, (n, _) in enumerate(boxes):
            rho, u, _ = inputs.random_lattice_fields(n, n, n, seed=b + 1, umax=0.03)
            ens.init(b, rho, u)
        ens.step(steps)
        ens.step(3)
        f = [ens.get_populations(b) for b in range(len(boxes))]
        ke = ens.energy()[0]
        assert ens.step_count == steps + 3
        ens.close()
        return f, ke

    (fa, ka), (fb, kb) = run("0"), run("1")
    assert np.array_equal(ka, kb)
    for a, b in zip(fa, fb):
        assert np.isfinite(a).all() and np.array_equal(a, b)


@pytest.mark.parametrize("boxes,q,precision", [
    ([(32, 1.9), (32, 1.5), (7, 1.2)], 19, "fp32"),  # 10 MB
    ([(32, 1.9), (32, 1.5), (7, 1.2)], 27, "fp32"),
    ([(32, 1.9), (32, 1.5)], 19, "fp64"),
    ([(96, 1.9), (96, 1.6), (64, 1.2)], 19, "fp32"),  # 309 MB
])
def test_ensemble_with_streaming_stores(boxes, q, precision, monkeypatch):
    """Ensembles that take streaming stores (below 48 MB or above 256 MiB) in
    boxes whose rows are whole 128-byte lines: bit for bit the single-step
    ensemble's."""
    def run(two):
        monkeypatch.setenv("LBM_TWO_STEP", two)
        ens = L.Ensemble(boxes, q=q, precision=precision)
        for b, (n, _) in enumerate(boxes):
            rho, u, _ = inputs.random_lattice_fields(n, n, n, seed=b + 1, umax=0.03)
            ens.init(b, rho, u)
        ens.step(7)
        f = [ens.get_populations(b) for b in range(len(boxes))]
        ens.close()
        return f

    for a, b in zip(run("0"), run("1")):
        assert np.isfinite(a).all() and np.array_equal(a, b)


def test_arrays_beyond_4_gib(monkeypatch):
    """Population arrays that start beyond 4 GiB from the first (384x400x384
    FP32, 4.5 GB a buffer): passes of two steps equal single steps, bit for
    bit."""
    import torch

    size = (384, 400, 384)
    shape = size[::-1]
    gen = torch.Generator(device="cuda").manual_seed(3)
    rho = 1.0 + 0.01 * torch.rand(shape, generator=gen, dtype=torch.float64, device="cuda")
    u = 0.05 * (torch.rand((3,) + shape, generator=gen, dtype=torch.float64, device="cuda") - 0.5)
    runs = []
    for two in ("0", "1"):
        monkeypatch.setenv("LBM_TWO_STEP", two)
        lat = L.Lattice(L.make_params(*size, precision="fp32", omega=1.7))
        lat.init(rho, u)
        lat.step(5)
        runs.append(lat.get_populations())
        lat.close()
    assert torch.isfinite(runs[0]).all()
    assert torch.equal(runs[0], runs[1])
