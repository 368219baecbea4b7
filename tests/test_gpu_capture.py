"""lbm_step and lbm_ensemble_step recorded into a HIP graph: replays of an even
number of steps advance the state like eager steps, bit for bit, also where
eager calls take two steps per pass over memory (a pass changes buffers once).
Eager work and synchronizations stand between the replays."""
import ctypes

import numpy as np
import pytest

from paper_2010_01628_amd import inputs
from paper_2010_01628_amd import lbm as L

pytestmark = pytest.mark.gpu

REPLAYS = 3


@pytest.mark.parametrize("size,mode", [((64, 20, 9), None), ((37, 19, 11), "1")])  # blocks, sweeps
@pytest.mark.parametrize("steps", [2, 4, 6])
def test_lattice(size, mode, steps, monkeypatch):
    import torch

    if mode is not None:
        monkeypatch.setenv("LBM_TWO_STEP", mode)
    rho, u, _ = inputs.random_lattice_fields(*size, seed=5, umax=0.05)
    st = torch.cuda.Stream()
    par = L.make_params(*size, precision="fp32", omega=1.7)
    lat = L.Lattice(par, stream=st)
    ref = L.Lattice(par)
    for x in (lat, ref):
        x.init(rho, u)
        x.step(steps)
    r = torch.zeros(lat.shape, dtype=torch.float64, device="cuda")
    v = torch.zeros((3,) + lat.shape, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        lat.step(steps)
        L.lbm_moments_noalloc(lat.h, r.data_ptr(), v.data_ptr(), None)
    for k in range(REPLAYS):
        graph.replay()
        torch.cuda.synchronize()
        ref.step(steps)
        want_r, want_v, _ = ref.moments()
        assert torch.equal(lat.get_populations(), ref.get_populations()), k
        assert torch.equal(r, want_r) and torch.equal(v, want_v), k
    lat.close()
    ref.close()


@pytest.mark.parametrize("steps", [2, 6])
def test_ensemble(steps, monkeypatch):
    import torch

    monkeypatch.setenv("LBM_TWO_STEP", "1")
    boxes = [(7, 1.9), (33, 1.7), (16, 1.5)]
    st = torch.cuda.Stream()
    es = [L.lbm_ensemble_create(boxes, 19, "fp32", st.cuda_stream) for _ in range(2)]
    for e in es:
        for b, (n, _) in enumerate(boxes):
            rho, u, _ = inputs.random_lattice_fields(n, n, n, seed=b + 1, umax=0.03)
            L._check(L.lib().lbm_ensemble_init(e, b, rho.ctypes.data, u.ctypes.data, 0))
        L._check(L.lib().lbm_ensemble_step(e, steps))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        L._check(L.lib().lbm_ensemble_step(es[0], steps))

    def pops(e):
        out = []
        for b, (n, _) in enumerate(boxes):
            f = np.zeros((19, n, n, n))
            L._check(L.lib().lbm_ensemble_get_populations(e, b, ctypes.c_void_p(f.ctypes.data), 0))
            out.append(f)
        return out

    for k in range(REPLAYS):
        graph.replay()
        torch.cuda.synchronize()
        L._check(L.lib().lbm_ensemble_step(es[1], steps))
        for a, b in zip(pops(es[0]), pops(es[1])):
            assert np.isfinite(a).all() and np.array_equal(a, b), k
    for e in es:
        L._check(L.lib().lbm_ensemble_destroy(e))
