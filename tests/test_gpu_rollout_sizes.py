"""Rollout losses and gradients on lattices that do not fill the training
kernels' blocks: node counts that are no multiple of 64 or 256, rows shorter
and longer than 64 nodes; and one network used with lattices of several sizes.
Node counts near the 1024 of test_gpu_rollout.py, whose checks and tolerances
these are (the BF16 effect on a gradient averages over as many nodes)."""
import numpy as np
import pytest

import test_gpu_rollout as R
from paper_2010_01628_amd import lbm as L

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[(67, 5, 3), (7, 11, 13), (129, 4, 2)], ids=lambda s: "x".join(map(str, s)))
def size(request, monkeypatch):
    for name, v in zip(("NX", "NY", "NZ"), request.param):
        monkeypatch.setattr(R, name, v)
    return request.param


def test_loss(orc, size):
    R.test_rollout_loss_matches_oracle(orc, 2)


def test_one_step(orc, size):
    R.test_one_step_rollout_is_the_one_step_gradient(orc)
    R.test_one_step_against_exact_model_gradient(orc)


def test_parameter_gradient(orc, size):
    R.test_rollout_parameter_gradient(orc, 2)


@pytest.mark.parametrize("steps", [1, 3])
def test_state_gradient(orc, size, steps):
    R.test_rollout_state_gradient(orc, steps)


def test_step_weights(orc, size):
    R.test_step_weights_and_per_step_losses(orc)


def test_energy(orc, size):
    """The energy term's value and its part of both gradients."""
    c = R.Case(orc, 3)
    c.set_energy_weight(2e5)
    loss, g, ds = c.gpu(want_dstate=True)
    want = c.loss(orc, bf16=True)
    assert abs(loss - want) / want < 1e-4
    gn = np.linalg.norm(g)
    assert abs(c.fd_theta(orc, g) - gn) <= R.GRAD_TOL * gn
    n2 = float(np.sum(ds * ds))
    h = 1e-7 * np.abs(c.f0).max() / np.abs(ds).max()
    assert abs(c.fd_state(orc, ds, h) - n2) <= R.GRAD_TOL * n2
    c.close()


def test_one_network_on_several_lattices(orc, monkeypatch):
    """A network's scratch, grown on a larger lattice or a longer rollout,
    serves smaller ones: results equal a fresh network's, bit for bit."""
    def run(case, net):
        case.lat.attach_mlp(net)
        net.zero_grad()
        net.set_energy_weight(2e5)
        loss, per, ds = case.lat.accumulate_rollout_grad(net, case.tgt, R.SIGMA, want_dstate=True, want_steps=True)
        state = case.lat.get_populations().cpu().numpy()
        assert np.array_equal(state, case.f0)  # the lattice's state is untouched
        return loss, per, ds.cpu().numpy(), net.grad()

    shared = None
    for (nx, ny, nz), steps in (((67, 5, 3), 3), ((7, 5, 3), 2), ((64, 8, 4), 1), ((9, 7, 5), 4), ((67, 5, 3), 3)):
        for name, v in (("NX", nx), ("NY", ny), ("NZ", nz)):
            monkeypatch.setattr(R, name, v)
        c = R.Case(orc, steps)
        if shared is None:
            shared = L.Mlp(c.P, R.SCALES)
        a, b = run(c, shared), run(c, c.mlp)
        assert a[0] == b[0]
        for x, y in zip(a[1:], b[1:]):
            assert np.isfinite(x).all() and np.array_equal(x, y)
        c.lat.attach_mlp(None)
        c.close()
    shared.close()
