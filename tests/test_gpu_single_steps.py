"""The single-step A-B kernels over several steps (LBM_TWO_STEP=0: without it
calls of two steps and more take passes of two on these sizes): their
addressing, row staging and wavefront cap bit for bit, and their states against
the FP64 oracle."""
import numpy as np
import pytest

from paper_2010_01628_amd import inputs
from paper_2010_01628_amd import lbm as L

from gpu_helpers import gpu_run, oracle_run, say

pytestmark = pytest.mark.gpu

CASES = [("fp64", 19, "central", False), ("fp32", 19, "central", False), ("fp32", 19, "central", True), ("fp16", 19, "central", False),
         ("bf16", 19, "central", True), ("fp32", 27, "central", True), ("fp32", 19, "raw", False), ("fp64", 27, "raw", False)]


@pytest.mark.parametrize("precision,q,moments,walls", CASES)
@pytest.mark.parametrize("var,value", [("LBM_OFF32", "0"), ("LBM_ROW_STAGING", "0"), ("LBM_WAVES_PER_SIMD", "0"),
                                       ("LBM_WAVES_PER_SIMD", "2"), ("LBM_XCD_CHUNK", "4")])
def test_launch_choices_are_bitwise_identical(precision, q, moments, walls, var, value, monkeypatch):
    nx, ny, nz = 64, 44, 16  # whole-row work-groups, ragged in y
    rho, u, F = inputs.random_lattice_fields(nx, ny, nz, seed=33, umax=0.05, fmax=1e-3)
    kw = dict(omega=1.8, force=F, walls=walls, q=q, moments=moments)
    monkeypatch.setenv("LBM_TWO_STEP", "0")
    a = gpu_run(nx, ny, nz, rho, u, 6, precision, "ab", **kw)
    monkeypatch.setenv(var, value)
    b = gpu_run(nx, ny, nz, rho, u, 6, precision, "ab", **kw)
    assert np.isfinite(a["f"]).all() and np.array_equal(a["f"], b["f"])


@pytest.mark.parametrize("size", [(64, 20, 9), (37, 19, 11)])  # staged rows, direct reads
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("walls", [False, True])
def test_against_oracle(orc, size, precision, walls, monkeypatch):
    steps = 6
    rho, u, F = inputs.random_lattice_fields(*size, seed=9, umax=0.05, fmax=1e-3)
    monkeypatch.setenv("LBM_TWO_STEP", "0")
    got = gpu_run(*size, rho, u, steps, precision, "ab", omega=1.8, force=F, walls=walls)
    ref = oracle_run(orc, rho, u, steps, omega=1.8, F=F, walls=walls)
    err = np.abs(got["f"] - ref["f"]).max()
    say(f"single steps {size} {precision} walls={walls}: max |f - f_oracle| = {err:.2e}")
    # per step: the stored deviations (below 0.02 here) rounded to the storage
    # type, unit roundoff eps, four roundings' worth after the collision's
    # recombination; the collision's arithmetic, some 16 roundings of moments of
    # deviations up to 0.2; the oracle's dense solve on values up to 1 in FP64
    eps = {"fp64": 2.0 ** -53, "fp32": 2.0 ** -24, "fp16": 2.0 ** -11, "bf16": 2.0 ** -8}[precision]
    arith = 2.0 ** -53 if precision == "fp64" else 2.0 ** -24
    assert err < steps * (4 * 0.02 * eps + 16 * 0.2 * arith + 64 * 2.0 ** -53)
