"""Which kernels the entry points launch, on which buffers and with how much
device memory, on the CPU: a child process loads the library over a HIP
runtime that records launches instead of running them (hip_recorder.cpp)."""
import json
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
STREAM = 0x1000  # any non-null stream

PREAMBLE = """
import ctypes, json, sys, types
import numpy as np
rec = ctypes.CDLL({shim!r}, mode=ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
rec.rec_arg.restype = ctypes.c_void_p
rec.rec_threads.restype = rec.rec_live_bytes.restype = rec.rec_peak_bytes.restype = ctypes.c_int64
sys.modules["torch"] = types.ModuleType("torch")  # its HIP runtime must not be the one that is bound
from paper_2010_01628_amd import lbm as L
L.lib()
STREAM = {stream}


def lattice(nx, ny, nz, **kw):
    return L.lbm_create(L.make_params(nx, ny, nz, **kw), STREAM)


def launched():
    # (kernel, its first two arguments) since the last call
    out = [(rec.rec_name(i).decode(), rec.rec_arg(i, 0), rec.rec_arg(i, 1)) for i in range(rec.rec_count())]
    rec.rec_clear()
    return out


def kinds():
    # what each launch since the last call is
    return ["block" if "k_step_pair_block" in n else "sweep" if "k_step_pair" in n or "k_ens_pair" in n
            else "single" if "k_step" in n or "k_ens_step" in n else "other" for n, _, _ in launched()]


def accesses(h):
    # two single steps: whether each streams, and whether it takes the planes downwards
    import re
    out = []
    for _ in range(2):
        launched()
        L.lbm_step(h, 1)
        i, name = [(i, rec.rec_name(i).decode()) for i in range(rec.rec_count())][-1]
        flags = [f == "1" for f in re.findall("Lb([01])E", name)]
        at = 1 if re.search("k_step_ab_rows|k_step_aa_odd_rows|k_step_mlp|k_mhd_step|k_sc_step|k_cg_step", name) else \
            0 if "k_phase_step" in name else 2
        out.append([flags[at], bool(rec.rec_rev(i))])
    return out
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    so = tmp_path_factory.mktemp("recorder") / "librecorder.so"
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-o", str(so), os.path.join(HERE, "hip_recorder.cpp")], check=True)

    def run(code, **env):
        full = {k: v for k, v in os.environ.items() if not k.startswith("LBM_")}
        full.update(env)
        body = PREAMBLE.format(shim=str(so), stream=STREAM) + textwrap.dedent(code)
        r = subprocess.run([sys.executable, "-c", body], cwd=ROOT, env=full, capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-3000:]
        return json.loads(r.stdout.splitlines()[-1])

    return run


def test_recorder_sees_the_default_paths(recorder):
    """Small A-B lattices take blocks, large ones sweeps, two steps to a
    launch; an odd step, AA and LBM_TWO_STEP=0 single steps."""
    code = """
    out = []
    for size, kw, n in (((64, 20, 9), {}, 6), ((64, 20, 9), {}, 7), ((200, 101, 75), {}, 5), ((64, 20, 9), dict(streaming="aa"), 3)):
        h = lattice(*size, **kw)
        launched()
        L.lbm_step(h, n)
        out.append(kinds())
        L.lbm_destroy(h)
    print(json.dumps(out))
    """
    assert recorder(code) == [["block"] * 3, ["block"] * 3 + ["single"], ["sweep"] * 2 + ["single"], ["single"] * 3]
    assert recorder(code, LBM_TWO_STEP="0") == [["single"] * n for n in (6, 7, 5, 3)]


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 6, 7, 10, 13])
def test_captured_steps_keep_the_buffer_parity(recorder, steps):
    """Recorded into a graph, lbm_step(n) and lbm_ensemble_step(n) leave the
    populations in the buffer that n single steps leave them in: a graph of an
    even number of steps can be replayed.  (A pass of two steps changes
    buffers once.)"""
    got = recorder(f"""
    n = {steps}
    out = []
    h = lattice(64, 20, 9)
    e = L.lbm_ensemble_create([(32, 1.5)] * 64, 19, L.LBM_FP64, STREAM)
    for step, obj in ((L.lbm_step, h), (L.lib().lbm_ensemble_step, e)):
        rec.rec_set_capturing(1)
        launched()
        step(obj, n)
        ls = launched()
        assert all(a == b for (_, _, a), (_, b, _) in zip(ls, ls[1:]))  # each launch reads what the one before wrote
        out.append([ls[0][1] == ls[-1][2], len(ls)])
        rec.rec_set_capturing(0)
        step(obj, 4)
        out[-1].append(kinds())
    print(json.dumps(out))
    """)
    for back, launches, eager in got:
        assert back == (steps % 2 == 0)
        assert launches < steps or steps < 4  # pairs are still taken
        assert eager in (["block"] * 2, ["sweep"] * 2)


@pytest.mark.parametrize("var,value,single", [
    ("LBM_OFF32", "0", True), ("LBM_OFF32", "1", False), ("LBM_ROW_STAGING", "0", True), ("LBM_ROW_STAGING", "1", True),
    ("LBM_XCD_CHUNK", "4", True), ("LBM_WAVES_PER_SIMD", "0", True), ("LBM_WAVES_PER_SIMD", "2", True)])
def test_single_step_variables_reach_single_steps(recorder, var, value, single):
    """A variable that picks a launch or an addressing of the single step
    takes single steps, so that it has the effect it is documented with;
    LBM_TWO_STEP=1 beside it takes passes of two steps all the same."""
    code = """
    out = []
    e = L.lbm_ensemble_create([(32, 1.5)] * 64, 19, L.LBM_FP64, STREAM)
    for h in (lattice(64, 20, 9), lattice(200, 101, 75)):
        launched()
        L.lbm_step(h, 6)
        out.append(kinds())
    L.lib().lbm_ensemble_step(e, 6)
    out.append(kinds())
    print(json.dumps(out))
    """
    singles = [["single"] * 6] * 3
    assert recorder(code, **{var: value}) == (singles if single else [["block"] * 3, ["sweep"] * 3, ["sweep"] * 3])
    assert recorder(code, LBM_TWO_STEP="1", **{var: value}) == [["sweep"] * 3] * 3


def test_tuned_launch_is_kept_per_plane_order(recorder):
    """lbm_tune's choice is kept for lattices whose single steps take the
    planes in the same order as the ones it was timed on: streaming accesses
    (cache_policy 1) always upwards, the default upwards and downwards in turn
    on this size in place."""
    got = recorder("""
    out = []
    for policy in (1, 0, 1, 0):
        h = lattice(96, 90, 80, streaming="aa", cache_policy=policy)
        L._check(L.lib().lbm_tune(h, 2, None, None, None, None))
        out.append(L.lbm_step_count(h) > 0)  # candidates were timed on steps
        L.lbm_destroy(h)
    print(json.dumps(out))
    """)
    assert got == [True, True, False, False]


@pytest.mark.parametrize("steps", [1, 3])
@pytest.mark.parametrize("dstate", [False, True])
def test_rollout_scratch(recorder, steps, dstate):
    """A rollout's gradient keeps its states, two adjoint states, a gradient
    per row of nodes and the losses' partial sums, and nothing else of the
    lattice's size."""
    got = recorder(f"""
    n, steps = 32, {steps}
    N = n ** 3
    h = lattice(n, n, n)
    m = L.lbm_mlp_create(None, np.ones(11, dtype=np.float32), STREAM)
    L.lbm_set_mlp(h, m)
    before = rec.rec_live_bytes()
    targets = np.ones((steps, 10, N), dtype=np.float32)
    out = np.zeros((19, N), dtype=np.float32)
    L.lbm_mlp_accumulate_rollout_grad(m, h, targets.ctypes.data, steps, np.ones(10), None,
                                      out.ctypes.data if {dstate} else None)
    print(json.dumps([rec.rec_live_bytes() - before, N, L.lbm_device_bytes(h)]))
    """)
    used, N, lattice_bytes = got
    state = lattice_bytes // 2  # (two buffers and small tables)
    allowed = 2 * 19 * 4 * N + steps * state + 4 * 1737 * N // 32 + steps * 8 * N // 64 + 65536
    assert used <= allowed, (used, allowed)


def test_benchmark_ensemble_takes_passes_of_two_steps(recorder):
    """The 64-box workload's plain ensembles take two steps to a pass (bench.py
    counts their bytes by that)."""
    got = recorder("""
    from paper_2010_01628_amd import inputs
    boxes = [(n, inputs.omega_from_nu(nu)) for n, nu, _ in inputs.ensemble_boxes()]
    out = []
    for q in (19, 27):
        e = L.lbm_ensemble_create(boxes, q, L.LBM_FP32, STREAM)
        launched()
        L.lib().lbm_ensemble_step(e, 4)
        out.append(kinds())
        L.lib().lbm_ensemble_destroy(e)
    print(json.dumps(out))
    """)
    assert got == [["sweep"] * 2] * 2


@pytest.mark.parametrize("size,kw,streams", [
    ((96, 64, 40), dict(), True), ((200, 64, 40), dict(precision="fp64"), True),     # rows of whole halves of lines
    ((100, 64, 40), dict(), False), ((201, 64, 40), dict(precision="fp64"), False),  # shared ones: all in the cache
    ((100, 100, 100), dict(), True), ((100, 100, 100), dict(streaming="aa"), False),  # state 152 and 76 MB, f 152
    ((180, 180, 100), dict(streaming="aa"), True), ((161, 160, 159), dict(streaming="aa"), False),  # f 492, 622 MB
    ((118, 52, 170), dict(precision="fp64"), True), ((150, 130, 110), dict(precision="fp64"), False),  # state 317, 652
    ((150, 130, 110), dict(), True), ((150, 130, 110), dict(q=27), True), ((180, 180, 100), dict(q=27), False),
    ((96, 64, 40), dict(precision="fp16"), False)])
def test_checkpoint_stores(recorder, size, kw, streams):
    """lbm_get_populations stores with the streaming hint where rows do not
    share half-lines, or where the state would leave the last-level cache, and
    not from 2-byte storage."""
    name = recorder(f"""
    h = lattice(*{size}, **{kw})
    f = np.zeros(27 * {size[0] * size[1] * size[2]})
    launched()
    L.lbm_get_populations(h, f.ctypes.data, True)
    print(json.dumps(launched()[0][0]))
    """)
    assert "k_get_pops" in name and ("Lb1EEEv" in name) == streams, name


@pytest.mark.parametrize("size,precision,streams", [
    ((96, 96, 90), "fp16", False), ((128, 128, 110), "bf16", True), ((201, 97, 93), "fp16", True),
    ((96, 96, 90), "fp32", False), ((128, 128, 110), "fp32", True), ((192, 160, 128), "fp32", True),  # 126, 274, 598 MB
    ((150, 130, 110), "fp32", True), ((201, 199, 100), "fp32", False), ((200, 200, 100), "fp32", False),  # 326, 608
    ((128, 128, 128), "fp64", False)])
def test_restore_loads(recorder, size, precision, streams):
    """lbm_set_populations reads arrays larger than the last-level cache with
    the streaming hint: into 2-byte storage, and into 4-byte storage on whole
    lines or where the state fits the cache."""
    name = recorder(f"""
    h = lattice(*{size}, precision={precision!r})
    f = np.zeros(19 * {size[0] * size[1] * size[2]})
    launched()
    L.lbm_set_populations(h, f.ctypes.data, True)
    print(json.dumps(launched()[0][0]))
    """)
    assert "k_set_pops" in name and ("Lb1EEEv" in name) == streams, name


MHD = dict(magnetic=dict(eta=0.1))
SC = dict(shan_chen=dict(G=-5.0))
CG = dict(colour=dict(alpha_red=7 / 9), walls_y=True)
PHASE = dict(phase=dict(rho_light=1.0, rho_heavy=10.0, sigma=1e-3, width=4.0, mobility=0.1))


@pytest.mark.parametrize("size,kw,streams", [
    ((64, 64, 64), dict(), True), ((64, 64, 80), dict(), False),                  # 20, 25 MB a buffer
    ((64, 64, 64), dict(q=27), True), ((64, 64, 80), dict(q=27), False),          # 28, 35 MB
    ((64, 64, 64), dict(precision="fp64"), False),
    ((160, 160, 128), dict(), True), ((161, 160, 128), dict(), False),            # 498 MB: whole lines, shared ones
    ((48, 300, 230), dict(), True), ((48, 300, 230), dict(walls_y=True), False),  # 503 MB: staged rows fill lines
    ((64, 64, 48), MHD, False),
    ((64, 64, 80), PHASE, False), ((170, 150, 141), PHASE, False), ((97, 90, 80), dict(precision="fp64", **PHASE), False),
    ((128, 128, 128), PHASE, True),
    ((64, 80, 80), SC, True), ((64, 64, 64), dict(precision="fp64", **SC), True), ((128, 80, 64), SC, False),
    ((80, 80, 64), dict(precision="fp64", **SC), False), ((96, 96, 96), SC, False),
    ((72, 72, 64), SC, True), ((75, 75, 75), SC, False), ((150, 140, 130), SC, False), ((201, 199, 150), SC, True),
    ((64, 64, 80), CG, True), ((128, 80, 64), CG, False), ((67, 66, 65), CG, False), ((150, 130, 110), CG, True)])
def test_single_steps_stream_where_it_pays(recorder, size, kw, streams):
    """Both sides of each bound of the rule for ordinary accesses, upwards
    (a lattice that alternates has ordinary ones anyway)."""
    got = recorder(f"""
    h = lattice(*{size}, **{kw})
    print(json.dumps(accesses(h)))
    """, LBM_TWO_STEP="0")
    assert got == [[streams, False]] * 2


@pytest.mark.parametrize("boxes,q,precision,want", [
    ([200], 27, "LBM_FP32", "single"), ([144], 27, "LBM_FP64", "single"), ([160], 19, "LBM_FP64", "single"),
    ([80] * 4, 27, "LBM_FP64", "single"), ([100] * 3, 27, "LBM_FP64", "single"),
    ([32] * 32, 27, "LBM_FP32", "single"), ([64], 19, "LBM_FP32", "single"),
    ([200], 19, "LBM_FP32", "sweep"), ([48] * 16, 19, "LBM_FP64", "sweep"), ([128] * 2, 27, "LBM_FP32", "sweep"),
    ([48, 64, 96, 33] * 4, 27, "LBM_FP32", "sweep")])
def test_ensemble_passes_where_they_are_faster(recorder, boxes, q, precision, want):
    """The ensemble's estimate counts rounds of whole blocks on each XCD's
    units: passes of two steps only where they are measured faster."""
    got = recorder(f"""
    e = L.lbm_ensemble_create([(n, 1.5) for n in {boxes}], {q}, L.{precision}, STREAM)
    launched()
    L.lib().lbm_ensemble_step(e, 4)
    print(json.dumps(kinds()))
    """)
    assert got == [want] * (4 if want == "single" else 2)
