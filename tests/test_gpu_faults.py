"""What the library does when a call of the HIP runtime fails under it, forced from the host
by a shim in a process of its own (hip_shim.c): it reports the error, and what it does
next is right."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
MALLOC, HOST_MALLOC, GRAPH_LAUNCH, KERNEL, ELAPSED = range(5)
ALL = 1 << 40
N, BOX = 48, 4.5
DT = BOX / N / 8


def make(cp, init=True, **glasma):
    g = dict(N=N, L_fm=BOX, n_sheets=1, tau_max_fm=400 * DT, seed=5)
    g.update(glasma)
    ctx = cp.Context(g, dict(n=500, mass_GeV=1.27, tau_form_fm=0.0, pT_max_GeV=3.0, seed=4), stream=None)
    if init:
        ctx.init_mv()
    return ctx


def evolve(ctx, steps):
    ctx.evolve((ctx.n + steps) * DT * (1 - 1e-12))


def state(ctx):
    return [ctx.get_state(k) for k in range(5)]


def check_same(ctx, ref):
    for a, b in zip(state(ctx), state(ref)):
        assert np.array_equal(a, b)


def failed_graph_launch(cp, shim):
    """A stretch whose launch failed leaves a graph of separate steps; the next call pipelines."""
    ctx, ref = make(cp), make(cp)
    shim.shim_fail(GRAPH_LAUNCH, 0, 1, 0)
    with pytest.raises(cp.CpicError):
        evolve(ctx, 20)
    assert ctx.n == 0
    evolve(ctx, 40)
    ref.step(40)
    check_same(ctx, ref)


def tuned(cp, shim, pair_ms, piped_ms):
    """Tune with the pipelined trial (the last 1 + 2 timings) answered with piped_ms and all others with pair_ms:
    the choice, and the kernels in the graph of a stretch of 16 steps."""
    for turn in (ALL, None):
        ctx, ref = make(cp), make(cp)
        ctx.step(3)
        turn = turn or timings - 3
        before = shim.shim_calls(ELAPSED)
        shim.shim_elapsed(pair_ms, turn, piped_ms)
        report = ctx.tune(2)
        timings = shim.shim_calls(ELAPSED) - before
    assert "step pipelined, four in a stretch" in report
    evolve(ctx, 13)                  # up to the reordering at step 16
    k0 = shim.shim_calls(KERNEL)
    evolve(ctx, 16)                  # one graph, captured now
    kernels = shim.shim_calls(KERNEL) - k0
    evolve(ctx, 40)
    ref.step(3 + 13 + 16 + 40)
    check_same(ctx, ref)
    return report.strip().splitlines()[-1], kernels


def tuner_keeps_the_faster_form(cp, shim):
    # per step: pairs 1 ms / 2, four pipelined steps 1 ms / 4, or 10 ms / 4
    piped_line, piped = tuned(cp, shim, 1.0, 1.0)
    line, separate = tuned(cp, shim, 1.0, 10.0)
    # 17 launches pipelined and 32 separate, besides the reordering's
    assert 17 <= piped <= 17 + 8 < 32 <= separate, (piped, separate)
    assert "pipelined step" in piped_line and "separate step" in line, piped_line + line


def failed_workspace(cp, shim):
    """No memory for the initial condition's work: an error, the state and the next launches untouched."""
    small, ctx, ref = make(cp), make(cp, n_sheets=40, init=False), make(cp, init=False)
    for c in (ctx, ref):
        c.load_state(small.state(), 0, small.get_state(cp.STATE_PARTICLES))
    evolve(ctx, 40)
    ref.step(40)
    shim.shim_fail(MALLOC, 0, ALL, 1 << 20)
    with pytest.raises(cp.CpicError):
        ctx.init_mv()
    shim.shim_fail(MALLOC, 0, 0, 0)
    check_same(ctx, ref)
    evolve(ctx, 20)
    ref.step(20)
    check_same(ctx, ref)
    ctx.init_mv()
    check_same(ctx, make(cp, n_sheets=40))


def failed_third_set(cp, shim):
    """No memory for the third buffer set: the steps stay separate launches, without an error."""
    ctx, ref = make(cp), make(cp)
    shim.shim_fail(MALLOC, 0, ALL, 1 << 20)
    k0 = shim.shim_calls(KERNEL)
    evolve(ctx, 64)
    assert shim.shim_calls(KERNEL) - k0 >= 32
    shim.shim_fail(MALLOC, 0, 0, 0)
    evolve(ctx, 40)
    ctx.sync()
    ref.step(104)
    check_same(ctx, ref)


def another_device_current(cp, shim):
    """The caller has another device current: the context's memory still comes from its own, and the caller's choice stays."""
    ctx, ref = make(cp, n_sheets=20, init=False), make(cp, n_sheets=20)
    shim.shim_set_device(1)
    ctx.init_mv()
    evolve(ctx, 64)
    got = state(ctx)
    ctx.load_state(dict(zip(("U", "phi", "E", "pi"), got)), ctx.n, got[4])
    evolve(ctx, 16)
    ctx.sync()
    assert shim.shim_device() == 1 and shim.shim_elsewhere() == 0
    shim.shim_set_device(0)
    ref.step(80)
    check_same(ctx, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("scenario", [failed_graph_launch, tuner_keeps_the_faster_form, failed_workspace, failed_third_set, another_device_current], ids=lambda f: f.__name__)
def test_forced_failure(scenario, tmp_path):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    so = str(tmp_path / "hip_shim.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", so, os.path.join(HERE, "hip_shim.c"), "-ldl"], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), scenario.__name__, so], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("done"), r.stdout[-2000:] + r.stderr[-3000:]


if __name__ == "__main__":
    shim_ = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)   # before anything loads the runtime
    shim_.shim_fail.argtypes = [ctypes.c_int, ctypes.c_long, ctypes.c_long, ctypes.c_size_t]
    shim_.shim_elapsed.argtypes = [ctypes.c_float, ctypes.c_long, ctypes.c_float]
    shim_.shim_elsewhere.restype = ctypes.c_long
    shim_.shim_calls.argtypes, shim_.shim_calls.restype = [ctypes.c_int], ctypes.c_long
    sys.path.insert(0, os.path.dirname(HERE))
    import paper_2303_05599_amd as cp_
    cp_.lib()
    globals()[sys.argv[1]](cp_, shim_)
    assert shim_.shim_calls(KERNEL) > 0, "the shim does not stand between the library and the runtime"
    print("done")
