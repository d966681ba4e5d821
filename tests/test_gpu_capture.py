"""Steps that the caller captures on the context's stream: `cpic_step` of an even number
of steps returns to the buffer it read, so its graph can be replayed, from wherever
the evolution before it has left the state.  `cpic_evolve` replays graphs of its own there, which
the runtime runs at once, whether it has met the stretch before or not."""
import ctypes

import numpy as np
import pytest

cp = pytest.importorskip("paper_2303_05599_amd")
torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
N, BOX = 48, 4.5
DT = BOX / N / 8


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    cp.lib()
    yield


def make(stream, nc=3):
    ctx = cp.Context(dict(N=N, L_fm=BOX, n_sheets=1, tau_max_fm=400 * DT, seed=5, n_colors=nc),
                     dict(n=500, mass_GeV=1.27, tau_form_fm=0.0, pT_max_GeV=3.0, seed=4), stream=stream)
    ctx.set_watchdog(0)
    ctx.init_mv()
    return ctx


def evolve(ctx, steps):
    ctx.evolve((ctx.n + steps) * DT * (1 - 1e-12))


def same(a, b):
    return all(np.array_equal(a.get_state(k), b.get_state(k)) for k in range(4))


@pytest.mark.parametrize("nc", [3, 2])
@pytest.mark.parametrize("before", [(33,), (34,), (35,), (34, 2), (40, 3, 5)])
def test_captured_steps_replay(before, nc):
    s = torch.cuda.Stream()
    a, b = make(ctypes.c_void_p(s.cuda_stream), nc), make(None, nc)
    for k in before:
        evolve(a, k)
        b.step(k)
    a.sync()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        a.step(4)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        b.step(4)
        assert same(a, b)
    del g
    a.close()
    b.close()


@pytest.mark.filterwarnings("ignore:The CUDA Graph is empty")
@pytest.mark.parametrize("before", [(16,), (16, 16), (32, 16), (20, 12), (64,)])
def test_evolve_on_a_captured_stream(before):
    s = torch.cuda.Stream()
    a, b = make(ctypes.c_void_p(s.cuda_stream)), make(None)
    for k in before:
        evolve(a, k)
        b.step(k)
    a.sync()
    for k in (16, 7):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            evolve(a, k)
        torch.cuda.synchronize()
        b.step(k)
        assert a.n == b.n and same(a, b)
        del g
    evolve(a, 25)
    b.step(25)
    assert same(a, b)
    a.close()
    b.close()
