"""Device memory that a context holds: what a call needs only while it runs is not kept by it."""
import concurrent.futures
import ctypes

import numpy as np
import pytest

cp = pytest.importorskip("paper_2303_05599_amd")
torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
SLACK = 4 << 20   # the allocator's granularity (2 MiB), at two places
stream = None     # one for all: the runtime keeps spill memory of its own per hardware queue


@pytest.fixture(scope="module", autouse=True)
def gpu():
    global stream
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    own = torch.cuda.Stream()
    stream = ctypes.c_void_p(own.cuda_stream)
    yield


def free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def make(N, sheets, prec, nc):
    L = 6.0 * min(1.0, N / 64)
    return cp.Context(dict(N=N, L_fm=L, n_sheets=sheets, tau_max_fm=400 * L / N / 8, precision=prec, seed=5, n_colors=nc),
                      dict(n=N * N // 3, mass_GeV=1.27, tau_form_fm=0.0, seed=4), stream=stream)


def held_by_calls(call, *args):
    """What the first of four contexts' calls leaves allocated, and what those of the others add; all is gone with the last one."""
    warm = make(*args)      # the runtime's own memory
    call(warm)
    warm.close()
    at_first = free()
    ctxs = [make(*args) for _ in range(4)]
    made = free()
    call(ctxs[0])
    first = made - free()
    for c in ctxs[1:]:
        call(c)
    others = made - free() - first
    for c in ctxs:
        c.close()
    assert at_first - free() <= SLACK
    return first, others


KEPT = 256 << 20  # blocks that wait for the next call, whatever the number of contexts


@pytest.mark.parametrize("N,sheets,prec,nc", [(96, 50, cp.FP64, 3), (96, 50, cp.FP32, 3), (324, 20, cp.FP64, 2),
                                              (576, 18, cp.FP64, 3), (576, 18, cp.FP32, 3)])
def test_initial_condition(N, sheets, prec, nc):
    first, others = held_by_calls(lambda c: c.init_mv(), N, sheets, prec, nc)
    assert first <= KEPT + SLACK and others <= SLACK


@pytest.mark.parametrize("N,prec,nc", [(96, cp.FP64, 3), (216, cp.FP32, 3), (324, cp.FP64, 2)])
def test_state_exchange(N, prec, nc):
    """Fields and particles read and installed; their chunks lie in memory that the context has anyway."""
    def call(ctx):
        ctx.init_mv()
        st, P = ctx.state(), ctx.get_state(cp.STATE_PARTICLES)
        ctx.load_state(st, 0, P)
    first, others = held_by_calls(call, N, 1, prec, nc)
    assert first <= KEPT + SLACK and others <= SLACK


def test_third_buffer_set():
    """Taken by an evolve of many steps while a quarter of the device's memory stays free, and not otherwise."""
    def run():
        ctx = make(144, 1, cp.FP64, 3)
        ctx.init_mv()
        before = free()
        ctx.evolve(64 * 6.0 / 144 / 8 * (1 - 1e-12))
        ctx.sync()
        assert ctx.n == 64
        held, P = before - free(), ctx.get_state(cp.STATE_PARTICLES)
        ctx.close()
        return held, P
    size = 144 * 144 * (68 + 8) * 8
    held, P = run()
    assert held >= size
    avail, total = torch.cuda.mem_get_info()
    filler = torch.empty(avail - total // 5, dtype=torch.uint8, device="cuda")
    try:
        held, Q = run()
    finally:
        del filler
        torch.cuda.empty_cache()
    assert held < size // 2 and np.array_equal(P, Q)


def test_threads():
    """Contexts used side by side on threads of their own: initial conditions, steps and exchange as one after the other."""
    sizes = [(48, 9, cp.FP64, 3), (96, 25, cp.FP64, 3), (96, 25, cp.FP32, 3), (144, 12, cp.FP64, 3), (128, 7, cp.FP64, 2), (216, 4, cp.FP32, 3)]

    def work(size):
        N, sheets, prec, nc = size
        L = 6.0 * min(1.0, N / 64)
        ctx = cp.Context(dict(N=N, L_fm=L, n_sheets=sheets, tau_max_fm=400 * L / N / 8, precision=prec, seed=5, n_colors=nc),
                         dict(n=N * N // 3, mass_GeV=1.27, tau_form_fm=0.0, seed=4), stream=None)
        for _ in range(2):
            ctx.init_mv()
            ctx.evolve(40 * L / N / 8 * (1 - 1e-12))
            ctx.load_state(ctx.state(), ctx.n, ctx.get_state(cp.STATE_PARTICLES))
        out = [ctx.get_state(k) for k in range(5)]
        ctx.close()
        return out

    alone = [work(s) for s in sizes]
    with concurrent.futures.ThreadPoolExecutor(len(sizes)) as ex:
        together = list(ex.map(work, sizes))
    for a, b in zip(alone, together):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("N,sheets,prec,nc", [(48, 1, cp.FP32, 3), (96, 9, cp.FP32, 3), (96, 9, cp.FP64, 3), (64, 4, cp.FP32, 2)])
def test_initial_condition_with_the_third_set(N, sheets, prec, nc):
    """Started again where a long run has left a third buffer set to work in: the same bits."""
    ctx = make(N, sheets, prec, nc)
    ctx.init_mv()
    first = [ctx.get_state(k) for k in range(5)]
    ctx.evolve(64 * 6.0 * min(1.0, N / 64) / N / 8 * (1 - 1e-12))
    ctx.init_mv()
    again = [ctx.get_state(k) for k in range(5)]
    ctx.close()
    assert all(np.array_equal(x, y) for x, y in zip(first, again))
