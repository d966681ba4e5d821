"""Steps inside a graph run pipelined (push of step n beside the field update of
step n + 1, three buffer sets, once 32 or 64 steps pay for the third): the same bits as
the same steps launched one by one, at the edges of the tiles and particle
groups, for stretches of one, two, an odd number and many steps, and after the
state has been read, saved and loaded from each of the three buffers."""
import numpy as np
import pytest

import inputs

cp = pytest.importorskip("paper_2303_05599_amd")
torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    cp.lib()
    yield


def make(N, prec, n, form, log, load=True, nc=3):
    L = 6.0 * N / 64
    ctx = cp.Context(dict(N=N, L_fm=L, n_sheets=1, tau_max_fm=256 * L / N / 8, precision=prec, reunit_every=5,
                          record_every=3, seed=7, n_colors=nc),
                     dict(n=n, mass_GeV=1.27, pT_max_GeV=3.0, tau_form_fm=form, color_update=cp.COLOR_LOG if log else cp.COLOR_ROTATE, seed=8))
    if nc == 2:
        ctx.init_mv()
        return ctx
    ctx.set_push_lanes(4)
    if load:
        ctx.load_state(inputs.random_state(N, 4), 0, inputs.random_particles(n, N, 5))
    return ctx


def state(ctx):
    return [ctx.get_state(k) for k in range(5)]


def run(ctx, N, steps, graph):
    dt = 6.0 * N / 64 / N / 8
    for k in steps:
        if graph:
            ctx.evolve((ctx.n + k) * dt * (1 - 1e-12))
        else:
            ctx.step(k)
    return state(ctx)


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N,n", [(4, 1), (6, 64), (12, 700), (18, 65), (27, 513), (48, 4000), (81, 700), (432, 3001), (768, 2000)])
def test_same_bits_as_single_steps(N, n, prec):
    log = n % 2
    for form in (0.0, 4.5 * 6.0 / 64 / 8):
        if N >= 432 and form:
            continue
        got = []
        for graph in (False, True):
            ctx = make(N, prec, n, form, log)
            run(ctx, N, (16, 18), graph)
            ctx.load_state(inputs.random_state(N, 4), 0, inputs.random_particles(n, N, 5))
            got.append(run(ctx, N, (1, 2, 3, 16, 7, 16, 18), graph))
            got[-1].append(ctx.observables())
            ctx.close()
        for a, b in zip(*got):
            assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N,n", [(4, 1), (16, 64), (27, 65), (96, 3001)])
def test_same_bits_for_two_colours(N, n, prec):
    for form in (0.0, 4.5 * 6.0 / 64 / 8):
        got = []
        for graph in (False, True):
            ctx = make(N, prec, n, form, 0, nc=2)
            got.append(run(ctx, N, (1, 2, 3, 16, 7, 16, 18), graph) + [ctx.observables()])
            ctx.close()
        for a, b in zip(*got):
            assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N,n", [(16, 200), (18, 1000), (432, 190001)])
def test_same_bits_with_paths(N, n, prec):
    """The light-like paths beside the gather push and beside the table push."""
    got = []
    for graph in (False, True):
        ctx = make(N, prec, n, 0.0, 0)
        ctx.enable_jets(x_offset=0.3)
        run(ctx, N, (16, 18), graph)
        ctx.load_state(inputs.random_state(N, 4), 0, inputs.random_particles(n, N, 5))
        got.append(run(ctx, N, (1, 2, 16, 7, 16, 13), graph))
        got[-1] += [ctx.observables(), ctx.jet_observables(), ctx.get_state(cp.STATE_JET_W), ctx.get_state(cp.STATE_JET_F)]
        ctx.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b, equal_nan=True)


@pytest.mark.parametrize("N,n,jets,mode", [(16, 384, False, cp.PUSH_GATHER), (16, 385, False, cp.PUSH_TABLE),
                                           (162, 16383, True, cp.PUSH_GATHER), (162, 16384, True, cp.PUSH_TABLE)])
def test_default_push(N, n, jets, mode):
    """Both lines of the rule, and that a choice of the caller stays."""
    for chosen in (None, cp.PUSH_GATHER, cp.PUSH_TABLE):
        ctx = cp.Context(dict(N=N, L_fm=6.0, n_sheets=1, tau_max_fm=0.1), dict(n=n, mass_GeV=1.27))
        if chosen is not None:
            ctx.set_push_mode(chosen)
        if jets:
            ctx.enable_jets()
        assert ctx.push_mode() == (mode if chosen is None else chosen)
        ctx.close()


@pytest.mark.parametrize("steps", [1, 2, 3, 4])
def test_saved_from_any_buffer(steps, tmp_path):
    """save, load, set_state and a change of the launch, from whichever buffer holds the state."""
    N, n = 18, 300
    ref, ctx = make(N, cp.FP64, n, 0.0, 0), make(N, cp.FP64, n, 0.0, 0)
    run(ref, N, (32, steps), False)
    run(ctx, N, (32, steps), True)
    path = str(tmp_path / "s.bin")
    ctx.save(path)
    want = run(ref, N, (21,), False)
    for a, b in zip(want, run(ctx, N, (21,), True)):
        assert np.array_equal(a, b)
    again = make(N, cp.FP64, n, 0.0, 0, False)
    again.load(path)
    again.set_launch(16, 16, 1, 1, 3)
    for a, b in zip(want, run(again, N, (21,), True)):
        assert np.array_equal(a, b)
    for c in (ref, ctx, again):
        c.close()
