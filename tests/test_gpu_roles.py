"""The field update with four wavefronts per 64 sites (the default up to 384^2)
against the thread-per-site tiles: the same operations in the same order, so the
same bits, at the edges of its 16 x 4 tiles and on both sides of the size rule."""
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


def evolve(N, prec, n, steps, tile, form=0.0):
    L = 6.0 * N / 64
    ctx = cp.Context(dict(N=N, L_fm=L, n_sheets=1, tau_max_fm=64 * L / N / 8, precision=prec, reunit_every=3, record_every=4, seed=7),
                     dict(n=n, mass_GeV=1.27, pT_max_GeV=3.0, tau_form_fm=form, seed=8))
    if tile:
        ctx.set_launch(32, 4, 1, 1, 3)
    P = inputs.random_particles(n, N, 5) if n else None
    ctx.load_state(inputs.random_state(N, 4), 0, P)
    ctx.step(steps)
    out = [ctx.get_state(k) for k in range(4)] + ([ctx.get_state(cp.STATE_PARTICLES)] if n else [])
    ctx.close()
    return out


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N", [4, 6, 16, 18, 27, 48, 81])
def test_same_bits_as_the_tiles(N, prec):
    """With particles formed at 0 (G stored at n = 0), formed later (no G at first) and without any."""
    for n, form in ((70, 0.0), (70, 4.5 * 6.0 / 64 / 8), (0, 0.0)):
        for a, b in zip(evolve(N, prec, n, 8, True, form), evolve(N, prec, n, 8, False, form)):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("N", [384, 432])
def test_size_rule(N):
    """The largest lattice of the rule and the next one: one step from the initial condition."""
    got = []
    for tile in (False, True):
        ctx = cp.Context(dict(N=N, L_fm=6.0, n_sheets=1, tau_max_fm=0.1, seed=3))
        if tile:
            ctx.set_launch(16, 16, 1, 1, 3)
        ctx.init_mv()
        ctx.step(2)
        got.append([ctx.get_state(k) for k in range(4)])
        ctx.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
