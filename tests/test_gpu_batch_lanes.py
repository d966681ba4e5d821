"""The default lanes and launch groups of single-precision batches (three lanes
where larger events do not do a third of the work) against one lane: the same bits."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("sizes", [(384, 384, 384, 288), (512, 384, 384, 384, 64), (512, 512, 64)])
def test_default_lanes(sizes):
    """No event above the group budget, one among smaller ones, and two that do most of it."""
    gl = [dict(N=N, L_fm=6.0 * min(1, N / 64), n_sheets=1, tau_max_fm=1.0, precision=cp.FP32, seed=10 + k, reunit_every=4)
          for k, N in enumerate(sizes)]
    pl = [dict(n=300 + 500 * k, mass_GeV=1.27, pT_max_GeV=2.0, tau_form_fm=0.0, seed=20 + k) for k in range(len(sizes))]
    got = []
    for lanes in (None, 1):
        b = cp.Batch(gl, pl)
        if lanes:
            b.set_lanes(lanes)
        b.init_mv()
        b.step(19)
        got.append([a for e, N in enumerate(sizes) for a in (b.get_state(e, cp.STATE_E, (2, N, N, 8)), b.observables(e),
                    b.get_state(e, cp.STATE_PARTICLES, (pl[e]["n"], 20)))])
        b.close()
    for a, c in zip(*got):
        assert np.array_equal(a, c)
