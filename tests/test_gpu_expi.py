"""The exponential of an algebra element in every range of its argument that takes
a number of terms of its own, through the drift of the first step, which multiplies
each link by exp(i eps E) (no kick at n = 0)."""
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


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("size", [1e-3, 0.17, 0.18, 0.4, 0.6, 0.75, 1.5, 3.0, 12.0])
def test_drift_of_the_links(size, prec):
    """n = 0: no kick; U <- exp(i 2 E) U with |2 E| = size on both sides of every bound (sqrt(4 c1 / 3)).
    Error: a few roundings of the entries, and of each squaring of the result for |Y| > 2."""
    N, L = 18, 6.0
    st = inputs.random_state(N, 5)
    rng = np.random.default_rng(6)
    E = rng.normal(size=(2, N, N, 8))
    E *= rng.uniform(0.9, 1.1, (2, N, N, 1)) * size / 2 / np.sqrt((E ** 2).sum(axis=-1, keepdims=True) / 3)
    st = dict(st, E=E, phi=np.zeros_like(st["phi"]), pi=np.zeros_like(st["pi"]))
    ctx = cp.Context(dict(N=N, L_fm=L, n_sheets=1, tau_max_fm=1.0, precision=prec))
    ctx.load_state(st, 0)
    U0, E0 = ctx.get_state(cp.STATE_U), ctx.get_state(cp.STATE_E)
    ctx.step(1)
    U1 = ctx.get_state(cp.STATE_U)
    ctx.close()
    l = np.zeros((8, 3, 3), complex)
    for k, a, b in ((0, 0, 1), (3, 0, 2), (5, 1, 2)):
        l[k][a, b] = l[k][b, a] = 1
        l[k + 1][a, b], l[k + 1][b, a] = -1j, 1j
    l[2] = np.diag([1, -1, 0])
    l[7] = np.diag([1, 1, -2]) / np.sqrt(3)
    Y = np.tensordot(E0, l, 1)     # 2 E^a T^a
    w, v = np.linalg.eigh(Y)
    want = (v * np.exp(1j * w)[..., None, :]) @ v.conj().swapaxes(-1, -2) @ U0.reshape(Y.shape)
    u = 2.0 ** -52 if prec == cp.FP64 else 2.0 ** -23
    squarings = max(0, int(np.ceil(np.log2(max(np.abs(w).max(), 1e-9)))))
    assert np.abs(U1.reshape(Y.shape) - want).max() <= 24 * u * 2 ** squarings
