"""State exchange on the device: every part, round trip, below and above the size that passes
straight through pinned memory, across chunks, after a reordering, in both gauge groups and precisions."""
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


def third_rows(U):
    """conj(r1 x r2), the products as the interchange documents them."""
    r1, r2 = U[..., 0, :], U[..., 1, :]
    out = U.copy()
    out[..., 2, :] = np.conj(np.cross(r1, r2))
    return out


# N = 18: every part below the direct size; 96: above it; 216: links in two chunks of 8 MB
@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N,n", [(18, 1), (18, 77), (96, 5000), (216, 60001)])
def test_round_trip(N, n, prec):
    real = np.float64 if prec == cp.FP64 else np.float32
    ctx = cp.Context(dict(N=N, L_fm=6.0 * N / 64, precision=prec, tau_max_fm=1.0), dict(n=n, mass_GeV=1.27, seed=3))
    st, P = inputs.random_state(N, 6), inputs.random_particles(n, N, 7)
    ctx.load_state(st, 1, P)
    got = ctx.state()
    for k in ("phi", "E", "pi"):
        assert np.array_equal(got[k], st[k].astype(real))
    rows = st["U"][..., :2, :]
    rounded = rows.real.astype(real) + 1j * rows.imag.astype(real).astype(np.float64)
    assert np.array_equal(got["U"][..., :2, :], rounded)
    assert np.max(np.abs(got["U"] - third_rows(got["U"]))) < 4e-16
    Q = ctx.get_state(cp.STATE_PARTICLES)
    assert np.array_equal(Q, P.astype(real))
    # p^tau from the constraint in both columns
    pt = ctx.get_state(cp.STATE_PTAU)
    a = 6.0 / 64 / 0.1973269804
    ref = np.sqrt(P[:, 3] ** 2 + P[:, 4] ** 2 + (0.125 * P[:, 5]) ** 2 + (1.27 * a) ** 2)
    assert np.allclose(pt[:, 1], ref, rtol=1e-15 if prec == cp.FP64 else 1e-7, atol=0)
    assert np.allclose(pt[:, 0], ref, rtol=1e-15 if prec == cp.FP64 else 2e-7, atol=0)
    # after steps (and a reordering) the rows are still the particles they were: the same run in another order
    order = np.random.default_rng(2).permutation(n)
    ctx.step(4)
    A = ctx.get_state(cp.STATE_PARTICLES)
    ctx.load_state(st, 1, P[order])
    ctx.step(4)
    B = ctx.get_state(cp.STATE_PARTICLES)
    assert np.array_equal(A[order], B)
    ctx.close()


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N", [12, 128])
def test_round_trip_su2(N, prec):
    real = np.float64 if prec == cp.FP64 else np.float32
    rng = np.random.default_rng(4)
    q = rng.normal(size=(2, N, N, 4))
    q /= np.linalg.norm(q, axis=-1, keepdims=True)
    q = q.astype(real).astype(np.float64)
    w, a1, a2, a3 = np.moveaxis(q, -1, 0)
    U = np.stack([np.stack([w + 1j * a3, a2 + 1j * a1], -1), np.stack([-a2 + 1j * a1, w - 1j * a3], -1)], -2)
    st = dict(U=U, phi=rng.normal(size=(N, N, 3)), E=rng.normal(size=(2, N, N, 3)), pi=rng.normal(size=(N, N, 3)))
    ctx = cp.Context(dict(N=N, n_colors=2, precision=prec, tau_max_fm=1.0), dict(n=200, mass_GeV=1.27))
    P = inputs.random_particles(200, N, 7)
    P[:, 9:14] = 0
    ctx.load_state(st, 0, P)
    got = ctx.state()
    assert np.array_equal(got["U"], U)
    for k in ("phi", "E", "pi"):
        assert np.array_equal(got[k], st[k].astype(real))
    assert np.array_equal(ctx.get_state(cp.STATE_PARTICLES), P.astype(real))
    ctx.close()
