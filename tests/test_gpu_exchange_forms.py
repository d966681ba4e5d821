"""Every part of the state in both directions where the form it crosses in changes: by a kernel or a
copy command (16 KiB of the device's arrays), in one chunk or several (8 MiB), rows that would share
the sets of the host's caches, few links and many, converted by one thread or more.  The values are
those of the interchange, third rows included, bit for bit."""
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
    """conj(r1 x r2), each product and sum rounded by itself in the order of the interchange."""
    a, b, out = U[..., 0, :], U[..., 1, :], U.copy()
    for j in range(3):
        j1, j2 = (j + 1) % 3, (j + 2) % 3

        def product(x, y):
            return x.real * y.real - x.imag * y.imag, x.real * y.imag + x.imag * y.real
        (pr, pi), (qr, qi) = product(a[..., j1], b[..., j2]), product(a[..., j2], b[..., j1])
        out[..., 2, j] = (pr - qr) + 1j * (qi - pi)
    return out


# algebra rows: 16 KiB at 16^2 (FP64) and 22.6^2 (FP32); 192 KiB of links at 26^2; 8 MiB of links' rows (30 of the
# 36) at 187^2 FP64 and 264^2 FP32, of algebra elements at 362^2 (FP64, interchange), 512^2 (FP32)
@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N", [4, 16, 18, 24, 27, 32, 128, 256, 288, 384, 576])
def test_three_colours(N, prec):
    real = np.float64 if prec == cp.FP64 else np.float32
    ctx = cp.Context(dict(N=N, L_fm=6.0 * N / 64, precision=prec, tau_max_fm=1.0))
    rng = np.random.default_rng(N)
    # (the exchange does not look at what it moves)
    st = {k: rng.normal(size=s).astype(real).astype(np.float64) for k, s in (("phi", (N, N, 8)), ("E", (2, N, N, 8)), ("pi", (N, N, 8)))}
    U = (rng.normal(size=(2, N, N, 3, 3, 2)).astype(real).astype(np.float64)).view(np.complex128)[..., 0]
    ctx.load_state(dict(st, U=U), 0)
    got = ctx.state()
    for k in st:
        assert np.array_equal(got[k], st[k]), k
    assert np.array_equal(got["U"], third_rows(U))
    ctx.close()


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N", [4, 16, 18, 24, 64, 324, 512, 1024])
def test_two_colours(N, prec):
    real = np.float64 if prec == cp.FP64 else np.float32
    rng = np.random.default_rng(N)
    w, x, y, z = rng.normal(size=(4, 2, N, N)).astype(real).astype(np.float64)
    U = np.stack([np.stack([w + 1j * z, y + 1j * x], -1), np.stack([-y + 1j * x, w - 1j * z], -1)], -2)
    st = {k: rng.normal(size=s).astype(real).astype(np.float64) for k, s in (("phi", (N, N, 3)), ("E", (2, N, N, 3)), ("pi", (N, N, 3)))}
    ctx = cp.Context(dict(N=N, n_colors=2, precision=prec, tau_max_fm=1.0))
    ctx.load_state(dict(st, U=U), 0)
    got = ctx.state()
    for k in st:
        assert np.array_equal(got[k], st[k]), k
    assert np.array_equal(got["U"], U)
    ctx.close()


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 3277, 52428, 52429, 120001])
def test_records(n, prec):
    real = np.float64 if prec == cp.FP64 else np.float32
    ctx = cp.Context(dict(N=16, L_fm=1.5, precision=prec, tau_max_fm=1.0), dict(n=n, mass_GeV=1.27))
    P = inputs.random_particles(n, 16, 7).astype(real).astype(np.float64)
    P[:, 0:2] = np.minimum(P[:, 0:2], 15.25)   # (a value of both precisions)
    P[:, 14:16] = np.floor(P[:, 0:2] + 0.5) % 16
    ctx.load_state(inputs.random_state(16, 6), 1, P)
    assert np.array_equal(ctx.get_state(cp.STATE_PARTICLES), P)
    ctx.close()


@pytest.mark.parametrize("prec", [cp.FP64, cp.FP32])
@pytest.mark.parametrize("N", [16, 27, 128, 324])
def test_paths(N, prec):
    """The paths' arrays against the sums of their squares that the device itself takes."""
    ctx = cp.Context(dict(N=N, L_fm=6.0 * N / 64, n_sheets=1, precision=prec, tau_max_fm=1.0, record_every=2, seed=3))
    ctx.enable_jets()
    ctx.init_mv()
    ctx.step(4)
    F, W = ctx.get_state(cp.STATE_JET_F), ctx.get_state(cp.STATE_JET_W)
    a = 6.0 / 64 / 0.1973269804
    dpx2 = np.sum(F[:, :, 0, :] ** 2) * 4.0 / 8 / (N * N * a * a)
    assert abs(ctx.jet_observables()[-1][1] / dpx2 - 1) < (1e-12 if prec == cp.FP64 else 1e-5)
    eye = np.einsum("yxij,yxkj->yxik", W, W.conj())
    assert np.max(np.abs(eye - np.eye(3))) < (1e-13 if prec == cp.FP64 else 1e-5)
    ctx.close()
