"""The initial condition's transforms and Wilson lines at the sizes where their
kernels change: one, two and more FFT stages, every radix first or last, rows
shorter and longer than a workgroup, partial column groups and row groups, one
and several sheet segments, several chunks of spectral planes.  Against the oracle at the 1e-12 of the
initial-condition parity."""
import numpy as np
import pytest

import oracle
from oracle import su2

cp = pytest.importorskip("paper_2303_05599_amd")
torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    cp.lib()
    yield


def library(N, L, uv, sheets, nc, prec=None):
    ctx = cp.Context(dict(N=N, L_fm=L, uv_GeV=uv, n_sheets=sheets, seed=21, n_colors=nc, precision=cp.FP64 if prec is None else prec, tau_max_fm=1.0))
    ctx.init_mv()
    first = ctx.state()
    ctx.init_mv()   # again in the kept workspace
    st = ctx.state()
    ctx.close()
    for k in st:
        assert np.array_equal(first[k], st[k])
    return st


def compare(st, ref, tol=TOL):
    for k in ("U", "pi"):
        rms = np.sqrt(np.mean(np.abs(ref[k]) ** 2))
        assert np.all(np.abs(st[k] - ref[k]) <= tol * np.maximum(np.abs(ref[k]), rms)), k
    assert not st["phi"].any() and not st["E"].any()


# (N, sheets, fraction of the modes along x that the UV cut keeps; > 1: all of them)
SIZES = [(4, 3, 0.3), (6, 2, 2.0), (8, 5, 0.6), (9, 3, 0.5), (12, 2, 0.4), (16, 40, 0.7), (18, 3, 0.3), (27, 7, 0.9), (32, 20, 2.0),
         (54, 2, 0.2), (64, 3, 0.5), (81, 2, 0.35), (128, 17, 0.3), (162, 2, 0.99), (256, 2, 0.1), (288, 3, 0.35)]


@pytest.mark.parametrize("nc", [3, 2])
@pytest.mark.parametrize("N,sheets,keep", SIZES)
def test_initial_condition(N, sheets, keep, nc):
    L = 6.0 * N / 64
    a = oracle.lattice_spacing(L, N)
    uv = 0.0 if keep > 1 else keep * np.pi / a
    mod = oracle if nc == 3 else su2
    ref = mod.mv_initial_condition(N, L, 2.0, 0.2, uv, sheets, 21)
    compare(library(N, L, uv, sheets, nc), ref)


def test_mode_on_the_cut():
    """A UV cut exactly at a mode along x keeps that column (|k| > Lambda is cut, not >=)."""
    N = 32
    L = 6.0 * N / 64
    a = oracle.lattice_spacing(L, N)
    for m in (1, 5, 16):
        uv = (2 * np.pi / N) * m / a
        ref = oracle.mv_initial_condition(N, L, 2.0, 0.2, uv, 2, 21)
        compare(library(N, L, uv, 2, 3), ref)


def test_float_run_rounds_the_double_result():
    a, b = (library(48, 4.5, 10.0, 3, 3, p) for p in (cp.FP64, cp.FP32))
    assert np.array_equal(a["pi"].astype(np.float32), b["pi"].astype(np.float32))
    assert np.array_equal(a["U"][..., :2, :].astype(np.complex64), b["U"][..., :2, :].astype(np.complex64))


@pytest.mark.parametrize("N,sheets,uv", [(512, 1, 10.0), (1024, 1, 10.0), (1024, 2, 0.0)])
def test_long_rows(N, sheets, uv):
    """Rows of 512 and 1024 sites (two sites per thread; with no cut one chunk holds one
    sheet): the tau = 0 condition holds on a sample of links with the oracle's nuclei, whose residual
    at a solution is at rounding."""
    L = 6.0
    a = oracle.lattice_spacing(L, N)
    st = library(N, L, uv, sheets, 3)
    UA, UB = (oracle.nucleus_links(N, 21, k, sheets, 2.0 * a, 0.2 * a, uv * a) for k in (0, 1))
    rng = np.random.default_rng(3)
    i, y, x = rng.integers(0, 2, 2000), rng.integers(0, N, 2000), rng.integers(0, N, 2000)
    W, U = (UA + UB)[i, y, x], st["U"][i, y, x]
    for k in range(2000):
        F = oracle.proj(W[k] @ (np.eye(3) + U[k].conj().T))
        assert np.max(np.abs(F)) < TOL
