"""Inputs that are not finite in the FP64 line-spectral form: results that are formed again
from their own terms are the right ones, and forming them stays a bounded amount of work
(a diverging run hands such inputs to every call). Measured on clean inputs the calls here
take under 0.1 ms; the limits of 100 ms leave room for the n m multiply-adds per point and
pair of lines on vector units, and none for a sum per thread and term."""
import numpy as np
import pytest
import torch

from paper_2012_11430_amd import api
from tests._close import assert_close

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _cn(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _timed(fn):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    a.record()
    out = fn()
    b.record()
    torch.cuda.synchronize()
    return out, a.elapsed_time(b)


def _fft_gradient(gS, d, n, U, s, V):
    L, E, m = 2 * n + 2, n + 1, U.shape[1]
    Z = np.zeros((L,) * d + (m,), dtype=complex)
    for l in range(d):
        at = tuple(slice(1, E + 1) if a == l else slice(0, E) for a in range(d))
        Z[at] += (U @ gS[l] / s).reshape((E,) * d + (m,))
    W = np.zeros_like(Z)
    W[(slice(0, E),) * d] = V.reshape((E,) * d + (m,))
    axes = tuple(range(d))
    g = np.fft.ifftn(np.sum(np.fft.fftn(Z, axes=axes) * np.conj(np.fft.fftn(W, axes=axes)), axis=-1))
    return np.roll(g, n, axis=axes).reshape(-1)


@pytest.mark.parametrize("d,n,m", [(2, 16, 5), (2, 63, 20), (3, 3, 32), (3, 12, 11)])
@pytest.mark.parametrize("where", ["U", "V", "gS"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_gradients_with_one_entry_not_finite(d, n, m, where, bad):
    rng = np.random.Generator(np.random.PCG64(8800 + 10 * n + d))
    N, E = (n + 1) ** d, n + 1
    U, V, gS, s = _cn(rng, N, m), _cn(rng, N, m), _cn(rng, d, m, m), rng.uniform(0.5, 2.0, m)
    ref = _fft_gradient(gS, d, n, U, s, V)
    row = np.ravel_multi_index((1,) * d, (E,) * d)
    hit = np.zeros((2 * n + 2,) * d, dtype=bool)          # points whose terms hold the entry
    rows = np.zeros((n + 2,) * d, dtype=bool)             # k' of a term with U[k' - e_l]
    cols = np.zeros((E,) * d, dtype=bool)
    if where == "U":
        U[row, m - 1] = bad
        for l in range(d):
            rows[tuple(1 + (a == l) for a in range(d))] = True
        cols[:] = True
    else:
        for l in range(d):
            rows[tuple(slice(1, E + 1) if a == l else slice(0, E) for a in range(d))] = True
        if where == "V":
            V[row, 0] = bad
            cols[(1,) * d] = True
        else:
            gS[0, 0, m - 1] = bad
            rows[:] = False
            rows[(slice(1, E + 1),) + (slice(0, E),) * (d - 1)] = True
            cols[:] = True
    for k in np.argwhere(rows):
        hit[tuple(slice(x, x + E) for x in k)] |= cols[(slice(None, None, -1),) * d]      # p + n = k - h + n
    print(f"gradient d={d} n={n} m={m} {where} {bad}", flush=True)
    args = (_dev(gS), d, n, _dev(U), _dev(s), _dev(V))
    api.build_S_adjoint(*args, prec="fp64")
    got, ms = _timed(lambda: api.build_S_adjoint(*args, prec="fp64"))
    print(f"  {ms:.2f} ms", flush=True)
    got = got.cpu().numpy()
    flat = hit.reshape(-1)
    assert np.array_equal(~np.isfinite(got), flat)
    if not flat.all():
        assert_close(got[~flat], ref[~flat], 1e-12, "points without the entry")
    assert ms < 100.0


@pytest.mark.parametrize("d,n,r", [(1, 40, 3), (1, 1000, 4), (2, 17, 9), (2, 63, 40), (3, 6, 12), (3, 12, 9), (3, 20, 1)])
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("where", ["f", "X"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_products_with_one_entry_not_finite(d, n, r, adjoint, where, bad):
    from tests.test_gpu_spectral import _fft_product
    rng = np.random.Generator(np.random.PCG64(8900 + 10 * n + d))
    N, E = (n + 1) ** d, n + 1
    grid, X = _cn(rng, (2 * n + 2) ** d), _cn(rng, N, r)
    ref = _fft_product(grid, d, n, X, adjoint)
    hit = np.zeros((N, r), dtype=bool)                    # results whose terms hold the entry
    if where == "X":
        X[N // 2, r - 1] = bad
        hit[:, r - 1] = True
    else:
        p = np.array([n // 2] + [-(n // 3)] * (d - 1))    # a sample f(p): T[k, k - p]
        grid[np.ravel_multi_index(tuple(p + n), (2 * n + 2,) * d)] = bad
        k = np.stack(np.meshgrid(*[np.arange(E)] * d, indexing="ij"), -1).reshape(-1, d)
        other = k + p if adjoint else k - p
        hit[np.all((other >= 0) & (other <= n), axis=1)] = True
    print(f"product d={d} n={n} r={r} adjoint={adjoint} {where} {bad}", flush=True)
    f, Xd = _dev(grid), _dev(X)
    api.toeplitz_mm(f, d, n, Xd, adjoint=adjoint)
    got, ms = _timed(lambda: api.toeplitz_mm(f, d, n, Xd, adjoint=adjoint))
    print(f"  {ms:.2f} ms", flush=True)
    got = got.cpu().numpy()
    assert np.array_equal(~np.isfinite(got), hit)
    if not hit.all():
        assert_close(got[~hit], ref[~hit], 1e-12, "results without the entry")
    assert ms < 100.0
