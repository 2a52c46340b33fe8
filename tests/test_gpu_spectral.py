"""The line-spectral FP64 S-build at the sizes where its tilings end: lines of less
than, exactly and just over a block of 8 frequency pairs and of 16 rows, one and two
column blocks of V, one to four row blocks of [U | shifted U], partial row blocks
split over the full ones, the fold of d = 1, the largest line count and the first
size past it (tile kernel). Reference: the oracle's dense matrices, and for N too
large for those the same products by zero-padded FFTs in numpy. Tolerance: the
suite's FP64 bound 1e-12 (normwise and entrywise): every sum is FP64 with at most
n + 1 terms per axis, so the error is a small multiple of (3 n) 2^-53 < 1e-13."""
import numpy as np
import pytest
import torch

from oracle import prony_oracle as O
from paper_2012_11430_amd import api
from tests._close import assert_close, assert_close_per_matrix

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = 1e-12


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _problem(d, n, m, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    N, G = (n + 1) ** d, (2 * n + 2) ** d
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)   # noqa: E731
    return cn(G), cn(N, m), rng.uniform(0.5, 2.0, m), cn(N, m)


def _fft_pencil(grid, d, n, U, s, V):
    """S_l, l = 0..d, by a circular convolution on the (2n+2)^d box: k - h + e_l lies in
    {-n..n+1} on every axis, where the residues modulo 2n + 2 are distinct."""
    L, axes = 2 * n + 2, tuple(range(1, d + 1))
    g = np.roll(grid.reshape((L,) * d), -n, axis=tuple(range(d)))      # point p at index p mod L
    pad = np.zeros((V.shape[1],) + (L,) * d, dtype=complex)
    box = (slice(None),) + (slice(0, n + 1),) * d
    pad[box] = V.T.reshape((-1,) + (n + 1,) * d)
    Z = np.fft.ifftn(np.fft.fftn(g)[None] * np.fft.fftn(pad, axes=axes), axes=axes)
    out = []
    for l in range(d + 1):
        lo = [1 if l == a else 0 for a in range(1, d + 1)]
        Y = Z[(slice(None),) + tuple(slice(x, x + n + 1) for x in lo)].reshape(V.shape[1], -1).T
        out.append(U.conj().T @ Y / s[None, :])
    return np.stack(out)


@pytest.mark.parametrize("d,n,m", [
    (1, 1, 1), (1, 14, 3), (1, 15, 8), (1, 16, 16), (1, 255, 17), (1, 576, 24), (1, 1023, 32),
    (2, 1, 1), (2, 6, 4), (2, 7, 8), (2, 8, 9), (2, 14, 16), (2, 15, 17), (2, 16, 25), (2, 23, 32), (2, 32, 24),
    (3, 1, 2), (3, 6, 7), (3, 7, 8), (3, 8, 9), (3, 9, 33 - 8), (3, 14, 16)])
@pytest.mark.parametrize("with_s0", [False, True])
def test_tile_edges_match_the_oracle(d, n, m, with_s0):
    grid, U, s, V = _problem(d, n, m, seed=7000 + 100 * d + n + m)
    print(f"spectral d={d} n={n} m={m} s0={with_s0}", flush=True)
    ref = O.pencil_matrices(grid, d, n, U, s, V, with_s0=with_s0)
    got = api.build_S(_dev(grid), d, n, _dev(U), _dev(s), _dev(V), with_s0=with_s0)
    assert_close_per_matrix(got.cpu().numpy(), ref, TOL, "row-major factors")
    again = api.build_S(_dev(grid), d, n, _dev(U.T).T, _dev(s), _dev(V.T).T, with_s0=with_s0)
    assert torch.equal(got, again)       # the strides do not enter the arithmetic


@pytest.mark.parametrize("d,n,m", [(1, 20000, 5), (1, 57599, 3), (1, 57600, 2), (2, 127, 20), (2, 239, 9), (2, 240, 4),
                                   (3, 20, 20), (3, 24, 10), (3, 31, 4)])
def test_large_shapes_match_padded_ffts(d, n, m):
    grid, U, s, V = _problem(d, n, m, seed=9000 + 100 * d + n + m)
    print(f"spectral d={d} n={n} m={m}", flush=True)
    ref = _fft_pencil(grid, d, n, U, s, V)
    got = api.build_S(_dev(grid), d, n, _dev(U), _dev(s), _dev(V), with_s0=True).cpu().numpy()
    assert_close_per_matrix(got, ref, TOL, f"d={d} n={n} m={m}")


def test_non_finite_columns_stay_in_their_columns():
    # a NaN or infinity in one column of V (or U) reaches that column (row) of every S_l only
    d, n, m = 2, 20, 20
    grid, U, s, V = _problem(d, n, m, seed=11)
    for bad in (np.nan, np.inf):
        Vb, Ub = V.copy(), U.copy()
        Vb[37, 3] = bad
        Ub[100, 18] = bad
        S = api.build_S(_dev(grid), d, n, _dev(Ub), _dev(s), _dev(Vb), with_s0=True).cpu().numpy()
        finite = np.isfinite(S)
        assert not finite[:, :, 3].any() and not finite[:, 18, :].any()
        keep = np.ones((m, m), dtype=bool)
        keep[:, 3] = keep[18, :] = False
        assert finite[:, keep].all()
        ref = O.pencil_matrices(grid, d, n, U, s, V, with_s0=True)
        np.testing.assert_allclose(S[:, keep], ref[:, keep], rtol=0, atol=1e-12 * np.abs(ref).max())


def _fft_product(grid, d, n, X, adjoint):
    """T X or T^* X by a circular convolution on the (2n+2)^d box (samples p <= n only)."""
    L, axes = 2 * n + 2, tuple(range(1, d + 1))
    g = grid.reshape((L,) * d).copy()
    for a in range(d):
        g[(slice(None),) * a + (L - 1,)] = 0.0                          # p = n + 1 is not read
    g = np.roll(g, -n, axis=tuple(range(d)))
    if adjoint:                                                        # conj(f(-p))
        g = np.conj(np.roll(np.flip(g, axis=tuple(range(d))), 1, axis=tuple(range(d))))
    pad = np.zeros((X.shape[1],) + (L,) * d, dtype=complex)
    box = (slice(None),) + (slice(0, n + 1),) * d
    pad[box] = X.T.reshape((-1,) + (n + 1,) * d)
    Y = np.fft.ifftn(np.fft.fftn(g)[None] * np.fft.fftn(pad, axes=axes), axes=axes)
    return Y[box].reshape(X.shape[1], -1).T


@pytest.mark.parametrize("d,n,r", [
    (1, 1, 2), (1, 14, 1), (1, 255, 16), (1, 576, 17), (1, 1023, 64), (1, 57599, 3), (1, 57600, 2),
    (2, 1, 1), (2, 7, 8), (2, 14, 9), (2, 15, 16), (2, 16, 33), (2, 31, 64), (2, 63, 40), (2, 95, 1), (2, 239, 5),
    (2, 240, 3), (3, 1, 5), (3, 6, 1), (3, 7, 8), (3, 8, 12), (3, 15, 7), (3, 16, 40), (3, 20, 1), (3, 24, 9), (3, 31, 3)])
def test_products_at_tile_edges(d, n, r):
    rng = np.random.Generator(np.random.PCG64(5000 + 100 * d + n + r))
    N, G = (n + 1) ** d, (2 * n + 2) ** d
    grid = rng.standard_normal(G) + 1j * rng.standard_normal(G)
    X = rng.standard_normal((N, r)) + 1j * rng.standard_normal((N, r))
    # the samples with a coordinate n + 1 are not read
    edge = np.zeros((2 * n + 2,) * d, dtype=bool)
    for a in range(d):
        edge[(slice(None),) * a + (2 * n + 1,)] = True
    dirty = grid.copy()
    dirty[edge.reshape(-1)] = np.nan
    big = torch.zeros((N, r + 3), dtype=torch.complex128, device=DEV)
    big[:, :r] = _dev(X)
    for adjoint in (False, True):
        print(f"spectral product d={d} n={n} r={r} adjoint={adjoint}", flush=True)
        ref = _fft_product(grid, d, n, X, adjoint)
        out = torch.full((N, r + 2), 7.0, dtype=torch.complex128, device=DEV)
        api.toeplitz_mm(_dev(dirty), d, n, big[:, :r], adjoint=adjoint, out=out[:, :r])
        got = out.cpu().numpy()
        assert_close(got[:, :r], ref, TOL, f"adjoint={adjoint}")
        assert np.all(got[:, r:] == 7.0)                 # nothing written past the r columns
        again = api.toeplitz_mm(_dev(grid), d, n, _dev(X), adjoint=adjoint)
        assert torch.equal(again, out[:, :r])


@pytest.mark.parametrize("shapes", [
    [(1, 63, 5), (1, 1023, 32), (2, 7, 3), (2, 63, 20), (3, 3, 9), (3, 15, 31), (2, 30, 16), (3, 8, 8)],
    [(2, 12, 4)],
    [(2, 240, 2), (2, 12, 4)]])      # an instance past the form: the whole batch on the tiles
def test_fp64_batches_match_single_builds(shapes):
    probs = [_problem(d, n, m, seed=300 + i) for i, (d, n, m) in enumerate(shapes)]
    dev = [(d, n, _dev(f), _dev(U), _dev(s), _dev(V)) for (d, n, m), (f, U, s, V) in zip(shapes, probs)]
    batch = api.Batch(dev, prec="fp64")
    batch.run()
    eager = [S.clone() for S in batch.S]
    for S, (d, n, f, U, s, V) in zip(eager, dev):
        ref = api.build_S(f, d, n, U, s, V)
        # the sums over groups of frequencies are grouped differently: rounding only
        assert_close_per_matrix(S.cpu().numpy(), ref.cpu().numpy(), TOL, f"d={d} n={n}")
    batch.capture()
    for rep in range(3):
        for S in batch.S:
            S.zero_()
        batch.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(eager, batch.S)), f"replay {rep}"
        (torch.randn(4096, device=DEV) * 3).sum().item()
    batch.close()


@pytest.mark.parametrize("d,n,r", [(1, 40, 3), (2, 9, 5), (2, 17, 1), (3, 5, 9)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_products_keep_non_finite_samples_to_their_rows(d, n, r, adjoint):
    """A NaN sample reaches the rows of T (or T^*) that hold it, and no others."""
    grid, _, _, X = _problem(d, n, r, seed=7700 + n)
    p = (n,) * (d - 1) + (2,)
    print(f"non-finite product d={d} n={n} r={r} adjoint={adjoint}", flush=True)
    at = np.ravel_multi_index(tuple(x + n for x in p), (2 * n + 2,) * d)
    bad = grid.copy()
    bad[at] = np.nan
    T = O.toeplitz(bad, d, n, 0)
    T = T.conj().T if adjoint else T
    hit = np.isnan(T).any(axis=1)
    assert 0 < hit.sum() < T.shape[0]
    got = api.toeplitz_mm(_dev(bad), d, n, _dev(X), adjoint=adjoint).cpu().numpy()
    assert np.array_equal(np.isnan(got).any(axis=1), hit) and np.array_equal(np.isnan(got).all(axis=1), hit)
    assert_close(got[~hit], T[~hit] @ X, TOL, "rows without the NaN")


@pytest.mark.parametrize("d,n,m", [
    (2, 1, 1), (2, 6, 4), (2, 7, 15), (2, 14, 16), (2, 15, 17), (2, 16, 32), (2, 31, 3), (2, 33, 20),
    (3, 1, 2), (3, 3, 16), (3, 6, 7), (3, 7, 17), (3, 8, 32), (3, 14, 9)])
def test_adjoint_at_tile_edges(d, n, m):
    """Row blocks of 16 lines (n + 2 rows), one and two column blocks, one to three blocks of
    the inverse transform's points. The sums hold N m terms on the way to a point of the grid,
    in line transforms of FP64: the error stays a small multiple of (3 n + m) 2^-53 < 1e-13."""
    _, U, s, V = _problem(d, n, m, seed=7800 + 100 * d + n + m)
    rng = np.random.Generator(np.random.PCG64(n))
    gS = rng.standard_normal((d, m, m)) + 1j * rng.standard_normal((d, m, m))
    print(f"spectral adjoint d={d} n={n} m={m}", flush=True)
    ref = O.pencil_adjoint(gS, d, n, U, s, V)
    got = api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64")
    assert_close(got.cpu().numpy(), ref, TOL, f"adjoint d={d} n={n} m={m}")
    col = api.build_S_adjoint(_dev(gS), d, n, _dev(U.T).T, _dev(s), _dev(V.T).T, prec="fp64")
    assert torch.equal(col, got)
    assert np.all(got.cpu().numpy()[ref == 0] == 0)       # points that no T_l holds


@pytest.mark.parametrize("d,n,m", [(2, 9, 3), (3, 4, 17)])
def test_adjoint_keeps_non_finite_rows_to_their_points(d, n, m):
    _, U, s, V = _problem(d, n, m, seed=7900 + n)
    rng = np.random.Generator(np.random.PCG64(n))
    gS = rng.standard_normal((d, m, m)) + 1j * rng.standard_normal((d, m, m))
    ref = O.pencil_adjoint(gS, d, n, U, s, V)
    U[1, 0] = np.nan
    hit = np.isnan(O.pencil_adjoint(gS, d, n, U, s, V))
    got = api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64").cpu().numpy()
    assert 0 < hit.sum() < hit.size
    assert np.array_equal(np.isnan(got), hit)
    assert_close(got[~hit], ref[~hit], TOL, "points without the NaN")


@pytest.mark.parametrize("shapes", [
    [(2, 7, 4), (2, 33, 20), (3, 4, 17), (2, 1, 1), (3, 8, 32), (2, 15, 16)],
    [(2, 9, 5), (1, 60, 7), (3, 3, 3)],       # d = 1: the tile kernels
])
def test_fp64_batched_adjoints_match_the_oracle(shapes):
    probs = [_problem(d, n, m, seed=8100 + 10 * d + n) for d, n, m in shapes]
    rng = np.random.Generator(np.random.PCG64(3))
    gS = [rng.standard_normal((d, m, m)) + 1j * rng.standard_normal((d, m, m)) for d, n, m in shapes]
    batch = api.Batch([(d, n, _dev(f), _dev(U), _dev(s), _dev(V)) for (d, n, m), (f, U, s, V) in zip(shapes, probs)],
                      prec="fp64")
    print(f"batched adjoint {shapes}", flush=True)
    for scale in (1.0, -2.0):                 # the second call reuses the batch's plan
        got = batch.adjoint(_dev(np.concatenate([scale * g.reshape(-1) for g in gS])))
        for (d, n, m), (f, U, s, V), g, x in zip(shapes, probs, gS, torch.split(got, batch.gf_sizes)):
            assert_close(x.cpu().numpy(), scale * O.pencil_adjoint(g, d, n, U, s, V), TOL, f"d={d} n={n} m={m}")
    batch.close()
