"""The error of FP64 results in line-spectral form, entry by entry against extended
precision, on samples of even size and on damped ones (0.75 per step, so that entries of one
result span many orders of magnitude).

Products and gradients: an entry's error is bounded by the norms of the lines (d = 3: planes)
along the transformed axes that meet in it, not by its own terms alone:
    |error| <= 4 sqrt(P') 2^-53 sum over the pairs of lines of |line of f|_2 |line of x|_2,
P' points of x's line. Three transforms round independently, each by about sqrt(P' / 2) 2^-53
of its line's norm (a random walk of partial sums); 4 covers the largest of many entries.
S-builds likewise, with the lines of U, f and V that meet: the sum over a line's frequencies
of the three transforms' products is at most |line of U|_2 |line of f|_1 |line of V|_2.

Direct FP64 ('fp64_direct'): |error| <= 4 sqrt(N) 2^-53 sum |terms| for every entry's own terms
(N of them, two to three roundings each; 4 as above)."""
import numpy as np
import pytest
import torch

from paper_2012_11430_amd import api

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
ROUND = 2.0 ** -53


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _box(d, lo, hi):
    return np.stack(np.meshgrid(*[np.arange(lo, hi)] * d, indexing="ij"), -1).reshape(-1, d)


def _problem(d, n, m, modulus):
    """Samples of m modes with noise of 1e-6 of each sample's size, singular factors of T."""
    rng = np.random.Generator(np.random.PCG64(10 * n + d))
    t, c = rng.random((m, d)), rng.uniform(0.5, 1.5, m) * np.exp(2j * np.pi * rng.random(m))
    power = lambda k, r: r ** k.sum(1)[:, None].astype(float) * np.exp(-2j * np.pi * (k @ t.T))   # noqa: E731
    f = power(_box(d, -n, n + 2), modulus) @ c
    f = f * (1 + 1e-6 * rng.standard_normal(f.size))
    Q, R = np.linalg.qr(power(_box(d, 0, n + 1), modulus))
    Q2, R2 = np.linalg.qr(power(_box(d, 0, n + 1), 1 / modulus))
    W, s, Xh = np.linalg.svd(R @ (c[:, None] * R2.conj().T))
    return rng, f, Q @ W, s, Q2 @ Xh.conj().T


def _ext(a, b):
    return np.dot(a.astype(np.clongdouble), b.astype(np.clongdouble))


def _lines(d, n):
    """Points of a line of x (P'), and I_n's index -> line; d = 1: folded lines."""
    N = (n + 1) ** d
    if d == 1:
        P = 16 * max(1, (int(np.sqrt(N)) + 8) // 16)
        return P, np.arange(N) // P
    return (n + 1) ** (d - 1), np.arange(N) // (n + 1) ** (d - 1)


@pytest.mark.parametrize("d,n", [(1, 300), (2, 15), (2, 24), (3, 7)])
@pytest.mark.parametrize("modulus", [1.0, 0.75])
@pytest.mark.parametrize("adjoint", [False, True])
def test_products_hold_the_bound_by_lines(d, n, modulus, adjoint):
    rng, f, U, s, V = _problem(d, n, 4, modulus)
    N, L = (n + 1) ** d, 2 * n + 2
    X = rng.standard_normal((N, 3)) + 1j * rng.standard_normal((N, 3))
    k = _box(d, 0, n + 1)
    flat = lambda p: np.ravel_multi_index(tuple((p + n).T), (L,) * d)      # noqa: E731
    T = np.stack([f[flat(k[i] - k)] for i in range(N)])
    A = T.conj().T if adjoint else T
    print(f"product d={d} n={n} modulus={modulus} adjoint={adjoint}", flush=True)
    got = api.toeplitz_mm(_dev(f), d, n, _dev(X), adjoint=adjoint).cpu().numpy()
    err = np.abs(got - _ext(A, X)).astype(float)
    P, line = _lines(d, n)
    nl = line[-1] + 1
    xs = np.sqrt(np.stack([np.sum(np.abs(X[line == a]) ** 2, axis=0) for a in range(nl)]))          # (lines, 3)
    # norms of the sample lines that the rows of one line meet: over all differences inside them
    fs = np.array([[np.sqrt(np.sum(np.abs(np.unique(A[np.ix_(line == a, line == b)])) ** 2)) for b in range(nl)]
                   for a in range(nl)])
    bound = 4 * np.sqrt(P) * ROUND * (fs @ xs)[line]
    print(f"  largest error / bound {np.max(err / bound):.2f}, / sum |terms| {np.max(err / (np.abs(A) @ np.abs(X))):.1e}", flush=True)
    assert np.all(err <= bound)


@pytest.mark.parametrize("d,n,m", [(2, 16, 5), (2, 24, 9), (3, 7, 20)])
@pytest.mark.parametrize("modulus", [1.0, 0.75])
def test_gradients_hold_the_bound_by_lines(d, n, m, modulus):
    rng, f, U, s, V = _problem(d, n, m, modulus)
    E, L = n + 1, 2 * n + 2
    gS = rng.standard_normal((d, m, m)) + 1j * rng.standard_normal((d, m, m))
    print(f"gradient d={d} n={n} m={m} modulus={modulus}", flush=True)
    got = api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64").cpu().numpy()
    Z = np.zeros((n + 2,) * d + (m,), dtype=np.clongdouble)
    size = np.zeros((n + 2,) * d + (m,))                  # of Z's own terms
    for l in range(d):
        at = tuple(slice(1, E + 1) if a == l else slice(0, E) for a in range(d))
        Z[at] += (_ext(U, gS[l]) / s.astype(np.longdouble)).reshape((E,) * d + (m,))
        size[at] += (np.abs(U) @ np.abs(gS[l]) / s).reshape((E,) * d + (m,))
    kz, Zf = _box(d, 0, n + 2), Z.reshape(-1, m)
    ref = np.zeros(L ** d, dtype=np.clongdouble)
    for h, v in zip(_box(d, 0, n + 1), V):
        ref[np.ravel_multi_index(tuple((kz - h + n).T), (L,) * d)] += np.dot(Zf, np.conj(v.astype(np.clongdouble)))
    zs = np.sqrt(np.sum(size.reshape(n + 2, -1, m) ** 2, axis=1))
    vs = np.sqrt(np.sum(np.abs(V.reshape(E, -1, m)) ** 2, axis=1))
    lines = np.zeros(L)
    for k1 in range(n + 2):
        for h1 in range(E):
            lines[k1 - h1 + n] += zs[k1] @ vs[h1]
    bound = np.repeat(4 * np.sqrt((n + 1) ** (d - 1)) * ROUND * lines, L ** (d - 1))
    err = np.abs(got - ref).astype(float)
    held = np.abs(ref) > 0
    print(f"  largest error / bound {np.max(err[held] / bound[held]):.2f}", flush=True)
    assert np.all(err <= bound)


@pytest.mark.parametrize("d,n,m", [(1, 300, 12), (2, 15, 9), (2, 24, 20), (3, 7, 10)])
@pytest.mark.parametrize("modulus", [1.0, 0.75])
def test_pencil_matrices_hold_the_bound_by_lines(d, n, m, modulus):
    rng, f, U, s, V = _problem(d, n, m, modulus)
    print(f"S d={d} n={n} m={m} modulus={modulus}", flush=True)
    got = api.build_S(_dev(f), d, n, _dev(U), _dev(s), _dev(V)).cpu().numpy()
    k, L = _box(d, 0, n + 1), 2 * n + 2
    P, line = _lines(d, n)
    nl = line[-1] + 1
    norms = lambda X: np.sqrt(np.stack([np.sum(np.abs(X[line == a]) ** 2, axis=0) for a in range(nl)]))   # noqa: E731
    for l in range(d):
        e = np.arange(d) == l
        T = np.stack([f[np.ravel_multi_index(tuple((k[i] - k + e + n).T), (L,) * d)] for i in range(len(k))])
        ref = _ext(U.conj().T, _ext(T, V)) / s.astype(np.longdouble)
        fs = np.array([[np.sum(np.abs(np.unique(T[np.ix_(line == a, line == b)]))) for b in range(nl)] for a in range(nl)])
        bound = 4 * np.sqrt(P) * ROUND * (norms(U).T @ fs @ norms(V)) / s
        err = np.abs(got[l] - ref).astype(float)
        print(f"  largest error / bound {np.max(err / bound):.2f}", flush=True)
        assert np.all(err <= bound)


@pytest.mark.parametrize("d,n,m", [(1, 300, 4), (2, 15, 5), (2, 24, 9), (3, 7, 10)])
@pytest.mark.parametrize("modulus", [1.0, 0.75])
def test_direct_results_hold_a_bound_by_their_own_terms(d, n, m, modulus):
    rng, f, U, s, V = _problem(d, n, m, modulus)
    print(f"direct d={d} n={n} m={m} modulus={modulus}", flush=True)
    k, N, L = _box(d, 0, n + 1), (n + 1) ** d, 2 * n + 2
    limit = 4 * np.sqrt(N) * ROUND
    block = lambda e: np.stack([f[np.ravel_multi_index(tuple((k[i] - k + e + n).T), (L,) * d)] for i in range(N)])  # noqa: E731
    X = rng.standard_normal((N, 3)) + 1j * rng.standard_normal((N, 3))
    T = block(0)
    for A, adjoint in ((T, False), (T.conj().T, True)):
        got = api.toeplitz_mm(_dev(f), d, n, _dev(X), adjoint=adjoint, prec="fp64_direct").cpu().numpy()
        ratio = np.max(np.abs(got - _ext(A, X)).astype(float) / (np.abs(A) @ np.abs(X)))
        print(f"  product {ratio:.1e}", flush=True)
        assert ratio <= limit
    S = api.build_S(_dev(f), d, n, _dev(U), _dev(s), _dev(V), prec="fp64_direct").cpu().numpy()
    for l in range(d):
        T = block(np.arange(d) == l)
        ref = _ext(U.conj().T, _ext(T, V)) / s.astype(np.longdouble)
        ratio = np.max(np.abs(S[l] - ref).astype(float) / (np.abs(U).T @ (np.abs(T) @ np.abs(V)) / s))
        print(f"  S_{l + 1} {ratio:.1e}", flush=True)
        assert ratio <= limit
    gS = rng.standard_normal((d, m, m)) + 1j * rng.standard_normal((d, m, m))
    got = api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64_direct").cpu().numpy()
    ref, terms = np.zeros(L ** d, dtype=np.clongdouble), np.zeros(L ** d)
    for l in range(d):
        Z = _ext(U, gS[l]) / s.astype(np.longdouble)
        A = np.abs(U) @ np.abs(gS[l]) / s
        for h in range(N):
            at = np.ravel_multi_index(tuple((k - k[h] + (np.arange(d) == l) + n).T), (L,) * d)
            ref[at] += np.dot(Z, np.conj(V[h].astype(np.clongdouble)))
            terms[at] += A @ np.abs(V[h])
    held = terms > 0
    ratio = np.max(np.abs(got - ref).astype(float)[held] / terms[held])
    print(f"  gradient {ratio:.1e}", flush=True)
    assert ratio <= limit
