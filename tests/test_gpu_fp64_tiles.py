"""The FP64 tile kernels, which serve what the line-spectral form does not: direct FP64, lines
of more than 240 points, captures that find only the tiles' workspace, batches with an instance
past the form. They reach every column-block form (pair and three-product blocks, one to four
fragments, tuned splits), products of one to 64 columns and gradients with d >= 2; each test checks through the profiling names that the tiles are what ran. References: padded
FFTs. Tolerance: the suite's FP64 bound 1e-12 normwise and entrywise, on data of even size
(sums of N = 58081 terms: 2^-53 sqrt(N) = 3e-14)."""
import ctypes
import functools

import numpy as np
import pytest
import torch

from oracle import prony_oracle as O
from paper_2012_11430_amd import _lib, api, autotune
from tests._close import assert_close, assert_close_per_matrix
from tests.test_gpu_nonfinite import _fft_gradient
from tests.test_gpu_spectral import _fft_pencil, _fft_product

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
TOL = 1e-12


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


@functools.lru_cache(maxsize=2)
def _problem(d, n, m, seed=0):
    rng = np.random.Generator(np.random.PCG64(1200 + 100 * d + n + m + seed))
    N, G = (n + 1) ** d, (2 * n + 2) ** d
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)   # noqa: E731
    return cn(G), cn(N, m), rng.uniform(0.5, 2.0, m), cn(N, m), cn(d, m, m)


def _ran(kernel, fn):
    """fn()'s result; asserts that it launched `kernel`."""
    api.profile_enable(DEV, kernel)
    try:
        out = fn()
        launches, _ = api.profile_read(DEV)
    finally:
        api.profile_enable(DEV, None)
    assert launches >= 1, f"{kernel} did not run"
    return out


@pytest.mark.parametrize("d,n,m", [(2, 240, 8), (2, 240, 9), (2, 240, 16), (2, 240, 17), (2, 240, 24), (2, 240, 25), (2, 240, 32),
                                   (1, 57600, 7), (1, 57600, 20), (1, 57600, 31)])
def test_builds_past_the_form_under_tuned_plans(d, n, m):
    f, U, s, V, _ = _problem(d, n, m)
    ref = _fft_pencil(f, d, n, U, s, V)
    args = (_dev(f), d, n, _dev(U), _dev(s), _dev(V))
    cus = torch.cuda.get_device_properties(DEV).multi_processor_count
    seen = set()
    try:
        for frag in (0, 1, 2, 4):
            for target in (0, cus, 8 * cus):
                autotune.register(DEV, d, n, m, "fp64", False, target, frag)
                p = autotune.plan(DEV, d, n, m, "fp64", with_s0=True)
                if (p["fragments"], p["workgroups"]) in seen:
                    continue
                seen.add((p["fragments"], p["workgroups"]))
                what = f"d={d} n={n} m={m} fragments {p['fragments']} workgroups {p['workgroups']}"
                print(what, flush=True)
                got = _ran("pencil_tiles", lambda: api.build_S(*args, with_s0=True))
                assert_close_per_matrix(got.cpu().numpy(), ref, TOL, what)
    finally:
        autotune.register(DEV, d, n, m, "fp64", False, 0, 0)
    assert len(seen) >= 2


@pytest.mark.parametrize("d,n,r", [(2, 240, 1), (2, 240, 2), (2, 240, 8), (2, 240, 9), (2, 240, 16), (2, 240, 33), (2, 240, 64),
                                   (1, 57600, 1), (1, 57600, 40)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_products_past_the_form(d, n, r, adjoint):
    f, X, *_ = _problem(d, n, r)
    print(f"product d={d} n={n} r={r} adjoint={adjoint}", flush=True)
    got = _ran("toeplitz_mv" if r == 1 else "toeplitz_mm_tiles",
               lambda: api.toeplitz_mm(_dev(f), d, n, _dev(X), adjoint=adjoint))
    assert_close(got.cpu().numpy(), _fft_product(f, d, n, X, adjoint), TOL, "product")


@pytest.mark.parametrize("d,n,m", [(2, 240, 5), (2, 240, 9), (2, 240, 17), (2, 240, 32)])
def test_gradients_past_the_form(d, n, m):
    _, U, s, V, gS = _problem(d, n, m)
    print(f"gradient d={d} n={n} m={m}", flush=True)
    got = _ran("adjoint_tiles", lambda: api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64"))
    assert_close(got.cpu().numpy(), _fft_gradient(gS, d, n, U, s, V), TOL, "gradient")


@pytest.mark.parametrize("chunks,fragments", [(0, 0), (2, 1), (4, 2)])
def test_batches_with_an_instance_past_the_form(chunks, fragments):
    shapes = [(2, 240, 2), (1, 200, 32), (2, 20, 9), (2, 33, 17), (3, 6, 31), (3, 8, 16), (2, 12, 4), (1, 63, 24)]
    probs = [_problem.__wrapped__(d, n, m, 7) for d, n, m in shapes]
    try:
        for d, n, m in shapes:
            autotune.register(DEV, d, n, m, "fp64", True, chunks, fragments)
        batch = api.Batch([(d, n, _dev(f), _dev(U), _dev(s), _dev(V)) for (d, n, m), (f, U, s, V, _) in zip(shapes, probs)],
                          prec="fp64")
        print(f"batch chunks {chunks} fragments {fragments}", flush=True)
        _ran("pencil_tiles_batched", batch.run)
        for S, (d, n, m), (f, U, s, V, _) in zip(batch.S, shapes, probs):
            assert_close_per_matrix(S.cpu().numpy(), _fft_pencil(f, d, n, U, s, V)[1:], TOL, f"d={d} n={n} m={m}")
        gf = _ran("adjoint_tiles_batched", lambda: batch.adjoint(_dev(np.concatenate([p[4].reshape(-1) for p in probs]))))
        for x, (d, n, m), (f, U, s, V, gS) in zip(torch.split(gf, batch.gf_sizes), shapes, probs):
            assert_close(x.cpu().numpy(), _fft_gradient(gS, d, n, U, s, V), TOL, f"gradient d={d} n={n} m={m}")
        batch.close()
    finally:
        for d, n, m in shapes:
            autotune.register(DEV, d, n, m, "fp64", True, 0, 0)


@pytest.mark.parametrize("d,n,m", [(3, 9, 9), (3, 12, 20), (3, 12, 32), (2, 31, 30)])
@pytest.mark.parametrize("fragments", [1, 2, 4])
def test_captures_that_find_only_the_tiles_workspace(d, n, m, fragments):
    """A handle whose workspace holds the tile plan (few partial rows: target 64) and not the
    line-spectral one captures the tiles; replays give the tiles' result."""
    lib = _lib.load()
    f, U, s, V, _ = _problem(d, n, m)
    fd, Ud, sd, Vd = _dev(f), _dev(U), _dev(s), _dev(V)
    z = _dev(np.exp(2j * np.pi * np.random.Generator(np.random.PCG64(1)).random((64, d))))
    gram = torch.empty(64 * 65, dtype=torch.complex128, device=DEV)
    out = torch.empty((d, m, m), dtype=torch.complex128, device=DEV)
    ref = O.pencil_matrices(f, d, n, U, s, V)
    ptr = lambda t: t.data_ptr()       # noqa: E731
    for columns in range(8, 65):       # one prony_coeffs call sizes a fresh handle's workspace
        bytes_ = 256 * columns * (columns + 1) * 16
        held = -(-(bytes_ + bytes_ // 4) // (1 << 20)) << 20
        h = ctypes.c_void_p()
        assert lib.prony_create(ctypes.byref(h), DEV.index or 0) == _lib.PRONY_OK
        try:
            assert lib.prony_tune_set_tile(h, d, n, m, _lib.PRONY_FP64, 0, fragments, 64) == _lib.PRONY_OK
            need = ctypes.c_size_t()
            assert lib.prony_build_S_plan(h, d, n, m, _lib.PRONY_FP64, 0, None, None, None, ctypes.byref(need)) == 0
            assert held < need.value, "no workspace size between the two forms"
            stream = torch.cuda.Stream(DEV)
            assert lib.prony_set_stream(h, stream.cuda_stream) == _lib.PRONY_OK
            assert lib.prony_coeffs(h, d, n, columns, ptr(z), ptr(fd), ptr(gram), ptr(gram), None) == _lib.PRONY_OK
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.stream(stream):
                with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
                    st = lib.prony_build_S(h, d, n, m, ptr(fd), ptr(Ud), m, 1, ptr(sd), ptr(Vd), m, 1, _lib.PRONY_FP64, 0,
                                           ptr(out))
            if st == _lib.PRONY_ECAPTURE:
                torch.cuda.synchronize()
                continue
            assert st == _lib.PRONY_OK
            print(f"captured d={d} n={n} m={m} fragments={fragments}: {held} of {need.value} bytes", flush=True)
            first = None
            for rep in range(3):
                out.zero_()
                g.replay()
                torch.cuda.synchronize()
                assert_close_per_matrix(out.cpu().numpy(), ref, TOL, f"replay {rep}")
                first = out.clone() if first is None else first
                assert torch.equal(out, first)
                (torch.randn(4096, device=DEV) * 3).sum().item()
            return
        finally:
            torch.cuda.synchronize()
            assert lib.prony_destroy(h) == _lib.PRONY_OK
    raise AssertionError("no capture succeeded")


# ---- direct FP64 ------------------------------------------------------------------------


def _direct_under_tuned_plans(d, n, m, f, U, s, V, with_s0=False, fragments=(0, 1, 2, 4), targets=(0, 1, 2, 3, 4, 8)):
    ref = _fft_pencil(f, d, n, U, s, V)[0 if with_s0 else 1:]
    args = (_dev(f), d, n, _dev(U), _dev(s), _dev(V))
    cus = torch.cuda.get_device_properties(DEV).multi_processor_count
    seen = set()
    try:
        for frag in fragments:
            for target in targets:
                autotune.register(DEV, d, n, m, "fp64", False, target * cus, frag)
                p = autotune.plan(DEV, d, n, m, "fp64", with_s0=with_s0)
                if (p["fragments"], p["workgroups"]) in seen:
                    continue
                seen.add((p["fragments"], p["workgroups"]))
                what = f"direct d={d} n={n} m={m} fragments {p['fragments']} workgroups {p['workgroups']}"
                print(what, flush=True)
                got = _ran("pencil_tiles", lambda: api.build_S(*args, prec="fp64_direct", with_s0=with_s0))
                assert_close_per_matrix(got.cpu().numpy(), ref, TOL, what)
    finally:
        autotune.register(DEV, d, n, m, "fp64", False, 0, 0)
    return args, got


@pytest.mark.parametrize("d,n,m", [(2, 63, 20), (3, 19, 30), (3, 20, 5), (3, 20, 20)])
def test_direct_builds_under_every_tuner_target(d, n, m):
    f, U, s, V, _ = _problem(d, n, m)
    _direct_under_tuned_plans(d, n, m, f, U, s, V)


@pytest.mark.parametrize("d,n,m", [(1, 1, 1), (1, 3, 4), (1, 63, 5), (1, 200, 32), (2, 1, 2), (2, 1, 4), (2, 4, 16), (2, 9, 17),
                                   (2, 20, 16), (2, 20, 32), (3, 1, 3), (3, 1, 8), (3, 3, 8), (3, 6, 31)])
def test_direct_builds_ragged_and_the_same_in_every_entry_point(d, n, m):
    f, U, s, V, _ = _problem(d, n, m)
    args, last = _direct_under_tuned_plans(d, n, m, f, U, s, V, with_s0=True, targets=(0, 2))
    out = torch.empty_like(last)
    one = api.build_S(*args, prec="fp64_direct", with_s0=True)
    assert torch.equal(api.build_S_noalloc(*args, out=out, prec="fp64_direct", with_s0=True), one)
    factors = api.Factors(d, n, *args[3:], prec="fp64_direct", with_s0=True)
    assert torch.equal(factors.build_S(args[0]), one)
    factors.close()


@pytest.mark.parametrize("d,n,r", [(1, 40, 1), (1, 300, 9), (2, 9, 1), (2, 9, 8), (2, 20, 17), (2, 35, 64), (2, 63, 40), (3, 6, 1),
                                   (3, 9, 16), (3, 12, 33), (3, 20, 1), (3, 20, 2)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_direct_products(d, n, r, adjoint):
    f, X, *_ = _problem(d, n, r)
    print(f"direct product d={d} n={n} r={r} adjoint={adjoint}", flush=True)
    got = _ran("toeplitz_mv" if r == 1 else "toeplitz_mm_tiles",
               lambda: api.toeplitz_mm(_dev(f), d, n, _dev(X), adjoint=adjoint, prec="fp64_direct"))
    assert_close(got.cpu().numpy(), _fft_product(f, d, n, X, adjoint), TOL, "product")


@pytest.mark.parametrize("d,n,m", [(1, 70, 9), (2, 1, 1), (2, 3, 5), (2, 12, 32), (2, 47, 16), (3, 2, 4), (3, 6, 20), (3, 12, 11)])
def test_direct_gradients(d, n, m):
    _, U, s, V, gS = _problem(d, n, m)
    print(f"direct gradient d={d} n={n} m={m}", flush=True)
    got = _ran("adjoint_tiles",
               lambda: api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64_direct"))
    assert_close(got.cpu().numpy(), _fft_gradient(gS, d, n, U, s, V), TOL, "gradient")


def test_direct_batches():
    shapes = [(2, 47, 16), (1, 70, 9), (2, 3, 5), (2, 12, 32), (3, 2, 4), (3, 6, 20), (1, 300, 32)]
    probs = [_problem.__wrapped__(d, n, m, 9) for d, n, m in shapes]
    batch = api.Batch([(d, n, _dev(f), _dev(U), _dev(s), _dev(V)) for (d, n, m), (f, U, s, V, _) in zip(shapes, probs)],
                      prec="fp64_direct")
    print("direct batch", flush=True)
    _ran("pencil_tiles_batched", batch.run)
    gf = _ran("adjoint_tiles_batched", lambda: batch.adjoint(_dev(np.concatenate([p[4].reshape(-1) for p in probs]))))
    for S, x, (d, n, m), (f, U, s, V, gS) in zip(batch.S, torch.split(gf, batch.gf_sizes), shapes, probs):
        assert_close_per_matrix(S.cpu().numpy(), _fft_pencil(f, d, n, U, s, V)[1:], TOL, f"d={d} n={n} m={m}")
        assert_close(x.cpu().numpy(), _fft_gradient(gS, d, n, U, s, V), TOL, f"gradient d={d} n={n} m={m}")
    batch.close()
