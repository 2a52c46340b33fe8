"""The smallest FP64 gradients (d >= 2, summed line by line) at the ends of their range:
lines of 2 to 15 points, one to eight K steps, fewer pairs of lines than waves and more; and
the line-spectral form at the same shapes, which batches take."""
import numpy as np
import pytest
import torch

from oracle import prony_oracle as O
from paper_2012_11430_amd import api
from tests._close import assert_close
from tests.test_gpu_nonfinite import test_gradients_with_one_entry_not_finite as one_entry_not_finite

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")
# tolerance: the suite's FP64 bound, on sums of at most d m (n+1)^d terms of one size
SHAPES = [(2, 1, 1), (2, 1, 4), (2, 2, 9), (2, 5, 5), (2, 6, 17), (2, 7, 8), (2, 13, 30), (2, 14, 16), (2, 14, 32), (2, 15, 3),
          (3, 1, 1), (3, 1, 8), (3, 2, 16), (3, 3, 20), (3, 3, 21), (3, 4, 12), (3, 5, 8), (3, 9, 4), (3, 10, 2)]


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _inputs(d, n, m):
    rng = np.random.Generator(np.random.PCG64(6100 + 100 * d + 10 * n + m))
    cn = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)   # noqa: E731
    return cn((n + 1) ** d, m), rng.uniform(0.5, 2.0, m), cn((n + 1) ** d, m), cn(d, m, m)


@pytest.mark.parametrize("d,n,m", SHAPES)
def test_ends_of_the_range(d, n, m):
    U, s, V, gS = _inputs(d, n, m)
    print(f"gradient d={d} n={n} m={m}", flush=True)
    ref = O.pencil_adjoint(gS, d, n, U, s, V)
    got = api.build_S_adjoint(_dev(gS), d, n, _dev(U), _dev(s), _dev(V), prec="fp64")
    assert_close(got.cpu().numpy(), ref, 1e-12, "gradient")
    assert np.all(got.cpu().numpy()[ref == 0] == 0)            # points that no T_l holds
    again = api.build_S_adjoint(_dev(gS), d, n, _dev(U.T).T, _dev(s), _dev(V.T).T, prec="fp64")
    assert torch.equal(got, again)                             # a fixed order, whatever the strides


def test_the_same_shapes_in_a_batch():
    cases = [(d, n, *_inputs(d, n, m)) for d, n, m in SHAPES]
    batch = api.Batch([(d, n, _dev(np.zeros((2 * n + 2) ** d, dtype=complex)), _dev(U), _dev(s), _dev(V))
                       for d, n, U, s, V, gS in cases], prec="fp64")
    got = batch.adjoint(torch.cat([_dev(c[-1]).reshape(-1) for c in cases]))
    for (d, n, U, s, V, gS), x in zip(cases, torch.split(got, batch.gf_sizes)):
        assert_close(x.cpu().numpy(), O.pencil_adjoint(gS, d, n, U, s, V), 1e-12, f"d={d} n={n} m={U.shape[1]}")
    batch.close()


@pytest.mark.parametrize("d,n,m", [(2, 1, 4), (2, 9, 5), (2, 14, 32), (3, 1, 8), (3, 3, 7)])
@pytest.mark.parametrize("where", ["U", "V", "gS"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_entries_not_finite_stay_with_their_points(d, n, m, where, bad):
    one_entry_not_finite(d, n, m, where, bad)
