"""The FP64 root of the fluxes against numpy's, which is correctly rounded.  Its error is 1/2 ulp and at most 2^-40 of one
(one Goldschmidt iteration and one residual correction, whose own error is 2^-94 of the root): 2^24 arguments at random
have to be equal, roots next to the middle of two numbers may round to either."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


def root(x):
    return dk.root_f64(torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).cuda()).cpu().numpy()


@pytest.mark.parametrize("lo,hi", [(-4, 4), (-960, 1024)])
def test_random_arguments(lo, hi):
    rng = np.random.default_rng(hi)
    for _ in range(4):
        x = np.ldexp(rng.uniform(0.5, 1.0, 1 << 22), rng.integers(lo + 1, hi + 1, 1 << 22))
        assert np.array_equal(root(x), np.sqrt(x))


def test_squares_and_midpoints():
    rng = np.random.default_rng(1)
    m = rng.integers(1 << 25, 1 << 26, 1 << 16).astype(np.float64)
    assert np.array_equal(root(m * m), m)                       # exact squares
    for x in (np.nextafter(m * m, 0), np.nextafter(m * m, np.inf)):
        assert np.array_equal(root(x), np.sqrt(x))              # 2^-53 of the root away from it
    # arguments whose root lies next to the middle of two numbers
    r = rng.integers(1 << 52, 1 << 53, 1 << 16)
    x = np.array([float(int(k) * int(k) + int(k)) for k in r])
    got, want = root(x), np.sqrt(x)
    assert np.all((got == want) | (got == np.nextafter(want, 0)) | (got == np.nextafter(want, np.inf)))


def test_ends_of_the_range():
    big, tiny = np.finfo(np.float64).max, np.finfo(np.float64).tiny
    x = np.array([0.0, -0.0, -1.0, -big, -np.inf, np.nan, np.inf, big])
    assert np.array_equal(root(x), np.array([0, 0, 0, 0, 0, 0, np.inf, np.sqrt(big)]))
    assert np.all(root(np.array([5e-324, tiny, 2.0 ** -1000])) <= 2.0 ** -500)
