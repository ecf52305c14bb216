"""Sectors of very small and very large values, where the squares of a row leave
float64's range: the values scale with the matrix, and both factors stay
orthonormal.  Every sector is a power of two times the same matrix, so that the
values are those of the unscaled sector times it, bit for bit."""
import numpy as np
import pytest

from tests.gpu_common import require_gpu
from tests.test_gpu_svd_graded import _factors, _tensor

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


SHAPES = [(14, 9), (40, 40), (33, 60), (130, 100), (150, 160)]


def _off(a):
    return float(np.max(np.abs(a - np.eye(len(a)))))


@pytest.mark.parametrize("shape", SHAPES)
def test_powers_of_two(shape):
    """Of 1e-161 to 1e-120 and 1e120 to 1e150: singular values exact multiples of
    the unscaled ones, |U^T U - 1| and |V V^T - 1| at most 50 max(m, n) eps (a
    column takes some 8 r rotations and r reflections of a few eps each, random
    in sign)."""
    x = np.random.default_rng(sum(shape)).standard_normal(shape)
    powers = [0, -535, -532, -528, -524, -519, -480, -400, 400, 480, 498]
    print("powers of two", shape, flush=True)
    base, *rest = _factors(_tensor([np.ldexp(x, e) for e in powers]))
    for e, (U, S, V) in zip([0] + powers[1:], [base] + rest):
        print(shape, e, "off", _off(U.T @ U), _off(V @ V.T), flush=True)
        assert np.array_equal(S, np.ldexp(base[1], e)), e
        assert max(_off(U.T @ U), _off(V @ V.T)) <= 50 * max(shape) * np.finfo(float).eps, e


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("tiny", [1e-156, 1e-158, 1e-160, 1e-161, 1e-170])
def test_tiny_rows_beside_large_ones(shape, tiny):
    """Half of the rows (of the longer side) are tiny: their reflections
    keep the factor that they go into orthonormal, and the large values are those
    of the other rows."""
    m, n = shape if shape[0] >= shape[1] else shape[::-1]
    x = np.random.default_rng(7).standard_normal((m, n))
    h = n // 2
    x[h:] *= tiny
    if shape[0] < shape[1]:
        x = x.T
    print("tiny rows", shape, tiny, flush=True)
    (U, S, V), = _factors(_tensor([x]))
    W = V.T if shape[0] >= shape[1] else U   # the factor of the shorter side
    print(shape, tiny, "off", _off(W.T @ W), flush=True)
    assert _off(W.T @ W) <= 50 * m * np.finfo(float).eps
    want = np.linalg.svd(x, compute_uv=False)[:h]
    assert np.max(np.abs(S[:h] - want)) <= 50 * m * np.finfo(float).eps * want[0]


def test_zero_and_infinite_sectors():
    """No scale exists for these: zero stays zero, and an infinity ends in NaN
    values of its own sector only."""
    rng = np.random.default_rng(1)
    a, b = np.ldexp(rng.standard_normal((30, 20)), -530), rng.standard_normal((25, 25))
    bad = rng.standard_normal((40, 30))
    bad[3, 4] = np.inf
    (_, s0, _), (_, s1, _), (_, s2, _), (_, s3, _) = _factors(_tensor([np.zeros((20, 12)), a, bad, b]))
    assert not s0.any() and not np.isfinite(s2).all()
    for x, s in ((a, s1), (b, s3)):
        e = 530 if x is a else 0
        want = np.linalg.svd(np.ldexp(x, e), compute_uv=False)
        assert np.max(np.abs(np.ldexp(s, e) - want)) <= 50 * max(x.shape) * np.finfo(float).eps * want[0]
