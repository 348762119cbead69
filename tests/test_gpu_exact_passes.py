"""Integer rank-1 filters on integer cells run as three exact passes: the result
is the dense integer sum's, bit for bit, at the edges of the rule (16-bit packed
sums, FP32 sums, 24-bit multiply-adds, dense) and of the tiles, for signed
factors, factors with zeros and volumes at their largest values."""
import numpy as np
import pytest

from _gpu import check_against_oracle, run_filter

pytestmark = pytest.mark.gpu


def _outer(u, v, t):
    return np.einsum("c,b,a->cba", t, v, u).astype(np.int32)


def _binomial(k):
    r = np.array([1], np.int64)
    for _ in range(k - 1):
        r = np.convolve(r, [1, 1])
    return r


def _filters(k):
    """(weights, divisor): box, binomial, one axis only, a signed derivative,
    unequal factors with zeros; weights of an 8-bit product and beyond."""
    one = np.ones(k, np.int64)
    at = np.zeros(k, np.int64)
    at[k // 2] = 1
    d = np.arange(k) - k // 2
    out = [(_outer(one, one, one), k ** 3), (_outer(one, at, at), k), (_outer(at, at, 2 * one), 3),
           (_outer(d, one, at), 2 * k), (_outer(at + d, one, 1 - at), 5)]
    if k <= 7:
        b = _binomial(k)
        out.append((_outer(b, b, at), int(b.sum()) ** 2))
        out.append((_outer(b, at, b), 7))
    return out


@pytest.mark.parametrize("mode", ["clamp", "wrap", "mirror", "border"])
@pytest.mark.parametrize("k", [3, 5, 7, 9, 11, 13, 15])
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
def test_exact(orc, dtype, k, mode):
    g = np.random.default_rng(1000 + k)
    mx = np.iinfo(dtype).max
    for i, (w, D) in enumerate(_filters(k)):
        shape = [(5, 18, 260), (9, 17, 61), (3, 33, 64), (20, 5, 7), (4, 6, 4)][i % 5]
        src = g.integers(0, mx + 1, shape).astype(dtype)
        src[:, : shape[1] // 2] = mx  # the largest sums
        out = run_filter(src, w, mode, divisor=D)
        check_against_oracle(orc, src, w, mode, out, divisor=D, what=f"{shape} k={k} filter {i}")


def test_exact_range_and_large(orc):
    """A range with unaligned columns, and uint8 3^3 above the direct kernel's
    size on rows of 4 n + 1 cells."""
    g = np.random.default_rng(5)
    src = g.integers(0, 256, (30, 130, 141)).astype(np.uint8)
    w, D = np.ones((3, 3, 3), np.int32), 27
    out = run_filter(src, w, "mirror", divisor=D)
    check_against_oracle(orc, src, w, "mirror", out, divisor=D)
    for dtype, k, roi in ((np.uint8, 5, ((4, 3, 1), (52, 40, 9))), (np.uint8, 5, ((3, 3, 1), (50, 40, 9))),
                          (np.uint16, 7, ((3, 1, 0), (61, 39, 8)))):
        src = g.integers(0, np.iinfo(dtype).max + 1, (10, 44, 64)).astype(dtype)
        w = np.ones((k, k, k), np.int32)
        out = run_filter(src, w, "wrap", divisor=k ** 3, roi=roi)
        check_against_oracle(orc, src, w, "wrap", out, divisor=k ** 3, roi=roi)
