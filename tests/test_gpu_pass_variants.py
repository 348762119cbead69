"""uint8 rank-1 integer filters in passes on the 8-bit dot products: every variant of
the kernel (v and t all 1, 1 at their ends, any; k = 3, 5, 7; unsigned and signed
weights) against the oracle, bit for bit: rows of one and of two tiles, one to many
planes, cells at their largest value, ranges."""
import numpy as np
import pytest

from _gpu import check_against_oracle, run_filter

pytestmark = pytest.mark.gpu

ENDS = {3: [1, 2, 1], 5: [1, 3, 2, 0, 1], 7: [1, 2, 0, 1, 3, 1, 1]}
ANY = {3: [2, 3, 1], 5: [2, 1, 0, 3, 2], 7: [2, 1, 1, 0, 1, 2, 3]}
SIGNED = {3: [-1, 0, 1], 5: [-1, -2, 0, 2, 1], 7: [-3, -2, -1, 0, 1, 2, 3]}


def _factors(k, kind):
    one, at = np.ones(k, int), (np.arange(k) == k // 2).astype(int)
    small = {3: ANY[3], 5: ENDS[5], 7: (np.arange(7) % 2)}[k]  # sums of at most 2048
    return {"ones": (3 * one if k == 3 else one, one, one),
            "ends": (small, ENDS[k], ENDS[k]),
            "any": (small, ANY[k], ANY[k]),
            "any y, ends z": (one, ANY[k], ENDS[k]),
            "one plane": (ANY[k], ENDS[k], 5 * at)}[kind]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("kind", ["ones", "ends", "any", "any y, ends z", "one plane"])
@pytest.mark.parametrize("k", [3, 5, 7])
def test_variant(orc, k, kind, signed):
    u, v, t = (np.asarray(f, np.int64) for f in _factors(k, kind))
    if signed:
        u = np.asarray(SIGNED[k], np.int64)
    w = (t[:, None, None] * v[None, :, None] * u[None, None, :]).astype(np.int32)
    assert np.abs(w).sum() <= 2048 and w.max() <= 127
    D = int(max(1, np.abs(w).sum() // (3 if signed else 1)))
    g = np.random.default_rng(10 * k + signed)
    for shape, mode, roi in (((1, 17, 64), "clamp", None), ((37, 19, 260), "mirror", None),
                             ((70, 5, 4), "wrap", None), ((9, 40, 516), "border", None),
                             ((23, 33, 128), "clamp", ((4, 3, 2), (120, 30, 22)))):
        src = g.integers(0, 256, shape).astype(np.uint8)
        src[:, : shape[1] // 2] = 255
        out = run_filter(src, w, mode, divisor=D, roi=roi)
        check_against_oracle(orc, src, w, mode, out, divisor=D, roi=roi,
                             what=f"{kind} k={k} {shape} {mode}")
