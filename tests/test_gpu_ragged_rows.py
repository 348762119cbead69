"""Resample and Flip where their vector forms can go wrong: rows around one
16-byte chunk (the last chunk moved back, rows that go by cells, in-place
middles), four-cell groups at the row's end, sources of 1 to 3 cells, uint8
sources around twice the destination (one 8-cell load or pairs), planes of
under 8 cells, and marches that skip, repeat or revisit source planes.
Tolerances as for the other resample and flip tests: exact halving and flips
bit for bit, interpolation within 2^-18 of the largest neighbour or its
rounding."""
import numpy as np
import pytest

from test_gpu_resample_flip import (DTYPES, _check_resample, _gpu_flip, _gpu_resample, _vol)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", DTYPES)
def test_resample_ragged(orc, dtype):
    g = np.random.default_rng(60 + DTYPES.index(dtype))
    for src_shape, dst_shape in [
            ((3, 4, 1), (4, 5, 6)), ((3, 4, 2), (4, 5, 7)), ((2, 3, 3), (5, 7, 9)),
            ((2, 2, 3), (3, 5, 4)), ((1, 3, 2), (2, 9, 1)), ((1, 1, 8), (1, 2, 4)),
            ((5, 9, 40), (4, 7, 20)), ((5, 9, 41), (4, 7, 20)), ((5, 9, 39), (4, 7, 20)),
            ((40, 3, 9), (97, 4, 7)), ((97, 3, 9), (40, 4, 7)), ((5, 3, 9), (70, 2, 11)),
            ((70, 3, 9), (5, 2, 11)), ((6, 5, 200), (5, 6, 255)), ((6, 5, 200), (7, 6, 257)),
            ((33, 1, 5), (33, 1, 4))]:
        src = _vol(g, src_shape, dtype)
        got = _gpu_resample(src, dst_shape)
        _check_resample(orc, src, got, f"{dtype.__name__} {src_shape}->{dst_shape}")


@pytest.mark.parametrize("dtype", DTYPES)
def test_halve_ragged(orc, dtype):
    g = np.random.default_rng(70 + DTYPES.index(dtype))
    for Xo in (1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33):
        src = _vol(g, (6, 10, 2 * Xo), dtype)
        got = _gpu_resample(src, (3, 5, Xo))
        _check_resample(orc, src, got, f"halve {dtype.__name__} {Xo}", exact_half=True)


@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("dtype", DTYPES)
def test_flip_ragged(dtype, inplace):
    g = np.random.default_rng(80 + DTYPES.index(dtype))
    for X in (1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 63, 64, 65):
        src = _vol(g, (5, 6 if X % 2 else 7, X), dtype)
        for axis in (0, 1, 2):
            got = _gpu_flip(src, axis, inplace=inplace)
            assert np.array_equal(got, np.flip(src, 2 - axis)), (X, axis)
