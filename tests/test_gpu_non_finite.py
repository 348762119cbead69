"""GPU checks of float32 cells that are not finite: every output whose filter reads
such a cell is not finite; the split precisions may spoil outputs up to 7 columns and
one row beyond, never a further plane; all others hold the bits that they hold with
a zero in the cell's place.  FP32 and the rank-1 passes spoil nothing beyond."""
import numpy as np
import pytest

from _gpu import run_filter

pytestmark = pytest.mark.gpu
BEYOND_X, BEYOND_Y = 7, 1


@pytest.fixture(autouse=True)
def _reset():
    from paper_2203_10213_amd import vkt
    rp = vkt.vktGetRowPairMinCells()
    yield
    vkt.vktSetRowPairMinCells(rp)
    vkt.vktSetSeparable(False)
    vkt.vktSetPrecision("auto")


def _check(shape, k, precision, cell, value, beyond):
    Z, Y, X = shape
    x, y, z = cell
    r = k // 2
    g = np.random.default_rng(k + x)
    src = g.standard_normal(shape).astype(np.float32)
    w = (np.abs(g.standard_normal((k, k, k))) + 0.1).astype(np.float32)
    src[z, y, x] = 0
    want = run_filter(src, w, "clamp", precision=precision)
    src[z, y, x] = value
    got = run_filter(src, w, "clamp", precision=precision)
    assert np.isfinite(want).all()
    dz, dy, dx = (np.abs(np.arange(n) - c) for n, c in ((Z, z), (Y, y), (X, x)))

    def box(bx, by):
        return ((dz <= r)[:, None, None] & (dy <= r + by)[None, :, None]
                & (dx <= r + bx)[None, None, :])

    assert not np.isfinite(got[box(0, 0)]).any()
    assert np.isfinite(got[~box(*beyond)]).all()
    ok = np.isfinite(got)
    assert np.array_equal(got[ok].view(np.uint32), want[ok].view(np.uint32))


# one row block of 16x16 tiles, two of them (k = 5, 7), 32x32 tiles (k >= 9), and the
# row-pair kernel (k = 5, and 7 with three products)
@pytest.mark.parametrize("value", [np.inf, np.nan])
@pytest.mark.parametrize("precision", ["auto", "splitbf16"])
@pytest.mark.parametrize("k,shape,pairs", [
    (5, (9, 40, 100), False), (7, (9, 40, 100), False), (5, (40, 200, 200), False),
    (7, (40, 200, 200), False), (5, (30, 150, 200), True), (7, (30, 150, 200), True),
    (9, (20, 70, 130), False), (11, (20, 70, 130), False), (13, (16, 40, 90), False),
    (15, (16, 40, 90), False)])
def test_split_precisions(k, shape, pairs, precision, value):
    from paper_2203_10213_amd import vkt
    if pairs:
        vkt.vktSetRowPairMinCells(0)
    Z, Y, X = shape
    # every place of a strip of two or three columns, and at the faces
    cells = [(X // 2 + i, Y // 2 + i % 2, Z // 2) for i in range(6)]
    cells += [(0, 0, 0), (X - 1, Y - 1, Z - 1), (X - 2, 1, Z - 1), (1, Y - 2, 0)]
    for cell in cells:
        _check(shape, k, precision, cell, np.float32(value), (BEYOND_X, BEYOND_Y))


@pytest.mark.parametrize("k,rank1", [(3, False), (5, False), (9, False), (5, True)])
def test_fp32_and_passes_spoil_nothing_beyond(k, rank1):
    from paper_2203_10213_amd import vkt
    for shape in ((9, 40, 100), (20, 120, 260)):
        Z, Y, X = shape
        for cell in ((X // 2, Y // 2, Z // 2), (0, 0, 0), (X - 1, Y - 1, Z - 1)):
            if not rank1:
                _check(shape, k, "fp32", cell, np.float32(np.inf), (0, 0))
                continue
            vkt.vktSetSeparable(True)
            g = np.random.default_rng(k)
            u = g.uniform(0.1, 1, k).astype(np.float32)
            w = (u[:, None, None] * u[None, :, None] * u[None, None, :]).astype(np.float32)
            src = g.standard_normal(shape).astype(np.float32)
            src[cell[2], cell[1], cell[0]] = np.inf
            got = run_filter(src, w, "clamp")
            r = k // 2
            d = [np.abs(np.arange(n) - c) <= r for n, c in zip(shape, cell[::-1])]
            reach = d[0][:, None, None] & d[1][None, :, None] & d[2][None, None, :]
            assert np.array_equal(~np.isfinite(got), reach)
