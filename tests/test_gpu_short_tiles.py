"""GPU check of the line between the 16x16 matrix-core kernel's two tiles: a range
too small for two workgroups per CU runs on the short tile, the whole volume on
the tall one.  A cell's sum has the same terms in the same order on both, so the
range equals the whole volume's cells bit for bit; and the range is checked
against the oracle."""
import numpy as np
import pytest

from _gpu import check_against_oracle, run_filter

pytestmark = pytest.mark.gpu

RANGES = [((0, 0, 0), (110, 75, 9)), ((1, 3, 10), (34, 20, 27)), ((77, 58, 59), (110, 75, 60)),
          ((32, 16, 5), (64, 32, 6))]


@pytest.mark.parametrize("precision", ["auto", "splitbf16"])
@pytest.mark.parametrize("k", [5, 7])
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16, np.float32])
def test_short_tile_equals_tall_tile(orc, dtype, k, precision):
    g = np.random.default_rng(7 * k)
    shape = (60, 75, 110)  # 540 (k = 5) and 720 one-plane slabs of the tall tile
    src = (g.standard_normal(shape).astype(np.float32) if dtype == np.float32
           else g.integers(0, np.iinfo(dtype).max + 1, shape).astype(dtype))
    w = np.abs(g.standard_normal((k, k, k))) + 0.1
    w = (w / w.sum()).astype(np.float32)
    whole = run_filter(src, w, "mirror", precision=precision)
    for first, last in RANGES:
        at = tuple(slice(a, b) for a, b in zip(first[::-1], last[::-1]))
        part = run_filter(src, w, "mirror", precision=precision, roi=(first, last))
        assert np.array_equal(part[at].view(np.uint8), whole[at].view(np.uint8)), (first, last)
    if precision == "auto":
        check_against_oracle(orc, src, w, "mirror", whole, what=f"{dtype.__name__} k={k}")
