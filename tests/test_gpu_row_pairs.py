"""The row-pair matrix-core kernel at the edges of its staging: quads of four
cells at the x faces (rows shorter than a quad, than a tile, a cell either side
of one 48- or 32-column tile), odd rows, rows that no vector store fits, and
ranges whose first column is no multiple of anything.  Tolerances are those of
the split path: integer cells 1 LSB, float32 1e-5 of sum |w||s| (6 products
1e-6)."""
import numpy as np
import pytest

from _gpu import check_against_oracle, run_filter

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _row_pairs_always():
    from paper_2203_10213_amd import vkt
    rp = vkt.vktGetRowPairMinCells()
    vkt.vktSetRowPairMinCells(0)
    yield
    vkt.vktSetPrecision("auto")
    vkt.vktSetRowPairMinCells(rp)


@pytest.mark.parametrize("mode", ["clamp", "wrap", "mirror", "border"])
@pytest.mark.parametrize("dtype,precision,k", [
    (np.uint8, "auto", 5), (np.uint16, "auto", 5), (np.float32, "splitbf16x6", 5),
    (np.float32, "splitbf16", 5), (np.float32, "splitbf16", 7)])
def test_face_quads(orc, dtype, precision, k, mode):
    g = np.random.default_rng(77 + k)
    w = g.standard_normal((k, k, k)).astype(np.float32)
    if dtype != np.float32:
        w = np.abs(w) / np.abs(w).sum()
    for X in (2, 3, 4, 5, 7, 31, 34, 46, 47, 48, 49, 51, 95, 100):
        shape = (3, 67 if X in (47, 49) else 5, X)
        src = (g.standard_normal(shape).astype(np.float32) if dtype == np.float32
               else g.integers(0, np.iinfo(dtype).max + 1, shape).astype(dtype))
        out = run_filter(src, w, mode, precision=precision)
        check_against_oracle(orc, src, w, mode, out,
                             tol=1e-6 if precision == "splitbf16x6" else 1e-5,
                             what=f"{shape} k={k} {mode}")
        if X > 40:
            roi = ((X // 2 - 19, 1, 0), (X - 2, 4, 3))
            out = run_filter(src, w, mode, precision=precision, roi=roi)
            check_against_oracle(orc, src, w, mode, out, roi=roi,
                                 tol=1e-6 if precision == "splitbf16x6" else 1e-5,
                                 what=f"{shape} k={k} {mode} range")
