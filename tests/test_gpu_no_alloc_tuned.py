"""GPU check of the allocation-free batched form where a tuning entry's tile does not
fit its scratch: the taller tile is taken with a slab depth of its own, not with
the one that was timed on the other tile.  In a process of its own, as the table is
read once per process."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROWS, Z = 700_000 * 32, 16  # one column: a 64 x 32 tile per 32 rows


def test_taller_tile_takes_its_own_depth(tmp_path):
    # uint8, k = 3, vector kernel, FP32 sums; edge 2^9 .. 2^10; 64 x 16 tiles in
    # slabs of 8: 2.8 M items of 8 bytes.  64 x 32 tiles in slabs of 8 are 1.4 M,
    # too many for 8 MiB; in slabs of 16, their own default, 0.7 M fit.
    f = tmp_path / "tune"
    f.write_text("0 3 0 0 9 8 1 64 16\n")
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__)], cwd=ROOT,
                       env=dict(os.environ, PYTHONPATH=ROOT, VKT_TUNE_CACHE=str(f)),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "all equal" in r.stdout, r.stdout + r.stderr


def _child():
    import torch
    from paper_2203_10213_amd import vkt
    assert vkt.vktDataFormatUInt8 == 0 and 2 ** 27 <= ROWS * Z < 2 ** 30
    vkt.vktSetStream(torch.cuda.current_stream())
    w = np.abs(np.random.default_rng(3).standard_normal((3, 3, 3)))
    f = vkt.vktFilterCreate((w / w.sum()).astype(np.float32))
    src = torch.randint(0, 256, (Z, ROWS, 1), dtype=torch.uint8, device="cuda",
                        generator=torch.Generator(device="cuda").manual_seed(5))
    got, want = torch.zeros_like(src), torch.zeros_like(src)
    hs, hg, hw = (vkt.volume_from_tensor(t) for t in (src, got, want))
    vkt.vktApplyFilter(hw, hs, f, "clamp")
    vkt.vktApplyFilterBatchedNoAlloc([hg], [hs], [f], "clamp")
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    print("all equal", flush=True)


if __name__ == "__main__":
    _child()
