"""GPU check of the tuning table's file (VKT_TUNE_CACHE): an entry counts only for
the tile that it was timed on.  Each run of the autotuner is a process of its own,
as the table is read once per process."""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DEPTH = 77  # a slab depth that the autotuner does not try


def _run(path):
    r = subprocess.run([sys.executable, "-u", os.path.abspath(__file__)], cwd=ROOT,
                       env=dict(os.environ, PYTHONPATH=ROOT, VKT_TUNE_CACHE=str(path)),
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "all equal" in r.stdout, r.stdout + r.stderr
    return [[int(v) for v in line.split()] for line in open(path)]


def _write(path, lines):
    path.write_text("".join(" ".join(str(v) for v in line) + "\n" for line in lines))


def test_entries_count_for_their_tile_only(tmp_path):
    f = tmp_path / "tune"
    fresh = _run(f)  # fmt k path flag size_class tz variant tx ty
    assert len(fresh) == 2 and all(len(line) == 9 for line in fresh)
    assert all(line[5] != DEPTH and line[7] > 0 and line[8] > 0 for line in fresh)
    deep = [line[:5] + [DEPTH] + line[6:] for line in fresh]
    _write(f, deep)
    assert _run(f) == deep  # taken as it is
    for stale in ([line[:7] for line in deep],                     # a file without tiles
                  [line[:7] + [line[7] + 16, line[8]] for line in deep],
                  [line[:8] + [2 * line[8]] for line in deep]):
        _write(f, stale)
        again = _run(f)
        assert [line[:5] for line in again] == [line[:5] for line in fresh]
        assert all(len(line) == 9 and line[5] != DEPTH for line in again)


def _child():
    import torch
    from paper_2203_10213_amd import vkt
    vkt.vktSetStream(torch.cuda.current_stream())
    vkt.vktSetAutotune(True)
    src = [torch.randn((100, 60 + 7 * i, 90), device="cuda") for i in range(4)]
    dst, want = [torch.zeros_like(s) for s in src], [torch.zeros_like(s) for s in src]
    f = []
    for k in (5, 3):
        w = np.abs(np.random.default_rng(k).standard_normal((k, k, k)))
        f += 2 * [vkt.vktFilterCreate((w / w.sum()).astype(np.float32))]
    hs, hd, hw = ([vkt.volume_from_tensor(t) for t in ts] for ts in (src, dst, want))
    vkt.vktApplyFilterBatched(hd, hs, f, "clamp")
    for h, s, g in zip(hw, hs, f):
        vkt.vktApplyFilter(h, s, g, "clamp")
    torch.cuda.synchronize()
    assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(dst, want))
    print("all equal", flush=True)


if __name__ == "__main__":
    _child()
