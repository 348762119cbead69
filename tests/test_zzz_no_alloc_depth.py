"""GPU check of the slab depth and tile rules of batches where no tuning entry
exists, through the allocation-free form (it plans as the cached form does, and
makes no plan or graph).  A result cell's sum has the same terms in the same order
on every slab depth and tile height, so all comparisons with single-volume calls
are bit for bit:

- a class with enough tiles for 64-plane slabs, depths at and about a slab's edge;
- a batch that only fits the form's scratch on the taller tile.

These tests come last on purpose: run just before test_zz_no_alloc, and with plans
of their own, they were followed by a host crash inside vktApplyFilterBatched whose
cause is not known."""
import numpy as np
import pytest

from _gpu import sentinel_like

pytestmark = pytest.mark.gpu


def _vol(torch, z, y, x, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if dtype == torch.float32:
        return torch.randn((z, y, x), generator=g, device="cuda")
    return torch.randint(0, 60000, (z, y, x), generator=g, device="cuda",
                         dtype=torch.int32).to(dtype)


def _weights(k):
    w = np.abs(np.random.default_rng(k).standard_normal((k, k, k))) + 0.1
    return (w / w.sum()).astype(np.float32)


@pytest.mark.parametrize("fmt,k,depths", [("uint16", 5, (63, 64, 65, 129)),
                                          ("float32", 7, (1, 64, 67, 130)),
                                          ("uint16", 7, (5, 64, 65, 128))])
def test_deep_slabs_equal_single_calls(fmt, k, depths):
    import torch
    from paper_2203_10213_amd import vkt
    vkt.vktSetPrecision("auto")
    vkt.vktSetAutotune(False)
    vkt.vktSetStream(torch.cuda.current_stream())
    dtype = getattr(torch, fmt)
    f = vkt.vktFilterCreate(_weights(k))
    src = [_vol(torch, z, 513, 390, dtype, z) for z in depths]
    got = [sentinel_like(s) for s in src]
    want = [sentinel_like(s) for s in src]
    hs = [vkt.volume_from_tensor(t) for t in src]
    hg = [vkt.volume_from_tensor(t) for t in got]
    hw = [vkt.volume_from_tensor(t) for t in want]
    vkt.vktApplyFilterBatchedNoAlloc(hg, hs, [f] * len(hs), "clamp")
    for d, s in zip(hw, hs):
        vkt.vktApplyFilter(d, s, f, "clamp")
    torch.cuda.synchronize()
    for h in hs + hg + hw:
        vkt.vktStructuredVolumeDestroy(h)
    vkt.vktFilterDestroy(f)
    vkt.vktSetStream(None)
    for g, w in zip(got, want):
        assert torch.equal(g.view(torch.uint8), w.view(torch.uint8))


def test_no_alloc_takes_the_taller_tile_where_the_shorter_does_not_fit():
    import torch
    from paper_2203_10213_amd import vkt
    vkt.vktSetPrecision("auto")
    vkt.vktSetAutotune(False)
    vkt.vktSetStream(torch.cuda.current_stream())
    f = vkt.vktFilterCreate(_weights(13))
    src = _vol(torch, 1, 40_000_000, 1, torch.float32, 3)
    got, want = sentinel_like(src), sentinel_like(src)
    hs, hg, hw = (vkt.volume_from_tensor(t) for t in (src, got, want))
    vkt.vktApplyFilter(hw, hs, f, "clamp")
    vkt.vktApplyFilterBatchedNoAlloc([hg], [hs], [f], "clamp")
    torch.cuda.synchronize()
    for h in (hs, hg, hw):
        vkt.vktStructuredVolumeDestroy(h)
    vkt.vktFilterDestroy(f)
    vkt.vktSetStream(None)
    assert torch.equal(got.view(torch.uint8), want.view(torch.uint8))
