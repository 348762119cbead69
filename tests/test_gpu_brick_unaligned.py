"""GPU parity of vktBrickDecompose where brick rows are not whole dwords, bit
for bit against the oracle: rows with 2 to 17 bytes inside the source (cells one
by one, 4-byte groups, 16-byte groups), rows of more items than a workgroup has
threads, more ghost cells than the volume has cells, brick rows that wrap more
than once per step of a workgroup, and a source and bricks that start at an odd
byte.  And a row past 2^30 cells, which takes the cell kernel."""
import numpy as np
import pytest

from _gpu import to_device

pytestmark = pytest.mark.gpu

CASES = [  # (Z, Y, X), brick (x, y, z), ghost (x, y, z)
    ((4, 5, 3), (3, 2, 2), (1, 1, 0)),          # 3 cells inside
    ((4, 5, 9), (5, 2, 2), (2, 1, 1)),
    ((3, 4, 15), (15, 3, 3), (0, 1, 0)),
    ((3, 4, 17), (17, 3, 3), (1, 0, 1)),
    ((5, 7, 33), (16, 3, 2), (1, 2, 1)),
    ((9, 11, 63), (21, 4, 5), (4, 3, 2)),
    ((3, 300, 5), (5, 299, 2), (1, 0, 2)),      # many short rows
    ((2, 3, 4501), (4500, 2, 2), (3, 1, 1)),    # over 256 items in a row
    ((2, 2, 3), (2, 1, 2), (7, 4, 5)),          # ghosts beyond the volume
]


@pytest.mark.parametrize("mode", ["clamp", "wrap", "mirror", "border"])
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
def test_unaligned_rows_match_oracle(orc, dtype, mode):
    from paper_2203_10213_amd import vkt
    g = np.random.default_rng(17)
    for shape, brick, ghost in CASES:
        src = g.integers(0, np.iinfo(dtype).max + 1, shape).astype(dtype)
        got = vkt.brick_decompose(to_device(src), brick, ghost, mode)
        vkt.vktSynchronize()
        want = orc.brick_decompose(src, brick, ghost, mode)
        for i, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a.cpu().numpy(), b), (shape, brick, ghost, i)


@pytest.mark.parametrize("mode", ["clamp", "border"])
def test_odd_byte_buffers(orc, mode):
    import torch
    from paper_2203_10213_amd import vkt
    src = np.random.default_rng(5).integers(0, 256, (6, 7, 64)).astype(np.uint8)
    want = orc.brick_decompose(src, (32, 4, 3), (2, 1, 1), mode)

    def odd(a):
        t = torch.full((a.size + 3,), 0xA5, dtype=torch.uint8, device="cuda")
        return t, t[1:1 + a.size].view(a.shape)
    held, s = odd(src)
    s.copy_(torch.from_numpy(src))
    bricks = [odd(w) for w in want]
    hs = vkt.volume_from_tensor(s)
    hb = [vkt.volume_from_tensor(v) for _, v in bricks]
    vkt.vktSetStream(torch.cuda.current_stream())
    vkt.vktBrickDecompose(hb, hs, (32, 4, 3), (2, 1, 1), mode)
    torch.cuda.synchronize()
    for (t, v), w in zip(bricks, want):
        assert np.array_equal(v.cpu().numpy(), w)
        assert t[0] == 0xA5 and (t[-2:] == 0xA5).all()
    for h in hb + [hs]:
        vkt.vktStructuredVolumeDestroy(h)
    vkt.vktSetStream(None)


def test_row_past_two_to_the_thirty():
    import torch
    from paper_2203_10213_amd import vkt
    n, b = (1 << 30) + 5, (1 << 28) + 3
    src = torch.randint(0, 256, (1, 1, n), dtype=torch.uint8, device="cuda")
    got = vkt.brick_decompose(src, (b, 1, 1), (1, 0, 0), "clamp")
    torch.cuda.synchronize()
    at = src.flatten()
    for i, v in enumerate(got):
        lo, hi = i * b - 1, min((i + 1) * b, n) + 1
        want = torch.cat([at[:1]] * (lo < 0) + [at[max(lo, 0):min(hi, n)]] + [at[-1:]] * (hi > n))
        assert torch.equal(v.flatten(), want)
