"""Malformed adjacency offsets: every row that is sound by itself is handled as if
the others were, and nothing outside the arrays is read or written."""
import numpy as np
import pytest
import torch

from paper_2608_17682_amd import voro

pytestmark = pytest.mark.gpu

TOP = 2 ** 31 - 1


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    voro.lib()
    return torch.device("cuda:0")


def i32(x):
    return (int(x) + 2 ** 31) % 2 ** 32 - 2 ** 31


# the row's offsets, of 40 ids; lengths are summed in 32 bits, as the library does
@pytest.mark.parametrize("name,off", [
    ("row that ends before it starts", [0, 10, 6, 25, 40]),
    ("row past the array's end", [0, 10, 60, 20, 40]),
    ("negative offset", [0, 10, -5, 20, 40]),
    # 10 + (TOP - 10) + 10 + (TOP - 10) + 12 = 10 in 32 bits: the row of 5 that
    # follows goes to [10, 15), behind sums that went up and down
    ("lengths beyond 2^31", [0, 10, TOP, 0, 10, TOP, 0, 12, 17, 40]),
])
# the malformed rows alone, at the start of a workgroup's 64 rows, and at their end
@pytest.mark.parametrize("before,after", [(0, 0), (0, 90), (60, 90)])
def test_sound_rows_are_reordered(dev, name, off, before, after):
    print(f"[gpu-case] malformed: {name}, {before} rows before and {after} after", flush=True)
    off = [0] * before + off + [off[-1]] * after     # the rows around are empty
    n, m = len(off) - 1, 40
    rng = np.random.default_rng(n)
    idx = rng.integers(-1, n + 2, m).astype(np.int32)   # ids outside [0, n) stay as they are
    # equal positions: the Morton order is the order of the cells
    ds = voro.DeviceScene(*(torch.from_numpy(a).to(dev) for a in (
        np.zeros((n, 3), np.float32), np.ones(n, np.float32), np.array(off, np.int32), idx,
        np.zeros((n, 2, 2, 4), np.float32))))
    out, perm, _ = voro.voro_morton_reorder(ds)
    np.testing.assert_array_equal(perm.cpu().numpy(), np.arange(n))
    got = out.nbr_idx.cpu().numpy()
    at = 0
    sound = 0
    for s, e in zip(off[:-1], off[1:]):
        if 0 <= s <= e <= m and 0 <= at <= m - (e - s):
            np.testing.assert_array_equal(got[at:at + e - s], idx[s:e])
            sound += e - s
        at = i32(at + max(0, i32(e - s)))
    assert sound >= 10
