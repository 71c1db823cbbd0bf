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


def test_overlapping_rows_longer_than_an_int_together(dev):
    # 32 cells of one position whose rows are all the same 2^26 ids (between them
    # rows that end before they start): a wave that stands in all of them cannot
    # stage 2^31 faces.  The one real face, of the first id, is at x = 0.5; the
    # cell behind it has no row, so each ray ends there, at its extent.
    m, n = 2 ** 26, 64
    print(f"[gpu-case] malformed: 32 rows of {m} ids", flush=True)
    idx = torch.full((m,), -1, dtype=torch.int32, device=dev)
    idx[0] = 1
    sites = torch.zeros((n, 3), device=dev)
    sites[1, 0] = 1.0
    off = torch.tensor([0, m] * (n // 2) + [0], dtype=torch.int32, device=dev)
    ds = voro.DeviceScene(sites, torch.full((n,), 0.5, device=dev), off, idx,
                          torch.ones((n, 2, 2, 4), device=dev))
    voro.voro_prepare(ds)
    R = n // 2
    o = torch.zeros((R, 3), device=dev)
    d = torch.zeros((R, 3), device=dev)
    d[:, 0] = 1.0
    start = torch.arange(0, n, 2, dtype=torch.int32, device=dev)
    k = torch.zeros(R, dtype=torch.int32, device=dev)
    rgb, T = voro.voro_render_fwd(ds, o, d, torch.full((R,), 2.0, device=dev), start,
                                  voro.default_params(lanes_per_ray=1), nsteps=k)
    assert k.tolist() == [2] * R
    # exp(-0.5 * 2) in two FP32 factors
    np.testing.assert_allclose(T.cpu().numpy(), np.exp(-1.0), rtol=1e-6)
    np.testing.assert_allclose(rgb.cpu().numpy(), 1.0 - np.exp(-1.0), rtol=1e-6)
