"""The ROI query where it can go wrong: every form it takes (many wavefronts
per ROI, one, and the unsorted scan behind small signature calls), ROIs at and
beyond the specimen's edge, cells too full to rank, long grids, types.
Against a NumPy FP32 evaluation of the membership test, with the rows in their
defined order: by grid cell (x fastest), then by atom index."""
import math

import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu
f32 = np.float32


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def members(pos, c, R):
    d = (pos - c).astype(f32)
    d64 = d.astype(np.float64)
    s = (d64[:, 0] * d64[:, 0]).astype(f32).astype(np.float64)
    s = (d64[:, 1] * d64[:, 1] + s).astype(f32).astype(np.float64)
    s = (d64[:, 2] * d64[:, 2] + s).astype(f32)
    return np.flatnonzero(s <= f32(float(f32(R)) ** 2)), d


def cells(pos, centres, R):
    """Grid cell of every atom: edge R/2 over the centres' box +- 1.5 R."""
    R = float(f32(R))
    h = 0.5 * R
    lo, hi = centres.min(0).astype(np.float64), centres.max(0).astype(np.float64)
    ext = hi - lo + 2 * (R + h)
    while np.prod(np.floor(ext / h) + 1) > 6.4e7:
        h *= 1.5
    o = (lo - (R + h if h == 0.5 * R else R + 0.5 * R)).astype(f32)
    n = np.floor(ext / h).astype(np.int64) + 1
    c = np.floor((pos - o) * f32(1.0 / h)).astype(np.int64)
    return c[:, 0] + n[0] * (c[:, 1] + n[1] * c[:, 2])


def check(pos, centres, R, types=None, mask=None, sample=None):
    ctx = nat.Context(0)
    kw = {} if types is None else {"types": dev(types), "type_mask": mask}
    off, rel = nat.ar_roi_gather(ctx, dev(pos), dev(centres), R, **kw)
    off, rel = off.cpu().numpy(), rel.cpu().numpy()
    key = cells(pos, centres, R)
    assert off[0] == 0 and off[-1] == len(rel)
    for r in range(len(centres)) if sample is None else sample:
        i, d = members(pos, centres[r], R)
        if types is not None:
            i = i[[0 <= t < 64 and (mask >> int(t)) & 1 == 1 for t in types[i]]]
        i = i[np.lexsort((i, key[i]))]
        got = rel[off[r]:off[r + 1]]
        assert np.array_equal(got[:, :3], d[i]) and not got[:, 3].any(), r


@pytest.mark.parametrize("n_roi", [1, 600])
def test_rows_and_order(n_roi):
    gen = np.random.default_rng(n_roi)
    pos = gen.uniform(-4, 4, (40000, 3)).astype(f32)
    centres = gen.uniform(-5.5, 5.5, (n_roi, 3)).astype(f32)
    check(pos, centres, 1.3)
    types = gen.integers(-1, 70, len(pos)).astype(np.int32)
    check(pos, centres, 1.3, types, (1 << 63) | 0b1011, range(0, n_roi, 7))


def test_full_cells_and_long_grids():
    gen = np.random.default_rng(3)
    crowd = np.concatenate([gen.normal(0, 0.02, (3000, 3)), gen.uniform(-2, 2, (3000, 3))]).astype(f32)
    check(crowd, gen.uniform(-1, 1, (20, 3)).astype(f32), 0.9)
    wire = gen.uniform(0, 1, (20000, 3)) * [3.0e5, 1.0, 1.0]
    centres = np.concatenate([wire[::400], wire[::300] + 0.4])
    check(wire.astype(f32), centres.astype(f32), 7.0)


def test_cells_of_a_hundred_thousand_atoms_keep_the_input_order():
    gen = np.random.default_rng(4)
    pos = np.concatenate([gen.normal(0.3, 0.001, (100000, 3)), gen.normal(0.8, 0.02, (20000, 3))]).astype(f32)
    check(pos[gen.permutation(len(pos))], gen.uniform(0.2, 0.4, (3, 3)).astype(f32), 0.9)


@pytest.mark.parametrize("n", [262143, 262144, 262145, 300001])
@pytest.mark.parametrize("shape", ["box", "crowd", "few cells", "many cells"])
def test_sort_by_parts(n, shape):
    """Either side of the line between the two sorts: even and crowded cells,
    fewer cells than parts, a part's most cells and beyond, types."""
    gen = np.random.default_rng(n)
    pos, R = gen.uniform(-8, 8, (n, 3)), 1.1
    centres = gen.uniform(-8, 8, (40, 3))
    if shape == "crowd":
        pos[: n // 8] = gen.normal(1.0, 0.05, (n // 8, 3))
        pos = pos[gen.permutation(n)]
    elif shape == "few cells":
        R, centres = 4.0, gen.uniform(-1, 1, (5, 3))
    elif shape == "many cells":
        R, centres = 0.22 if n % 2 else 0.1, gen.uniform(-8, 8, (40, 3))
    pos, centres = pos.astype(f32), centres.astype(f32)
    check(pos, centres, R, sample=range(0, len(centres), 4))
    types = gen.integers(-1, 70, n).astype(np.int32)
    check(pos, centres, R, types, (1 << 63) | 0b1011, range(0, len(centres), 9))


def test_more_rois_than_row_counts_are_kept_for():
    gen = np.random.default_rng(4)
    pos = gen.uniform(-3, 3, (5000, 3)).astype(f32)
    centres = gen.uniform(-3, 3, (262200, 3)).astype(f32)
    check(pos, centres, 0.5, sample=[0, 1, 1000, 131072, 262199])


def test_small_signature_calls_count_the_same_atoms():
    """The unsorted scan (up to 32768 atoms and 4e6 tests) and the grid just past it."""
    gen = np.random.default_rng(5)
    dirs = gen.normal(size=(5, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(f32)
    ctx = nat.Context(0)
    for n, n_roi in ((0, 2), (1, 1), (1025, 3), (32768, 128), (32769, 1), (30000, 140)):
        pos = gen.uniform(-3, 3, (n, 3)).astype(f32)
        centres = gen.uniform(-3, 3, (n_roi, 3)).astype(f32)
        want = [len(members(pos, c, 1.5)[0]) for c in centres]
        img, cnt = nat.araullo_signatures(ctx, dev(pos), dev(centres), 1.5, dev(dirs), 256, [[8, 12]])
        assert cnt.cpu().tolist() == want
        if n:
            off, rel = nat.ar_roi_gather(ctx, dev(pos), dev(centres), 1.5)
            assert torch.equal(nat.araullo_signatures_csr(ctx, rel, off, 1.5, dev(dirs), 256, [[8, 12]]), img)
    for bad in ([math.inf, 0, 0], [math.nan] * 3):
        with pytest.raises(nat.AraulloError, match="finite"):
            nat.araullo_signatures(ctx, dev(np.zeros((4, 3), f32)), dev(np.array([bad], f32)), 1.5, dev(dirs), 256,
                                   [[8, 12]])
