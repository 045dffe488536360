"""Rows padded to the height of the tile that a dense indexing call takes: calls
of 1 to 3 row blocks of 128 against libraries that take the 128-row tiles rank
as a tile set by hand does, whose rows are padded to 256."""
import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu


# (n_roi, n_lib, n_dir): 128 x 128 tiles from 768 64-tiles on, 128 x 256 from 256 128-tiles on, 256 x 256 past
# that, and for long libraries of short rows (112 + K / 128 tiles of 256, K / 256 for 32 candidates)
@pytest.mark.parametrize("n_roi, n_lib, n_dir", [
    (65, 25000, 23), (100, 30000, 23), (128, 32768, 23), (129, 16300, 23), (257, 10900, 23), (129, 28600, 23),
    (129, 28900, 23), (384, 21800, 23), (385, 16300, 23), (64, 60000, 23), (128, 65536, 23), (100, 33000, 1290),
    (128, 33500, 1290), (100, 66000, 23)])
def test_padded_rows(n_roi, n_lib, n_dir):
    gen = torch.Generator(device="cuda").manual_seed(n_roi + n_lib)
    refs, rois = (torch.rand((n, 2, n_dir), generator=gen, device="cuda") for n in (n_lib, n_roi))
    ctx = nat.Context(0)
    lib = nat.Library(ctx, refs)
    for k, cand in ((4, 16), (20, 32), (64, 64)):
        got = nat.index_orientations_ex(ctx, rois, lib, k, cand)
        nat.ar_index_set_tile(ctx, 4, 4, 4, 32)
        want = nat.index_orientations_ex(ctx, rois, lib, k, cand)
        nat.ar_index_set_tile(ctx, 0, 0, 0, 0)
        for g, w in zip(got, want):
            assert torch.equal(g, w), (k, cand)
