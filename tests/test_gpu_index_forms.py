"""The forms a dense indexing call can take (wavefront tiles and smaller
workgroup tiles for small calls) against a tile set by hand: every form sums
the correlations in the same order, so indices, scores and candidates are
equal.  Ragged sizes, libraries smaller than the candidate list, images that
are not numbers, windows past the registers of the normalisation."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu


def images(gen, n, n_win, n_dir):
    return gen.gamma(2.0, 1.0, (n, n_win, n_dir)).astype(np.float32)


def call(ctx, lib, rois, k, cand):
    return [x.cpu() for x in nat.index_orientations_ex(ctx, rois, lib, k, cand)]


# (n_roi, n_lib): one wavefront tile each way; the edges of the 32 and 64 tiles
# and of the forms (tiles per 256 CUs): 32 ROIs to 65536 rows, 64-tiles to 768,
# 128 x 128 to 256 and 128 x 256 to 256
@pytest.mark.parametrize("n_roi, n_lib", [
    (1, 1), (3, 40), (32, 257), (33, 300), (16, 1000), (32, 65536), (32, 65537), (33, 8192), (33, 8193), (65, 6000),
    (300, 2500), (768, 4096), (769, 4096), (1024, 4096), (1025, 4000), (1030, 7000), (1100, 7200)])
def test_small_calls_rank_as_the_tiles_do(n_roi, n_lib):
    gen = np.random.default_rng(n_roi + n_lib)
    n_dir = int(gen.integers(20, 40))
    dev = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    ctx = nat.Context(0)
    refs = dev(images(gen, n_lib, 2, n_dir))
    lib = nat.Library(ctx, refs)
    rois = images(gen, n_roi, 2, n_dir)
    if n_roi > 2:
        rois[1, 1, 3] = np.nan
        rois[2, 0, 5] = np.inf
        rois[n_roi // 2] = 0
    for k, cand in ((1, 16), (16, 16), (20, 32), (64, 64)):
        got = call(ctx, lib, dev(rois), k, cand)
        nat.ar_index_set_tile(ctx, 4, 4, 4, 32)
        want = call(ctx, lib, dev(rois), k, cand)
        nat.ar_index_set_tile(ctx, 0, 0, 0, 0)
        for g, w in zip(got, want):
            assert np.array_equal(g.numpy(), w.numpy(), equal_nan=g.is_floating_point()), (k, cand)


@pytest.mark.parametrize("n_dir", [1, 63, 1001, 10242, 10241, 11000])
def test_candidates_match_the_normalised_images(n_dir):
    """An image among the references is at distance 0 from itself, also where the array starts off 8 bytes."""
    gen = np.random.default_rng(n_dir)
    refs = torch.from_numpy(images(gen, 300, 4, n_dir)).cuda()
    at = torch.from_numpy(gen.integers(0, 300, 40)).cuda()
    ctx = nat.Context(0)
    lib = nat.Library(ctx, refs)
    flat = torch.empty(40 * 4 * n_dir + 1, device="cuda")[1:].view(40, 4, n_dir)
    for rois in (refs[at].contiguous(), flat.copy_(refs[at])):
        idx, score = nat.index_orientations(ctx, rois, lib, k=1)
        if n_dir > 1:
            assert torch.equal(idx[:, 0].long(), at) and not score.any().item()
        else:   # every image is x (1 / x), 1 within 2^-23: any of them may rank first
            assert score.max().item() <= 4 * 2.0 ** -44
