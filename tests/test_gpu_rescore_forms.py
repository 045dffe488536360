"""The rescoring with four and with sixteen wavefronts per ROI: a ROI gets the
same candidates and the same scores in a call on either side of the rule that
chooses (two ROIs per CU, long rows, candidate counts)."""
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dir,n_win", [(1, 1), (63, 2), (642, 4), (8193, 1), (8192, 4)])
def test_dense(n_dir, n_win):
    gen = torch.Generator(device="cuda").manual_seed(n_dir)
    refs = torch.rand((90, n_win, n_dir), generator=gen, device="cuda")
    rois = torch.rand((1100, n_win, n_dir), generator=gen, device="cuda")
    rois[7] = refs[3]
    rois[8, 0, 0] = float("nan")
    ctx = nat.Context(0)
    lib = nat.Library(ctx, refs)
    for k in (1, 20, 64):
        many = nat.index_orientations(ctx, rois, lib, k)
        for a, b in ((0, 64), (500, 1012), (1093, 1100)):
            few = nat.index_orientations(ctx, rois[a:b].contiguous(), lib, k)
            assert torch.equal(many[0][a:b], few[0])
            assert torch.equal(many[1][a:b].nan_to_num(-1.0), few[1].nan_to_num(-1.0))


@pytest.mark.parametrize("n_hat", [50, 300])
def test_sparse(n_hat):
    gen = torch.Generator(device="cuda").manual_seed(n_hat)
    dirs = torch.from_numpy(synth.icosphere(2)).cuda()
    quats = torch.randn((300, 4), generator=gen, device="cuda", dtype=torch.float64)
    ctx = nat.Context(0)
    lut = nat.SparseLUT(ctx, torch.rand((1, 4, 162), generator=gen, device="cuda"), dirs, quats, [300], n_hat)
    rois = torch.rand((2500, 4, 162), generator=gen, device="cuda")
    for k in (1, 32):
        many = nat.index_orientations_sparse(ctx, rois, lut, k)
        for a in (0, 1024, 2400):
            few = nat.index_orientations_sparse(ctx, rois[a:a + 64].contiguous(), lut, k)
            assert torch.equal(many[0][a:a + 64], few[0]) and torch.equal(many[1][a:a + 64], few[1])


@pytest.mark.parametrize("n_dir", [2, 510, 512, 514, 1022, 1024, 1026])
def test_windows_about_the_registers(n_dir):
    """The normalised windows of either kernel form (1024 directions, and the pairs of a thread): an image among the
    references is at distance 0 from itself, two scaled copies of it as well."""
    gen = torch.Generator(device="cuda").manual_seed(n_dir)
    refs = torch.rand((70, 2, n_dir), generator=gen, device="cuda") + 0.1
    ctx = nat.Context(0)
    lib = nat.Library(ctx, refs)
    for scale in (1.0, 4.0, 0.125):
        idx, score = nat.index_orientations(ctx, refs * scale, lib, 1)
        assert torch.equal(idx[:, 0].long(), torch.arange(70, device="cuda")) and not score.any().item()


@pytest.mark.parametrize("n_dir", [12, 255, 256, 511, 766, 767, 768, 1026])
def test_sparse_codes_about_the_registers(n_dir):
    """Every image of the look-up table's own orientations scores 0 against its own entry."""
    gen = torch.Generator(device="cuda").manual_seed(n_dir)
    dirs = torch.randn((n_dir, 3), generator=gen, device="cuda")
    dirs = (dirs / dirs.norm(dim=1, keepdim=True)).contiguous()
    ref = torch.rand((1, 2, n_dir), generator=gen, device="cuda") + 0.01
    ident = torch.tensor([[1.0, 0, 0, 0]], dtype=torch.float64, device="cuda")
    ctx = nat.Context(0)
    lut = nat.SparseLUT(ctx, ref, dirs, ident, [1], min(2 * n_dir, 300))
    rois = torch.cat([ref, 2 * ref, torch.rand((20, 2, n_dir), generator=gen, device="cuda"), 0.25 * ref])
    idx, score = nat.index_orientations_sparse(ctx, rois.contiguous(), lut, 1)
    assert not idx.any().item()
    assert score[[0, 1, -1]].abs().max().item() <= 2.0 ** -40 * 300 and score[2:-1].min().item() > 0
