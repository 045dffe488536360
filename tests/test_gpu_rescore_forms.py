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
