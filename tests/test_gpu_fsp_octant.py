"""The octant form of the reciprocal-space grid where it can go wrong: grid
edges whose half is not a multiple of the 32-column tile (L = 32, 96), several
tiles per axis (L = 128), atom counts around the 16-atom slice, the 32-atom
step and the 512-atom stage, and coordinates of the largest phases.  Bar: every
point within 1e-5 N_w of the FP64 oracle, the bar of every whole spectrum."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,sizes", [(32, [15, 16, 17, 31, 32, 33, 479, 481, 1025]), (96, [1, 33, 0]), (128, [5]),
                                     (160, [2])])
def test_octant_edges(orc, L, sizes):
    from paper_2009_00735_amd import native as nat
    gen = np.random.default_rng(900 + L)
    rois = [gen.uniform(-2.5, 2.5, (n, 3)).astype(np.float32) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rel = np.zeros((int(off[-1]), 4), np.float32)
    rel[:, :3] = np.concatenate(rois)
    ctx = nat.Context(0)
    out = torch.full((len(rois), L, L, L), -1.0, device="cuda")
    amp = nat.ar_fsp_amplitudes(ctx, torch.from_numpy(rel).cuda(), torch.from_numpy(off).cuda(), L, 10.0,
                                out=out).cpu().numpy()
    for r, x in enumerate(rois):
        ref = orc.fsp_grid(x, L, 10.0) if len(x) else np.zeros((L, L, L))
        err = np.abs(amp[r] - ref).max()
        assert err <= 1e-5 * max(len(x), 1), (L, len(x), err)
