"""The reciprocal grid's amplitudes are not shrunk: the FP16 parts that the
factors are split into leave a remainder of either sign, so the amplitudes'
mean error (their projection on the exact ones) stays below 2^-23, half a unit
in the last place of an FP32 value, as with FP32 factors.  Parts cut toward
zero shrink every amplitude by 0.5 to 0.8 of 2^-22."""
import math

import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,n_atoms", [(32, 130), (64, 2000), (64, 4001)])
def test_mean_error_has_no_side(L, n_atoms):
    gen = torch.Generator(device="cuda").manual_seed(L + n_atoms)
    x = torch.zeros((n_atoms, 4), device="cuda")
    x[:, :3] = 4 * torch.rand((n_atoms, 3), generator=gen, device="cuda") - 2
    off = torch.tensor([0, n_atoms], device="cuda")
    amp = nat.ar_fsp_amplitudes(nat.Context(0), x, off, L, 10.0)[0].double()
    k = (torch.arange(L, device="cuda", dtype=torch.float64) - L // 2) * (20.0 / L)
    wave = [2 * math.pi * k[:, None] * x[:, a].double()[None] for a in range(3)]
    wave = [torch.complex(p.cos(), p.sin()) for p in wave]
    ref = torch.stack([((wave[0][a] * wave[1]) @ wave[2].T).abs() for a in range(L)])
    mean = float(((amp - ref) * ref).sum() / (ref * ref).sum())
    assert abs(mean) <= 2.0 ** -23, mean * 2 ** 22
    assert float((amp - ref).norm() / ref.norm()) <= 1e-6
