"""The gradient on either side of the line between its two kernels: large calls
and small ones of the same ROIs agree, one and four frequencies, tiles beyond
the atoms of one stage."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_freq", [1, 3, 4])
@pytest.mark.parametrize("n_atoms", [1, 250, 1025])
def test_large_calls_score_as_small_ones(n_freq, n_atoms):
    gen = np.random.default_rng(n_freq + n_atoms)
    n_dir, part = 1537, 8                      # 7 tiles, the last of one direction
    n_roi = 12288 // 7 + 3                     # past the line; parts of 8 ROIs lie before it
    dirs = gen.normal(size=(n_dir, 3))
    dirs /= np.linalg.norm(dirs, axis=1, keepdims=True)
    atoms = np.zeros((part * n_atoms, 4), np.float32)
    atoms[:, :3] = gen.uniform(-1, 1, (len(atoms), 3))
    q = gen.normal(size=(part, 4))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    dev = lambda a, t=torch.float32: torch.from_numpy(np.ascontiguousarray(a)).to(t).cuda()  # noqa: E731
    freqs, targets = dev(gen.uniform(1, 4, (1, n_freq))), dev(gen.uniform(0, 1, (1, n_freq, n_dir)))
    ctx = nat.Context(0)

    def run(reps, n):
        rel = dev(atoms).repeat(reps, 1)
        off = torch.arange(n + 1, dtype=torch.int64, device="cuda") * n_atoms
        return nat.ar_sf_score_grad(ctx, rel[:n * n_atoms].contiguous(), off, dev(q).repeat(reps, 1)[:n].contiguous(),
                                    torch.zeros(n, dtype=torch.int32, device="cuda"), dev(dirs), freqs, targets)

    score, grad = run(1, part)
    reps = -(-n_roi // part)
    big_score, big_grad = run(reps, n_roi)
    want_s, want_g = score.repeat(reps)[:n_roi], grad.repeat(reps, 1)[:n_roi]
    # both forms keep 22 bits of every sine and sum in FP32: their sums of up to
    # 1025 terms and 1537 directions differ by rounding, far below 1e-4 of the largest gradient
    assert (big_score - want_s).abs().max().item() <= 1e-5 * want_s.abs().max().item()
    bound = 1e-4 * want_g.abs().max().item()
    if n_atoms == 1:   # |F| = 1 whatever the orientation: no gradient but the rounding of its terms, each
        # 2 |e| 2 pi f |x| (|S Q| + |C P|) <= 8 pi f |x| with f <= 4 and |x| <= sqrt(3), in 22 bits
        bound = 2.0 ** -22 * n_freq * n_dir * 8 * np.pi * 4 * 3 ** 0.5
    assert (big_grad - want_g).abs().max().item() <= bound
