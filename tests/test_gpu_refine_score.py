"""The refinement's acceptance compares scores formed in one way: the J it
returns is, bit for bit, the one of the score-and-gradient call at the returned
orientation, whether the last trial was taken or not."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_freq", range(1, 9))
def test_final_score_is_the_trials(n_freq):
    gen = np.random.default_rng(n_freq)
    n_roi, n_atoms = 24, 300
    dirs = torch.from_numpy(synth.icosphere(3)).cuda()
    rel = np.zeros((n_roi * n_atoms, 4), np.float32)
    rel[:, :3] = gen.uniform(-1, 1, (len(rel), 3))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rois = [dev(rel), torch.arange(n_roi + 1, device="cuda") * n_atoms]
    rest = [torch.zeros(n_roi, dtype=torch.int32, device="cuda"), dirs,
            dev(gen.uniform(2, 8, (1, n_freq)).astype(np.float32)),
            dev(gen.uniform(0, 0.3, (1, n_freq, len(dirs))).astype(np.float32))]
    q0 = dev(gen.normal(size=(n_roi, 4)).astype(np.float32))
    q0 = q0 / q0.norm(dim=1, keepdim=True)
    ctx = nat.Context(0)
    taken = 0
    for steps in (1, 2, 5):
        q = q0.clone()
        J = nat.ar_refine_orientations(ctx, *rois, q, *rest, steps=steps, a0=0.01)
        again = nat.ar_sf_score_grad(ctx, *rois, q, *rest)[0]
        assert torch.equal(J, again), steps
        if steps == 1:
            taken = int((q != q0).any(1).sum())
    assert taken > 0   # some last trial was accepted
