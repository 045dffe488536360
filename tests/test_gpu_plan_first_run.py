"""A plan's first run on a new context, captured in a graph before anything else
has used the context's tables."""
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins,windows", [(256, [[8, 9], [10, 11]]), (1024, [[16, 60]]), (4096, [[16, 19]])])
def test_first_run_is_captured(nbins, windows):
    gen = torch.Generator(device="cuda").manual_seed(nbins)
    rel = torch.rand((300, 4), generator=gen, device="cuda") - 0.5
    off = torch.tensor([0, 100, 300], device="cuda")
    dirs = torch.from_numpy(synth.icosphere(1)).cuda()
    plan = nat.SignaturePlan(nat.Context(0), 2, 300, len(dirs), nbins, len(windows))
    got = [plan.run(rel, off, 1.0, dirs, windows) for _ in range(3)]
    want = nat.araullo_signatures_csr(nat.Context(0), rel, off, 1.0, dirs, nbins, windows)
    assert all(torch.equal(g, want) for g in got)
