"""ROIs of more atoms than the 16-bit histogram counts hold at once: the spans
they go through lie at fixed atoms, so every stage size writes the same bits,
also those that do not divide a span (1792, 2304, 2816, 3328, 3584)."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins", [256, 512, 1024, 2048])
def test_every_stage_writes_the_same_images(nbins):
    gen = np.random.default_rng(nbins)
    n_dir, sizes = 19, [61440, 61441, 62000, 200003]
    d = gen.normal(size=(n_dir, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rel = np.zeros((sum(sizes), 4), np.float32)
    rel[:, :3] = gen.uniform(-0.55, 0.55, (len(rel), 3))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rel, dirs = dev(rel), dev(d.astype(np.float32))
    off = dev(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64))
    w = [[16, 19], [18, 21], [26, 31], [30, 36]]
    ctx = nat.Context(0)
    want = nat.araullo_signatures_csr(ctx, rel, off, 1.0, dirs, nbins, w)
    plan = nat.SignaturePlan(ctx, len(sizes), len(rel), n_dir, nbins, len(w))
    for stage in range(256, 4097, 256):
        plan.set_config(n_dir, stage, 2)
        assert torch.equal(plan.run(rel, off, 1.0, dirs, w), want), stage
