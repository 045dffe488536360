"""One score per orientation: J is the same, bit for bit, formed alone, beside a
gradient, through torch.autograd, without allocation, and in a batch of any
size, and the gradient does not depend on the batch either."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import refine, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_freq", range(1, 9))
def test_score_does_not_depend_on_the_call(n_freq):
    gen = np.random.default_rng(n_freq)
    sizes = [130, 0, 1, 700, 1025, 33]
    dirs = torch.from_numpy(synth.icosphere(4)).cuda()           # 1281 evaluated: the last tile holds one
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rel = np.zeros((sum(sizes), 4), np.float32)
    rel[:, :3] = gen.uniform(-1.2, 1.2, (len(rel), 3))
    q = gen.normal(size=(len(sizes), 4)).astype(np.float32)
    f = dev(gen.uniform(1, 9, (1, n_freq)).astype(np.float32))
    T = dev(gen.uniform(0, 0.6, (1, n_freq, len(dirs))).astype(np.float32))
    ctx = nat.Context(0)

    def args(reps):
        off = np.concatenate([[0], np.cumsum(sizes * reps)]).astype(np.int64)
        return (dev(np.tile(rel, (reps, 1))), dev(off), dev(np.tile(q, (reps, 1))),
                torch.zeros(len(off) - 1, dtype=torch.int32, device="cuda"), dirs, f, T)

    a = args(1)
    J, g = nat.ar_sf_score_grad(ctx, *a)
    assert torch.equal(nat.ar_sf_score_grad(ctx, *a, grad=False)[0], J)
    s, h = torch.empty_like(J), torch.empty_like(g)
    nat.ar_sf_score_grad_noalloc(ctx, *a, s, h)
    assert torch.equal(s, J) and torch.equal(h, g)
    leaf = a[2].clone().requires_grad_(True)
    score = refine.sf_score(ctx, leaf, a[0], a[1], *a[3:])
    score.sum().backward()
    with torch.no_grad():
        alone = refine.sf_score(ctx, leaf, a[0], a[1], *a[3:])
    assert torch.equal(score.detach(), J) and torch.equal(alone, J) and torch.equal(leaf.grad, g)
    big = nat.ar_sf_score_grad(ctx, *args(400))
    assert torch.equal(big[0], J.repeat(400)) and torch.equal(big[1], g.repeat(400, 1))
