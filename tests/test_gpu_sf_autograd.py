"""The autograd form of the structure-factor score: the gradient kept from the
forward pass is the adjoint's, for every way the forward pass can run (with a
gradient, under no_grad, for inputs that need none, twice backward, through
saved-tensor hooks), and inputs changed in place between the passes are
refused."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import refine, synth

pytestmark = pytest.mark.gpu


def case():
    gen = np.random.default_rng(5)
    sizes = [40, 0, 300]
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    rel = np.zeros((sum(sizes), 4), np.float32)
    rel[:, :3] = gen.uniform(-1, 1, (sum(sizes), 3))
    dirs = torch.from_numpy(synth.icosphere(2)).cuda()
    freqs = torch.tensor([[4.0, 7.0]], device="cuda")
    targets = torch.rand((1, 2, len(dirs)), device="cuda")
    q = torch.from_numpy(gen.normal(size=(3, 4)).astype(np.float32)).cuda()
    return nat.Context(0), q, [torch.from_numpy(rel).cuda(), off, torch.zeros(3, dtype=torch.int32, device="cuda"), dirs,
                               freqs, targets]


def test_gradient_of_every_forward():
    ctx, q, args = case()
    J, g = nat.ar_sf_score_grad(ctx, args[0], args[1], q, *args[2:])
    scale = torch.tensor([2.0, -1.0, 0.5], device="cuda")
    p = q.clone().requires_grad_(True)
    s = refine.sf_score(ctx, p, *args)
    assert torch.equal(s, J)
    (s * scale).sum().backward(retain_graph=True)
    assert torch.equal(p.grad, scale[:, None] * g)
    (s * scale).sum().backward()
    assert torch.equal(p.grad, 2 * scale[:, None] * g)
    with torch.no_grad():
        plain = refine.sf_score(ctx, p, *args)
    assert not plain.requires_grad and torch.allclose(plain, J, rtol=1e-5)
    assert not refine.sf_score(ctx, q, *args).requires_grad
    p = q.clone().requires_grad_(True)
    with torch.autograd.graph.save_on_cpu():
        s = refine.sf_score(ctx, p, *args)
    s.sum().backward()
    assert torch.equal(p.grad, g)
    strided = q.t().contiguous().t().requires_grad_(True)        # not contiguous
    refine.SFScore.apply(strided, ctx, *args).sum().backward()
    assert torch.equal(strided.grad, g)


def test_inputs_changed_between_the_passes_are_refused():
    ctx, q, args = case()
    p = q.clone().requires_grad_(True)
    s = refine.sf_score(ctx, p, *args)
    args[5].mul_(2.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        s.sum().backward()
