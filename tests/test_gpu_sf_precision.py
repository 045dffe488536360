"""The gradient's matrix-core form is no further from FP64 than the FP32 form
that large calls take: the same ROIs in a call on either side of the line (one
and four frequencies, 12288 tiles), each against the gradient in FP64."""
import math

import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


def exact(q, x, n, f, T):
    q = q.double().requires_grad_(True)
    w, a, b, c = (q / q.norm()).unbind()
    M = torch.stack([1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                     2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                     2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)]).reshape(3, 3)
    t = 2 * math.pi * (n.double() @ M.T) @ x.double().T
    J = 0.0
    for i in range(len(f)):
        C, S = torch.cos(f[i].double() * t).sum(1), torch.sin(f[i].double() * t).sum(1)
        J = J + ((torch.sqrt(C * C + S * S) / len(x) - T[i].double()) ** 2).sum()
    J.backward()
    return q.grad


@pytest.mark.parametrize("n_freq", [1, 4])
@pytest.mark.parametrize("radius", [0.8, 1.2, 1.6, 2.0, 2.5])
def test_no_further_from_fp64_than_fp32(n_freq, radius):
    gen = np.random.default_rng(int(100 * radius) + n_freq)
    n_roi, a = 32, 0.405
    c = np.arange(-int(radius / a) - 2, int(radius / a) + 3)
    cells = np.stack(np.meshgrid(c, c, c, indexing="ij"), -1).reshape(-1, 1, 3)
    sites = (cells + np.array([[0, 0, 0], [0, .5, .5], [.5, 0, .5], [.5, .5, 0]])).reshape(-1, 3) * a
    rows = []
    for _ in range(n_roi):
        p = sites[gen.random(len(sites)) < 0.5]
        p = (p + 0.05 * gen.normal(size=p.shape)) @ np.linalg.qr(gen.normal(size=(3, 3)))[0]
        rows.append(torch.from_numpy(p[(p * p).sum(1) <= radius * radius].astype(np.float32)).cuda())
    n = torch.from_numpy(synth.icosphere(3)).cuda()
    f = torch.tensor([4.2767, 4.9383, 6.9838, 8.1892][:n_freq], device="cuda")
    T = torch.from_numpy(gen.uniform(0, 0.4, (n_freq, len(n))).astype(np.float32)).cuda()
    q = torch.from_numpy(gen.normal(size=(n_roi, 4)).astype(np.float32)).cuda()
    ctx = nat.Context(0)

    def grad(reps):
        off = torch.tensor([0] + [len(x) for x in rows] * reps, device="cuda").cumsum(0)
        rel = torch.nn.functional.pad(torch.cat(rows), (0, 1)).repeat(reps, 1)
        z = torch.zeros(n_roi * reps, dtype=torch.int32, device="cuda")
        return nat.ar_sf_score_grad(ctx, rel, off, q.repeat(reps, 1), z, n, f[None], T[None])[1][:n_roi].double()

    want = torch.stack([exact(q[r], x, n, f, T) for r, x in enumerate(rows)])
    small, large = grad(1), grad(12288 // (3 * n_roi))
    assert float((small - want).norm()) <= float((large - want).norm())
