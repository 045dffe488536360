"""The structure-factor gradient of every frequency count against FP64, held to
1e-3 of its own length, the bar of the adjoint against finite differences (J to
1e-5 of itself): atom counts around the 32-atom step and the 1024-atom stage,
several stages, a mesh whose last tile is short and one without antipodes."""
import math

import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


def exact(q, x, dirs, f, T):
    q = q.clone().requires_grad_(True)
    w, a, b, c = (q / q.norm()).unbind()
    M = torch.stack([1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                     2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                     2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)]).reshape(3, 3)
    t = 2 * math.pi * (dirs @ M.T) @ x.T
    J = torch.zeros((), dtype=torch.float64)
    for i in range(len(f)):
        C, S = torch.cos(f[i] * t).sum(1), torch.sin(f[i] * t).sum(1)
        J = J + ((torch.sqrt(C * C + S * S) / len(x) - T[i]) ** 2).sum()
    J.backward()
    return J.detach(), q.grad


@pytest.mark.parametrize("n_dir", [100, 642])
@pytest.mark.parametrize("n_freq", range(1, 9))
def test_gradient_relative_to_its_length(n_freq, n_dir):
    gen = np.random.default_rng(100 * n_freq + n_dir)
    sizes = [33, 700, 1025, 2049]
    rel = np.zeros((sum(sizes), 4), np.float32)
    rel[:, :3] = gen.uniform(-1.2, 1.2, (len(rel), 3))
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    dirs = synth.icosphere(3) if n_dir == 642 else gen.normal(size=(n_dir, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)
    f = gen.uniform(1.0, 9.0, (1, n_freq)).astype(np.float32)
    T = gen.uniform(0.0, 0.6, (1, n_freq, n_dir)).astype(np.float32)
    q = gen.normal(size=(len(sizes), 4)).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    J, g = nat.ar_sf_score_grad(nat.Context(0), dev(rel), dev(off), dev(q),
                                torch.zeros(len(sizes), dtype=torch.int32, device="cuda"), dev(dirs), dev(f), dev(T))
    wide = lambda a: torch.from_numpy(a).double()  # noqa: E731
    for r in range(len(sizes)):
        ref, gref = exact(wide(q[r]), wide(rel[off[r]:off[r + 1], :3]), wide(dirs), wide(f[0]), wide(T[0]))
        bar = 1e-3 * float(gref.norm())
        assert bar < 0.05 * float(gref.abs().max())           # a wrong gradient cannot pass
        assert float((g[r].cpu().double() - gref).norm()) <= bar, sizes[r]
        assert abs(float(J[r]) - float(ref)) <= 1e-5 * float(ref)
