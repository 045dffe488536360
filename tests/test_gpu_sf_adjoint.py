"""The structure-factor gradient's matrix-core sums where they can go wrong:
atom counts around the 32-atom step and the 1024-atom stage (and none), last
tiles and groups of directions that are partly past the list, every class of
frequency count, and coordinates whose FP16 parts need the scale.

Reference: the score and its gradient in FP64 by torch.autograd.  Bars: J
relative 1e-5 (the bar of the score).  Gradient: every sum C, S, P, Q carries
at most 1e-5 of its N terms' size (phases of up to 20 turns rounded at 2^-24,
sine and cosine, FP32 accumulation), a term of dJ/dR is at most
2 |e| 2 pi f X 2 in size (X the largest coordinate) and dR/dq at most 4, so
4 * 4e-5 of the sum of those sizes bounds it."""
import math

import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


def score64(q, x, dirs, f, T):
    w, a, b, c = (q / q.norm()).unbind()
    M = torch.stack([1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                     2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                     2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)]).reshape(3, 3)
    t = 2 * math.pi * (dirs @ M.T) @ x.T
    J = torch.zeros((), dtype=torch.float64)
    size = 0.0
    for i in range(len(f)):
        C, S = torch.cos(f[i] * t).sum(1), torch.sin(f[i] * t).sum(1)
        e = torch.sqrt(C * C + S * S) / len(x) - T[i]
        J = J + (e * e).sum()
        size += float((2 * e.abs()).sum()) * 2 * math.pi * float(f[i].abs()) * 2 * float(x.abs().max())
    return J, size


@pytest.mark.parametrize("n_dir", [18, 100, 300, 642])
@pytest.mark.parametrize("n_freq,scale", [(1, 1.0), (4, 1.0), (4, 3e-4), (4, 5e5), (7, 1.0), (8, 1.0)])
def test_gradient_matches_float64(n_dir, n_freq, scale):
    gen = np.random.default_rng(1000 * n_dir + 10 * n_freq)
    sizes = [0, 1, 31, 32, 33, 700, 1023, 1025, 2049]
    xs = [(gen.uniform(-1.2, 1.2, (n, 3)) * scale).astype(np.float32) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rel = np.zeros((int(off[-1]), 4), np.float32)
    rel[:, :3] = np.concatenate(xs)
    rel[:, 3] = 7.0                                   # never read
    dirs = synth.icosphere(3) if n_dir == 642 else gen.normal(size=(n_dir, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)
    f = (gen.uniform(1.0, 9.0, (2, n_freq)) / scale).astype(np.float32)
    T = gen.uniform(0.0, 0.6, (2, n_freq, n_dir)).astype(np.float32)
    q = gen.normal(size=(len(sizes), 4)).astype(np.float32)
    ph = (np.arange(len(sizes)) % 2).astype(np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    J, g = nat.ar_sf_score_grad(nat.Context(0), dev(rel), dev(off), dev(q), dev(ph), dev(dirs), dev(f), dev(T))
    J, g = J.double().cpu(), g.double().cpu()
    for r, x in enumerate(xs):
        t64 = torch.from_numpy(T[ph[r]]).double()
        if not len(x):
            assert abs(float(J[r]) - float((t64 * t64).sum())) <= 1e-5 * float((t64 * t64).sum())
            assert float(g[r].abs().max()) == 0.0
            continue
        q64 = torch.from_numpy(q[r]).double().requires_grad_(True)
        ref, size = score64(q64, torch.from_numpy(x).double(), torch.from_numpy(dirs).double(),
                            torch.from_numpy(f[ph[r]]).double(), t64)
        ref.backward()
        assert abs(float(J[r]) - float(ref)) <= 1e-5 * float(ref), (sizes[r], float(J[r]), float(ref))
        bar = 4 * 4e-5 * size / float(q64.detach().norm())
        assert float((g[r] - q64.grad).abs().max()) <= bar, (sizes[r], g[r], q64.grad, bar)
