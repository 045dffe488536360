"""The sparse indexer's normalisation where its registers end (10240 nodes, 8
ROIs per group), each window's maximum in the first or the last nodes, and the
ranking of its candidates, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth
from test_gpu_sparse import build, check_index, dev, phases_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_dir, n_roi, k", [(9, 1, 4), (1025, 8, 16), (10239, 9, 16), (10240, 3, 1), (10241, 8, 32),
                                             (12000, 11, 16)])
def test_edges_of_the_registers(orc, n_dir, n_roi, k):
    gen = np.random.default_rng(n_dir)
    dirs = gen.normal(size=(n_dir, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)
    counts, n_hat = [40, 23], min(60, n_dir)
    ref = gen.gamma(2.0, 1.0, (2, 4, n_dir)).astype(np.float32)
    q = synth.library_orientations(sum(counts), 8)
    ctx = nat.Context(0)
    lut, si, sv, nodes = build(nat, ctx, ref, dirs, q, counts, n_hat)
    S = gen.gamma(2.0, 1.0, (n_roi, 4, n_dir)).astype(np.float32)
    S[:, 0, -1] = S[:, 1, 0] = 50.0   # the maxima: last node, first node, wherever they fall, none
    S[:, 3] = 0.0
    idx, score = nat.index_orientations_sparse(ctx, dev(S), lut, k)
    check_index(orc, S, si, sv, phases_of(counts), nodes, idx.cpu().numpy(), score.cpu().numpy(), k)
