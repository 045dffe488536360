"""Batches whose kernels need more work items than one grid holds (2^32; past it
a grid wraps around): every call still answers, each ROI as in a small batch."""
import numpy as np
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


def repeated(a, n):
    """The rows of a over and over, n of them."""
    return a.repeat((-(-n // len(a)), *[1] * (a.dim() - 1)))[:n].contiguous()


def assert_repeats(got, want):
    whole = len(got) // len(want) * len(want)
    assert bool((got[:whole].view(-1, *want.shape) == want).all())
    assert torch.equal(got[whole:], want[:len(got) - whole])


@pytest.mark.parametrize("n_roi", [2 ** 22 + 3, 2 ** 24 - 1, 2 ** 26 + 3])
def test_dense_indexing(n_roi):
    gen = torch.Generator(device="cuda").manual_seed(n_roi)
    ctx = nat.Context(0)
    refs = torch.rand((40, 1, 12), generator=gen, device="cuda")
    rois = torch.rand((61, 1, 12), generator=gen, device="cuda")
    lib = nat.Library(ctx, refs)
    want = nat.index_orientations(ctx, rois, lib, 2)
    got = nat.index_orientations(ctx, repeated(rois, n_roi), lib, 2)
    for g, w in zip(got, want):
        assert_repeats(g, w)


def test_many_references():
    n_lib = 2 ** 24 + 300
    gen = torch.Generator(device="cuda").manual_seed(5)
    refs = torch.rand((n_lib, 1, 12), generator=gen, device="cuda")
    rois = refs[-61:].clone()
    ctx = nat.Context(0)
    idx, score = nat.index_orientations(ctx, rois, nat.Library(ctx, refs), 1)
    assert idx[:, 0].tolist() == list(range(n_lib - 61, n_lib)) and not bool(score.any())


@pytest.mark.parametrize("n_lib,n_roi", [(50, 2 ** 22 + 3), (20000, 3355443)])   # ten chunks: 419431 groups
def test_sparse_indexing(n_lib, n_roi):
    gen = torch.Generator(device="cuda").manual_seed(1)
    ctx = nat.Context(0)
    dirs = torch.from_numpy(synth.icosphere(0)).cuda()
    quats = torch.randn((n_lib, 4), generator=gen, device="cuda", dtype=torch.float64)
    lut = nat.SparseLUT(ctx, torch.rand((1, 1, 12), generator=gen, device="cuda"), dirs, quats, [n_lib], 8)
    rois = torch.rand((61, 1, 12), generator=gen, device="cuda")
    want = nat.index_orientations_sparse(ctx, rois, lut, 2)
    got = nat.index_orientations_sparse(ctx, repeated(rois, n_roi), lut, 2)
    for g, w in zip(got, want):
        assert_repeats(g, w)


def test_sparse_table():
    n_lib = 2 ** 32 // 642 + 5
    gen = torch.Generator(device="cuda").manual_seed(6)
    dirs = torch.from_numpy(synth.icosphere(3)).cuda()
    ref = torch.rand((1, 1, len(dirs)), generator=gen, device="cuda")
    q = torch.randn((7, 4), generator=gen, device="cuda", dtype=torch.float64)
    ctx = nat.Context(0)
    want = nat.SparseLUT(ctx, ref, dirs, q, [7], len(dirs)).export()
    got = nat.SparseLUT(ctx, ref, dirs, repeated(q, n_lib), [n_lib], len(dirs)).export()
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert_repeats(got[2], want[2])


def test_roi_query():
    n_roi = 2 ** 26 + 5
    pos = torch.tensor([[0.1, 0.2, 0.0], [0.4, 0.0, 0.1], [5.0, 5.0, 5.0]], device="cuda")
    base = torch.tensor([[0.0, 0.0, 0.0], [9.0, 0.0, 0.0], [5.0, 5.1, 5.0]], device="cuda")
    ctx = nat.Context(0)
    want = nat.ar_roi_gather(ctx, pos, base, 1.0)
    off, rel = nat.ar_roi_gather(ctx, pos, repeated(base, n_roi), 1.0)[:2]
    assert_repeats(off[1:] - off[:-1], want[0][1:] - want[0][:-1])
    assert_repeats(rel, want[1])


def test_adaptive_grid():
    n_roi = 2 ** 24 + 3
    gen = torch.Generator(device="cuda").manual_seed(7)
    images = torch.rand((61, 1, 3), generator=gen, device="cuda")
    centres = torch.rand((61, 3), generator=gen, device="cuda")
    counts = torch.ones(n_roi, dtype=torch.int32, device="cuda")
    ctx = nat.Context(0)
    small = nat.ar_refine_roi_grid(ctx, centres, images, counts[:61], 1, 0.97, 0.5, 7)
    kept = len(small[0])
    assert 0 < kept <= 20 * 343
    out, parent = nat.ar_refine_roi_grid(ctx, repeated(centres, n_roi), repeated(images, n_roi), counts, 1, 0.97, 0.5, 7)
    assert_repeats(out, small[0])
    first = torch.arange(0, n_roi, 61, device="cuda", dtype=torch.int32)
    assert torch.equal(parent, (first[:, None] + small[1]).flatten()[:len(parent)])
    assert len(parent) >= n_roi // 61 * kept


@pytest.mark.parametrize("n_atoms,n_roi", [(0, 2 ** 22 + 1), (1, 2 ** 22), (1, 2 ** 24 + 5)])
def test_signatures_of_hardly_any_atoms(n_atoms, n_roi):
    gen = np.random.default_rng(n_atoms)
    dirs = gen.normal(size=(3, 3))
    dirs = torch.from_numpy((dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)).cuda()
    pos = torch.zeros((n_atoms, 3), device="cuda")
    base = torch.tensor([[0.1, 0.2, 0.0], [9.0, 0.0, 0.0], [0.0, -0.4, 0.3]], device="cuda")
    ctx = nat.Context(0)
    want = nat.araullo_signatures(ctx, pos, base, 1.0, dirs, 256, [[8, 12]])
    assert want[1].tolist() == [n_atoms, 0, n_atoms]
    got = nat.araullo_signatures(ctx, pos, repeated(base, n_roi), 1.0, dirs, 256, [[8, 12]])
    for g, w in zip(got, want):
        assert_repeats(g, w)


def test_structure_factors():
    n_roi = 2 ** 24 + 9
    gen = torch.Generator(device="cuda").manual_seed(3)
    dirs = torch.randn((3, 3), generator=gen, device="cuda")
    dirs = dirs / dirs.norm(dim=1, keepdim=True)
    rel = torch.rand((3, 4), generator=gen, device="cuda")
    off = torch.tensor([0, 2, 2], device="cuda") + 3 * torch.arange(-(-n_roi // 3), device="cuda")[:, None]
    off = torch.cat([off.flatten(), torch.tensor([3 * len(off)], device="cuda")])[:n_roi + 1].contiguous()
    rel = rel.repeat(-(-n_roi // 3), 1)
    q = torch.randn((3, 4), generator=gen, device="cuda")
    phase = torch.zeros(n_roi, dtype=torch.int32, device="cuda")
    f, T = torch.tensor([[4.0]], device="cuda"), torch.rand((1, 1, 3), generator=gen, device="cuda")
    ctx = nat.Context(0)

    def calls(n):
        a = (ctx, rel, off[:n + 1].contiguous(), repeated(q, n), phase[:n].contiguous(), dirs, f)
        s64 = nat.ar_sf_score_f64(*a[:3], a[3].double(), *a[4:6], f.double(), T.double())
        return *nat.ar_sf_score_grad(*a, T), nat.ar_sf_score_grad(*a, T, grad=False)[0], nat.ar_sf_amplitudes(*a), s64

    small, large = calls(3), calls(n_roi)
    for g, w in zip(large, small):
        assert_repeats(g, w)


def test_rotated_references():
    n_lib = 2 ** 32 // 10242 + 5
    gen = torch.Generator(device="cuda").manual_seed(4)
    dirs = torch.from_numpy(synth.icosphere(5)).cuda()
    ref = torch.rand((1, 1, len(dirs)), generator=gen, device="cuda")
    q = torch.randn((3, 4), generator=gen, device="cuda", dtype=torch.float64)
    ctx = nat.Context(0)
    phase = torch.zeros(n_lib, dtype=torch.int32, device="cuda")
    want = nat.ar_rotate_reference(ctx, ref, dirs, q, phase[:3].contiguous())
    assert_repeats(nat.ar_rotate_reference(ctx, ref, dirs, repeated(q, n_lib), phase), want)


def test_reciprocal_grids():
    """1920000 grids of L = 32 fill most of the card's memory (252 GB)."""
    n_roi, L = 1920000, 32
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < n_roi * L ** 3 * 4 + 2 ** 32:
        pytest.skip("needs 256 GB of free device memory")
    gen = torch.Generator(device="cuda").manual_seed(2)
    rows = [3, 0, 1, 2]
    rel = torch.rand((6, 4), generator=gen, device="cuda")
    first = torch.tensor([0, 3, 3, 4], device="cuda")
    off = (first + 6 * torch.arange(n_roi // 4, device="cuda")[:, None]).flatten()
    off = torch.cat([off, torch.tensor([6 * (n_roi // 4)], device="cuda")])
    ctx = nat.Context(0)
    want = nat.ar_fsp_amplitudes(ctx, rel, off[:5].contiguous(), L, 10.0)
    assert want[:, L // 2, L // 2, L // 2].tolist() == pytest.approx(rows)
    out = torch.empty((n_roi, L, L, L), device="cuda")
    out[:, 0, 0, 0] = out[:, -1, -1, -1] = -1.0
    nat.ar_fsp_amplitudes(ctx, rel.repeat(n_roi // 4, 1), off, L, 10.0, out=out)
    for part in out.view(-1, 4, L, L, L).split(4000):
        assert bool((part == want).all())
    del out, part
    torch.cuda.empty_cache()
