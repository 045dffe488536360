"""The window products on the matrix cores where they can go wrong: direction
counts that leave a pass partly empty, every histogram size of that form (and
4096 bins and a 33-bin span, which take the FFT), ROIs without atoms, around
the 64-atom slots and the 4096-atom stage, and bins that hold more counts than
one FP16 operand (many atoms on one lattice plane).  Against the FP64 oracle
with the image bar every image is held to."""
import numpy as np
import pytest
import torch

from parity_bars import assert_images

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nbins,n_dir", [(256, 33), (512, 17), (1024, 7), (2048, 2), (4096, 1)])
@pytest.mark.parametrize("windows", [[[1, 1]], [[16, 19], [18, 21], [26, 31], [30, 36]], [[5, 20], [21, 36]],
                                     [[4, 8], [30, 36]]])
def test_windows_match_the_oracle(orc, nbins, n_dir, windows):
    from paper_2009_00735_amd import native as nat
    gen = np.random.default_rng(nbins + n_dir)
    R = 1.0
    # balls of atoms far apart, and two ROIs of atoms crowded onto few planes
    sizes = [0, 1, 63, 64, 65, 700, 2500, 5000, 4500]
    centres = np.array([[5.0 * i, 0.0, 0.0] for i in range(len(sizes))], np.float32)
    pos = []
    for i, n in enumerate(sizes):
        p = gen.normal(size=(n, 3))
        p *= (0.95 * R * gen.random(n) ** (1 / 3) / np.maximum(np.linalg.norm(p, axis=1), 1e-9))[:, None]
        if i == 7:
            p[:] = [0.1, -0.2, 0.05]                       # one point: 5000 counts in one bin
        if i == 8:
            p = np.array([[0.3, 0.1, 0.0], [-0.2, 0.1, 0.4]])[gen.integers(0, 2, n)]
        pos.append((p + centres[i]).astype(np.float32))
    pos = np.concatenate(pos)
    d = gen.normal(size=(n_dir, 3))
    dirs = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    w = np.array(windows, np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    ctx = nat.Context(0)
    img, cnt = nat.araullo_signatures(ctx, dev(pos), dev(centres), R, dev(dirs), nbins, w)
    ref, rcnt = orc.signatures(pos, centres, R, dirs, nbins, w)
    assert np.array_equal(cnt.cpu().numpy(), rcnt) and list(rcnt) == sizes
    assert_images(img.cpu().numpy(), ref, rcnt[:, None, None], f"{nbins} bins, {n_dir} directions")
    # the batched plan and the gathered form write the same bits
    off, rel = nat.ar_roi_gather(ctx, dev(pos), dev(centres), R)
    assert torch.equal(nat.araullo_signatures_csr(ctx, rel, off, R, dev(dirs), nbins, w), img)
    plan = nat.SignaturePlan(ctx, len(sizes), len(rel), n_dir, nbins, len(w))
    for cap in (256, 4096):
        plan.set_config(min(3, n_dir), cap, 2)
        assert torch.equal(plan.run(rel, off, R, dev(dirs), w), img)


@pytest.mark.parametrize("nbins", [256, 1024, 2048])
def test_more_atoms_than_the_histograms_hold_at_once(orc, nbins):
    """ROIs past 65535 atoms go through the 16-bit halves in spans."""
    from paper_2009_00735_amd import native as nat
    gen = np.random.default_rng(nbins)
    ball = gen.normal(size=(70000, 3))
    ball *= (0.9 * gen.random(70000) ** (1 / 3) / np.linalg.norm(ball, axis=1))[:, None]
    point = np.tile([[7.1, 0.2, -0.3]], (130001, 1))
    pos = np.concatenate([ball, point]).astype(np.float32)
    centres = np.array([[0.0, 0.0, 0.0], [7.0, 0.0, 0.0]], np.float32)
    d = gen.normal(size=(5, 3))
    dirs = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    w = np.array([[16, 19], [18, 21], [26, 31], [30, 36]], np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    img, cnt = nat.araullo_signatures(nat.Context(0), dev(pos), dev(centres), 1.0, dev(dirs), nbins, w)
    ref, rcnt = orc.signatures(pos, centres, 1.0, dirs, nbins, w)
    assert cnt.cpu().tolist() == [70000, 130001] == list(rcnt)
    assert_images(img.cpu().numpy(), ref, rcnt[:, None, None])
