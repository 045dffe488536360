"""Plans, libraries and look-up tables closed after their context: garbage
collection may take a cycle's objects in any order."""
import pytest
import torch

from paper_2009_00735_amd import native as nat
from paper_2009_00735_amd import synth

pytestmark = pytest.mark.gpu


def _plan(ctx, dirs, ref, quats):
    return nat.SignaturePlan(ctx, 2, 300, len(dirs), 256, 2)


def _library(ctx, dirs, ref, quats):
    return nat.Library(ctx, ref)


def _lut(ctx, dirs, ref, quats):
    return nat.SparseLUT(ctx, ref[:1], dirs, quats, [len(quats)], 8)


@pytest.mark.parametrize("make", [_plan, _library, _lut])
def test_closed_after_its_context(make):
    gen = torch.Generator(device="cuda").manual_seed(3)
    dirs = torch.from_numpy(synth.icosphere(1)).cuda()
    ref = torch.rand((40, 2, len(dirs)), generator=gen, device="cuda")
    quats = torch.nn.functional.normalize(torch.randn((40, 4), generator=gen, device="cuda", dtype=torch.float64))
    other = nat.Context(0)
    rel = torch.rand((50, 4), generator=gen, device="cuda") - 0.5
    off = torch.tensor([0, 50], device="cuda")
    want = nat.araullo_signatures_csr(other, rel, off, 1.0, dirs, 256, [[8, 10]])
    for _ in range(4):
        ctx = nat.Context(0)
        obj = make(ctx, dirs, ref, quats)
        ctx.close()
        held = [bytearray(b"\xff" * 4096) for _ in range(64)]   # what the context held is written over
        obj.close()
        # a device set from the freed context would be reported by the next launch
        got = nat.araullo_signatures_csr(other, rel, off, 1.0, dirs, 256, [[8, 10]])
        assert torch.equal(got, want) and len(held) == 64
