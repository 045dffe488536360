"""Device memory that the ROI query keeps: two records of 16 bytes per atom in
either form of its sort, and the cell grid."""
import pytest
import torch

from paper_2009_00735_amd import native as nat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [200000, 6000000])
def test_workspace_per_atom(n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    pos = 40 * torch.rand((n, 3), generator=gen, device="cuda")
    centres = torch.tensor([[5.0, 5.0, 5.0], [35.0, 35.0, 35.0]], device="cuda")
    ctx = nat.Context(0)
    nat.ar_roi_gather(ctx, pos[:1000].contiguous(), centres, 2.0)   # the code is loaded, the grid allocated
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    off = torch.zeros(3, dtype=torch.int64, device="cuda")
    total = nat.ctypes.c_int64()
    nat._call("ar_roi_gather", ctx.handle, pos.data_ptr(), n, centres.data_ptr(), 2, 2.0, off.data_ptr(), None, 0,
              nat.ctypes.byref(total), torch.cuda.current_stream().cuda_stream)
    held = before - torch.cuda.mem_get_info()[0]
    # and 2 MB of page rounding for each of six buffers, 4 bytes of counts per 8 atoms
    assert held <= 32.5 * n + 6 * 2 ** 21, held / n
