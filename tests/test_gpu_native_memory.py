"""A call whose output cannot be allocated: the allocator's own error, and nothing held afterwards."""
import gc
import sys

import pytest

from paper_2207_10741_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("given", [True, False])
def test_a_failed_allocation_holds_no_workspace(given):
    """An output of 2 TB, refused by the allocator's own limit; the workspace given, or one that was kept (rows of 2^20 channels: the
    sizes that decide about a workspace stay small)."""
    torch = G.torch_mod()
    small = B.conv_desc(1, 8, 8, 8, 8, in_dtype=B.BF16)
    huge = B.conv_desc(1, 1024, 1024, 8, 1 << 20, in_dtype=B.BF16)
    x = torch.zeros((1, 8, 8, 8), dtype=torch.bfloat16, device=G.dev())
    w = torch.zeros((8, 3, 3, 8), dtype=torch.bfloat16, device=G.dev())
    mask = torch.ones((1, 8, 8), dtype=torch.uint8, device=G.dev())
    need = B.workspace_bytes(huge)
    assert need <= B._WORKSPACE_MOST
    ws = torch.empty((need,), dtype=torch.uint8, device=G.dev()) if given else None
    if not given:
        B.focused_conv2d(small, x, w, mask_in=mask)                 # (the extension is bound, a workspace kept)
        key = (B._current_raw_stream(), x.device.index)
        ws = B._kept.__dict__[key] = torch.empty((need,), dtype=torch.uint8, device=G.dev())
    held = sys.getrefcount(ws)
    torch.cuda.set_per_process_memory_fraction(0.5)
    try:
        for _ in range(3):
            with pytest.raises(torch.cuda.OutOfMemoryError):
                B.focused_conv2d(huge, x, w, mask_in=mask, workspace=ws if given else None)
            gc.collect()
            assert sys.getrefcount(ws) == held
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        B._kept.__dict__.clear()
    out = B.focused_conv2d(small, x, w, mask_in=mask)
    torch.cuda.synchronize()
    assert not out.any()
