"""Fills the card up to a given number of free bytes (for tests of what a
context does when its optional vectors do not fit)."""
import contextlib

from tests.gpu_util import torch_cuda


@contextlib.contextmanager
def free_bytes(n: int):
    """Within the block about n bytes of the card are free (untouched tensors
    hold the rest, 16 GiB apiece)."""
    torch = torch_cuda()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hold = []
    while (rest := torch.cuda.mem_get_info()[0] - n) > (4 << 20):
        hold.append(torch.empty(min(rest, 16 << 30), dtype=torch.uint8, device="cuda"))
    try:
        yield
    finally:
        hold.clear()
        torch.cuda.empty_cache()
