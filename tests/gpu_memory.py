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
    rest = torch.cuda.mem_get_info()[0] - n
    assert rest >= 0, "the card has less free memory than the test wants to leave"
    hold = []
    while rest > 0:
        take = min(rest, 16 << 30)
        hold.append(torch.empty(take, dtype=torch.uint8, device="cuda"))
        rest -= take
    try:
        yield
    finally:
        hold.clear()
        torch.cuda.empty_cache()
