"""The trees' fold tiles at the end of the accepted range: a star of 2^31 - 1
nodes, whose last tiles' entry numbers pass the largest int.  Its numbers are
known: n - 1 descendants and height 1 at the root, 0 elsewhere.  About 85 GB of
device memory."""
import pytest
import torch

from gpu_util import say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu


def test_largest_star():
    n = (1 << 31) - 1
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GB of free device memory")
    child_ptr = torch.full((n + 1,), n - 1, dtype=torch.int32, device="cuda")
    child_ptr[0] = 0
    child = torch.arange(1, n, dtype=torch.int32, device="cuda")
    tree = wc.DeviceTree(n, child, child_ptr, child)  # the parents are not read in grid mode
    out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    own = wc.Context(0)  # its pool grows to some 50 GB and goes with it
    try:
        for call, root in ((own.tree_descendants, n - 1), (own.tree_height, 1)):
            say(f"largest star: {call.__name__}")
            call(tree, mode="grid", out=out)
            torch.cuda.synchronize()
            assert int(out[0]) == root
            assert not out[1:].any()
            out.fill_(-7)
    finally:
        own.close()
        del child_ptr, child, tree, out
        torch.cuda.empty_cache()
