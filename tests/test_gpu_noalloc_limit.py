"""wc_spmv_noalloc at the end of what it takes: the largest matrix of the wave and
block modes whose documented workspace fits the fixed array (bit for bit as
wc_spmv), and the next one, which is refused."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_1606_08150_amd import wc

pytestmark = pytest.mark.gpu
CHUNKS = 1198199  # 64-entry chunks: 20 bytes for each of 2 CHUNKS + 1, 16 for each of CHUNKS + 1 rows, 9.25 KiB besides


@pytest.mark.parametrize("mode", ["wave", "block"])
def test_largest_accepted(ctx, mode):
    n, m = 700, 64 * CHUNKS + 63
    gen = torch.Generator(device="cuda").manual_seed(1)
    ptr = torch.linspace(0, m, n + 1, dtype=torch.float64, device="cuda").int()
    ptr[2:40] = ptr[40]  # one long row
    ptr[n] = m
    col = torch.randint(0, n, (m + 1,), dtype=torch.int32, device="cuda", generator=gen)
    val, x = torch.rand(m + 1, device="cuda", generator=gen), torch.rand(n, device="cuda", generator=gen)
    tune = wc.make_tune(items_per_lane=1)
    a = wc.DeviceCSR(n, ptr, col[:m])
    say(f"noalloc limit mode={mode} m={m}")
    y = wc.spmv_noalloc(a, val[:m], x, torch.empty(n, device="cuda"), mode=mode, tune=tune).cpu().numpy()
    ref = ctx.spmv(a, val[:m], x, mode=mode, tune=tune).cpu().numpy()
    assert np.array_equal(y.view(np.uint32), ref.view(np.uint32))
    ptr[n] = m + 1
    with pytest.raises(wc.WcError) as ei:
        wc.spmv_noalloc(wc.DeviceCSR(n, ptr, col), val, x, torch.empty(n, device="cuda"), mode=mode, tune=tune)
    assert ei.value.status == -1
