"""LP_PLACE_LDS keeps a workgroup-kernel tableau in LDS whenever it fits beside the
kernel's least window of two pivots, however many LPs share the launch; by default
a tableau whose window would hold fewer than four goes to device memory.  FP64
sizes that leave room for two or three pivots in a CU's 160 KB."""
import numpy as np
import pytest

from paper_1802_08557_amd import workloads as W
from helpers import assert_parity, oracle_solve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_08557_amd import lpbatch
    c = lpbatch.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("m,n", [(80, 232), (290, 65), (20, 796)])
def test_lds_whenever_it_fits(ctx, m, n):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    bt = W.uniform_batch(300, m, n, seed=m + n)  # more LPs than CUs
    ref = oracle_solve(bt)
    for num in (300, 40):
        sub = bt.subset(range(num))
        dev = DeviceBatch.from_host(sub)
        got = []
        for placement, where in ((1, 3), (0, 2)):
            print(f"[gpu] placement {placement} {num} of {m}x{n}", flush=True)
            s = ctx.solve(dev, stats=True, sync=True, placement=placement)
            got.append([v.cpu().numpy() for v in (s.status, s.obj, s.x, s.stats)])
            assert np.all(got[-1][3][:, 6] == where)
        assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(got[0][:3], got[1][:3]))
        if num == 300:
            assert_parity(bt, *got[0][:3], ref)
