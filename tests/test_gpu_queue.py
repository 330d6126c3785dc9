"""Work queues of the persistent launches: every LP solved exactly once for
batches around the queue's number of counters and the resident workgroups, and
the counters back at zero for the next call."""
import numpy as np
import pytest

from paper_1802_08557_amd import workloads as W
from helpers import assert_parity, oracle_solve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_08557_amd.lpbatch import Context
    c = Context(0)
    yield c
    c.close()


# 16 counters per queue; 8192 one-wavefront workgroups fill 256 CUs.
@pytest.mark.parametrize("num", [1, 15, 16, 17, 33, 8191, 8193, 20000])
def test_every_lp_once_and_counters_reset(ctx, num):
    import torch
    from paper_1802_08557_amd.lpbatch import DeviceBatch, Solution
    bt = W.uniform_batch(num, 6, 5, seed=num)
    ref = oracle_solve(bt)
    dev = DeviceBatch.from_host(bt)
    for precision in (0, 1, 0):
        print(f"[gpu] queue num={num} precision={precision}", flush=True)
        out = Solution(torch.full((num,), -7, dtype=torch.int32, device="cuda"),
                       torch.full((5 * num,), float("nan"), dtype=torch.float64, device="cuda"),
                       torch.full((num,), float("nan"), dtype=torch.float64, device="cuda"), None)
        s = ctx.solve(dev, precision=precision, out=out, sync=True)
        assert_parity(bt, s.status.cpu().numpy(), s.obj.cpu().numpy(), s.x.cpu().numpy(), ref)
        assert np.all(s.status.cpu().numpy() == 0)
