"""FP64 certificate with 64 and with 256 threads per LP: the choice follows the LPs per
CU and the bound on the LU block, for batches of one size and of mixed sizes, and
must not show in the results.  A batch of more than two LPs per CU against its first
LPs alone, bit for bit, and against the oracle."""
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


# Sizes on both sides of the lines at blocks of 96 and 128, LPs on both sides of two and
# four to a CU (256 of them).
@pytest.mark.parametrize("lo,hi,num", [(66, 76, 700), (90, 100, 700), (90, 100, 1100), (120, 132, 1100), (80, 80, 700)])
def test_threads_do_not_show(ctx, lo, hi, num):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    bt = W.uniform_batch(num, lo, lo, seed=lo) if lo == hi else W.uneven_batch(num, seed=lo + num, lo=lo, hi=hi)
    print(f"[gpu] certificate {num} of {lo}..{hi}", flush=True)
    solve = lambda b: [v.cpu().numpy() for v in (lambda s: (s.status, s.obj, s.x, s.stats))(
        ctx.solve(DeviceBatch.from_host(b), precision=1, stats=True, sync=True))]
    st, obj, x, stats = solve(bt)
    assert_parity(bt, st, obj, x, oracle_solve(bt))
    first = bt.subset(range(60))
    st1, obj1, x1, stats1 = solve(first)
    assert np.array_equal(st1, st[:60]) and np.array_equal(stats1[:, 5], stats[:60, 5])
    assert np.array_equal(obj1, obj[:60], equal_nan=True)
    assert np.array_equal(x1, x[:len(x1)], equal_nan=True)
