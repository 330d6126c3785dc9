"""FP64 certificate of batches of mixed sizes (256 threads per LP): LU blocks that
fit LDS and ones in device memory, all statuses, against the oracle; and the
same LPs one at a time (64 threads per LP; at most 64 rows or columns would go to
the one-wavefront certificate instead), bit for bit."""
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


@pytest.mark.parametrize("lo,hi", [(60, 70), (100, 140), (240, 300)])
def test_mixed_sizes(ctx, lo, hi):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    bt = W.uneven_batch(40, seed=lo + hi, lo=lo, hi=hi, frac_infeasible=0.2, frac_unbounded=0.1)
    print(f"[gpu] certificate mixed {lo}..{hi}", flush=True)
    ref = oracle_solve(bt)
    s = ctx.solve(DeviceBatch.from_host(bt), precision=1, stats=True, sync=True)
    st, obj, x, stats = [v.cpu().numpy() for v in (s.status, s.obj, s.x, s.stats)]
    assert_parity(bt, st, obj, x, ref)
    assert set(np.unique(st)) >= {0, 1, 2}
    coff = bt.offsets()[2]
    big = [k for k in range(40) if min(bt.m[k], bt.n[k]) > 64][:8]
    assert big
    for k in big:
        one = bt.subset([k])
        r = ctx.solve(DeviceBatch.from_host(one), precision=1, stats=True, sync=True)
        assert int(r.status[0]) == st[k] and int(r.stats[0, 5]) == stats[k, 5]
        np.testing.assert_array_equal(r.x.cpu().numpy(), x[coff[k]:coff[k + 1]])
        np.testing.assert_array_equal(r.obj.cpu().numpy(), obj[k:k + 1])
