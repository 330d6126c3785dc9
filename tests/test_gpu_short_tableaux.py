"""Tableaux of few rows.  The workgroup kernel updates one of at most twelve rows
pivot by pivot when it lies in LDS and through windows of pivots when it lies in
device memory: both against the oracle and bit for bit against each other, at the
edges of the rule, with surplus columns, artificials and both pricing rules."""
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


def solve(ctx, bt, **kw):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    print(f"[gpu] short {bt.name} N={bt.num_lps} {kw}", flush=True)
    s = ctx.solve(DeviceBatch.from_host(bt), stats=True, sync=True, **kw)
    return [v.cpu().numpy() for v in (s.status, s.obj, s.x, s.stats)]


@pytest.mark.parametrize("pricing", [0, 1])
@pytest.mark.parametrize("m,n", [(1, 65), (3, 100), (4, 511), (5, 64), (7, 129), (8, 65), (8, 300), (12, 65), (13, 65), (12, 129), (16, 100)])
def test_lds_and_memory_agree(ctx, m, n, pricing):
    for bt in (W.uniform_batch(9, m, n, seed=m + n), W.phase1_batch(9, m, n, seed=5 * m + n)):
        ref = oracle_solve(bt, pricing=pricing)
        first = None
        for kw in (dict(block_threads=64, placement=1), dict(placement=2), dict(block_threads=256), dict(),
                   dict(block_threads=512, placement=2)):
            st, obj, x, stats = solve(ctx, bt, pricing=pricing, **kw)
            assert_parity(bt, st, obj, x, ref)
            if first is None:
                first = (st, obj, x, stats)
            assert np.array_equal(st, first[0])
            assert np.array_equal(obj, first[1], equal_nan=True) and np.array_equal(x, first[2], equal_nan=True)
            assert np.array_equal(stats[:, :3], first[3][:, :3])
