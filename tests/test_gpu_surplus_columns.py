"""The wavefront kernel with room for a surplus column in every row: all->= LPs at
the edge of its 64 columns take it in batches of one round and of many."""
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
    print(f"[gpu] surplus {bt.name} N={bt.num_lps} {kw}", flush=True)
    s = ctx.solve(DeviceBatch.from_host(bt), stats=True, sync=True, **kw)
    return [v.cpu().numpy() for v in (s.status, s.obj, s.x, s.stats)]


@pytest.mark.parametrize("N", [1, 40, 9000])
@pytest.mark.parametrize("m,n", [(1, 1), (1, 63), (32, 32), (63, 1), (40, 24), (40, 25)])
def test_every_row_with_a_surplus_column(ctx, m, n, N):
    rng = np.random.default_rng(m + 100 * n)
    # x >= lower limits and x <= upper limits by rows alone: minimise a positive cost.
    A = rng.uniform(1.0, 10.0, (N, m, n))
    b = rng.uniform(100.0, 1000.0, (N, m))
    bt = W.Batch(A.ravel(), b.ravel(), -rng.uniform(1.0, 10.0, N * n), np.ones(N * m, np.int8),
                 np.full(N, m, np.int32), np.full(N, n, np.int32), f"covering_{m}x{n}")
    st, obj, x, stats = solve(ctx, bt)
    assert np.all(st == 0)
    if m + n <= 64 and N <= 40:  # larger batches only where it costs no LPs in flight
        assert np.all(stats[:, 6] == 1)  # the wavefront kernel took every LP
    st2, obj2, x2, stats2 = solve(ctx, bt, block_threads=64)
    assert np.array_equal(st, st2) and np.array_equal(obj, obj2) and np.array_equal(x, x2)
    assert np.array_equal(stats[:, :3], stats2[:, :3])
    if N <= 40:
        assert_parity(bt, st, obj, x, oracle_solve(bt))
