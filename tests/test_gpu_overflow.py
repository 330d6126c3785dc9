"""Tableau entries past the type's range.  A pivot whose column or row holds an
infinity must leave the row and column it replaces alone, wherever its update of
the other entries happens: LPs with entries of 1e-305 to 1e305 (single precision:
1e-44 to 1e44) through the one-wavefront kernel and through workgroup-kernel
windows in device memory, bit for bit as the workgroup kernel's pivot-by-pivot
update (tableaux of up to twelve rows in LDS).  (The plain method is no reference
for such LPs: a variable at -1e-55 is within its tolerances and moves a row with
an entry of 1e55.)"""
import numpy as np
import pytest

from paper_1802_08557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_08557_amd import lpbatch
    c = lpbatch.Context(0)
    yield c
    c.close()


def extreme(N, m, n, seed, span):
    """A third of the entries 10^+-[0.4 span, span], a fifth 0, the rest 0.1 to 10;
    right-hand sides down to 10^-span (the ratios then make pivot rows overflow);
    <=, >= and = rows."""
    rng = np.random.default_rng(seed)
    u = lambda *s: rng.uniform(0.0, 1.0, s)
    A = np.where(u(N, m, n) < 0.3, 10.0 ** (span * np.sign(u(N, m, n) - 0.5) * (0.4 + 0.6 * u(N, m, n))),
                 10.0 ** (2.0 * u(N, m, n) - 1.0))
    A = np.where(u(N, m, n) < 0.3, -A, A) * (u(N, m, n) >= 0.2)
    b = 10.0 ** (2.0 * u(N, m)) * np.where(u(N, m) < 0.3, 10.0 ** (-span * u(N, m)), 1.0)
    c = 10.0 * u(N, n) - 2.0
    sense = np.where(u(N, m) < 0.25, 1, np.where(u(N, m) < 0.1, 2, 0)).astype(np.int8)
    return W.Batch(A.reshape(-1), b.reshape(-1), c.reshape(-1), sense.reshape(-1), np.full(N, m, np.int32),
                   np.full(N, n, np.int32), f"extreme_{m}x{n}")


def solve(ctx, dev, **kw):
    print(f"[gpu] overflow {dev.num_lps} {kw}", flush=True)
    s = ctx.solve(dev, stats=True, sync=True, **kw)
    return [v.cpu().numpy() for v in (s.status, s.obj, s.x, s.stats)]


# Spans past the range of each tableau type (the single-precision solve's pivots
# are counted in the statistics whatever its FP64 certificate says).
@pytest.mark.parametrize("precision,span", [(0, 305.0), (1, 44.0)])
@pytest.mark.parametrize("m,n", [(8, 7), (12, 9)])
def test_windows_match_pivot_by_pivot(ctx, m, n, precision, span):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    dev = DeviceBatch.from_host(extreme(20000, m, n, m + n, span))
    st, obj, x, stats = solve(ctx, dev, precision=precision, block_threads=64, placement=1)
    assert precision or np.all(stats[:, 6] == 3)
    assert precision or np.isnan(obj[st == 0]).any()  # some right-hand sides did overflow
    for kw in (dict(), dict(block_threads=64, placement=2), dict(block_threads=256, placement=2)):
        st2, obj2, x2, stats2 = solve(ctx, dev, precision=precision, **kw)
        assert np.array_equal(stats[:, :3], stats2[:, :3]), np.flatnonzero((stats[:, :3] != stats2[:, :3]).any(1))[:5]
        if precision == 0:
            assert np.array_equal(st, st2)
            assert np.array_equal(obj, obj2, equal_nan=True) and np.array_equal(x, x2, equal_nan=True)


# Steepest edge: more rows than columns (the pivot column's owners past the last
# column take part in every sweep), weights and keys that overflow.
@pytest.mark.parametrize("m,n,N", [(8, 7, 20000), (12, 4, 20000), (60, 9, 4000), (100, 11, 2000)])
def test_steepest_edge_matches_workgroup_kernel(ctx, m, n, N):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    dev = DeviceBatch.from_host(extreme(N, m, n, m * n, 305.0))
    st, obj, x, stats = solve(ctx, dev, pricing=1, block_threads=64)
    for kw in (dict(), dict(block_threads=256, placement=2)):
        st2, obj2, x2, stats2 = solve(ctx, dev, pricing=1, **kw)
        assert np.array_equal(st, st2), np.flatnonzero(st != st2)[:5]
        assert np.array_equal(obj, obj2, equal_nan=True) and np.array_equal(x, x2, equal_nan=True)
        assert np.array_equal(stats[:, :3], stats2[:, :3])
