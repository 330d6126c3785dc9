"""Deferred pivots.  The one-wavefront kernel: sizes at the edges of its 16 x 16
tiles and 64-row blocks, LPs of fewer and of many more pivots than one window
holds, one and two phases.  Status and objective against the oracle; status,
x, objective and pivot counts bit for bit against the workgroup kernel, whose
sweeps are organised differently.  The workgroup kernel: sizes at the edges of
its tiles, wavefronts and thread counts, windows from three pivots (an LP whose
vectors nearly fill LDS) to thirty-two, tableaux in LDS and in device memory,
against the oracle and bit for bit against each other."""
import numpy as np
import pytest

from paper_1802_08557_amd import workloads as W
from helpers import assert_parity, oracle_solve

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 64), (128, 1), (15, 17), (16, 16), (17, 15), (31, 48), (32, 49), (33, 33), (48, 20),
         (49, 64), (63, 47), (64, 64), (65, 16), (80, 32), (96, 33), (113, 48), (127, 40), (128, 64)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_08557_amd import lpbatch
    c = lpbatch.Context(0)
    yield c
    c.close()


def gaussian(N, m, n, seed):
    """A ~ N(0,1), b ~ U[1,100], c ~ U[-1,10], all <=: tens to hundreds of pivots."""
    rng = np.random.default_rng(seed)
    return W.Batch(rng.standard_normal(N * m * n), rng.uniform(1.0, 100.0, N * m), rng.uniform(-1.0, 10.0, N * n),
                   np.zeros(N * m, np.int8), np.full(N, m, np.int32), np.full(N, n, np.int32), f"gaussian_{m}x{n}")


def solve(ctx, bt, **kw):
    from paper_1802_08557_amd.lpbatch import DeviceBatch
    print(f"[gpu] window {bt.name} {kw}", flush=True)
    s = ctx.solve(DeviceBatch.from_host(bt), stats=True, sync=True, **kw)
    return [v.cpu().numpy() for v in (s.status, s.obj, s.x, s.stats)]


@pytest.mark.parametrize("pricing", [0, 1])
@pytest.mark.parametrize("m,n", SIZES)
def test_windows_match_workgroup_kernel(ctx, m, n, pricing):
    for bt in (gaussian(24, m, n, 100 * m + n), W.uniform_batch(12, m, n, seed=m + n),
               W.phase1_batch(12, m, n, seed=7 * m + n)):
        ref = oracle_solve(bt, pricing=pricing)
        st, obj, x, stats = solve(ctx, bt, pricing=pricing)
        assert_parity(bt, st, obj, x, ref)
        st2, obj2, x2, stats2 = solve(ctx, bt, pricing=pricing, block_threads=64)
        assert np.array_equal(st, st2)
        assert np.array_equal(obj, obj2, equal_nan=True) and np.array_equal(x, x2, equal_nan=True)
        assert np.array_equal(stats[:, :3], stats2[:, :3])
        if not bt.sense.any():
            assert np.all(stats[:, 6] == 1)
        st3, obj3, x3, _ = solve(ctx, bt, pricing=pricing, precision=1)
        assert_parity(bt, st3, obj3, x3, ref)


BLOCK_SIZES = [(1, 65), (130, 1), (15, 66), (65, 64), (129, 17), (97, 255), (256, 100), (128, 129), (257, 70)]


@pytest.mark.parametrize("m,n", BLOCK_SIZES)
def test_workgroup_windows(ctx, m, n):
    for bt in (gaussian(6, m, n, 10 * m + n), W.phase1_batch(6, m, n, seed=3 * m + n)):
        ref = oracle_solve(bt)
        first = None
        for kw in (dict(), dict(placement=2), dict(block_threads=64), dict(block_threads=128, placement=1),
                   dict(block_threads=512, placement=2), dict(block_threads=256)):
            st, obj, x, stats = solve(ctx, bt, **kw)
            assert_parity(bt, st, obj, x, ref)
            if first is None:
                first = (st, obj, x, stats)
            assert np.array_equal(st, first[0])
            assert np.array_equal(obj, first[1], equal_nan=True) and np.array_equal(x, first[2], equal_nan=True)
            assert np.array_equal(stats[:, :3], first[3][:, :3])
        st, obj, x, _ = solve(ctx, bt, precision=1)
        assert_parity(bt, st, obj, x, ref)


@pytest.mark.parametrize("precision", [0, 1])
def test_workgroup_window_of_three(ctx, precision):
    bt = W.uniform_batch(1, 1700, 1700, seed=5)
    ref = oracle_solve(bt)
    st, obj, x, stats = solve(ctx, bt, precision=precision)
    assert_parity(bt, st, obj, x, ref)
    assert np.all(stats[:, 6] == 2)
