"""Closed-form box LP at the edges of its tiles (64 directions, chunks of at most
32 columns): the maximiser bit for bit, the value within the rounding bound of
an n-term sum, infinite and NaN bounds as the closed form gives them."""
import numpy as np
import pytest

from oracle import hyperbox_max
from paper_1802_08557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_08557_amd import lpbatch
    ctx = lpbatch.Context(0)
    yield torch, ctx
    ctx.close()


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("N,n", [(63, 1), (64, 2), (65, 31), (128, 32), (129, 33), (64, 64), (191, 65), (5, 97)])
def test_tile_edges(env, N, n, shared):
    torch, ctx = env
    print(f"[gpu] box N={N} n={n} shared={shared}", flush=True)
    lo, hi, l = W.hyperbox_batch(N, n, seed=7 * N + n)
    if shared:
        lo, hi = lo[0], hi[0]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    val, x = ctx.hyperbox_support(t(lo), t(hi), t(l), want_x=True)
    only, none = ctx.hyperbox_support(t(lo), t(hi), t(l))
    val, x, only = val.cpu().numpy(), x.cpu().numpy(), only.cpu().numpy()
    assert none is None
    want, h = hyperbox_max(lo if not shared else lo[None, :], hi if not shared else hi[None, :], l)
    np.testing.assert_array_equal(x, np.broadcast_to(h, x.shape))
    assert np.all(np.abs(val - want) <= 2 * n * np.finfo(np.float64).eps * np.sum(np.abs(l * h), axis=-1))
    np.testing.assert_array_equal(val, only)


def test_bounds_not_taken_do_not_count(env):
    torch, ctx = env
    N, n = 70, 20
    lo, hi, l = W.hyperbox_batch(N, n, seed=2)
    l = np.where(l == 0, 1.0, l)
    lo2, hi2 = np.where(l < 0, lo, np.nan), np.where(l < 0, np.inf, hi)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    a, _ = ctx.hyperbox_support(t(lo), t(hi), t(l))
    b, _ = ctx.hyperbox_support(t(lo2), t(hi2), t(l))
    np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
