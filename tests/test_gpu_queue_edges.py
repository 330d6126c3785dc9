"""Launches around one round of resident workgroups: a launch with a worker for every
LP uses no queue and no prefetch, one LP more brings both in.  The wavefront kernels
hold one to eight workgroups per SIMD, so every multiple of 1,024 up to 8,192 (256 CUs
of four SIMDs) and its neighbours are tried: every LP solved, twice on one
context, in both precisions."""
import numpy as np
import pytest

from paper_1802_08557_amd import workloads as W
from helpers import assert_parity, oracle_solve

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1802_08557_amd.lpbatch import Context, DeviceBatch
    c = Context(0)
    bt = W.uniform_batch(8193, 6, 5, seed=11)
    yield c, bt, oracle_solve(bt), DeviceBatch.from_host(bt)
    c.close()


@pytest.mark.parametrize("num", [k * 1024 + d for k in range(1, 9) for d in (-1, 0, 1)])
def test_every_lp_once(env, num):
    import torch
    from paper_1802_08557_amd.lpbatch import DeviceBatch, Solution
    ctx, bt, ref, dev = env
    part = DeviceBatch(dev.A[:num * 30], dev.b[:num * 6], dev.c[:num * 5], dev.sense[:num * 6], dev.m[:num], dev.n[:num])
    lps = W.Batch(bt.A[:num * 30], bt.b[:num * 6], bt.c[:num * 5], bt.sense[:num * 6], bt.m[:num], bt.n[:num], "part")
    for precision in (0, 1, 0, 1):
        print(f"[gpu] queue edges num={num} precision={precision}", flush=True)
        out = Solution(torch.full((num,), -7, dtype=torch.int32, device="cuda"),
                       torch.full((5 * num,), float("nan"), dtype=torch.float64, device="cuda"),
                       torch.full((num,), float("nan"), dtype=torch.float64, device="cuda"), None)
        s = ctx.solve(part, precision=precision, out=out, sync=True)
        assert_parity(lps, s.status.cpu().numpy(), s.obj.cpu().numpy(), s.x.cpu().numpy(), ref, idx=np.arange(num))
