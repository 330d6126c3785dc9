"""The autotuner against the launch it replaces: a mixed batch, whose sample of a few
LPs per CU favours other launches than the whole batch does, and a batch of one
size.  Kernel times; a tuned solve may be a fifth slower at most, the rest being
noise between launches."""
import pytest

from paper_1802_08557_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("name", ["mixed", "uniform"])
def test_tuned_launch_is_no_slower(name, precision):
    import torch
    from paper_1802_08557_amd.lpbatch import Context, DeviceBatch
    bt = W.uneven_batch(6000, seed=5, lo=10, hi=250) if name == "mixed" else W.uniform_batch(3000, 117, 100, seed=6)
    dev = DeviceBatch.from_host(bt)
    best = {}
    for tuned in (False, True):
        ctx = Context(0)
        if tuned:
            ctx.solve(dev, precision=precision, autotune=True, sync=True)
            print(f"[gpu] {name} precision={precision} table {ctx.tuning()}", flush=True)
        for _ in range(5):
            ctx.solve(dev, precision=precision, time_kernels=True)
            torch.cuda.synchronize()
            ms = sum(t for k, t in ctx.kernel_times() if k in ("simplex_block_fp64", "simplex_block_fp32"))
            best[tuned] = min(best.get(tuned, ms), ms)
        ctx.close()
    print(f"[gpu] {name} precision={precision} untuned {best[False]:.3f} ms, tuned {best[True]:.3f} ms", flush=True)
    assert best[True] <= 1.2 * best[False]
