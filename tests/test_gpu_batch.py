"""The batched path at the sizes where its launches change, against the oracle."""
import numpy as np
import pytest

from gpu_util import compare, gpu_batch, log, new_ctx, oracle_batch
from workload import device, gen

MiB = 1 << 20


@pytest.mark.gpu
@pytest.mark.parametrize("group,n", [(1, 5000), (3, 20000), (64, 100000)])
def test_groups_beyond_the_first_ones(group, n):
    """More groups than wavefronts, so that most are claimed from the parts' cursors: every request is
    translated once.  A second pass finds every accessed/dirty bit set and issues no atomic."""
    import torch  # noqa: F401  (the HIP runtime that the library then shares)
    sp = gen.spec("C1", mem_bytes=128 * MiB, n_requests=n, len_lo=8, len_hi=600, p_np=0.05, mix=(0.7, 0.3, 0.0),
                  seed=4500 + group)
    w = gen.make_workload(sp)
    ctx = new_ctx(group=group)
    try:
        dw = device.load(ctx, w)
        got = gpu_batch(w, ctx=ctx, dw=dw)
        assert compare(f"group {group}", got, oracle_batch(w)) == []
        ctx.set_profiling(True, counters=True)
        ctx.reset_stats()
        st = gpu_batch(w, ctx=ctx, dw=dw)[4]["stats"]
        log(f"group {group}: {n} requests, {st['pages_walked']} pages, {st['ad_atomics']} atomics in a second pass")
        assert st["pages_walked"] > 0.9 * n and st["ad_atomics"] == 0
    finally:
        ctx.close()
