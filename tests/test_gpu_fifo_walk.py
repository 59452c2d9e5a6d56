"""The translation cache of the per-request path where a request's lookups are
more than a wavefront's, against the oracle's sequential FIFO and, every byte
and bit, against the walk by one wavefront (the one that counts)."""
import numpy as np
import pytest

from gpu_util import log, new_ctx
from oracle import Oracle
from workload import device, gen

PAGES = (1, 2, 5, 9, 10, 11, 17, 40, 41, 63, 64, 65, 130, 1023, 1024, 1025, 2000)


def _world(levels, ept, entries):
    sp = gen.spec("C1", mem_bytes=256 << 20, levels=levels, ept=ept, p_np=0.0007, mix=(0.8, 0.2, 0.0), vmas_per_proc=4,
                  n_requests=0, seed=4800 + levels + 10 * ept)
    w = gen.make_workload(sp, requests=False)
    rng = np.random.default_rng(100 * levels + entries)
    rows, host = [], 0
    for base, size in ((int(x), int(y)) for x, y in w.procs[0].vmas):
        at = int(rng.integers(100, size // 4096 - 2200))
        for _ in range(60):  # ranges that overlap the pages the ones before left in the cache
            n = int(rng.choice(PAGES[:11] if rng.random() < 0.8 else PAGES))
            first = at + int(rng.integers(-90, 90))
            ln = max(1, n * 4096 - int(rng.integers(0, 4096)))
            rows.append((base + first * 4096, host, ln, 0, int(rng.integers(0, 2)), (0, 0, 0), 0))
            host += ln
            if rng.random() < 0.7:
                at = max(100, min(size // 4096 - 2200, first + n))
    w.requests = np.array(rows, gen.REQ_DTYPE)
    w.epoch_end = np.array([len(rows)], np.uint64)
    w.pool_bytes = (host + 4095) & ~4095
    return w


@pytest.mark.gpu
@pytest.mark.parametrize("levels,ept,entries", [(3, False, 10), (4, False, 1), (4, False, 16), (5, False, 9),
                                                (4, True, 10)])
def test_cache_over_long_requests(levels, ept, entries):
    import torch
    import paper_1304_3771_amd as dv
    w = _world(levels, ept, entries)
    o = Oracle.from_workload(w)
    o.fifo_reset(entries)
    er, _ = o.batch(w.requests)
    seen = []
    for counters in (False, True):
        ctx = new_ctx(fifo_entries=entries)
        try:
            dw = device.load(ctx, w)
            ctx.set_profiling(counters, counters=counters)
            ctx.fifo_flush()
            res = torch.zeros(dw.n * 24, dtype=torch.uint8, device="cuda")
            steps = []
            for i, r in enumerate(dw.reqs_host):
                f = ctx.copy_to_guest if r["dir"] else ctx.copy_from_guest
                f(0, int(r["gva"]), int(r["host"]), int(r["len"]), res.data_ptr() + 24 * i)
                steps.append(ctx.fifo_counts(0))
            ctx.sync()
            assert np.array_equal(res.cpu().numpy().view(dv.RESULT_DTYPE), er)
            assert steps[-1] == o.fifo_counts(0)
            assert np.array_equal(dw.pool.cpu().numpy(), o.pool)
            seen.append((steps, device.read_arenas(ctx, dw)[0]))
        finally:
            ctx.close()
    log(f"levels {levels} ept {ept} entries {entries}: {dw.n} requests, {int((er['code'] != 0).sum())} faults, "
        f"(hits, misses) {seen[0][0][-1]}")
    assert seen[0][0] == seen[1][0]
    assert np.array_equal(seen[0][1], seen[1][1])
    assert entries == 1 or seen[0][0][-1][0] > 0  # one entry: the oracle, too, finds none held
