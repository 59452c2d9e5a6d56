"""The routes that a copy can take leave the same accessed and dirty bits, with
2 MiB regions that start anywhere in a pass of 64 pages."""
import numpy as np
import pytest

from gpu_util import gpu_batch, log, new_ctx
from workload import device, gen

MiB = 1 << 20


@pytest.mark.gpu
@pytest.mark.parametrize("levels", [3, 4, 5])
def test_routes_leave_the_same_bits(levels):
    import torch
    import paper_1304_3771_amd as dv
    sp = gen.spec("C1", mem_bytes=256 * MiB, levels=levels, mix=(0.8, 0.2, 0.0), vmas_per_proc=2, n_requests=0,
                  seed=4700 + levels)
    w = gen.make_workload(sp, requests=False)
    # regions from the VMAs' ends downwards, so that no request shares its last region with another
    regions = [b + s - i * 4 * MiB for b, s in ((int(x), int(y)) for x, y in w.procs[0].vmas)
               for i in range(1, s // (4 * MiB) - 1)]
    regions = [(r + 2 * MiB - 1) & ~(2 * MiB - 1) for r in regions]
    rows, host = [], 0
    for i, k in enumerate((1, 29, 30, 31, 32, 62, 63, 64, 65, 94, 95, 127, 128)):
        for d in (0, 1):  # k pages before the last region's start, and one or three in it
            n = (k + 1 + 2 * d) * 4096 - 100
            rows.append((regions[2 * i + d] - k * 4096 + 50, host, n, 0, d, (0, 0, 0), 0))
            host += n
    w.requests = np.array(rows, gen.REQ_DTYPE)
    w.epoch_end = np.array([len(rows)], np.uint64)
    w.pool_bytes = (host + 4095) & ~4095
    seen = {}
    for name, cfg in (("plain", {}), ("batch", {}), ("fifo", dict(fifo_entries=10)), ("batch by group=1", dict(group=1))):
        ctx = new_ctx(**cfg)
        try:
            dw = device.load(ctx, w)
            res = torch.zeros(len(rows) * 24, dtype=torch.uint8, device="cuda")
            if "batch" in name:
                res = np.asarray(gpu_batch(w, ctx=ctx, dw=dw)[0]).view(dv.RESULT_DTYPE)
            else:
                for i, r in enumerate(dw.reqs_host):
                    f = ctx.copy_to_guest if r["dir"] else ctx.copy_from_guest
                    f(0, int(r["gva"]), int(r["host"]), int(r["len"]), res.data_ptr() + 24 * i)
                ctx.sync()
                res = res.cpu().numpy().view(dv.RESULT_DTYPE)
            seen[name] = (res, device.read_arenas(ctx, dw)[0], dw.pool.cpu().numpy())
        finally:
            ctx.close()
    for name, got in seen.items():
        bad = [int((a.view(np.uint8) != b.view(np.uint8)).sum()) for a, b in zip(got, seen["plain"])]
        log(f"levels {levels}, {name}: bytes that differ from the per-request copies' {bad}")
        assert bad == [0, 0, 0]
