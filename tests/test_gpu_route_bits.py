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


@pytest.mark.gpu
@pytest.mark.parametrize("n,levels,vms",
                         [(1024, 4, 1), (1025, 5, 2), (2049, 3, 1), (3073, 4, 4), (4096, 4, 1), (4097, 5, 1)])
def test_small_batches_leave_the_same_bits(n, levels, vms):
    """A one-epoch batch, whose requests a wavefront (or a workgroup: the long ones) walks one by one up to 4,096,
    and the same batch walked in groups, as it is while the device counters are on."""
    import torch  # noqa: F401  (the HIP runtime that the library then shares)
    sp = gen.spec("C1", mem_bytes=256 * MiB, levels=levels, n_vms=vms, mix=(0.75, 0.25, 0.0), p_np=0.001, rho=0.5,
                  vmas_per_proc=4, n_requests=n, len_lo=24, len_hi=16384, seed=4900 + n)
    w = gen.make_workload(sp)
    rng = np.random.default_rng(n)
    r = w.requests.copy()
    # one epoch: the odd VMAs are written, each page by one request, the even ones read
    written = set()
    for i, (asid, gva, ln) in enumerate(zip(r["asid"].tolist(), r["gva"].tolist(), r["len"].tolist())):
        vma = next(k for k, (b, s) in enumerate(w.procs[asid].vmas.tolist()) if b <= gva < b + s)
        r["dir"][i] = vma & 1
        pages = {(asid, p) for p in range(gva >> 12, ((gva + max(ln, 1) - 1) >> 12) + 1)}
        if vma & 1 and pages & written:
            r["len"][i] = 0
        elif vma & 1:
            written |= pages
    big = np.flatnonzero((rng.random(n) < 0.04) & (r["dir"] == 0))[:150]  # up to 2.5 MiB
    for i in big:
        base, size = (int(x) for x in w.procs[int(r["asid"][i])].vmas[0])
        ln = int(rng.integers(60, 640)) * 4096
        r["gva"][i] = base + int(rng.integers(0, size - ln))
        r["len"][i] = ln
    r["host"] = np.concatenate([[0], np.cumsum(r["len"].astype(np.uint64))[:-1]])
    w.requests, w.epoch_end, w.pool_bytes = r, np.array([n], np.uint64), (int(r["len"].sum()) + 4095) & ~4095
    seen = []
    for counters in (False, True):
        ctx = new_ctx()
        try:
            dw = device.load(ctx, w)
            ctx.set_profiling(counters, counters=counters)
            res, faults, arenas, pool, _ = gpu_batch(w, ctx=ctx, dw=dw)
            seen.append((res, faults, pool, *arenas))
        finally:
            ctx.close()
    bad = [int((a.view(np.uint8) != b.view(np.uint8)).sum()) for a, b in zip(*seen)]
    log(f"{n} requests, {len(big)} long, {len(seen[0][1])} faults: bytes that differ {bad}")
    assert bad == [0] * len(bad)
