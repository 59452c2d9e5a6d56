"""The per-request copy at the sizes where its launch changes: a request of one
page, around the longest one copied in one launch, around a wavefront's and a
workgroup's round of pages, and past it, with faults in between -- against the
oracle, every byte."""
import numpy as np
import pytest

from gpu_util import log, new_ctx
from oracle import Oracle
from workload import device, gen

PAGES = (1, 2, 16, 39, 40, 41, 64, 65, 1023, 1024, 1025, 2000)


def _world(levels, ept):
    sp = gen.spec("C1", mem_bytes=256 << 20, levels=levels, ept=ept, p_np=0.0007, mix=(0.8, 0.2, 0.0), vmas_per_proc=4,
                  n_requests=0, seed=4100 + levels + 10 * ept)
    return gen.make_workload(sp, requests=False)


@pytest.mark.gpu
@pytest.mark.parametrize("levels,ept", [(3, False), (4, False), (5, False), (4, True)])
def test_plain_copy_sizes(levels, ept):
    import torch
    import paper_1304_3771_amd as dv
    w = _world(levels, ept)
    rng = np.random.default_rng(levels)
    rows, host = [], 0
    for pages in PAGES:
        for d in (0, 1):
            for cut in (0, 1):  # whole pages; ragged first and last page
                base, size = (int(x) for x in w.procs[0].vmas[rng.integers(0, 4)])
                n = pages * 4096
                gva = base + int(rng.integers(0, (size - n) // 4096 + 1)) * 4096
                if cut:
                    gva += int(rng.integers(1, 2000))
                    n = max(1, n - int(rng.integers(2000, 4000)))
                rows.append((gva, host, n, 0, d, (0, 0, 0), 0))
                host += n + int(rng.integers(0, 64))
    w.requests = np.array(rows, gen.REQ_DTYPE)
    w.epoch_end = np.array([len(rows)], np.uint64)
    w.pool_bytes = (host + 4095) & ~4095
    o = Oracle.from_workload(w)
    er, _ = o.batch(w.requests)
    log(f"plain sizes: levels {levels} ept {ept}: {int((er['code'] != 0).sum())} of {len(rows)} requests fault")
    assert 0 < int((er["code"] != 0).sum()) < len(rows) // 2
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        res = torch.zeros(len(rows) * 24, dtype=torch.uint8, device="cuda")
        for i, r in enumerate(dw.reqs_host):
            f = ctx.copy_to_guest if r["dir"] else ctx.copy_from_guest
            f(0, int(r["gva"]), int(r["host"]), int(r["len"]), res.data_ptr() + 24 * i)
        ctx.sync()
        got = res.cpu().numpy().view(dv.RESULT_DTYPE)
        assert np.array_equal(got, er), next((i, got[i], er[i]) for i in range(len(rows)) if got[i] != er[i])
        assert np.array_equal(device.read_arenas(ctx, dw)[0], o.arenas[0])
        assert np.array_equal(dw.pool.cpu().numpy(), o.pool)
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["prot", "pae_prot", "ept_faults", "lvl5_1g", "multi_vm"])
def test_plain_copy_faults(name):
    """Every fault code, large leaves and several processes, one request at a time."""
    import torch
    import paper_1304_3771_amd as dv
    import pins
    w = gen.make_workload(pins.small_specs()[name])
    o = Oracle.from_workload(w)
    er, _ = o.batch(w.requests)
    log(f"plain {name}: {w.n_requests} requests, codes {sorted(set(er['code'].tolist()))}")
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        res = torch.zeros(dw.n * 24, dtype=torch.uint8, device="cuda")
        for i, r in enumerate(dw.reqs_host):
            f = ctx.copy_to_guest if r["dir"] else ctx.copy_from_guest
            f(int(r["asid"]), int(r["gva"]), int(r["host"]), int(r["len"]), res.data_ptr() + 24 * i)
        ctx.sync()
        assert np.array_equal(res.cpu().numpy().view(dv.RESULT_DTYPE), er)
        for a, b in zip(device.read_arenas(ctx, dw), o.arenas):
            assert np.array_equal(a, b)
        assert np.array_equal(dw.pool.cpu().numpy(), o.pool)
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("copy_wg", [64, 256, 1024])
def test_plain_copy_launch_shapes(copy_wg):
    """Around the longest copy that is launched in small workgroups (32 pages per CU), both ways."""
    import torch
    import paper_1304_3771_amd as dv
    sp = gen.spec("C1", mem_bytes=128 << 20, mix=(0.5, 0.5, 0.0), vmas_per_proc=1, p_np=0.0, n_requests=0, seed=4190)
    w = gen.make_workload(sp, requests=False)
    edge = 32 * torch.cuda.get_device_properties(0).multi_processor_count
    base, size = (int(x) for x in w.procs[0].vmas[0])
    rows, host = [], 0
    for pages in (41, edge, edge + 1):
        for d in (0, 1):
            assert pages * 4096 <= size
            rows.append((base + 17, host, pages * 4096 - 40, 0, d, (0, 0, 0), 0))
            host += pages * 4096
    w.requests = np.array(rows, gen.REQ_DTYPE)
    w.epoch_end = np.array([len(rows)], np.uint64)
    w.pool_bytes = host
    o = Oracle.from_workload(w)
    er, _ = o.batch(w.requests)
    ctx = new_ctx(copy_wg=copy_wg)
    try:
        dw = device.load(ctx, w)
        res = torch.zeros(len(rows) * 24, dtype=torch.uint8, device="cuda")
        for i, r in enumerate(dw.reqs_host):
            f = ctx.copy_to_guest if r["dir"] else ctx.copy_from_guest
            f(0, int(r["gva"]), int(r["host"]), int(r["len"]), res.data_ptr() + 24 * i)
        ctx.sync()
        assert np.array_equal(res.cpu().numpy().view(dv.RESULT_DTYPE), er)
        assert np.array_equal(device.read_arenas(ctx, dw)[0], o.arenas[0])
        assert np.array_equal(dw.pool.cpu().numpy(), o.pool)
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["ept", "ept_pae", "ept_lvl5", "ept_1g"])
def test_plain_copy_ept(name):
    """Behind an EPT, where a walk remembers its last level-2 table: tables and pages in one GiB and in two,
    1 GiB leaves, every depth."""
    test_plain_copy_faults(name)
