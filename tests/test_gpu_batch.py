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


def _run(ctx, dw, n, ends, faults=True, reps=1, stream=None):
    import torch
    import paper_1304_3771_amd as dv
    res = torch.zeros(max(n, 1) * 24, dtype=torch.uint8, device="cuda")
    fl = torch.full((max(n, 1) * 24,), 0x5A, dtype=torch.uint8, device="cuda") if faults else None
    nf = torch.full((1,), -1, dtype=torch.int64, device="cuda") if faults else None
    torch.cuda.synchronize()
    for _ in range(reps):
        ctx.submit_batch(dw.reqs, n, res, ends, fl, nf, stream=stream)
    ctx.sync(stream)
    k = int(nf.item()) if faults else 0
    if faults:
        assert bool((fl[k * 24:] == 0x5A).all()), "written past the fault list"
    return (res.cpu().numpy()[:n * 24].view(dv.RESULT_DTYPE),
            fl.cpu().numpy()[:k * 24].view(dv.FAULT_DTYPE) if faults else None)


@pytest.mark.gpu
@pytest.mark.parametrize("copy_wg", [64, 512, 1024])
def test_one_epoch_batches(copy_wg):
    """One-epoch batches of the sizes at the edges of the fault list's passes and of its limit, back to back on
    one stream (each clears the counters of the next), between a multi-epoch batch and per-request copies."""
    import torch  # noqa: F401
    sp = gen.spec("C1", mem_bytes=64 * MiB, n_requests=17000, len_lo=8, len_hi=200, p_np=0.3, rho=0.9, seed=4600)
    w = gen.make_workload(sp)
    assert len(w.epoch_end) == 1
    exp = oracle_batch(w)
    ctx = new_ctx(copy_wg=copy_wg)
    try:
        dw = device.load(ctx, w)
        for n in (1, 63, 64, 65, 511, 513, 1024, 8191, 8192, 8193, 16384, 16385, 17000, 256):
            r, f = _run(ctx, dw, n, None)
            e = exp[1][exp[1]["req_index"] < n]
            log(f"copy_wg {copy_wg}: {n} requests, {len(f)} faults")
            assert np.array_equal(r, exp[0][:n]) and np.array_equal(f, e), n
            if n == 65:  # other users of the stream's counters
                _run(ctx, dw, 4000, np.array([1000, 1000, 4000], np.uint64))
                q = dw.reqs_host[0]
                res = torch.zeros(24, dtype=torch.uint8, device="cuda")
                ctx.copy_from_guest(0, int(w.procs[0].vmas[0][0]), int(dw.pool.data_ptr()), 300000, res)
                del q
                dw.pool.copy_(torch.from_numpy(w.pool_image()))
            if n == 513:
                _run(ctx, dw, n, None, faults=False)
        got = (*_run(ctx, dw, 17000, None), device.read_arenas(ctx, dw), dw.pool.cpu().numpy())
        assert compare("one epoch", got, exp) == []
    finally:
        ctx.close()


@pytest.mark.gpu
def test_one_epoch_batch_under_capture():
    """A caller's own capture of a one-epoch batch, replayed between eager ones."""
    import torch
    sp = gen.spec("C1", mem_bytes=64 * MiB, n_requests=3000, len_lo=8, len_hi=400, p_np=0.2, rho=0.9, seed=4601)
    w = gen.make_workload(sp)
    exp = oracle_batch(w)
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        st = torch.cuda.Stream()
        n = dw.n
        import paper_1304_3771_amd as dv
        res = torch.zeros(n * 24, dtype=torch.uint8, device="cuda")
        fl = torch.zeros(n * 24, dtype=torch.uint8, device="cuda")
        nf = torch.zeros(1, dtype=torch.int64, device="cuda")
        torch.cuda.synchronize()
        ctx.submit_batch(dw.reqs, n, res, None, fl, nf, stream=st)  # sizes the workspace
        ctx.sync(st)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            ctx.submit_batch(dw.reqs, n, res, None, fl, nf, stream=st)
        for k in range(6):
            res.zero_(), fl.zero_(), nf.zero_()
            torch.cuda.synchronize()
            if k % 2:
                with torch.cuda.stream(st):
                    g.replay()
            else:
                ctx.submit_batch(dw.reqs, n, res, None, fl, nf, stream=st)
            ctx.sync(st)
            torch.cuda.synchronize()
            m = int(nf.item())
            got = (res.cpu().numpy().view(dv.RESULT_DTYPE), fl.cpu().numpy()[:m * 24].view(dv.FAULT_DTYPE),
                   device.read_arenas(ctx, dw), dw.pool.cpu().numpy())
            assert compare(f"capture, pass {k}", got, exp) == []
    finally:
        ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("levels,ept,cfg", [
    (4, False, {}), (3, False, {}), (5, False, {}), (4, True, {}),
    (4, False, dict(seg_chunks=4)), (5, False, dict(seg_chunks=64, inline_bytes=256)),
    (4, False, dict(xlat_wg=64)), (4, False, dict(xlat_wg=192, copy_wg=64)), (4, False, dict(tiny_queue=64)),
])
def test_one_request_per_wavefront(levels, ept, cfg, monkeypatch):
    """A one-epoch batch small enough for a wavefront a request: requests of one page to several rounds of a
    workgroup's wavefronts, every fault code, merged segments, lane copies, a queue that overflows."""
    import torch  # noqa: F401
    sp = gen.spec("C1", mem_bytes=256 * MiB, levels=levels, ept=ept, procs_per_vm=2, n_vms=2, n_requests=400, len_lo=16,
                  len_hi=3 * MiB, len_kind="loguniform", p_np=0.002, p_readonly=0.002, p_supervisor=0.002,
                  ept_np=0.002 * ept, ept_ro=0.002 * ept, ept_mis=0.002 * ept, mix=(0.7, 0.3, 0.0), rho=0.9,
                  seed=4700 + levels + 10 * ept)
    w = gen.make_workload(sp)
    w.requests["asid"][::97] = 99  # unknown processes
    w.requests["gva"][5::89] = np.uint64(1 << 63)  # not canonical
    w.requests["len"][7::101] = 0
    exp = oracle_batch(w)
    pages = (w.requests["len"] >> 12) + 1
    log(f"levels {levels} ept {ept} {cfg}: {len(w.epoch_end)} epochs, {int((pages > 128).sum())} requests of over 128 "
        f"pages, codes {np.bincount(exp[0]['code'])}")
    assert len(w.epoch_end) == 1 and (pages > 512).sum() > 5
    cfg = dict(cfg)
    if cfg.pop("tiny_queue", 0):
        monkeypatch.setenv("DEVIRT_SEG_CAP", "64")
    assert compare(f"{cfg}", gpu_batch(w, cfg=cfg, repeat=1), exp) == []
