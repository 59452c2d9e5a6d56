"""Map batches by the order of their pages: ascending ones, which need no page
set, and ones that leave that order at the edges of a wavefront or workgroup;
lacking tables whose first map is invalid; many calls in a row, whose pools
share the staging buffer -- against the oracle."""
import numpy as np
import pytest

import pins
from gpu_util import log, new_ctx
from oracle import Oracle
from oracle.oracle import EPT_MAP_DTYPE, MAP_DTYPE
from test_gpu_map import _gpu_ept_map, _gpu_map, _same
from workload import device, gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


TOP = {3: 3 << 30, 4: 1 << 46, 5: 1 << 55}


def _pages(rng, n, kind):
    """Page numbers (from a region's base): runs that cross 2 MiB and, at times, 1 GiB."""
    run = np.cumsum(np.where(rng.random(n) < 0.02, rng.integers(1, 3000, n), 1))
    p = run.astype(np.uint64)
    if kind == "duplicate":  # neighbours at a workgroup's edge, and far apart
        if n > 256:
            p[256] = p[255]
        p[-1] = p[0]
    elif kind == "swapped" and n > 64:
        p[[63, 64]] = p[[64, 63]]
    elif kind == "shuffled":
        p = rng.permutation(np.concatenate([p[: n - n // 4], p[: n // 4]]))
    return p


@pytest.mark.parametrize("levels", [3, 4, 5])
@pytest.mark.parametrize("kind", ["ascending", "duplicate", "swapped", "shuffled", "invalid"])
def test_guest_map_order(levels, kind):
    sp = gen.spec("C1", mem_bytes=128 << 20, levels=levels, n_requests=0, seed=4800 + levels)
    w = gen.make_workload(sp, requests=False)
    rng = np.random.default_rng(levels)
    pool = pins.usable_frames(w, 0, pins.free_frames(w, 0, 6000, rng))
    o = Oracle.from_workload(w)
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        at = 0
        for k, n in enumerate((1, 64, 65, 257, 3000)):
            m = np.zeros(n, MAP_DTYPE)
            m["gva"] = np.uint64(TOP[levels] + k * (128 << 20)) + (_pages(rng, n, kind) << np.uint64(12))
            m["gpa"] = rng.integers(0, 1 << 15, n).astype(np.uint64) << np.uint64(12)
            m["flags"] = rng.integers(0, 2, n)
            if kind == "invalid":  # the map that would bring a table, and every fifth one
                first = np.nonzero(np.diff(m["gva"] >> np.uint64(21), prepend=0))[0]
                m["gva"][first[::2]] += np.uint64(8)
                m["gpa"][first[1::2]] = np.uint64(1 << 52)
                m["gpa"][::5] |= np.uint64(1)
            r, used = _gpu_map(ctx, 0, m, pool[at:])
            er, eused = o.map_pages(0, m, pool[at:])
            log(f"levels {levels} {kind}: {n} maps, {used} tables, {int((er['code'] == 0).sum())} succeed")
            _same(f"{kind} {n}", r, used, er, eused, device.read_arenas(ctx, dw), o.arenas)
            at += used
    finally:
        ctx.close()


@pytest.mark.parametrize("kind", ["ascending", "duplicate", "shuffled", "invalid"])
def test_ept_map_order(kind):
    sp = gen.spec("C1", mem_bytes=64 << 20, ept=True, n_requests=0, seed=4810)
    w = gen.make_workload(sp, requests=False)
    rng = np.random.default_rng(3)
    pool = pins.ept_map_batch(w, 0, 400, rng)[1]
    o = Oracle.from_workload(w)
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        at = 0
        for k, n in enumerate((1, 65, 300)):
            m = np.zeros(n, EPT_MAP_DTYPE)
            m["gpa"] = np.uint64((8 + k) << 30) + (_pages(rng, n, kind) << np.uint64(12))
            m["hpa"] = rng.integers(0, 1 << 14, n).astype(np.uint64) << np.uint64(12)
            m["flags"] = 3
            if kind == "invalid":
                m["flags"][::7] = 2  # write without read
                m["gpa"][::5] |= np.uint64(64)
            r, used = _gpu_ept_map(ctx, 0, m, pool[at:])
            er, eused = o.ept_map_pages(0, m, pool[at:])
            _same(f"EPT {kind} {n}", r, used, er, eused, device.read_arenas(ctx, dw), o.arenas)
            at += used
    finally:
        ctx.close()


def test_many_maps_share_the_staging():
    """Calls in a row without waiting, with pools of very different sizes (the staging buffer turns over and
    grows while earlier calls still read it)."""
    import torch
    import paper_1304_3771_amd as dv
    sp = gen.spec("C1", mem_bytes=256 << 20, n_requests=0, seed=4820)
    w = gen.make_workload(sp, requests=False)
    rng = np.random.default_rng(5)
    pool = pins.usable_frames(w, 0, pins.free_frames(w, 0, 24000, rng))
    o = Oracle.from_workload(w)
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        calls, at = [], 0
        for k in range(60):
            n = int(rng.integers(1, 6000)) if k % 7 == 0 else int(rng.integers(1, 80))
            m = np.zeros(n, MAP_DTYPE)
            m["gva"] = np.uint64((1 << 46) + (k << 31)) + (_pages(rng, n, "ascending") << np.uint64(12))
            m["gpa"] = rng.integers(0, 1 << 16, n).astype(np.uint64) << np.uint64(12)
            size = int(rng.integers(200, 4000)) if k != 40 else len(pool) - at
            size = min(max(size, n // 100 + 200), len(pool) - at)
            er, eused = o.map_pages(0, m, pool[at:at + size])
            dm = torch.from_numpy(m.view(np.uint8).reshape(-1).copy()).cuda()
            calls.append((m, pool[at:at + size].copy(), er, eused, dm, torch.zeros(n * 24, dtype=torch.uint8, device="cuda"),
                          torch.zeros(1, dtype=torch.int64, device="cuda")))
            at += eused
        torch.cuda.synchronize()
        for m, p, er, eused, dm, res, used in calls:
            ctx.map_pages(0, dm, len(m), p, res, used)
        torch.cuda.synchronize()
        for i, (m, p, er, eused, dm, res, used) in enumerate(calls):
            assert int(used.item()) == eused, (i, int(used.item()), eused)
            assert np.array_equal(res.cpu().numpy().view(dv.RESULT_DTYPE), er), i
        assert np.array_equal(device.read_arenas(ctx, dw)[0], o.arenas[0])
        log(f"{len(calls)} map calls, {at} tables")
    finally:
        ctx.close()
