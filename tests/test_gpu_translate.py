"""devirt_translate at the sizes where its launch changes (a wavefront's round,
a workgroup, the larger workgroups and their grid) and where its table of
2 MiB blocks ends -- records and accessed/dirty bits against the oracle."""
import numpy as np
import pytest

from gpu_util import log, new_ctx
from oracle import Oracle
from workload import device, gen

GiB = 1 << 30


def _shifted(w, off):
    """The world with its guest-physical space moved up by `off` bytes."""
    for v in w.vms:
        v.slots["gpa"] += np.uint64(off)
        v.pt_data += np.where(v.pt_data & np.uint64(1), np.uint64(off), np.uint64(0))
        v.pt_gfn = v.pt_gfn + np.uint64(off >> 12)
    for p in w.procs:
        p.cr3 += off
    return w


def _addresses(rng, w, asid, n, lim):
    """Mapped addresses, page runs, and some anywhere; the last ones not canonical."""
    p = w.procs[asid]
    g = p.leaf_va[rng.integers(0, len(p.leaf_va), n)] + rng.integers(0, 4096, n, dtype=np.uint64)
    k = min(n, 64)
    g[:k] = p.leaf_va[0] + (np.arange(k, dtype=np.uint64) << np.uint64(12))
    far = rng.random(n) < 0.1
    g[far] = rng.integers(0, lim, int(far.sum()), dtype=np.uint64)
    if n > 8:
        g[-3:] = (lim - 1, lim, (1 << 64) - 1)
    return g


def _check(w, sizes, flags_of, seed):
    import torch
    import paper_1304_3771_amd as dv
    rng = np.random.default_rng(seed)
    ctx = new_ctx()
    try:
        dw = device.load(ctx, w)
        o = Oracle.from_workload(w)
        lim = {3: 1 << 32, 4: 1 << 47, 5: 1 << 56}[w.procs[0].levels]
        for n, flags in zip(sizes, flags_of):
            asid = int(rng.integers(0, len(w.procs)))
            g = _addresses(rng, w, asid, n, lim)
            out = torch.full((n * 24 + 24,), 0x5A, dtype=torch.uint8, device="cuda")
            ctx.translate(asid, torch.from_numpy(g.view(np.int64)).cuda(), n, flags, out)
            ctx.sync()
            x = out.cpu().numpy()
            assert np.all(x[n * 24:] == 0x5A), f"n {n}: written past the last record"
            x, e = x[:n * 24].view(dv.XLAT_DTYPE), o.translate(asid, g, flags)
            log(f"translate n {n} flags {flags}: codes {np.bincount(e['code'])}")
            bad = np.nonzero((x.view(np.uint8).reshape(-1, 24) != e.view(np.uint8).reshape(-1, 24)).any(axis=1))[0]
            assert not len(bad), f"n {n} flags {flags} address {int(bad[0])}: {hex(int(g[bad[0]]))} " \
                                 f"gpu {x[bad[0]]} oracle {e[bad[0]]}"
        for a, b in zip(device.read_arenas(ctx, dw), o.arenas):
            assert np.array_equal(a, b), "accessed/dirty bits differ"
    finally:
        ctx.close()


SIZES = (1, 63, 64, 65, 255, 257, 4097, 196608, 196609, 400000)


@pytest.mark.gpu
@pytest.mark.parametrize("levels,ept", [(3, False), (4, False), (5, False), (4, True), (5, True)])
def test_translate_sizes(levels, ept):
    sp = gen.spec("C1", mem_bytes=256 << 20, levels=levels, ept=ept, p_np=0.05, mix=(0.6, 0.4, 0.0), procs_per_vm=2,
                  p_readonly=0.05, p_supervisor=0.05, ept_np=0.02 * ept, ept_ro=0.02 * ept, ept_mis=0.02 * ept,
                  n_requests=0, seed=4200 + levels + 10 * ept)
    _check(gen.make_workload(sp, requests=False), SIZES, [i % 4 for i in range(len(SIZES))], levels)


@pytest.mark.gpu
@pytest.mark.parametrize("levels", [4, 5])
@pytest.mark.parametrize("off", [6 * GiB - (32 << 20), 9 * GiB, 1 << 42])
def test_translate_past_the_block_table(levels, off):
    """Guest-physical addresses across and beyond the last 2 MiB block held in LDS."""
    sp = gen.spec("C1", mem_bytes=64 << 20, levels=levels, p_np=0.05, mix=(0.6, 0.4, 0.0), n_slots=12, n_requests=0,
                  seed=4300 + levels)
    w = gen.make_workload(sp, requests=False)
    _check(_shifted(w, off), (5000, 5000, 300000), (0, 3, 1), levels)


@pytest.mark.gpu
def test_translate_one_gib_leaves():
    sp = gen.spec("C1", mem_bytes=5 * GiB, levels=5, p_np=0.0, mix=(0.1, 0.1, 0.8), mapped_frac=0.5, n_requests=0,
                  seed=4400)
    _check(gen.make_workload(sp, requests=False), (3000, 3000), (0, 3), 1)
