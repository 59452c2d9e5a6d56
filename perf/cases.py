"""Work that a user of this library has it do, as cases that can be timed.

A case names one call (or one burst of calls) of the data path on a synthetic
guest: a per-request copy, a translation of many addresses, a batched
submission, a map batch, or a burst through the serving loop.  `prepare`
builds what such a program holds before the call -- a context with its VMs,
memslots or EPTs, processes with real page tables, host buffers, descriptors
-- from a seed; `run` makes the call; its outputs are everything the call
writes: result records, fault lists, host buffers and guest memory (which
holds the accessed/dirty bits and the tables that map batches write).

Guests follow the repository's workload recipe: memslots cut at random page
boundaries and laid out in the arena in a random order behind guard gaps, VMAs
of 2 MiB units that are one 2 MiB leaf or 512 4 KiB leaves on randomly placed
frames, a share of leaves not present.  Each process has VMAs whose buffers
are only read by the device and VMAs that are only written, with host buffers
split the same way, so a pass repeated on one state gives the same outputs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1304_3771_amd as dv

PAGE, MiB, GiB = 4096, 1 << 20, 1 << 30
UNIT = 2 * MiB
U = np.uint64
USER_LIMIT = {3: 1 << 32, 4: 1 << 47, 5: 1 << 56}


# ------------------------------------------------------------------- cases
def listed():
    return [
        # a 64-bit input event delivered into a guest's read() buffer: the smallest operation there is
        dict(name="copy_event_24B", kind="copy", to_guest=True, bytes=24, levels=4, ept=False, fifo=0, static=False),
        # a GPU command buffer fetched from the guest (an ioctl submit): an odd size, unaligned on both sides
        dict(name="copy_cmdbuf_100KB", kind="copy", to_guest=False, bytes=100001, levels=4, ept=False, fifo=0,
             static=False),
        # a 1920x1080 YUYV camera frame delivered into the guest
        dict(name="copy_frame_4MB", kind="copy", to_guest=True, bytes=4147200, levels=4, ept=False, fifo=0,
             static=False),
        # the pages of one buffer list translated for writing, with accessed/dirty bits
        dict(name="translate_1k_write", kind="translate", n=1000, run=16, write=True, set_ad=True, levels=4,
             ept=False, mem_mib=1024),
        # translation as a service: millions of scattered addresses, a tenth of them anywhere in the user range
        dict(name="translate_4M_read", kind="translate", n=4 * MiB, run=1, write=False, set_ad=False, levels=4,
             ept=False, mem_mib=4096),
        # the same for a guest behind an EPT (two software walks), page runs, with accessed/dirty bits
        dict(name="translate_1M_ept", kind="translate", n=1000003, run=16, write=True, set_ad=True, levels=4,
             ept=True, mem_mib=4096),
        # one small guest's operations of a moment: a batch that is all latency
        dict(name="batch_256_small", kind="batch", n=256, lo=8, hi=4096, vms=1, procs=1, mem_mib=64, levels=4,
             ept=False, share_2m=0.0, p_np=0.10, reuse=False),
        # an ordinary batch of a guest under the 32-bit PAE tables: a few thousand requests
        dict(name="batch_8k_pae", kind="batch", n=8191, lo=64, hi=65536, vms=1, procs=1, mem_mib=2048, levels=3,
             ept=False, share_2m=0.3, p_np=0.05, reuse=False),
        # the repository's headline workload: one 4 GiB guest, a million requests of 64 B - 64 KiB
        dict(name="batch_1M_64KiB", kind="batch", n=1000000, lo=64, hi=65536, vms=1, procs=1, mem_mib=4096,
             levels=4, ept=False, share_2m=0.3, p_np=0.05, reuse=False),
        # many VMs with 5-level paging and buffers up to 1 MiB, host buffers reused from epoch to epoch
        dict(name="batch_fleet_5level", kind="batch", n=400000, lo=16, hi=1 << 20, vms=16, procs=2, mem_mib=1024,
             levels=5, ept=False, share_2m=0.35, p_np=0.03, reuse=True),
        # a driver's mmap: a large fresh region whose tables are all new
        dict(name="map_128k_fresh", kind="map", n=131072, fresh=True, ept=False, levels=4),
        # serving: a burst of operations of many guest threads (input events, audio periods, command buffers,
        # camera frames) through the serving loop, waited for
        dict(name="serve_burst_2k", kind="serve", n=2048, vms=4, mem_mib=2048, levels=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["copy", "copy", "translate", "translate", "batch", "batch", "batch", "map", "serve"])
    levels, ept = rng.choice([3, 4, 4, 5]), rng.random() < 0.25
    if kind == "copy":
        return dict(kind=kind, to_guest=rng.random() < 0.5, bytes=_log(rng, 16, 8 << 20), levels=levels, ept=ept,
                    fifo=rng.choice([0, 0, 10]), static=rng.random() < 0.25)
    if kind == "translate":
        write = rng.random() < 0.5
        return dict(kind=kind, n=_log(rng, 64, 8 << 20), run=rng.choice([1, 4, 16, 256]), write=write,
                    set_ad=write and rng.random() < 0.7, levels=levels, ept=ept,
                    mem_mib=rng.choice([256, 1024, 2048]))
    if kind == "batch":
        hi = rng.choice([4096, 65536, 1 << 20])
        vms = rng.choice([1, 1, 4, 16])
        n = _log(rng, 32, {4096: 1000000, 65536: 600000, 1 << 20: 120000}[hi])
        return dict(kind=kind, n=n, lo=rng.choice([8, 64]), hi=hi, vms=vms, procs=rng.choice([1, 2, 4]),
                    mem_mib=rng.choice([512, 1024]), levels=levels, ept=ept, share_2m=rng.choice([0.0, 0.2, 0.35]),
                    p_np=rng.choice([0.0, 0.03, 0.05, 0.10]), reuse=vms > 1)
    if kind == "map":
        return dict(kind=kind, n=_log(rng, 1, 1 << (16 if levels == 3 else 18)), fresh=rng.random() < 0.5,
                    ept=rng.random() < 0.4, levels=levels)
    return dict(kind=kind, n=_log(rng, 16, 4096), vms=4, mem_mib=2048, levels=rng.choice([4, 5]))


# ------------------------------------------------------------------- guests
class Guest:
    """A context, closed when the last tensor over its guest memory is gone."""

    def __init__(self):
        self.ctx = dv.Context(0)
        self.server = None

    def __del__(self):
        if self.server is not None:
            self.server.stop()
        self.ctx.close()


class _Arena:
    """Guest memory as an array on the device; keeps its guest open."""

    def __init__(self, guest, vm):
        ptr, nbytes = guest.ctx.vm_arena(vm)
        self.guest = guest
        self.__cuda_array_interface__ = dict(shape=(nbytes // 8,), typestr="<i8", data=(ptr, False), version=2)


def _arena(guest, vm):
    return torch.as_tensor(_Arena(guest, vm), device="cuda:0")


def _u64(rng, n):
    return rng.integers(0, 1 << 63, n, dtype=U) << U(1) | rng.integers(0, 2, n, dtype=U)


class VM:
    """One VM: memory, GPA layout, processes; `vmas[p]` = [(base, bytes)] of process p."""

    def __init__(self, guest, rng, gen, mem, levels, ept, procs, share_2m, p_np, n_slots=16, n_vmas=4, spare=0):
        ctx = guest.ctx
        self.mem, self.levels, nfr, nblk = mem, levels, mem // PAGE, mem // UNIT
        # GPA -> arena: memslots in a random order behind guard gaps, or an EPT over shuffled 2 MiB blocks
        # (one in sixteen mapped by 4 KiB leaves)
        if ept:
            self.block = rng.permutation(nblk).astype(U)
            small = np.sort(rng.choice(nblk, max(1, nblk // 16), replace=False))
            n_pd = -(-mem // GiB)
            n_tab = 2 + n_pd + len(small)
            size = mem + n_tab * PAGE
        else:
            cuts = np.sort(rng.choice(np.arange(1, nfr), n_slots - 1, replace=False))
            lo = np.concatenate([[0], cuts]).astype(np.int64)
            cnt = np.diff(np.concatenate([lo, [nfr]]))
            order = rng.permutation(n_slots)
            gap = rng.integers(0, 17, n_slots)
            self.slot_lo, self.slot_off = lo, np.zeros(n_slots, np.int64)
            self.slot_off[order] = np.cumsum(gap) + np.concatenate([[0], np.cumsum(cnt[order])[:-1]])
            size = (nfr + 16 * n_slots) * PAGE
        self.vm = ctx.vm_create(size)
        self.memory = _arena(guest, self.vm)
        self.memory.random_(generator=gen)
        frames = self.memory.view(-1, 512)
        if ept:
            tab = np.zeros((n_tab, 512), U)
            base = U(mem)
            tab[0, 0] = base + U(PAGE) | U(7)
            tab[1, :n_pd] = base + U(PAGE) * (U(2) + np.arange(n_pd, dtype=U)) | U(7)
            leaf = (self.block * U(UNIT)) | U(0x80 | 6 << 3 | 7)
            pt = base + U(PAGE) * (U(2 + n_pd) + np.arange(len(small), dtype=U))
            tab[2 + n_pd:] = (self.block[small][:, None] * U(UNIT) + np.arange(512, dtype=U) * U(PAGE)) | U(6 << 3 | 7)
            leaf[small] = pt | U(7)
            tab[2:2 + n_pd].reshape(-1)[:nblk] = leaf
            frames[mem // PAGE:mem // PAGE + n_tab] = torch.from_numpy(tab.view(np.int64)).cuda()
            ctx.vm_set_ept(self.vm, mem)
            self.ept = True
        else:
            for i in range(n_slots):
                ctx.memslot_set(self.vm, i, int(lo[i]) * PAGE, int(cnt[i]) * PAGE, int(self.slot_off[i]) * PAGE)
            self.ept = False
        # guest frames: half of memory is mapped; 2 MiB leaves take whole blocks, 4 KiB leaves and tables the rest
        units = max(n_vmas, int(0.5 * nblk) // procs)
        two = [np.sort(rng.choice(units, int(round(share_2m * units)), replace=False)) for _ in range(procs)]
        blocks = rng.permutation(nblk)
        n2 = sum(len(t) for t in two)
        rest = (blocks[n2:, None] * 512 + np.arange(512)).reshape(-1)
        rest = rest[rng.permutation(len(rest))].astype(U)
        self.procs, self.cr3s, self.vmas = [], [], []
        tabs, gfns = [], []
        k2 = k4 = 0
        for p in range(procs):
            vmas = self._vmas(rng, units, n_vmas)
            va = np.concatenate([U(b) + np.arange(n // UNIT, dtype=U) * U(UNIT) for b, n in vmas])
            is2 = np.zeros(units, bool)
            is2[two[p]] = True
            va4 = (va[~is2][:, None] + np.arange(512, dtype=U) * U(PAGE)).reshape(-1)
            va2 = va[is2]
            fr4, k4 = rest[k4:k4 + len(va4)], k4 + len(va4)
            fr2, k2 = blocks[k2:k2 + len(va2)].astype(U) * U(512), k2 + len(va2)
            ids = {lv: np.unique((va4 if lv == 1 else va) >> U(12 + 9 * lv)) for lv in range(1, levels + 1)}
            ids[levels] = np.zeros(1, U)
            gfn = {}
            for lv in ids:
                gfn[lv], k4 = rest[k4:k4 + len(ids[lv])], k4 + len(ids[lv])
            data = {lv: np.zeros((len(ids[lv]), 512), U) for lv in ids}
            slot = int(rng.integers(0, 128)) * 4 if levels == 3 else 0  # a PAE root table is 4 entries
            ign = U(0x0E00) | U(0 if levels == 3 else 0x7FF0000000000000)
            for lv in range(2, levels + 1):
                child = ids[lv - 1]
                root = levels == 3 and lv == 3
                e = gfn[lv - 1] << U(12) | U(1 if root else 7) | _u64(rng, len(child)) & (U(0x0E00) if root else ign)
                at = (child & U(511)).astype(np.int64) + (slot if root else 0)
                data[lv][np.searchsorted(ids[lv], child >> U(9)) if lv < levels else 0, at] = e
            for lv, v, f, ps in ((1, va4, fr4, 0), (2, va2, fr2, 0x80)):
                e = f << U(12) | U(7 | ps) | _u64(rng, len(v)) & ign
                e = np.where(rng.random(len(v)) < p_np, _u64(rng, len(v)) & ~U(1), e)
                at = ((v >> U(12 + 9 * (lv - 1))) & U(511)).astype(np.int64)
                data[lv][np.searchsorted(ids[lv], v >> U(12 + 9 * lv)), at] = e
            for lv in ids:
                tabs.append(data[lv])
                gfns.append(gfn[lv])
            cr3 = (int(gfn[levels][0]) << 12) + 8 * slot
            self.procs.append(ctx.process_create(self.vm, cr3, levels))
            self.cr3s.append(cr3)
            self.vmas.append(vmas)
        self.spare = np.sort(rest[k4:k4 + spare]) << U(12)  # free guest frames, ascending
        at = self.arena_offset(np.concatenate(gfns) << U(12)) >> U(12)
        frames[torch.from_numpy(at.view(np.int64)).cuda()] = \
            torch.from_numpy(np.concatenate(tabs).view(np.int64)).cuda()

    def _vmas(self, rng, units, n):
        cnt = np.full(n, units // n)
        cnt[:units % n] += 1
        if self.levels == 3:
            gap = (3 * GiB - 4 * MiB) // UNIT - units
            cut = np.sort(rng.integers(0, gap + 1, n))
            base = 4 * MiB + (cut + np.concatenate([[0], np.cumsum(cnt)[:-1]])) * UNIT
        else:
            cell = -(-int(cnt.max()) * UNIT // GiB) + 1
            base = GiB + rng.choice((USER_LIMIT[self.levels] // 4) // (cell * GiB), n, replace=False) * cell * GiB
        return [(int(b), int(c) * UNIT) for b, c in zip(base, cnt)]

    def arena_offset(self, gpa):
        if self.ept:
            return self.block[(gpa // U(UNIT)).astype(np.int64)] * U(UNIT) + gpa % U(UNIT)
        fr = (gpa >> U(12)).astype(np.int64)
        i = np.searchsorted(self.slot_lo, fr, side="right") - 1
        return ((fr - self.slot_lo[i] + self.slot_off[i]).astype(U) << U(12)) + (gpa & U(0xFFF))


def _rngs(seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    return np.random.default_rng(seed), gen


def _bytes(gen, n):
    t = torch.empty((n + 7) // 8, dtype=torch.int64, device="cuda:0")
    t.random_(generator=gen)
    return t


def _records(n, words):
    return torch.zeros((n, words), dtype=torch.int64, device="cuda:0")


def _upload(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1).view(np.int64)).cuda()


# ------------------------------------------------------------------ requests
def _lengths(rng, lo, hi, n):
    return np.minimum(hi, np.floor(lo * (hi / lo) ** rng.random(n))).astype(np.int64)


def _place(rng, region, size, base, length, rho):
    """Epochs and guest addresses of requests in `region`s (VMAs) of `size`
    bytes at `base`: in each epoch a region's requests lie one after another
    at random gaps and fill at most a `rho` share of it.  Returns (order,
    epoch ends, gva in that order)."""
    n = len(region)
    total = np.bincount(region, length, len(size))
    ne = max(1, int(np.ceil((total / (rho * size)).max())))
    by = np.argsort(region, kind="stable")
    cum = np.cumsum(length[by])
    first = np.searchsorted(region[by], np.arange(len(size)))
    before = np.concatenate([[0], cum])[first]
    epoch = np.zeros(n, np.int64)
    epoch[by] = np.minimum(ne - 1, (cum - length[by] - before[region[by]]) * ne // np.maximum(1, total[region[by]])
                           .astype(np.int64))
    order = np.argsort(epoch, kind="stable")
    region, length, epoch = region[order], length[order], epoch[order]
    g = epoch * len(size) + region
    by = np.argsort(g, kind="stable")
    gs, ls = g[by], length[by]
    start = np.concatenate([[0], np.nonzero(np.diff(gs))[0] + 1])
    of = np.repeat(np.arange(len(start)), np.diff(np.concatenate([start, [n]])))
    cum = np.cumsum(ls) - ls
    cum -= cum[start][of]
    free = size[region[by]] - np.add.reduceat(ls, start)[of]
    u = rng.random(n)
    u = u[np.lexsort((u, g))]
    gva = np.zeros(n, U)
    gva[by] = (base[region[by]] + (u * (free + 1)).astype(np.int64).clip(0, free) + cum).astype(U)
    return order, np.cumsum(np.bincount(epoch, minlength=ne)).astype(U), gva


def _room(n, mix):
    """Bytes that the host buffers of one side of n requests fit in, whatever the seed: eight standard deviations
    above the mean.  mix: (share of the requests, shortest, longest), lengths log-uniform."""
    lo, hi = (np.array([m[k] for m in mix], float) for k in (1, 2))
    share, ln = np.array([m[0] for m in mix]), np.log(np.maximum(hi / lo, 1 + 1e-9))
    mean = n * float((share * (hi - lo + 1e-9 * lo) / ln).sum())
    var = n * float((share * (hi ** 2 - lo ** 2 + 2e-9 * lo ** 2) / (2 * ln)).sum())
    return int(mean + 8 * math.sqrt(var) + hi.max()) + 64 * n


def _requests(rng, gen, vms, length, to_guest, rho, reuse, room):
    """Descriptors over the VMs' processes: (records, epoch ends, read pool, written pool).  room: bytes of the
    host buffers into the guest and out of it."""
    n = len(length)
    asid = np.array([a for v in vms for a in v.procs])
    vmas = np.array([x for v in vms for x in v.vmas], np.int64)  # (process, VMA, (base, bytes))
    proc = rng.integers(0, len(asid), n)
    half = vmas.shape[1] // 2  # the first VMAs are written by the device, the others read
    region = proc * 2 * half + np.where(to_guest, 0, half) + rng.integers(0, half, n)
    flat = vmas.reshape(-1, 2)
    length = np.maximum(1, np.minimum(length, flat[region, 1] // 4))
    order, ends, gva = _place(rng, region, flat[:, 1], flat[:, 0], length, rho)
    length, to_guest, proc = length[order], to_guest[order], proc[order]
    span = length + rng.integers(0, 64, n)
    host, pools = np.zeros(n, U), []
    for side, size in ((True, room[0]), (False, room[1])):
        at = np.nonzero(to_guest == side)[0]
        cum = np.cumsum(span[at])
        if reuse and len(at):  # every epoch starts at the pool's first byte again
            e = np.searchsorted(ends, at, side="right")
            new = np.concatenate([[0], np.nonzero(np.diff(e))[0] + 1])
            cum -= np.repeat(cum[new] - span[at][new], np.diff(np.concatenate([new, [len(at)]])))
        if reuse:  # an epoch places at most a rho share of the VMAs, and one request more in each
            k = len(asid) * half
            size = min(size, int(rho * flat[:, 1].sum()) // 2 + k * int(flat[:, 1].max() // 4) + 64 * n)
        pool = _bytes(gen, size)
        assert cum.max(initial=0) <= size
        host[at] = U(pool.data_ptr()) + (cum - length[at]).astype(U)
        pools.append(pool)
    r = np.zeros(n, dv.REQUEST_DTYPE)
    r["gva"], r["host"], r["len"], r["asid"], r["dir"] = gva, host, length, asid[proc], to_guest
    return r, ends, pools[0], pools[1]


# ------------------------------------------------------------------- prepare
def prepare(case, seed):
    rng, gen = _rngs(seed)
    g = Guest()
    make = {"copy": _prepare_copy, "translate": _prepare_translate, "batch": _prepare_batch, "map": _prepare_map,
            "serve": _prepare_serve}[case["kind"]]
    return dict(case=case, guest=g, **make(case, g, rng, gen))


def _prepare_copy(c, g, rng, gen):
    v = VM(g, rng, gen, 256 * MiB, c["levels"], c["ept"], 1, 0.3, 0.0)
    g.ctx.set_config(fifo_entries=c["fifo"])
    base, size = v.vmas[0][int(rng.integers(0, 4))]
    n = c["bytes"]
    buf = _bytes(gen, n + 64)
    return dict(vm=v, asid=v.procs[0], gva=base + int(rng.integers(0, size - n + 1)), buf=buf,
                host=buf.data_ptr() + int(rng.integers(0, 64)), res=_records(1, 3))


def _prepare_translate(c, g, rng, gen):
    v = VM(g, rng, gen, c["mem_mib"] * MiB, c["levels"], c["ept"], 1, 0.3, 0.05)
    n, run = c["n"], c["run"]
    vma = np.array(v.vmas[0], np.int64)
    k = -(-n // run)
    pick = rng.integers(0, 4, k)
    page = vma[pick, 0] // PAGE + (rng.random(k) * (vma[pick, 1] // PAGE - run)).astype(np.int64)
    gva = ((page[:, None] + np.arange(run)).reshape(-1)[:n].astype(U) << U(12)) + rng.integers(0, PAGE, n, dtype=U)
    if run == 1:  # a tenth anywhere in the user range
        at = rng.random(n) < 0.1
        gva[at] = rng.integers(0, USER_LIMIT[c["levels"]], int(at.sum()), dtype=U)
    flags = (dv.XLAT_WRITE if c["write"] else 0) | (dv.XLAT_SET_AD if c["set_ad"] else 0)
    return dict(vm=v, asid=v.procs[0], gvas=_upload(gva), flags=flags, out=_records(n, 3))


def _vms(c, g, rng, gen, procs, share_2m, p_np):
    return [VM(g, rng, gen, c["mem_mib"] * MiB, c["levels"], c.get("ept", False), procs, share_2m, p_np,
               n_slots=16 if c["vms"] == 1 else 8) for _ in range(c["vms"])]


def _prepare_batch(c, g, rng, gen):
    vms = _vms(c, g, rng, gen, c["procs"], c["share_2m"], c["p_np"])
    n = c["n"]
    room = _room(n, [(0.5, c["lo"], c["hi"])])
    r, ends, src, dst = _requests(rng, gen, vms, _lengths(rng, c["lo"], c["hi"], n), rng.random(n) < 0.5, 0.5,
                                  c["reuse"], (room, room))
    return dict(vms=vms, reqs=_upload(r), ends=ends, src=src, dst=dst, res=_records(n, 3), faults=_records(n, 3),
                n_faults=_records(1, 1))


def _prepare_map(c, g, rng, gen):
    n = c["n"]
    v = VM(g, rng, gen, 512 * MiB, c["levels"], c["ept"], 1, 0.3 if c["fresh"] else 0.0, 0.0, spare=n // 128 + 4096)
    if c["ept"]:  # the EPT half: guest-physical pages of the VM put on arena pages
        if c["fresh"]:
            page = GiB // PAGE + np.sort(rng.choice(max(2 * n, 512), n, replace=False))
        else:  # pages behind 4 KiB EPT leaves only (a 2 MiB leaf is never split)
            sm = np.nonzero(_ept_small(v))[0]
            page = np.sort((sm[:, None] * 512 + np.arange(512)).reshape(-1)[rng.integers(0, len(sm) * 512, n)])
        m = np.zeros(n, dv.EPT_MAP_DTYPE)
        m["gpa"] = page.astype(U) * U(PAGE)
        m["hpa"] = rng.integers(0, v.mem // PAGE, n).astype(U) * U(PAGE)
        m["flags"] = dv.EPT_R | dv.EPT_W
        pool = v.arena_offset(v.spare)
        # the EPT's level-3 entries that fresh regions hang off
        clear = v.memory[(v.mem + PAGE) // 8 + 1:(v.mem + PAGE) // 8 + 9] if c["fresh"] else None
        return dict(vm=v, maps=_upload(m), pool=pool, res=_records(n, 3), used=_records(1, 1), clear=clear)
    top = {3: 3 * GiB, 4: USER_LIMIT[4] // 2, 5: USER_LIMIT[5] // 2}[c["levels"]]
    if c["fresh"]:  # runs of 16 - 4096 pages at 2 MiB-aligned addresses, under one entry of the root table
        runs, left = [], n
        while left:
            runs.append(min(left, _lengths(rng, 16, 4096, 1)[0]))
            left -= runs[-1]
        cnt = -(-np.array(runs) // 512)
        room = (GiB if c["levels"] == 3 else 64 * GiB) // UNIT - int(cnt.sum())
        gap = np.sort(rng.integers(0, max(1, room), len(runs)))
        base = top + (gap + np.cumsum(cnt) - cnt) * UNIT
        gva = np.concatenate([U(b) + np.arange(k, dtype=U) * U(PAGE) for b, k in zip(base, runs)])
        shift = {3: 30, 4: 39, 5: 48}[c["levels"]]
        at = int(v.arena_offset(np.array([v.cr3s[0]], U))[0]) // 8 + ((top >> shift) & (3 if c["levels"] == 3 else 511))
        clear = v.memory[at:at + 1]
    else:
        vma = np.array(v.vmas[0], np.int64)
        pick = rng.integers(0, 4, n)
        gva = (vma[pick, 0] + rng.integers(0, vma[pick, 1] // PAGE) * PAGE).astype(U)
        clear = None
    m = np.zeros(n, dv.MAP_DTYPE)
    m["gva"], m["gpa"] = gva, rng.integers(0, v.mem // PAGE, n).astype(U) * U(PAGE)
    m["flags"] = dv.MAP_WRITE if c["fresh"] else rng.integers(0, 2, n)
    return dict(vm=v, asid=v.procs[0], maps=_upload(m), pool=v.spare, res=_records(n, 3), used=_records(1, 1),
                clear=clear)


def _ept_small(v):
    """Which 2 MiB blocks of the VM's memory lie behind 4 KiB EPT leaves."""
    pd = v.memory[(v.mem + 2 * PAGE) // 8:][:v.mem // UNIT].cpu().numpy()
    return pd & 0x80 == 0


SERVE_CLASSES = ((0.60, 24, 24, True), (0.25, 4096, 4096, False), (0.14, 16384, 262144, False),
                 (0.01, 4147200, 4147200, True))  # share, bytes from, to, into the guest


def _prepare_serve(c, g, rng, gen):
    vms = _vms(c, g, rng, gen, 4, 0.3, 0.0)
    n = c["n"]
    cls = rng.choice(4, n, p=[s[0] for s in SERVE_CLASSES])
    lo, hi, to = (np.array(x) for x in list(zip(*SERVE_CLASSES))[1:])
    length = np.floor(lo[cls] * (hi[cls] / lo[cls]) ** rng.random(n)).astype(np.int64)
    room = [_room(n, [s[:3] for s in SERVE_CLASSES if s[3] == side]) for side in (True, False)]
    r, ends, src, dst = _requests(rng, gen, vms, length, to[cls], 0.9, False, room)
    r["tag"] = np.arange(n)  # a guest thread each
    g.server = g.ctx.server_start(max_inflight=8192, pool_bytes=4 * GiB, max_batch=4096, streams=3)
    return dict(vms=vms, reqs=r, src=src, dst=dst)


# ----------------------------------------------------------------------- run
def run(state):
    return RUN[state["case"]["kind"]](state, state["guest"].ctx)


def _run_copy(s, ctx):
    c = s["case"]
    if c["static"]:
        ctx.copy_static(s["asid"], s["gva"], s["host"], c["bytes"], dv.TO_GUEST if c["to_guest"] else dv.FROM_GUEST,
                        s["res"])
    elif c["to_guest"]:
        ctx.copy_to_guest(s["asid"], s["gva"], s["host"], c["bytes"], s["res"])
    else:
        ctx.copy_from_guest(s["asid"], s["gva"], s["host"], c["bytes"], s["res"])
    return dict(res=s["res"], host=s["buf"], guest=s["vm"].memory)


def _run_translate(s, ctx):
    ctx.translate(s["asid"], s["gvas"], s["case"]["n"], s["flags"], s["out"])
    return dict(out=s["out"], guest=s["vm"].memory)


def _run_batch(s, ctx):
    ctx.submit_batch(s["reqs"], s["case"]["n"], s["res"], s["ends"], s["faults"], s["n_faults"])
    return dict(res=s["res"], faults=s["faults"], n_faults=s["n_faults"], host=s["dst"],
                guest=[v.memory for v in s["vms"]])


def _run_map(s, ctx):
    if s["clear"] is not None:
        s["clear"].zero_()  # the region is unmapped again: its tables go back to the pool
    if s["case"]["ept"]:
        ctx.ept_map_pages(s["vm"].vm, s["maps"], s["case"]["n"], s["pool"], s["res"], s["used"])
    else:
        ctx.map_pages(s["asid"], s["maps"], s["case"]["n"], s["pool"], s["res"], s["used"])
    return dict(res=s["res"], used=s["used"], guest=s["vm"].memory)


def _run_serve(s, ctx):
    srv = s["guest"].server
    srv.submit(s["reqs"])
    srv.drain()
    done = srv.poll(s["case"]["n"])
    done = done[np.argsort(done["ticket"])]
    return dict(bytes_done=done["bytes_done"], code=done["code"], host=s["dst"], guest=[v.memory for v in s["vms"]])


RUN = {"copy": _run_copy, "translate": _run_translate, "batch": _run_batch, "map": _run_map, "serve": _run_serve}


# ---------------------------------------------------------------------- work
def _copied(lo, hi, share_2m, p_np):
    """Expected bytes copied and pages walked of a request: log-uniform length, each leaf missing with p_np."""
    length = lo * (hi / lo) ** ((np.arange(256) + 0.5) / 256)
    done = lambda step: sum(np.clip(length - k * step, 0, step) * (1 - p_np) ** (k + 1)  # noqa: E731
                            for k in range(int(hi / step) + 1))
    b = float(np.mean((1 - share_2m) * done(PAGE) + share_2m * done(UNIT)))
    return b, b / PAGE + 1


def work(case):
    """Bytes moved: copied bytes read and written once, one leaf entry read per
    page, descriptors read, records written; a map writes its leaf and result,
    a new table its 4 KiB."""
    c = case
    if c["kind"] == "copy":
        return dict(bytes=2 * c["bytes"] + 8 * (c["bytes"] // PAGE + 1) + 24, flops=0)
    if c["kind"] == "translate":
        return dict(bytes=c["n"] * (8 + 24 + 8), flops=0)
    if c["kind"] == "map":
        return dict(bytes=c["n"] * (24 + 24 + 8) + (c["n"] // 512 * PAGE if c["fresh"] else 0), flops=0)
    if c["kind"] == "batch":
        b, pages = _copied(c["lo"], c["hi"], c["share_2m"], c["p_np"])
    else:
        each = [(s[0], *_copied(s[1], s[2], 0.3, 0.0)) for s in SERVE_CLASSES]
        b, pages = (sum(x[0] * x[k] for x in each) for k in (1, 2))
    return dict(bytes=c["n"] * (2 * b + 8 * pages + 32 + 24), flops=0)
