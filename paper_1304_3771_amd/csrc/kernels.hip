// gfx950 kernels of the guest-memory translate-and-copy path.
//
// The operation (section 4.2 of the paper): a buffer at a guest virtual
// address is translated page by page -- a software walk of the guest's page
// tables (x86-64 4- or 5-level, or the 32-bit PAE format of the paper's
// prototype, section 6.2) to a guest-physical address, then the VM's memslots
// to the host address (KVM style), or, for a VM described by an extended page
// table, a second software walk of that EPT (the paper's path for other
// hypervisors) -- and its bytes are copied between the guest memory image
// ("arena") and a host buffer.  A fault ends the operation with everything
// before the faulting byte copied, so the operation can be re-executed
// (section 6.6).
//
// Work decomposition (wave64 throughout):
//   translate  one wavefront owns a group of consecutive requests.  A wave
//              prefix sum over their page counts flattens the group's pages;
//              each pass gives every lane one page.  Lanes that start a 2 MiB
//              region ("heads") resolve the upper levels -- the levels above
//              2 through a per-wavefront LDS cache of 1 GiB regions, level 2
//              by a load -- and hand the result to the rest of the region with
//              cross-lane shuffles; every lane then reads its own leaf entry,
//              so neighbouring lanes read neighbouring PTEs in one cache line.
//              Because a group's pages are walked in order, the first fault
//              of each request is exact (ballot + find-first-set) before any
//              side effect: A/D bits are OR-ed only into entries on the paths
//              of pages that will be copied.  Copy segments (runs of pages
//              whose guest side is contiguous in the arena) are appended to a
//              long or a short queue, each split into parts with a counter of
//              their own, with one wave-aggregated atomic per pass and queue.
//   copy       a wavefront takes each long segment, a 16-lane quarter each
//              short one; stores are 16-byte aligned, the source misalignment
//              is absorbed with one neighbour dword and a byte funnel shift,
//              never with a read-modify-write of bytes outside the segment.
//   faults     the ordered fault list is a tile count, a single-workgroup
//              scan and a ballot/mbcnt scatter.
//   map pages  one lane per map walks the tables as they are; device hash
//              sets collect the distinct tables the batch lacks and the last
//              map of each page; the new tables are ordered by rank in LDS
//              tiles (long lists: tiles, then merge rounds), zeroed,
//              linked, and the leaves written -- four launches.
#include <cstring>

#include "dv_internal.h"

namespace dv {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// Global-address-space views: the copy path and the table walks address HBM
// through integers, so without these the compiler emits flat instructions
// (which also count against the LDS counter and serialise with shuffles).
// (The host compilation pass only parses device functions; it gets no qualifier.)
#if defined(__HIP_DEVICE_COMPILE__)
#define DV_GLOBAL __attribute__((address_space(1)))
#else
#define DV_GLOBAL
#endif
typedef DV_GLOBAL u32x4 g_u32x4;
typedef DV_GLOBAL uint8_t g_u8;
typedef DV_GLOBAL uint64_t g_u64;
typedef DV_GLOBAL unsigned int g_u32;

template <class T>
__device__ __forceinline__ T *gp(uint64_t a) {
    return (T *)(uintptr_t)a;
}
template <class T, class P>
__device__ __forceinline__ T *gp(P *a) {
    return (T *)(uintptr_t)a;
}

constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr int kCacheWays = 16;  // 1 GiB-region cache entries per wavefront

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

__device__ __forceinline__ uint64_t mask_le(int lane) {
    return lane >= 63 ? ~0ull : ((2ull << lane) - 1ull);
}
__device__ __forceinline__ uint64_t mask_lt(int lane) { return lane <= 0 ? 0ull : ((1ull << lane) - 1ull); }

__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}
__device__ __forceinline__ uint64_t uniform_u64(uint64_t x) {
    uint32_t lo = uniform_u32((uint32_t)x), hi = uniform_u32((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t shfl64(uint64_t x, int src) {
    return __shfl((unsigned long long)x, src);
}
__device__ __forceinline__ uint32_t shfl32(uint32_t x, int src) { return (uint32_t)__shfl((int)x, src); }

__device__ __forceinline__ uint64_t load_entry(const uint8_t *arena, uint64_t off) {
    return *gp<const g_u64>(arena + off);
}

// OR bits into the low dword of a page-table entry (A and D live in bits 5, 6).
__device__ __forceinline__ void or_entry(uint8_t *arena, uint64_t off, uint32_t bits) {
    __hip_atomic_fetch_or(gp<g_u32>(arena + off), bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t now_ns(const DBatch &b) {
    uint64_t t = wall_clock64();
    uint64_t t0 = *b.t0;
    return (t - t0) * b.ns_num / b.ns_den;
}

// ------------------------------------------------------------------ memslots
// The translate kernels keep a copy of every VM's sorted memslots in LDS when
// they fit (at most kLdsVms VMs, kLdsSlots slots in all: 12 KiB).  A walk looks
// a memslot up for every table it reads and for the data page; from LDS that
// is a few LDS reads instead of a dependent load of the 2 MiB index.
constexpr uint32_t kLdsSlots = 512;
constexpr uint32_t kLdsVms = 64;
__shared__ DSlot g_lds_slot[kLdsSlots];
__shared__ uint32_t g_lds_off[kLdsVms + 1];

// Fills the workgroup's copy; entered by every thread.  Returns (uniformly)
// whether the slots are in LDS.
__device__ bool lds_slots_load(const DView &V) {
    if (V.nvm > kLdsVms) return false;
    typedef DV_GLOBAL DVm g_vm;
    typedef DV_GLOBAL DSlot g_slot;
    const g_vm *vms = gp<const g_vm>(V.vms);
    if (threadIdx.x < 64) {  // one wavefront: exclusive prefix sum of the slot counts
        const uint32_t lane = threadIdx.x;
        const uint32_t cnt = lane < V.nvm ? vms[lane].nslots : 0u;
        uint32_t incl = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t t = (uint32_t)__shfl((int)incl, lane >= (uint32_t)d ? (int)lane - d : (int)lane);
            if (lane >= (uint32_t)d) incl += t;
        }
        if (lane < V.nvm) g_lds_off[lane] = incl - cnt;
        if (lane == V.nvm - 1) g_lds_off[V.nvm] = incl;
        if (V.nvm == 0 && lane == 0) g_lds_off[0] = 0;
    }
    __syncthreads();
    const uint32_t total = g_lds_off[V.nvm];
    if (total > kLdsSlots) return false;
    for (uint32_t t = threadIdx.x; t < total; t += blockDim.x) {
        uint32_t vm = 0;
        while (vm + 1 < V.nvm && g_lds_off[vm + 1] <= t) ++vm;
        g_lds_slot[t] = gp<const g_slot>(vms[vm].slots)[t - g_lds_off[vm]];
    }
    __syncthreads();
    return true;
}

// A VM's table entry as a translate kernel uses it (lds: its slots are in LDS).
__device__ __forceinline__ DVm load_vm(const DView &V, uint32_t vm, bool lds) {
    DVm v = gp<const DV_GLOBAL DVm>(V.vms)[vm];
    v.lds_base = lds ? g_lds_off[vm] : kLdsNone;
    return v;
}

// GPA -> arena offset (section 4.2: the guest-physical address is turned into
// the host address backing it, as KVM does with its memslots).
__device__ __forceinline__ bool slot_lookup(const DVm &v, uint64_t gpa, uint64_t &hpa) {
    if (v.lds_base != kLdsNone) {  // binary search of the LDS copy
        const DSlot *sl = g_lds_slot + v.lds_base;
        uint32_t lo = 0, hi = v.nslots;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (sl[mid].gpa <= gpa)
                lo = mid + 1;
            else
                hi = mid;
        }
        if (lo == 0 || gpa >= sl[lo - 1].end) return false;
        hpa = sl[lo - 1].arena_off + (gpa - sl[lo - 1].gpa);
        return true;
    }
    uint64_t blk = gpa >> 21;
    if (blk < v.index_len) {
        uint64_t e = gp<const g_u64>(v.index)[blk];
        if (e & 2) {
            hpa = gpa + (e & ~0xFFFull);
            return true;
        }
        if (!(e & 1)) return false;
    } else if (v.index_complete) {
        return false;
    }
    typedef DV_GLOBAL DSlot g_slot;
    const g_slot *slots = gp<const g_slot>(v.slots);
    uint32_t lo = 0, hi = v.nslots;
    while (lo < hi) {
        uint32_t mid = (lo + hi) >> 1;
        if (slots[mid].gpa <= gpa)
            lo = mid + 1;
        else
            hi = mid;
    }
    if (lo == 0) return false;
    DSlot s = slots[lo - 1];
    if (gpa >= s.end) return false;
    hpa = s.arena_off + (gpa - s.gpa);
    return true;
}

// ------------------------------------------------------------------ EPT
// Hypervisors other than KVM finish the translation with a second software
// walk, of the extended page table that describes the guest-physical space
// (section 4.2; EPT in section 2.2).  The EPT is 4-level and lives in the
// arena; entry addresses are arena offsets.  Per level, top-down: not
// present (bits 2:0 clear) is a violation; write without read, or any of
// bits 7:3 in a table entry, is a misconfiguration; read and write are
// AND-ed down the walk.  At the leaf: a memory type of 2, 3 or 7, reserved
// bits of a large leaf, or a page outside the arena is a misconfiguration,
// then a missing permission is a violation.  Addresses at or above 2^48 are
// violations.  Every table and page the walk yields lies inside the arena.
constexpr uint32_t kNeedR = 1, kNeedW = 2, kNeedTable = 3;  // a guest table frame may take A/D writes

struct XRes {
    uint64_t hpa;
    uint32_t code;
};

// The level-2 table that a lane's last EPT walk went through, and the rights
// above it.  The tables and the page of one guest walk mostly lie in one GiB,
// where only the first EPT walk needs all four of its dependent loads.
// Back-to-back calls behind an EPT: 24 B 7.0 -> 6.3 us, 100 KB 8.1 -> 7.4,
// batches of 1,000 requests of up to 4 KiB 16.5 -> 15.3, 5-level 17.6 -> 16.1,
// 64 of up to 1 MiB 29.2 -> 26.2.
struct EptUpper {
    uint64_t gib = ~0ull, table;  // guest-physical address / 1 GiB; the table's arena offset
    uint32_t perm;
};

// Inlined: out of line, the call convention costs the translate kernels a
// wave of occupancy even when no VM has an EPT.
__device__ __forceinline__ XRes ept_walk(uint8_t *arena, uint64_t arena_bytes, uint64_t root, uint64_t gpa,
                                      uint32_t need, EptUpper *up = nullptr) {
    XRes r{0, DEVIRT_EPT_VIOLATION};
    if (gpa >> 48) return r;
    uint64_t table = root;
    uint64_t perm = 3;
    const bool known = up && up->gib == gpa >> 30;
    if (known) {
        table = up->table;
        perm = up->perm;
    }
    for (int lvl = known ? 2 : 4; lvl >= 1; --lvl) {
        const uint32_t sh = 12u + 9u * (uint32_t)(lvl - 1);
        const uint64_t e = load_entry(arena, table + 8 * ((gpa >> sh) & 511));
        if (!(e & 7)) return r;
        r.code = DEVIRT_EPT_MISCONFIG;
        if ((e & 3) == 2) return r;
        perm &= e;
        const bool leaf = lvl == 1 || ((lvl == 3 || lvl == 2) && (e & 0x80));
        if (!leaf) {
            if (e & 0xF8) return r;
            table = e & kAddrMask;
            if (table >= arena_bytes || arena_bytes - table < 4096) return r;
            r.code = DEVIRT_EPT_VIOLATION;
            if (up && lvl == 3) *up = EptUpper{gpa >> 30, table, (uint32_t)perm & 3u};
            continue;
        }
        const uint64_t mt = (e >> 3) & 7;
        if (mt == 2 || mt == 3 || mt == 7) return r;
        const uint64_t low = (1ull << sh) - 1;
        if (e & low & ~0xFFFull) return r;
        const uint64_t h = (e & kAddrMask) | (gpa & low);
        const uint64_t pg = h & ~0xFFFull;
        if (pg >= arena_bytes || arena_bytes - pg < 4096) return r;
        r.code = DEVIRT_EPT_VIOLATION;
        if (need & ~perm & 3) return r;
        r.hpa = h;
        r.code = DEVIRT_OK;
        return r;
    }
    return r;
}

// GPA -> arena offset for an access that needs `need`: the memslots, or the
// EPT walk when the VM has one.
__device__ __forceinline__ uint32_t gpa_xlat(const DVm &v, uint64_t gpa, uint32_t need, uint64_t &hpa,
                                             EptUpper *up = nullptr) {
    if (v.ept_root == kNoEpt) return slot_lookup(v, gpa, hpa) ? DEVIRT_OK : DEVIRT_NO_MEMSLOT;
    const XRes r = ept_walk(v.arena, v.arena_bytes, v.ept_root, gpa, need, up);
    if (r.code == DEVIRT_OK) hpa = r.hpa;
    return r.code;
}

// ------------------------------------------------------------ upper levels
// Result of walking the levels above the page directory for one 1 GiB region
// (x86-64: level 5 (LA57), level 4, level 3).
struct CEnt {
    uint64_t key;      // (asid << 27) | (gva >> 30); ~0 when empty
    uint64_t base;     // table: GPA of the level-2 table; 1 GiB leaf: frame GPA
    uint64_t path[3];  // arena offsets of the entries read, top level first
    uint32_t info;     // code:4 level:4 leaf1g:1 u:1 w:1 npath:2 abits:3 dbit:1
    uint32_t pad;
};
__device__ __forceinline__ uint32_t ci_code(uint32_t i) { return i & 15u; }
__device__ __forceinline__ uint32_t ci_level(uint32_t i) { return (i >> 4) & 15u; }
__device__ __forceinline__ uint32_t ci_leaf(uint32_t i) { return (i >> 8) & 1u; }
__device__ __forceinline__ uint32_t ci_u(uint32_t i) { return (i >> 9) & 1u; }
__device__ __forceinline__ uint32_t ci_w(uint32_t i) { return (i >> 10) & 1u; }
__device__ __forceinline__ uint32_t ci_np(uint32_t i) { return (i >> 11) & 3u; }
__device__ __forceinline__ uint32_t ci_abits(uint32_t i) { return (i >> 13) & 7u; }
constexpr uint32_t kCiDbit = 1u << 16;

template <int LEVELS>
__device__ __forceinline__ void walk_upper_t(const DVm &v, uint64_t cr3, uint64_t gva, CEnt &c) {
    uint64_t table = cr3 & kAddrMask;
    uint32_t u = 1, w = 1, abits = 0;
    c.path[0] = c.path[1] = c.path[2] = 0;
#pragma unroll
    for (int i = 0; i < LEVELS - 2; ++i) {
        const int lvl = LEVELS - i;
        const uint32_t shift = 12 + 9 * (lvl - 1);
        uint64_t th;
        const uint32_t xc = gpa_xlat(v, table, kNeedTable, th);
        if (xc) {
            c.info = xc | (lvl << 4) | (i << 11) | (abits << 13);
            return;
        }
        uint64_t eoff = th + 8 * ((gva >> shift) & 511);
        uint64_t e = load_entry(v.arena, eoff);
        c.path[i] = eoff;
        if (e & kA) abits |= 1u << i;
        if (!(e & kP)) {
            c.info = DEVIRT_NOT_PRESENT | (lvl << 4) | ((i + 1) << 11) | (abits << 13);
            return;
        }
        u &= (uint32_t)(e >> 2) & 1u;
        w &= (uint32_t)(e >> 1) & 1u;
        if (lvl >= 4 && (e & kPS)) {
            c.info = DEVIRT_RESERVED | (lvl << 4) | ((i + 1) << 11) | (abits << 13);
            return;
        }
        if (lvl == 3 && (e & kPS)) {
            if (e & 0x3FFFE000ull) {  // bits 29:13 of a 1 GiB leaf are reserved
                c.info = DEVIRT_RESERVED | (3u << 4) | ((i + 1) << 11) | (abits << 13);
                return;
            }
            c.base = e & kAddrMask & ~((1ull << 30) - 1);
            c.info = DEVIRT_OK | (1u << 8) | (u << 9) | (w << 10) | ((i + 1) << 11) | (abits << 13) |
                     ((e & kD) ? kCiDbit : 0u);
            return;
        }
        table = e & kAddrMask;
    }
    c.base = table;
    c.info = DEVIRT_OK | (u << 9) | (w << 10) | ((LEVELS - 2) << 11) | (abits << 13);
}

// PAE, the paper's 32-bit platform (section 6.2): one read of the 4-entry
// root table at CR3 bits 31:5, indexed by address bits 31:30.  Its entries
// grant every permission and take no accessed bit, so the cached path is
// empty; bits 2:1, 8:5 and 63:52 are reserved.
__device__ __forceinline__ void walk_upper_pae(const DVm &v, uint64_t cr3, uint64_t gva, CEnt &c) {
    c.path[0] = c.path[1] = c.path[2] = 0;
    uint64_t th;
    const uint32_t xc = gpa_xlat(v, cr3 & 0xFFFFFFE0ull, kNeedTable, th);
    if (xc) {
        c.info = xc | (3u << 4);
        return;
    }
    const uint64_t e = load_entry(v.arena, th + 8 * ((gva >> 30) & 3));
    if (!(e & kP)) {
        c.info = DEVIRT_NOT_PRESENT | (3u << 4);
        return;
    }
    if (e & kPaeRootRsvd) {
        c.info = DEVIRT_RESERVED | (3u << 4);
        return;
    }
    c.base = e & kAddrMask;
    c.info = DEVIRT_OK | (1u << 9) | (1u << 10);  // u = w = 1, no path entries
}

__device__ __forceinline__ void walk_upper(const DVm &v, uint64_t cr3, uint32_t levels, uint64_t gva, CEnt &c) {
    if (levels == 5)
        walk_upper_t<5>(v, cr3, gva, c);
    else if (levels == 3)
        walk_upper_pae(v, cr3, gva, c);
    else
        walk_upper_t<4>(v, cr3, gva, c);
}

__device__ __forceinline__ uint64_t user_limit(uint32_t levels) {
    return levels == 5 ? (1ull << 56) : levels == 3 ? (1ull << 32) : (1ull << 47);
}

__device__ __forceinline__ uint32_t cache_slot(uint64_t key) {
    uint64_t h = key ^ (key >> 7) ^ (key >> 17) ^ (key >> 29);
    return (uint32_t)h & (kCacheWays - 1);
}

// Look up (or fill) the 1 GiB-region cache for the calling lanes with
// `want` set.  Cross-lane safe: only the lane that wins a slot writes it.
// Must be called by the whole wavefront (uniform control flow).
__device__ __forceinline__ void cache_resolve(CEnt *cache, uint32_t *owner, bool want, uint64_t key,
                                              const DVm &v, uint64_t cr3, uint32_t levels, uint64_t gva, CEnt &c,
                                              uint32_t &slot, bool &hit) {
    const int lane = lane_id();
    hit = false;
    slot = cache_slot(key);
    if (want) {
        c = cache[slot];
        hit = (c.key == key);
        if (!hit) {
            walk_upper(v, cr3, levels, gva, c);
            c.key = key;
        }
    }
    bool miss = want && !hit;
    if (miss) owner[slot] = (uint32_t)lane;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (miss && owner[slot] == (uint32_t)lane) cache[slot] = c;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------- copying
// 16 output bytes from the 20-byte window (c.x c.y c.z c.w nx), starting at
// byte a (0..3); v_alignbyte takes the shift per lane.
__device__ __forceinline__ u32x4 funnel4(u32x4 c, uint32_t nx, uint32_t a) {
    u32x4 r;
    r.x = __builtin_amdgcn_alignbyte(c.y, c.x, a);
    r.y = __builtin_amdgcn_alignbyte(c.z, c.y, a);
    r.z = __builtin_amdgcn_alignbyte(c.w, c.z, a);
    r.w = __builtin_amdgcn_alignbyte(nx, c.w, a);
    return r;
}

__device__ __forceinline__ void store16(g_u32x4 *p, u32x4 v, bool nt) {
    if (nt)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// 16 bytes read at a 4-byte aligned address (one global_load_dwordx4).
typedef u32x4 u32x4_w4 __attribute__((aligned(4)));
typedef DV_GLOBAL u32x4_w4 g_u32x4_w4;

// Copy of n bytes by a group of G consecutive lanes of one wavefront; l is
// the lane's index in its group.  G = 64: the whole wavefront, arguments
// wave-uniform.  G = 16: each quarter of the wavefront copies its own
// segment, so a wavefront keeps four short segments in flight.
//
// The destination is written as aligned 16-byte blocks, with byte stores for
// the unaligned head and the tail (< 16 bytes each): no store touches a byte
// outside [dst, dst+n).  Block i takes its bytes from the 20-byte window at
// sa + 16 i, where sa is the 4-byte aligned address a bytes below the first
// body byte: the lane loads 16 bytes and takes the next dword from the next
// lane of its group (or, for the group's last lane, from the first lane of
// the next row).  Every load lies in an aligned dword that holds at least one
// source byte.  A pass moves 4 rows of G blocks and issues all of its loads
// before any store.
template <int G>
__device__ __forceinline__ void copy_span(uint8_t *dst_, const uint8_t *src_, uint32_t n, bool nt, int l) {
    constexpr int R = 4;
    if (n == 0) return;
    g_u8 *__restrict__ dst = gp<g_u8>(dst_);
    const g_u8 *__restrict__ src = gp<const g_u8>(src_);
    uint32_t h = (16u - (uint32_t)((uintptr_t)dst_ & 15u)) & 15u;
    if (h > n) h = n;
    const int32_t m = (int32_t)((n - h) >> 4);  // whole 16-byte destination blocks
    const uint32_t t = (n - h) & 15u;
    const uint32_t a = (uint32_t)((uintptr_t)(src_ + h) & 3u);
    const g_u8 *__restrict__ sa = src + h - a;
    g_u8 *__restrict__ db = dst + h;
    const uint32_t tail_off = h + 16u * (uint32_t)m;
    const int lane = lane_id();
    const int nb = (lane & ~(G - 1)) | ((lane + 1) & (G - 1));  // next lane of the group, cyclically
    int32_t b0 = 0;
    do {
        const bool first = b0 == 0;
        const bool last = b0 + R * G >= m;
        const int32_t rem = m - b0 - l;  // block b0 + l + G*u exists when G*u < rem
        const g_u8 *__restrict__ ps = sa + 16 * (int64_t)(b0 + l);
        g_u32x4 *pd = (g_u32x4 *)(db + 16 * (int64_t)(b0 + l));
        uint8_t hb = 0, tb = 0;
        if (first && (uint32_t)l < h) hb = src[l];
        if (last && (uint32_t)l < t) tb = src[tail_off + l];
        u32x4 cur[R];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            cur[u] = (u32x4){0u, 0u, 0u, 0u};
            if (G * u < rem)
                cur[u] = *(const g_u32x4_w4 *)(ps + 16 * G * u);
            else if (a != 0 && G * u == rem)  // block m: only its first dword is needed
                cur[u].x = *(const g_u32 *)(ps + 16 * G * u);
        }
        uint32_t ex = 0;  // first dword of block b0 + R*G, for the group's last lane
        if (a != 0 && l == G - 1 && R * G <= rem + G - 1) ex = *(const g_u32 *)(ps + 16 * (G * (R - 1) + 1));
        if (first && (uint32_t)l < h) dst[l] = hb;
        uint32_t rot[R];
#pragma unroll
        for (int u = 0; u < R; ++u) rot[u] = (uint32_t)__shfl((int)cur[u].x, nb);
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint32_t nx = (l == G - 1) ? (u + 1 < R ? rot[u + 1 < R ? u + 1 : 0] : ex) : rot[u];
            if (G * u < rem) store16(pd + G * u, funnel4(cur[u], nx, a), nt);
        }
        if (last && (uint32_t)l < t) dst[tail_off + l] = tb;
        b0 += R * G;
    } while (b0 < m);
}

// Whole-wavefront copy (all arguments wave-uniform).
__device__ __forceinline__ void copy_wave(uint8_t *dst, const uint8_t *src, uint32_t n, bool nt) {
    copy_span<64>(dst, src, n, nt, lane_id());
}

// Copy by one lane (short segments).
__device__ __forceinline__ void copy_lane(uint8_t *dst_, const uint8_t *src_, uint32_t n) {
    g_u8 *dst = gp<g_u8>(dst_);
    const g_u8 *src = gp<const g_u8>(src_);
    for (uint32_t i = 0; i < n; ++i) dst[i] = src[i];
}

// ------------------------------------------------------ translate a group
// One wavefront, requests [r0, r0+gn) (or one request passed by value).
// Must be entered by all 64 lanes.
struct GroupOut {
    unsigned long long pages, hits, misses, segs, inl, atomics, spills;
};

// Requests of more than B.large_pages pages ("large"): in the batched path a
// group leaves them to k_translate_large, where the wavefronts of a workgroup
// walk one large request together.
enum : uint32_t {
    kLargeKeep = 0,   // walk them here
    kLargeDefer = 1,  // put them on the epoch's large list; their results come later
    kLargeSkip = 2,   // leave them alone (spill pass: a large request spills on its own)
};

// Workgroup-shared state of a large request walked by several wavefronts.
struct CoopShared {
    uint32_t ff[3];   // per round, rotating: the request's first faulting page (kNone: none)
    uint32_t fcode, flevel;
    uint64_t flo;     // that page's first byte in the request
    uint32_t queued;  // segments queued
    uint32_t spilled;
};

// Returns (wave-uniformly) true when some run of the group found its queue
// part full while B.spill_mode is set: such runs are neither queued nor
// copied, and the caller puts the group on the epoch's spill list.
//
// kCoop: the wavefronts of a workgroup walk one large request (gn = 1)
// together, round by round: in each round wavefront w takes pages
// [64 w, 64 w + 64) of the round's 64 W.  The walk of a round has no side
// effects; the request's first faulting page is then agreed in LDS (cs), and
// only pages before it get A/D bits and copies, as in the one-wavefront walk.
// All wavefronts run the same rounds (barriers inside); the result is written
// by wavefront 0.  e0: the epoch's first request (slot of the large list).
template <bool kPlain, bool kCoop>
__device__ bool process_group(const DView &V, const DBatch &B, uint64_t r0, uint32_t gn,
                              const devirt_request &preq, uint32_t epoch, CEnt *cache, uint32_t *owner,
                              bool coop_all, uint32_t large_mode, uint64_t e0, DEpochCtr *ctr, GroupOut &st,
                              CoopShared *cs) {
    const int lane = lane_id();
    const uint32_t nw = kCoop ? (blockDim.x >> 6) : 1u;    // wavefronts walking the request
    const uint32_t wv = kCoop ? (threadIdx.x >> 6) : 0u;   // this one
    // this wavefront's part of the segment queues
    const uint32_t qpart = kPlain ? 0u : (uint32_t)((blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) % kQParts);
    const uint64_t pcap = B.part_cap;
    // ---- load and validate the group's requests (lane k owns request k)
    uint64_t gva = 0, host = 0, cr3 = 0;
    uint32_t len = 0, asid = 0, dir = 0, vm = 0, levels = 4, code0 = 0, nch = 0;
    if ((uint32_t)lane < gn) {
        devirt_request rq;
        if (kPlain) {
            rq = preq;
        } else {
            const g_u32x4 *p = gp<const g_u32x4>(B.reqs + r0 + lane);
            u32x4 a = p[0], b = p[1];
            rq.gva = ((uint64_t)a.y << 32) | a.x;
            rq.host = ((uint64_t)a.w << 32) | a.z;
            rq.len = b.x;
            rq.asid = b.y;
            rq.dir = (uint8_t)(b.z & 0xFF);
        }
        gva = rq.gva;
        host = rq.host;
        len = rq.len;
        asid = rq.asid;
        dir = rq.dir ? 1u : 0u;
        if (asid >= V.nproc) {
            code0 = DEVIRT_INVALID;
        } else {
            DProc p = gp<const DV_GLOBAL DProc>(V.procs)[asid];
            vm = p.vm;
            levels = p.levels;
            cr3 = p.cr3;
            if (len != 0) {
                uint64_t lim = user_limit(levels);
                if (gva >= lim || (uint64_t)len > lim - gva)
                    code0 = DEVIRT_NONCANONICAL;
                else
                    nch = (uint32_t)(((gva + len - 1) >> 12) - (gva >> 12) + 1);
            }
        }
    }
    // large requests left to k_translate_large (or to their own spill entry)
    bool large = false;
    if (!kPlain && !kCoop && large_mode != kLargeKeep && B.large_pages && nch > B.large_pages) {
        large = true;
        nch = 0;
    }
    if (!kPlain && !kCoop && large_mode == kLargeDefer) {
        const uint64_t lm = __ballot(large);
        if (lm) {
            uint32_t lb = 0;
            if (lane == 0) lb = atomicAdd(&ctr[epoch].large_n, (uint32_t)__popcll(lm));
            lb = shfl32(lb, 0);
            if (large) gp<g_u64>(B.large)[e0 + lb + (uint32_t)__popcll(lm & mask_lt(lane))] = r0 + (uint64_t)lane;
        }
    }
    // ---- wave exclusive prefix sum of page counts
    uint32_t incl = nch;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = shfl32(incl, lane >= d ? lane - d : lane);
        if (lane >= d) incl += t;
    }
    const uint32_t start = incl - nch;
    const uint32_t total = shfl32(incl, 63);

    // ---- per-request path: the process's translation cache, a FIFO whose
    // slots live in lanes 0..cap-1 (section 4.2).  A page held in it (and,
    // for a write into the guest, held from a write) is not walked: its
    // translation comes from the slot, and the bits a walk would set are
    // already set.  Lookups are replayed in page order after each pass, so
    // hits, misses and evictions are those of a sequential FIFO.
    const uint32_t cap = B.fifo_entries;
    const bool use_fifo = kPlain && B.fifo != nullptr && cap != 0 && total > 0;
    DFifo *fifo = nullptr;
    uint64_t fv = ~0ull, fh = 0;
    uint32_t f_occ = 0, f_wr = 0, f_n = 0, f_head = 0;
    unsigned long long f_hits = 0, f_miss = 0;
    if (use_fifo) {
        fifo = B.fifo + uniform_u32(asid);  // kPlain: lane 0 holds the request
        if (uniform_u64(*gp<const g_u64>(&fifo->gen)) == B.xlat_gen) {
            f_n = uniform_u32(*gp<const g_u32>(&fifo->n));
            f_head = uniform_u32(*gp<const g_u32>(&fifo->head));
            f_wr = uniform_u32(*gp<const g_u32>(&fifo->written));
            if ((uint32_t)lane < cap) {
                fv = gp<const g_u64>(fifo->vpn)[lane];
                fh = gp<const g_u64>(fifo->hpa)[lane];
            }
            for (uint32_t k = 0; k < f_n; ++k) f_occ |= 1u << ((f_head + k) % cap);
        }
    }

    // per-request (owner lane) state
    uint32_t ff = kNone, fcode = 0, flevel = 0, queued = 0;
    uint64_t flo = 0;
    bool spilled = false;

    // kCoop: round r is walked by min(nw, 2^r) wavefronts, so that a request
    // faulting early is walked little past its fault (as by one wavefront),
    // and one that keeps going soon has every wavefront on it
    uint32_t round = 0, nr = 1;
    for (uint32_t rb = 0; rb < total; rb += 64 * nr, ++round) {
        nr = kCoop ? (round < 5 && (1u << round) < nw ? (1u << round) : nw) : 1u;  // wavefronts this round
        const uint32_t base = rb + 64 * wv;
        const uint32_t c = base + (uint32_t)lane;
        const bool active = wv < nr && c < total;
        // owner of page c: the last request whose start <= c
        int j = 0;
#pragma unroll
        for (int s = 32; s >= 1; s >>= 1) {
            int cand = j + s;
            int idx = cand < (int)gn ? cand : (int)gn - 1;
            uint32_t sj = shfl32(start, idx);
            if (cand < (int)gn && sj <= c) j = cand;
        }
        const uint64_t j_gva = shfl64(gva, j);
        const uint64_t j_host = shfl64(host, j);
        const uint64_t j_cr3 = shfl64(cr3, j);
        const uint32_t j_len = shfl32(len, j);
        const uint32_t j_meta = shfl32(dir | (levels << 1) | (vm << 4), j);
        const uint32_t j_asid = shfl32(asid, j);
        const uint32_t j_start = shfl32(start, j);
        const uint32_t j_ff = kCoop ? kNone : shfl32(ff, j);  // kCoop: rounds end at the first fault
        const uint32_t j_dir = j_meta & 1u, j_levels = (j_meta >> 1) & 7u, j_vm = j_meta >> 4;
        const bool work = active && j_ff == kNone;

        const uint32_t k = c - j_start;  // page index inside the request
        const uint64_t page = (j_gva & ~0xFFFull) + ((uint64_t)k << 12);
        const uint64_t lo = page > j_gva ? page : j_gva;
        const uint64_t end = j_gva + j_len;
        const uint64_t hi = page + 4096 < end ? page + 4096 : end;

        // pages the translation cache holds (as of the start of this pass) skip the walk
        bool fhit = false;
        uint64_t fhpa = 0;
        if (use_fifo) {
            for (uint32_t e = 0; e < cap; ++e) {
                const uint64_t ve = uniform_u64(shfl64(fv, (int)e));
                const uint64_t he = uniform_u64(shfl64(fh, (int)e));
                if (work && ((f_occ >> e) & 1u) && ve == (lo >> 12) && (!j_dir || ((f_wr >> e) & 1u))) {
                    fhit = true;
                    fhpa = he;
                }
            }
        }
        const bool walkl = work && !fhit;

        // ---- heads: first lane of each (request, 2 MiB region) run of walking lanes
        const int prev = lane > 0 ? lane - 1 : 0;
        const uint32_t p_work = shfl32(walkl ? 1u : 0u, prev);
        const uint32_t p_j = shfl32((uint32_t)j, prev);
        const uint64_t p_lo = shfl64(lo, prev);
        const bool head = walkl && (lane == 0 || !p_work || p_j != (uint32_t)j || (p_lo >> 21) != (lo >> 21));
        const uint64_t head_mask = __ballot(head);

        DVm vmv;
        if (work) vmv = load_vm(V, j_vm, V.lds != 0);
        // upper levels through the cache (heads only)
        CEnt ce;
        ce.info = 0;
        ce.base = 0;
        ce.path[0] = ce.path[1] = ce.path[2] = 0;
        uint32_t cslot;
        bool chit;
        const uint64_t key1 = ((uint64_t)j_asid << 27) | (lo >> 30);
        cache_resolve(cache, owner, head, key1, vmv, j_cr3, j_levels, lo, ce, cslot, chit);
        if (head) {
            if (chit)
                st.hits++;
            else
                st.misses++;
        }
        // level 2 (heads): rkind 0 = 4 KiB table, 1 = 2 MiB leaf, 2 = 1 GiB leaf
        uint32_t rcode = 0, rlevel = 0, rkind = 0, ru = 0, rw = 0, rhas = 0;
        uint64_t rbase = 0, pde_off = 0;
        if (head) {
            rcode = ci_code(ce.info);
            rlevel = ci_level(ce.info);
            ru = ci_u(ce.info);
            rw = ci_w(ce.info);
            if (rcode == 0) {
                if (ci_leaf(ce.info)) {
                    rkind = 2;
                    rbase = ce.base;
                } else {
                    uint64_t th;
                    const uint32_t xc = gpa_xlat(vmv, ce.base, kNeedTable, th);
                    if (xc) {
                        rcode = xc;
                        rlevel = 2;
                    } else {
                        pde_off = th + 8 * ((lo >> 21) & 511);
                        uint64_t e = load_entry(vmv.arena, pde_off);
                        // bits already set cost no atomic below: the 512 entries of a 1 GiB
                        // guest share 32 cache lines, on which atomics take turns (600,000
                        // requests of up to 4 KiB to one guest: 794 us of translation with
                        // an atomic per region and request, 70 without)
                        rhas = (uint32_t)e & (uint32_t)(kA | kD);
                        if (!(e & kP)) {
                            rcode = DEVIRT_NOT_PRESENT;
                            rlevel = 2;
                        } else if (j_levels == 3 && (e & kPaeRsvd)) {
                            rcode = DEVIRT_RESERVED;
                            rlevel = 2;
                        } else {
                            ru &= (uint32_t)(e >> 2) & 1u;
                            rw &= (uint32_t)(e >> 1) & 1u;
                            if (e & kPS) {
                                if (e & 0x1FE000ull) {  // bits 20:13 of a 2 MiB leaf are reserved
                                    rcode = DEVIRT_RESERVED;
                                    rlevel = 2;
                                } else {
                                    rkind = 1;
                                    rbase = e & kAddrMask & ~((1ull << 21) - 1);
                                }
                            } else {
                                uint64_t pt;
                                const uint32_t xc1 = gpa_xlat(vmv, e & kAddrMask, kNeedTable, pt);
                                if (xc1) {
                                    rcode = xc1;
                                    rlevel = 1;
                                } else {
                                    rkind = 0;
                                    rbase = pt;
                                }
                            }
                        }
                    }
                }
            }
        }
        // ---- broadcast the region result from each head to its lanes
        const int h = 63 - __clzll(head_mask & mask_le(lane));
        const int hsrc = (head_mask & mask_le(lane)) ? h : lane;
        const uint32_t r_packed =
            shfl32(rcode | (rlevel << 4) | (rkind << 8) | (ru << 10) | (rw << 11), hsrc);
        const uint64_t r_base = shfl64(rbase, hsrc);

        // ---- leaf step (every walking lane)
        uint32_t code = 0, level = 0, shift = 0;
        uint64_t gpa = 0, hpa = 0, leaf_off = 0, leaf_e = 0;
        if (fhit) hpa = fhpa + (lo & 0xFFFull);
        if (walkl) {
            code = r_packed & 15u;
            level = (r_packed >> 4) & 15u;
            const uint32_t kind = (r_packed >> 8) & 3u;
            uint32_t u = (r_packed >> 10) & 1u, w = (r_packed >> 11) & 1u;
            uint32_t leaf_level = 0;
            uint64_t frame = 0;
            if (code == 0) {
                if (kind == 0) {
                    leaf_off = r_base + 8 * ((lo >> 12) & 511);
                    leaf_e = load_entry(vmv.arena, leaf_off);
                    if (!(leaf_e & kP)) {
                        code = DEVIRT_NOT_PRESENT;
                        level = 1;
                    } else if (j_levels == 3 && (leaf_e & kPaeRsvd)) {
                        code = DEVIRT_RESERVED;
                        level = 1;
                    } else {
                        u &= (uint32_t)(leaf_e >> 2) & 1u;
                        w &= (uint32_t)(leaf_e >> 1) & 1u;
                        frame = leaf_e & kAddrMask;
                        shift = 12;
                        leaf_level = 1;
                    }
                } else {
                    frame = r_base;
                    shift = kind == 1 ? 21 : 30;
                    leaf_level = kind == 1 ? 2 : 3;
                }
            }
            if (code == 0) {
                gpa = frame | (lo & ((1ull << shift) - 1));
                if (!u) {
                    code = DEVIRT_PROT_USER;
                    level = leaf_level;
                } else if (j_dir && !w) {
                    code = DEVIRT_PROT_WRITE;
                    level = leaf_level;
                } else {
                    const uint32_t xc = gpa_xlat(vmv, gpa, j_dir ? kNeedW : kNeedR, hpa);
                    if (xc) {
                        code = xc;
                        level = 0;
                    }
                }
            }
        }
        st.pages += __popcll(__ballot(work));

        // ---- first fault per request, pages that will be copied
        const uint64_t fmask = __ballot(work && code != 0);
        const uint32_t jfirst = j_start > base ? j_start - base : 0u;  // first lane of request j
        const uint64_t jmask = mask_le(lane) & ~mask_lt((int)jfirst);
        uint32_t ffr = kNone;  // kCoop: the request's first faulting page, agreed by the workgroup
        if (kCoop) {
            if (lane == 0 && fmask)
                atomicMin(&cs->ff[round % 3], base + (uint32_t)(__ffsll((unsigned long long)fmask) - 1));
            __syncthreads();
            ffr = uniform_u32(*(volatile uint32_t *)&cs->ff[round % 3]);
            if (threadIdx.x == 0) cs->ff[(round + 2) % 3] = kNone;  // every wave is done reading it
            if (work && c == ffr) {
                cs->fcode = code;
                cs->flevel = level;
                cs->flo = lo;
            }
        }
        const bool copied = kCoop ? (work && code == 0 && c < ffr) : (work && code == 0 && (fmask & jmask) == 0);
        // (pages served by the translation cache need no A/D: their filling walk set them)
        const uint64_t cmask = __ballot(copied && !fhit);
        const uint64_t cto_mask = __ballot(copied && !fhit && j_dir);

        // owner lanes pick up their request's first fault in this pass
        if (!kCoop) {
            const bool own = (uint32_t)lane < gn && nch > 0 && ff == kNone;
            uint64_t my = 0;
            if (own) {
                uint32_t a = start > base ? start - base : 0u;
                uint32_t b = start + nch - base;  // may exceed 64
                if (start < base + 64 && start + nch > base) {
                    uint64_t hi_m = b >= 64 ? ~0ull : ((1ull << b) - 1);
                    my = fmask & hi_m & ~mask_lt((int)a);
                }
            }
            const int f = my ? (__ffsll((unsigned long long)my) - 1) : lane;
            const uint32_t f_code = shfl32(code, f);
            const uint32_t f_level = shfl32(level, f);
            const uint64_t f_lo = shfl64(lo, f);
            if (own && my) {
                ff = base + (uint32_t)f - start;
                fcode = f_code;
                flevel = f_level;
                flo = f_lo;
            }
        }

        // ---- translation cache: this pass's lookups in page order, up to and
        // including the request's first faulting page (kPlain: one request)
        if (use_fifo) {
            uint64_t lk = __ballot(work);
            if (fmask) lk &= mask_le(__ffsll((unsigned long long)fmask) - 1);
            const uint64_t okm = __ballot(work && code == 0);
            const uint64_t pg = hpa - (lo & 0xFFFull);  // the page's arena offset (lanes that translated)
            while (lk) {
                const int jl = __ffsll((unsigned long long)lk) - 1;
                lk &= lk - 1;
                const uint64_t v = uniform_u64(shfl64(lo >> 12, jl));
                const uint64_t hp = uniform_u64(shfl64(pg, jl));
                const bool wrj = uniform_u32(shfl32(j_dir, jl)) != 0;
                const uint64_t em = __ballot((uint32_t)lane < cap && ((f_occ >> lane) & 1u) && fv == v);
                const int slot = em ? __ffsll((unsigned long long)em) - 1 : -1;
                if (slot >= 0 && (!wrj || ((f_wr >> slot) & 1u))) {
                    f_hits++;
                    continue;
                }
                f_miss++;
                if (!((okm >> jl) & 1ull)) continue;  // a failed walk inserts nothing
                if (slot >= 0) {                      // held from reads: now written
                    f_wr |= 1u << slot;
                    continue;
                }
                uint32_t tail;
                if (f_n == cap) {  // full: the oldest entry leaves
                    tail = f_head;
                    f_head = (f_head + 1) % cap;
                } else {
                    tail = (f_head + f_n) % cap;
                    f_n++;
                }
                if ((uint32_t)lane == tail) {
                    fv = v;
                    fh = hp;
                }
                f_occ |= 1u << tail;
                f_wr = (f_wr & ~(1u << tail)) | ((wrj ? 1u : 0u) << tail);
            }
        }

        // ---- A/D: leaf of 4 KiB pages per lane; region-level entries by heads
        uint32_t atomics = 0;
        if (copied && leaf_off) {
            const uint32_t want = (uint32_t)kA | (j_dir ? (uint32_t)kD : 0u);
            if (((uint32_t)leaf_e & want) != want) {
                or_entry(vmv.arena, leaf_off, want);
                atomics++;
            }
        }
        if (head) {
            const int nh_bit = __ffsll((unsigned long long)(head_mask & ~mask_le(lane)));
            const int nh = nh_bit ? nh_bit - 1 : 64;
            // (known defect, see last_head_lost: with no later head nh is 64, which
            // mask_lt's shift does not cover)
            const uint64_t rmask = mask_lt(nh) & ~mask_lt(lane);
            if (cmask & rmask) {
                const bool rto = (cto_mask & rmask) != 0;
                // level-2 entry (a table pointer or a 2 MiB leaf)
                if (rkind == 0 || rkind == 1) {
                    uint32_t want = (uint32_t)kA | ((rkind == 1 && rto) ? (uint32_t)kD : 0u);
                    if ((rhas & want) != want) {
                        or_entry(vmv.arena, pde_off, want);
                        atomics++;
                    }
                }
                // levels 5..3 from the cached walk
                const uint32_t np = ci_np(ce.info), ab = ci_abits(ce.info);
                uint32_t mark = 0;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    if ((uint32_t)i < np) {
                        uint32_t want = (uint32_t)kA;
                        const bool is_leaf = rkind == 2 && (uint32_t)i + 1 == np;
                        bool need = !((ab >> i) & 1u);
                        if (is_leaf && rto) {
                            want |= (uint32_t)kD;
                            need = need || !(ce.info & kCiDbit);
                        }
                        if (need) {
                            or_entry(vmv.arena, ce.path[i], want);
                            atomics++;
                        }
                        mark |= 1u << (13 + i);
                        if (is_leaf && rto) mark |= kCiDbit;
                    }
                }
                if (cache[cslot].key == key1) atomicOr(&cache[cslot].info, mark);
            }
        }
        st.atomics += atomics;

        // ---- copy segments: runs of pages whose guest side is contiguous
        uint8_t *const arena = work ? vmv.arena : nullptr;
        const uint64_t gptr = (uint64_t)(uintptr_t)arena + hpa;
        const uint64_t hptr = j_host + (lo - j_gva);
        const uint32_t nbytes = (uint32_t)(hi - lo);
        const uint32_t p_copied = shfl32(copied ? 1u : 0u, prev);
        const uint64_t p_gptr = shfl64(gptr, prev);
        const uint32_t p_n = shfl32(nbytes, prev);
        const bool cont = copied && lane > 0 && p_copied && p_j == (uint32_t)j && p_gptr + p_n == gptr &&
                          (k % B.seg_chunks) != 0;
        const bool rhead = copied && !cont;
        const uint64_t cont_mask = __ballot(cont);
        // run [lane, e): e = first later lane that does not continue the run
        const int e_bit = __ffsll((unsigned long long)(~cont_mask & ~mask_le(lane)));
        const int e = e_bit ? e_bit - 1 : 64;
        const int last = rhead ? e - 1 : lane;
        const uint64_t l_end = shfl64(lo + nbytes, last);
        const uint32_t run = rhead ? (uint32_t)(l_end - lo) : 0u;
        uint64_t src = 0, dst = 0;
        if (rhead) {
            src = j_dir ? hptr : gptr;
            dst = j_dir ? gptr : hptr;
        }
        const bool small = rhead && !coop_all && run <= B.inline_bytes;
        if (small) copy_lane((uint8_t *)dst, (const uint8_t *)src, run);
        const bool want_q = rhead && !small && !coop_all;
        const bool is_short = run <= kShortRun;
        const uint64_t lmask = __ballot(want_q && !is_short);
        const uint64_t smask = __ballot(want_q && is_short);
        bool coop = rhead && coop_all;
        uint32_t q_ok = 0;
        if (lmask | smask) {
            uint32_t lbase = 0, sbase = 0;
            if (lane == 0) {
                if (lmask) lbase = atomicAdd(&ctr[epoch].q[qpart][0], (uint32_t)__popcll(lmask));
                if (smask) sbase = atomicAdd(&ctr[epoch].q[kQParts + qpart][0], (uint32_t)__popcll(smask));
            }
            lbase = shfl32(lbase, 0);
            sbase = shfl32(sbase, 0);
            if (want_q) {
                const uint64_t qm = is_short ? smask : lmask;
                const uint64_t pos = (uint64_t)(is_short ? sbase : lbase) + (uint64_t)__popcll(qm & mask_lt(lane));
                if (pos < pcap) {
                    DSeg sg;
                    sg.src = src;
                    sg.dst = dst;
                    sg.len = run;
                    sg.req = (uint32_t)(r0 + (uint64_t)j);
                    sg.pad = 0;
                    gp<DV_GLOBAL DSeg>(is_short ? B.shorts : B.segs)[qpart * pcap + pos] = sg;
                    q_ok = 1;
                } else if (B.spill_mode) {
                    spilled = true;  // queue full: the spill pass copies it
                } else {
                    coop = true;  // queue full: the wavefront copies it below
                }
            }
        }
        st.segs += __popcll(__ballot(q_ok != 0));
        st.inl += __popcll(__ballot(small || coop));  // inline and queue-overflow copies
        // per-request count of queued segments (for completion times)
        {
            const uint64_t okm = __ballot(q_ok != 0);
            if ((uint32_t)lane < gn && nch > 0 && start < base + 64 && start + nch > base) {
                uint32_t a = start > base ? start - base : 0u;
                uint32_t b = start + nch - base;
                uint64_t hi_m = b >= 64 ? ~0ull : ((1ull << b) - 1);
                queued += (uint32_t)__popcll(okm & hi_m & ~mask_lt((int)a));
            }
        }
        uint64_t cm = __ballot(coop);
        while (cm) {
            const int l = __ffsll((unsigned long long)cm) - 1;
            const uint64_t s = uniform_u64(shfl64(src, l)), d = uniform_u64(shfl64(dst, l));
            const uint32_t n = uniform_u32(shfl32(run, l));
            copy_wave((uint8_t *)d, (const uint8_t *)s, n, B.nontemporal != 0);
            cm &= cm - 1;
        }
        if (kCoop && ffr != kNone) {  // workgroup-uniform
            ff = ffr;
            break;
        }
    }
    bool any_spill = __ballot(spilled) != 0;
    if (kCoop) {
        // the request's outcome, from the workgroup's shared state
        if (lane == 0) {
            if (queued) atomicAdd(&cs->queued, queued);
            if (any_spill) atomicOr(&cs->spilled, 1u);
        }
        __syncthreads();
        any_spill = *(volatile uint32_t *)&cs->spilled != 0;
        queued = *(volatile uint32_t *)&cs->queued;
        if (ff != kNone) {
            fcode = *(volatile uint32_t *)&cs->fcode;
            flevel = *(volatile uint32_t *)&cs->flevel;
            flo = *(volatile uint64_t *)&cs->flo;
        }
    }

    // ---- results (owner lanes; a large request's come from k_translate_large)
    if ((uint32_t)lane < gn && !large && wv == 0) {
        devirt_result r;
        r.pad = 0;
        if (code0) {
            r.bytes_done = 0;
            r.fault_gva = gva;
            r.code = code0;
            r.level = 0;
        } else if (ff == kNone) {
            r.bytes_done = len;
            r.fault_gva = 0;
            r.code = 0;
            r.level = 0;
        } else {
            r.bytes_done = flo - gva;
            r.fault_gva = flo;
            r.code = fcode;
            r.level = (uint16_t)flevel;
        }
        gp<DV_GLOBAL devirt_result>(B.res)[kPlain ? 0 : r0 + lane] = r;
        if (!kPlain && B.t_done) {
            B.pending[r0 + lane] = queued;
            if (queued == 0) B.t_done[r0 + lane] = now_ns(B);
        }
    }
    if (use_fifo) {
        if ((uint32_t)lane < cap) {
            gp<g_u64>(fifo->vpn)[lane] = fv;
            gp<g_u64>(fifo->hpa)[lane] = fh;
        }
        if (lane == 0) {
            *gp<g_u32>(&fifo->written) = f_wr;
            *gp<g_u32>(&fifo->n) = f_n;
            *gp<g_u32>(&fifo->head) = f_head;
            *gp<g_u64>(&fifo->gen) = B.xlat_gen;
            *gp<DV_GLOBAL unsigned long long>(&fifo->hits) += f_hits;
            *gp<DV_GLOBAL unsigned long long>(&fifo->misses) += f_miss;
        }
    }
    return any_spill;
}

// ------------------------------------------------------------------ kernels
constexpr uint32_t kCtrLines = sizeof(DEpochCtr) / (4 * kLineWords);  // counters of an epoch: word 0 of every line

__global__ void k_reset(DBatch b, uint32_t n_epochs) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *b.t0 = wall_clock64();
    static_assert(sizeof(DEpochCtr) % (4 * kLineWords) == 0, "counters on lines of their own");
    for (; i < n_epochs * kCtrLines; i += gridDim.x * blockDim.x) ((uint32_t *)b.ctr)[(uint64_t)i * kLineWords] = 0;
}

__device__ __forceinline__ void flush_counters(DCounters *c, const GroupOut &st) {
    if (!c) return;
    unsigned long long v[7] = {st.pages, st.hits, st.misses, st.segs, st.inl, st.atomics, st.spills};
    // lane-local partial sums -> one atomic per counter per wavefront
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        unsigned long long x = v[i];
        for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d);
        v[i] = x;
    }
    if (lane_id() == 0) {
        atomicAdd(&c->pages_walked, v[0] / 64);
        atomicAdd(&c->cache_hits, v[1]);
        atomicAdd(&c->cache_misses, v[2]);
        atomicAdd(&c->segments, v[3] / 64);
        atomicAdd(&c->inline_segments, v[4] / 64);
        atomicAdd(&c->ad_atomics, v[5]);
        atomicAdd(&c->spilled_groups, v[6] / 64);
    }
}

// direct != 0: the translating wavefronts copy their runs themselves and
// nothing is queued (one launch for a small batch).
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_translate_groups(DView v, DBatch b, uint64_t r0, uint64_t r1, uint32_t epoch, int direct) {
    extern __shared__ uint8_t smem[];
    v.lds = lds_slots_load(v) ? 1u : 0u;
    const int wave = threadIdx.x >> 6;
    CEnt *cache = (CEnt *)smem + wave * kCacheWays;
    uint32_t *owner = (uint32_t *)((CEnt *)smem + (blockDim.x >> 6) * kCacheWays) + wave * kCacheWays;
    if ((threadIdx.x & 63) < kCacheWays) cache[threadIdx.x & 63].key = ~0ull;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint64_t n = r1 - r0;
    const uint32_t G = b.group;
    const uint64_t ngroups = (n + G - 1) / G;
    GroupOut st = {0, 0, 0, 0, 0, 0, 0};
    devirt_request dummy = {};
    // Each wavefront takes group (its global index) first, without an atomic;
    // further groups come from its part's cursor, numbered after those first
    // ones.  (One cursor for all served a claim every 13 ns, whatever the
    // group: 600,000 requests of up to 4 KiB took 989 us in groups of 8 and
    // 337 us in groups of 64.)  The next claim is issued before the current
    // group is translated, so its round trip overlaps the group's own loads.
    // When every group is some wavefront's first, no claim is made at all (and
    // the cursors are not read).
    const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    const bool claim = ngroups > nwaves;
    uint64_t gi = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (uint64_t)wave;
    const uint32_t parts = nwaves < kQParts ? (uint32_t)nwaves : kQParts, part = (uint32_t)(gi % parts);
    while (gi < ngroups) {
        uint32_t g = 0;
        if (claim && lane_id() == 0) g = atomicAdd(&b.ctr[epoch].cursor[part][0], 1u);
        const uint64_t gs = r0 + gi * G;
        const uint32_t gn = (uint32_t)((r1 - gs) < G ? (r1 - gs) : G);
        if (process_group<false, false>(v, b, gs, gn, dummy, epoch, cache, owner, direct != 0,
                                        direct ? kLargeKeep : kLargeDefer, r0, b.ctr, st, nullptr)) {
            st.spills++;
            if (lane_id() == 0) {
                const uint32_t k = atomicAdd(&b.ctr[epoch].spill_n, 1u);
                gp<g_u64>(b.spill)[r0 + k] = gs;  // at most one slot per group of [r0, r1)
            }
        }
        if (!claim) break;
        gi = nwaves + part + (uint64_t)parts * uniform_u32(shfl32(g, 0));
    }
    flush_counters(b.counters, st);
}

// The epoch's large requests (listed by k_translate_groups), one per
// workgroup at a time: its wavefronts walk the request's pages together (see
// process_group), so a request of thousands of pages takes a few rounds
// instead of one wavefront's many passes.  Queue overflow is handled as in
// k_translate_groups; a request that spills goes on the spill list alone.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_translate_large(DView v, DBatch b, uint64_t r0, uint32_t epoch) {
    extern __shared__ uint8_t smem[];
    __shared__ CoopShared cs;
    const int wave = threadIdx.x >> 6;
    CEnt *cache = (CEnt *)smem + wave * kCacheWays;
    uint32_t *owner = (uint32_t *)((CEnt *)smem + (blockDim.x >> 6) * kCacheWays) + wave * kCacheWays;
    const uint32_t n = uniform_u32(*gp<const g_u32>(&b.ctr[epoch].large_n));
    if (n == 0) return;
    v.lds = lds_slots_load(v) ? 1u : 0u;
    if ((threadIdx.x & 63) < kCacheWays) cache[threadIdx.x & 63].key = ~0ull;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    GroupOut st = {0, 0, 0, 0, 0, 0, 0};
    devirt_request dummy = {};
    for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
        const uint64_t r = uniform_u64(gp<const g_u64>(b.large)[r0 + k]);
        if (threadIdx.x == 0) {
            cs.ff[0] = cs.ff[1] = cs.ff[2] = kNone;
            cs.queued = 0;
            cs.spilled = 0;
        }
        __syncthreads();
        const bool sp = process_group<false, true>(v, b, r, 1, dummy, epoch, cache, owner, false, kLargeKeep, r0,
                                                   b.ctr, st, &cs);
        if (b.counters && threadIdx.x == 0) atomicAdd(&b.counters->large_requests, 1ull);
        if (sp && threadIdx.x == 0) {
            st.spills++;
            const uint32_t i = atomicAdd(&b.ctr[epoch].spill_n, 1u);
            gp<g_u64>(b.spill)[r0 + i] = r | kSpillOne;
        }
        __syncthreads();  // cs is reused for the next request
    }
    flush_counters(b.counters, st);
}

// The ordered fault list of a small batch, by one workgroup beside the copy
// (every result is final once the translation is done), and the counters of
// the stream's next one-epoch batch.  A batch of a few hundred requests is
// bound by its launches: with clearing, counting, scanning and scattering as
// launches of their own 256 requests took 32.1 us a batch, now 16.9; 8,191
// requests of up to 64 KiB 62 us, now 49.
__device__ void copy_tail(const devirt_result *res_, const CopyTail &t) {
    constexpr int Q = 8;  // results per lane and pass: one round trip for 8192 in a workgroup of 1024
    __shared__ uint32_t s_cnt[Q * 16];
    const int lane = lane_id();
    const uint32_t wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (uint32_t k = threadIdx.x; k < kCtrLines; k += blockDim.x)
        ((uint32_t *)t.clear)[(uint64_t)k * kLineWords] = 0;
    if (!t.faults && !t.n_faults) return;
    typedef const DV_GLOBAL devirt_result g_res;
    g_res *res = gp<g_res>(res_);
    const uint32_t n = (uint32_t)t.n;  // at most kTailFaults with a list
    uint32_t carry = 0;
    for (uint32_t base = 0; base < n; base += Q * blockDim.x) {
        uint32_t code[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t i = base + q * blockDim.x + threadIdx.x;
            code[q] = i < n ? res[i].code : 0u;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint64_t m = __ballot(code[q] != 0);
            if (lane == 0) s_cnt[q * nw + wave] = (uint32_t)__popcll(m);
        }
        __syncthreads();
        // the counts, in request order, are (q, wavefront): lane l sums entries 2 l and 2 l + 1
        const uint32_t ne = Q * nw;
        const uint32_t a = 2u * lane < ne ? s_cnt[2 * lane] : 0u, b = 2u * lane + 1 < ne ? s_cnt[2 * lane + 1] : 0u;
        uint32_t incl = a + b;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t x = shfl32(incl, lane >= d ? lane - d : lane);
            if (lane >= d) incl += x;
        }
        const uint32_t excl = incl - a - b, total = shfl32(incl, 63);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const uint32_t e = q * nw + wave;
            const uint32_t before = shfl32(excl, (int)(e >> 1)) + ((e & 1) ? shfl32(a, (int)(e >> 1)) : 0u);
            const uint64_t m = __ballot(code[q] != 0);
            if (code[q] != 0 && t.faults) {
                const uint32_t i = base + q * blockDim.x + threadIdx.x;
                devirt_fault f;
                f.req_index = i;
                f.fault_gva = res[i].fault_gva;
                f.code = code[q];
                f.level = res[i].level;
                f.pad = 0;
                gp<DV_GLOBAL devirt_fault>(t.faults)[carry + before + (uint32_t)__popcll(m & mask_lt(lane))] = f;
            }
        }
        carry += total;
        __syncthreads();  // s_cnt is used again
    }
    if (threadIdx.x == 0 && t.n_faults) *t.n_faults = carry;
}

// Copy of one epoch's queued segments.  The copy is bound by the bytes it
// keeps in flight: hence at most 64 VGPRs, so that 8 wavefronts (the most a
// SIMD holds) stay resident, and short segments a 16-lane quarter each, so
// that a wavefront keeps up to four of them in flight.
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8)))
k_copy(DBatch b, uint32_t epoch, CopyTail tail) {
    uint32_t blk = blockIdx.x, blks = gridDim.x;
    if (tail.n) {
        if (blk == 0) {
            copy_tail(b.res, tail);
            return;
        }
        --blk;
        --blks;
    }
    const uint64_t waves = (uint64_t)blks * (blockDim.x >> 6);
    const uint64_t w0 = uniform_u64((uint64_t)blk * (blockDim.x >> 6) + (threadIdx.x >> 6));
    const bool nt = b.nontemporal != 0;
    const int lane = lane_id();
    const uint64_t pcap = b.part_cap;
    // lane p < 32: part p of the long queue; lane 32 + p: part p of the short
    // queue.  Exclusive scan of the part counts within each half, by the
    // workgroup's first wavefront for all of them: every count is a line of
    // its own, and a wavefront copies only a few segments.
    __shared__ uint32_t s_excl[64], s_n[2];
    if (threadIdx.x < 64) {
        uint32_t cnt = b.ctr[epoch].q[lane][0];
        if (cnt > pcap) cnt = (uint32_t)pcap;
        uint32_t incl = cnt;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const uint32_t t = shfl32(incl, (lane & 31) >= d ? lane - d : lane);
            if ((lane & 31) >= d) incl += t;
        }
        s_excl[lane] = incl - cnt;
        if ((lane & 31) == 31) s_n[lane >> 5] = incl;
    }
    __syncthreads();
    const uint32_t excl = s_excl[lane];
    const uint32_t nlong = uniform_u32(s_n[0]);
    const uint32_t nshort = uniform_u32(s_n[1]);
    const bool lo_half = lane < 32;
    // queue index s lies in the last part whose exclusive start is <= s
    // (parts are in lane order, so those lanes form a prefix of the half)

    // long segments: one per wavefront
    const DV_GLOBAL DSeg *segs = gp<const DV_GLOBAL DSeg>(b.segs);
    for (uint64_t s = w0; s < nlong; s += waves) {
        const int p = 63 - __clzll(__ballot(lo_half && excl <= (uint32_t)s));
        const uint64_t i = (uint64_t)p * pcap + (s - (uint32_t)__builtin_amdgcn_readlane((int)excl, p));
        const DSeg sg = segs[i];
        copy_wave((uint8_t *)uniform_u64(sg.dst), (const uint8_t *)uniform_u64(sg.src), uniform_u32(sg.len), nt);
        if (b.t_done && lane == 0) {
            uint32_t old = atomicSub(&b.pending[sg.req], 1u);
            if (old == 1) b.t_done[sg.req] = now_ns(b);
        }
    }
    // short segments: one per 16-lane quarter, four per wavefront per round
    const DV_GLOBAL DSeg *sh = gp<const DV_GLOBAL DSeg>(b.shorts);
    const int q = lane >> 4, l = lane & 15;
    for (uint64_t s0 = 4 * w0; s0 < nshort; s0 += 4 * waves) {
        uint64_t i = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t sk = (uint32_t)s0 + (uint32_t)k;
            const int p = 63 - __clzll(__ballot(!lo_half && excl <= sk) >> 32);
            const uint64_t ik = (uint64_t)p * pcap + (sk - (uint32_t)__builtin_amdgcn_readlane((int)excl, 32 + p));
            if (q == k) i = ik;
        }
        const bool mine = s0 + (uint64_t)q < nshort;
        uint64_t src = 0, dst = 0;
        uint32_t len = 0, req = 0;
        if (mine) {
            src = sh[i].src;
            dst = sh[i].dst;
            len = sh[i].len;
            req = sh[i].req;
        }
        copy_span<16>((uint8_t *)dst, (const uint8_t *)src, len, nt, l);
        if (mine && b.t_done && l == 0) {
            uint32_t old = atomicSub(&b.pending[req], 1u);
            if (old == 1) b.t_done[req] = now_ns(b);
        }
    }
}

// Spill pass of one epoch: the groups whose runs did not all fit the queues
// while translation ran during an earlier epoch's copies.  Launched after the
// previous epoch's copy and this epoch's translation, and before the next
// epoch's copy, so that it runs beside the epoch's own copy: every payload
// byte still moves in epoch order.  Each group is translated again (same
// results: page tables change only in A/D bits, which are OR-ed) and its
// wavefront copies every run of it; a run the copy kernel also moves gets the
// same bytes twice, since nothing else in the epoch touches them (batch
// precondition).
__global__ void __launch_bounds__(256) k_spill(DView v, DBatch b, uint64_t r0, uint64_t r1, uint32_t epoch) {
    extern __shared__ uint8_t smem[];
    const int wave = threadIdx.x >> 6;
    CEnt *cache = (CEnt *)smem + wave * kCacheWays;
    uint32_t *owner = (uint32_t *)((CEnt *)smem + (blockDim.x >> 6) * kCacheWays) + wave * kCacheWays;
    const uint32_t n = uniform_u32(*gp<const g_u32>(&b.ctr[epoch].spill_n));
    if (n == 0) return;
    if ((threadIdx.x & 63) < kCacheWays) cache[threadIdx.x & 63].key = ~0ull;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    GroupOut st = {0, 0, 0, 0, 0, 0, 0};
    devirt_request dummy = {};
    for (uint64_t i = (uint64_t)blockIdx.x * (blockDim.x >> 6) + (uint64_t)wave; i < n; i += nwaves) {
        const uint64_t e = uniform_u64(gp<const g_u64>(b.spill)[r0 + i]);
        if (e & kSpillOne) {  // a large request, alone
            process_group<false, false>(v, b, e & ~kSpillOne, 1, dummy, epoch, cache, owner, true, kLargeKeep, r0,
                                        b.ctr, st, nullptr);
        } else {  // a group; its large requests spill on their own
            const uint32_t gn = (uint32_t)((r1 - e) < b.group ? (r1 - e) : b.group);
            process_group<false, false>(v, b, e, gn, dummy, epoch, cache, owner, true, kLargeSkip, r0, b.ctr, st,
                                        nullptr);
        }
    }
    flush_counters(b.counters, st);
}

__global__ void __launch_bounds__(64) k_plain(DView v, DBatch b, devirt_request req, int inline_copy) {
    __shared__ CEnt cache[kCacheWays];
    __shared__ uint32_t owner[kCacheWays];
    if (threadIdx.x < kCacheWays) cache[threadIdx.x].key = ~0ull;
    if (threadIdx.x < 2 * kQParts) b.ctr[0].q[threadIdx.x][0] = 0;
    if (threadIdx.x == 0) *b.t0 = wall_clock64();
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    GroupOut st = {0, 0, 0, 0, 0, 0, 0};
    process_group<true, false>(v, b, 0, 1, req, 0, cache, owner, inline_copy != 0, kLargeKeep, 0, b.ctr, st, nullptr);
    flush_counters(b.counters, st);
}

// ------------------------------------------------- one request, one workgroup
// The memslots of one VM as a wavefront holds them: lane i has slot i.
struct SlotLanes {
    uint64_t gpa, end, off;
};

// Arena offset of the (few) table addresses `table` of the lanes with `run`
// set: each distinct one is looked up once, by all lanes together (the slots
// are sorted, so the ones that start at or below it form a prefix).  Whole
// wavefront.  0, or the code of a table that cannot be reached.
__device__ __forceinline__ uint32_t table_xlat(const DVm &vm, const SlotLanes &sl, bool run, uint64_t table,
                                               EptUpper &up, uint64_t &th) {
    uint32_t code = DEVIRT_OK;
    if (vm.ept_root != kNoEpt) {
        if (run) code = gpa_xlat(vm, table, kNeedTable, th, &up);
        return code;
    }
    uint64_t todo = __ballot(run);
    while (todo) {
        const int lead = __ffsll((unsigned long long)todo) - 1;
        const uint64_t g = uniform_u64(shfl64(table, lead));
        const uint64_t below = __ballot(sl.gpa <= g);
        const int k = below ? 63 - __clzll(below) : 0;
        const uint64_t gpa = uniform_u64(shfl64(sl.gpa, k)), end = uniform_u64(shfl64(sl.end, k));
        const uint64_t off = uniform_u64(shfl64(sl.off, k));
        const bool mine = run && table == g;
        if (mine) {
            th = off + (g - gpa);
            if (!below || g >= end) code = DEVIRT_NO_MEMSLOT;
        }
        todo &= ~__ballot(mine);
    }
    return code;
}

// What a lane's walk of one page found: the outcome, the arena offset of its
// first byte, and the entries read (arena offset and low dword, top level
// first; the first `n` of them lie on the path).
template <int LEVELS>
struct PageWalk {
    uint32_t code, level, leaf;
    uint64_t hpa;
    uint64_t off[LEVELS];
    uint32_t lo[LEVELS];
};

// Every lane with `act` set walks its own page: neighbouring lanes share the
// upper levels, whose loads then fall on one address.  Whole wavefront.
template <int LEVELS>
__device__ __forceinline__ void page_walk(const DVm &vm, const SlotLanes &sl, const DSlot *slots, uint64_t cr3,
                                          uint64_t gva, bool write, bool act, PageWalk<LEVELS> &r) {
    bool run = act;
    uint32_t u = 1, w = 1;
    uint64_t table = LEVELS == 3 ? (cr3 & 0xFFFFFFE0ull) : (cr3 & kAddrMask), gpa = 0;
    r.code = DEVIRT_OK;
    r.level = r.leaf = 0;
    r.hpa = 0;
    EptUpper up;
#pragma unroll
    for (int i = 0; i < LEVELS; ++i) {
        const int lvl = LEVELS - i;
        const uint32_t sh = 12 + 9 * (lvl - 1);
        const bool root = LEVELS == 3 && lvl == 3;  // a PAE root entry: no rights, no accessed bit
        uint64_t th = 0;
        const uint32_t xc = table_xlat(vm, sl, run, table, up, th);
        r.off[i] = ~0ull;
        r.lo[i] = 0;
        if (run) {
            if (xc) {
                r.code = xc;
                r.level = lvl;
                run = false;
            } else {
                r.off[i] = th + 8 * (root ? ((gva >> 30) & 3) : ((gva >> sh) & 511));
                const uint64_t e = load_entry(vm.arena, r.off[i]);
                r.lo[i] = (uint32_t)e;
                if (!root) {
                    u &= (uint32_t)(e >> 2) & 1u;
                    w &= (uint32_t)(e >> 1) & 1u;
                }
                const uint64_t low = (1ull << sh) - 1;
                const bool ps = !root && lvl >= 2 && (e & kPS);
                run = false;
                if (!(e & kP)) {
                    r.code = DEVIRT_NOT_PRESENT;
                    r.level = lvl;
                } else if ((LEVELS == 3 && (e & (root ? kPaeRootRsvd : kPaeRsvd))) ||
                           (ps && (lvl >= 4 || (e & low & ~0x1FFFull)))) {  // a large leaf's bits above the PAT bit
                    r.code = DEVIRT_RESERVED;
                    r.level = lvl;
                } else if (lvl == 1 || ps) {
                    r.leaf = lvl;
                    gpa = (e & kAddrMask & ~low) | (gva & low);
                } else {
                    table = e & kAddrMask;
                    run = true;
                }
            }
        }
    }
    if (r.leaf) {
        if (!u) {
            r.code = DEVIRT_PROT_USER;
            r.level = r.leaf;
        } else if (write && !w) {
            r.code = DEVIRT_PROT_WRITE;
            r.level = r.leaf;
        } else if (vm.ept_root != kNoEpt) {
            r.code = gpa_xlat(vm, gpa, write ? kNeedW : kNeedR, r.hpa, &up);
        } else {  // binary search of the slots in LDS
            uint32_t a = 0, b = vm.nslots;
            while (a < b) {
                const uint32_t mid = (a + b) >> 1;
                if (slots[mid].gpa <= gpa)
                    a = mid + 1;
                else
                    b = mid;
            }
            if (a == 0 || gpa >= slots[a - 1].end)
                r.code = DEVIRT_NO_MEMSLOT;
            else
                r.hpa = slots[a - 1].arena_off + (gpa - slots[a - 1].gpa);
        }
    }
}

// Known defect, kept so that every path leaves the same bytes: process_group's
// run of a pass's last 2 MiB region ends at lane 30 (a shift by 64 in mask_lt),
// so a last region that starts in lane 31 or later gets its accessed and dirty
// bits above level 1 only from a pass that continues it.  The kernels that took
// over its requests one at a time leave out the same bits: whether this lane's
// page lies in such a region.  A pass is 64 consecutive pages, a lane each; a
// region starts anew behind a page that is not walked.  To be mended in all of
// them at once.
__device__ __forceinline__ bool last_head_lost(uint64_t gva, bool walked) {
    const int lane = lane_id();
    const uint64_t wm = __ballot(walked), p = gva >> 12;
    const bool head = walked && (lane == 0 || !((wm >> (lane - 1)) & 1) || ((p - 1) ^ p) >> 9 != 0);
    const uint64_t heads = __ballot(head);
    const int last = heads ? 63 - __clzll(heads) : 0;
    return last >= 31 && lane >= last;
}

// The same for page c of a request that shared process_group's passes with the
// others of its group: the request's pages have places [start, start + total)
// among the group's; follows: a later request of the group has pages, which
// then begin at start + total.
__device__ __forceinline__ bool last_head_lost(uint64_t gva, uint32_t c, uint32_t total, uint32_t start, bool follows) {
    const uint32_t p = start + c, pass = p & ~63u, end = start + total;
    if (follows && end <= pass + 63) return false;
    const uint32_t first = start > pass ? start : pass, last = end - 1 < pass + 63 ? end - 1 : pass + 63;
    const uint64_t p0 = gva >> 12, region = (p0 + (last - start)) & ~511ull;  // the last region's first page
    const uint32_t r = start + (region > p0 ? (uint32_t)(region - p0) : 0u);
    const uint32_t head = (r > first ? r : first) - pass;
    return head >= 31 && p - pass >= head;
}

// The process's translation cache as one request finds it (section 4.2): a
// FIFO whose slots lie in lanes 0..cap-1 of every wavefront.  The request's
// pages are distinct and ascend, so what a lookup in page order finds depends
// on the slots held before it alone: every page that was not held when its
// turn came is inserted, and slot q of the queue leaves with insertion number
// cap - n + q + 1.
struct FifoLook {
    uint64_t gen;
    uint64_t v, h;           // the lane's slot: page number, arena offset of the page
    uint32_t idx;            // the request's page that it holds (kNone: none of them)
    uint32_t n, head, written, cap;
    uint64_t hits, misses;   // counted so far
    uint64_t held;           // slots that are held when their page's turn comes
    uint64_t hit;            // slots whose page is not walked
};

// Pages inserted before page i's turn (uniform).
__device__ __forceinline__ uint32_t fifo_inserts(const FifoLook &f, uint32_t i) {
    return i - (uint32_t)__popcll(f.held & __ballot(f.idx < i));
}

__device__ __forceinline__ void fifo_load(const PlainArgs &a, FifoLook &f) {
    const uint32_t lane = (uint32_t)lane_id();
    const DFifo *q = a.fifo;
    f.gen = *gp<const g_u64>(&q->gen);
    f.n = *gp<const g_u32>(&q->n);
    f.head = *gp<const g_u32>(&q->head);
    f.written = *gp<const g_u32>(&q->written);
    f.hits = *gp<const DV_GLOBAL unsigned long long>(&q->hits);
    f.misses = *gp<const DV_GLOBAL unsigned long long>(&q->misses);
    f.v = ~0ull;
    f.h = 0;
    if (lane < a.fifo_entries) {
        f.v = gp<const g_u64>(q->vpn)[lane];
        f.h = gp<const g_u64>(q->hpa)[lane];
    }
}

__device__ __forceinline__ void fifo_look(const PlainArgs &a, uint32_t total, FifoLook &f) {
    const uint32_t lane = (uint32_t)lane_id(), cap = a.fifo_entries;
    f.cap = cap;
    f.n = uniform_u32(f.n);
    f.head = uniform_u32(f.head);
    f.written = uniform_u32(f.written);
    if (uniform_u64(f.gen) != a.xlat_gen) f.n = f.head = f.written = 0;  // emptied since
    if (f.n > cap) {  // it had more slots: the ones that are left, oldest first
        f.head += f.n;
        f.n = cap;
    }
    if (f.head >= cap) f.head %= cap;
    const uint32_t place = lane >= f.head ? lane - f.head : lane + cap - f.head;  // in the queue, oldest first
    const uint64_t d = f.v - (a.gva >> 12);
    const bool in = lane < cap && place < f.n && d < total;
    f.idx = in ? (uint32_t)d : kNone;
    f.held = f.hit = 0;
    const uint64_t im = __ballot(in);
    if (!im) return;
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t k = 0; k < kFifoMax; ++k)
        rank += (uint32_t)__builtin_amdgcn_readlane((int)f.idx, (int)k) < f.idx ? 1u : 0u;
    const uint32_t leaves = cap - f.n + place + 1;
    // held, were every slot before it held: most often so, or none after it is
    f.held = __ballot(in && f.idx - rank < leaves);
    const uint32_t held = (uint32_t)__popcll(f.held);
    if (__ballot(((f.held >> lane) & 1) && rank >= held)) {
        f.held = 0;
        for (uint32_t r = 0; r < (uint32_t)__popcll(im); ++r)  // in page order
            f.held |= __ballot(in && rank == r && f.idx - (uint32_t)__popcll(f.held) < leaves);
    }
    // a page is left unwalked if its slot is held as the page's pass of 64 begins
    uint64_t pass = f.held;
    for (uint64_t m = im & ~f.held; m; m &= m - 1) {
        const int k = __ffsll((unsigned long long)m) - 1;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)f.idx, k) & ~63u;
        if (fifo_inserts(f, first) < (uint32_t)__builtin_amdgcn_readlane((int)leaves, k)) pass |= 1ull << k;
    }
    f.hit = a.dir ? pass & f.written : pass;
}

// Shared state of k_plain_walk's workgroup.
struct PlainShared {
    DSlot slots[kSlotRow];
    uint64_t page[64 * kPlainWaves];  // a round's pages: address of their first byte in guest memory
    uint32_t ff;                      // the request's first faulting page (kNone: none)
    uint32_t fcode, flevel;
    uint64_t flo;
    uint64_t fifo_v[kFifoMax], fifo_h[kFifoMax];  // what each slot of the translation cache was given last
};

template <int LEVELS, bool FIFO>
__device__ void plain_pages(const PlainArgs &a, const DVm &vm, const SlotLanes &sl, FifoLook &fifo, PlainShared &sh) {
    const int lane = lane_id();
    const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint64_t end = a.gva + a.len;
    const uint32_t total = (uint32_t)(((end - 1) >> 12) - (a.gva >> 12) + 1);
    uint32_t ff = kNone;
    if (FIFO) fifo_look(a, total, fifo);
    for (uint32_t base = 0; base < total && ff == kNone; base += 64 * waves) {
        const uint32_t c = base + threadIdx.x;
        const uint64_t page = (a.gva & ~0xFFFull) + ((uint64_t)c << 12);
        const uint64_t lo = page > a.gva ? page : a.gva, hi = page + 4096 < end ? page + 4096 : end;
        const bool act = c < total;
        PageWalk<LEVELS> w;
        w.code = DEVIRT_OK;
        w.leaf = 0;
        bool walk = act;
        uint64_t held = 0;  // which of the 64 pages are held when their turn comes
        if (FIFO) {
            const uint32_t at = fifo.idx - (base + 64 * wave);
            const uint64_t here = (fifo.held | fifo.hit) & __ballot(fifo.idx != kNone && at < 64);
            uint64_t hit = 0;
            for (uint64_t m = here; m; m &= m - 1) {
                const int k = __ffsll((unsigned long long)m) - 1;
                const int l = __builtin_amdgcn_readlane((int)at, k);
                held |= ((fifo.held >> k) & 1) << l;
                hit |= ((fifo.hit >> k) & 1) << l;
            }
            if (hit) {  // their places go from the slots' lanes to the pages'
                walk = act && !((hit >> lane) & 1);
                if ((here & fifo.hit) >> lane & 1) sh.page[64 * wave + at] = fifo.h;
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        }
        if (FIFO ? __ballot(walk) != 0 : base + 64 * wave < total)
            page_walk<LEVELS>(vm, sl, sh.slots, a.cr3, lo, a.dir != 0, walk, w);
        if (FIFO && act && !walk) w.hpa = sh.page[threadIdx.x] + (lo & 0xFFFull);
        // the first fault of the round, agreed before any byte or bit changes
        const uint64_t fm = __ballot(act && w.code != DEVIRT_OK);
        if (fm && lane == 0) atomicMin(&sh.ff, base + 64 * wave + (uint32_t)__ffsll((unsigned long long)fm) - 1);
        const uint64_t gptr = (uint64_t)(uintptr_t)vm.arena + w.hpa;
        if (a.inline_copy) sh.page[threadIdx.x] = gptr;
        __syncthreads();
        ff = uniform_u32(*(volatile uint32_t *)&sh.ff);
        if (act && c == ff) {
            sh.fcode = w.code;
            sh.flevel = w.level;
            sh.flo = lo;
        }
        const uint32_t stop = ff < total ? ff : total;  // pages [base, stop) of this round are copied
        if (a.inline_copy) {  // a wavefront per page
            for (uint32_t k = base + wave; k < stop && k < base + 64 * waves; k += waves) {
                const uint64_t pk = (a.gva & ~0xFFFull) + ((uint64_t)k << 12);
                const uint64_t kl = pk > a.gva ? pk : a.gva, kh = pk + 4096 < end ? pk + 4096 : end;
                const uint64_t g = uniform_u64(sh.page[k - base]), h = a.host + (kl - a.gva);
                copy_wave((uint8_t *)(a.dir ? g : h), (const uint8_t *)(a.dir ? h : g), (uint32_t)(kh - kl),
                          a.nontemporal != 0);
            }
        } else if (act && c < stop) {
            const uint64_t h = a.host + (lo - a.gva);
            DSeg sg;
            sg.src = a.dir ? h : gptr;
            sg.dst = a.dir ? gptr : h;
            sg.len = (uint32_t)(hi - lo);
            sg.req = 0;
            sg.pad = 0;
            gp<DV_GLOBAL DSeg>(a.segs)[c] = sg;
        }
        // A/D of the copied pages' paths: an entry shared with the previous
        // lane is left to that lane
        if (base + 64 * wave < stop) {
            const bool lost = last_head_lost(page, walk);
#pragma unroll
            for (int i = 0; i < LEVELS; ++i) {
                const int lvl = LEVELS - i;
                const uint64_t prev = shfl64(w.off[i], lane > 0 ? lane - 1 : 0);
                if (LEVELS == 3 && lvl == 3) continue;
                const uint32_t want = (uint32_t)kA | (w.leaf == (uint32_t)lvl && a.dir ? (uint32_t)kD : 0u);
                if (walk && c < stop && lvl >= (int)w.leaf && (lane == 0 || prev != w.off[i]) &&
                    (w.lo[i] & want) != want && !(lvl > 1 && lost))
                    or_entry(vm.arena, w.off[i], want);
            }
            if (FIFO) {  // the last pages inserted so far, each in its slot
                const uint32_t to = stop < base + 64 * waves ? stop : base + 64 * waves;
                const bool near = act && c < to && !((held >> lane) & 1) && c + 2 * fifo.cap >= to;
                if (__ballot(near)) {
                    const uint32_t t = fifo_inserts(fifo, base + 64 * wave) + (uint32_t)lane -
                                       (uint32_t)__popcll(held & mask_lt(lane));
                    if (near && t + fifo.cap >= fifo_inserts(fifo, to)) {
                        const uint32_t slot = (fifo.head + fifo.n + t) % fifo.cap;
                        sh.fifo_v[slot] = page >> 12;
                        sh.fifo_h[slot] = w.hpa - (lo & 0xFFFull);
                    }
                }
            }
        }
        if (base + 64 * waves < total) __syncthreads();  // sh.page and sh.ff are used again
    }
    if (!a.inline_copy && threadIdx.x < 2 * kQParts)
        a.ctr->q[threadIdx.x][0] = threadIdx.x ? 0 : (ff < total ? ff : total);
    if (FIFO || ff != kNone) __syncthreads();  // workgroup-uniform
    if (FIFO && wave == 0) {
        const uint32_t cap = fifo.cap, stop = ff < total ? ff : total, seen = ff < total ? ff + 1 : total;
        const uint32_t ins = fifo_inserts(fifo, stop), l = (uint32_t)lane;
        const bool mine = (fifo.held >> lane) & 1, wr = (fifo.written >> (l & 31)) & 1;
        const uint32_t hits = (uint32_t)__popcll(__ballot(mine && fifo.idx < seen && (!a.dir || wr)));
        const bool fresh = l < cap && (ins >= cap || (l + 2 * cap - (fifo.head + fifo.n) % cap) % cap < ins);
        const uint64_t wm = __ballot(l < cap && (fresh ? a.dir != 0 : wr || (a.dir && mine && fifo.idx < stop)));
        DFifo *q = a.fifo;
        if (l < cap) {
            gp<g_u64>(q->vpn)[l] = fresh ? sh.fifo_v[l] : fifo.v;
            gp<g_u64>(q->hpa)[l] = fresh ? sh.fifo_h[l] : fifo.h;
        }
        if (lane == 0) {
            const uint32_t all = fifo.n + ins;
            *gp<g_u32>(&q->written) = (uint32_t)wm;
            *gp<g_u32>(&q->n) = all < cap ? all : cap;
            *gp<g_u32>(&q->head) = all > cap ? (fifo.head + (all - cap)) % cap : fifo.head;
            *gp<g_u64>(&q->gen) = a.xlat_gen;
            *gp<DV_GLOBAL unsigned long long>(&q->hits) = fifo.hits + hits;
            *gp<DV_GLOBAL unsigned long long>(&q->misses) = fifo.misses + (seen - hits);
        }
    }
    if (threadIdx.x == 0) {
        devirt_result r;
        r.pad = 0;
        r.bytes_done = ff == kNone ? a.len : sh.flo - a.gva;
        r.fault_gva = ff == kNone ? 0 : sh.flo;
        r.code = ff == kNone ? (uint32_t)DEVIRT_OK : sh.fcode;
        r.level = ff == kNone ? (uint16_t)0 : (uint16_t)sh.flevel;
        *gp<DV_GLOBAL devirt_result>(a.res) = r;
    }
}

// One request by one workgroup: a round walks 64 pages a wavefront, agrees on
// the request's first faulting page, then sets A/D bits and either copies the
// pages itself (inline: every walk ends before any byte moves) or lists them
// for k_copy.
//
// Bound by latency: the dependent loads of one walk, each level waiting for
// the one above.  So every page of a round is walked at once by a lane of its
// own, without a cache between the levels; the memslots come with the VM's
// record, a lane each, and a table's slot is found by one ballot; and what the
// process id names is a kernel argument.  Back-to-back calls, against one
// wavefront that took the request 64 pages at a time through the walk cache
// and copied it alone up to 16 pages: 24 B 8.2 -> 5.5 us, 32 KiB 13.4 -> 5.8,
// 100 KB 12.7 -> 6.7, 1 MiB 29.7 -> 8.8, 4,147,200 B 76.9 -> 10.2; behind an
// EPT 24 B 8.9 -> 6.3, 4,147,200 B 88.8 -> 12.7.
//
// FIFO: with the process's translation cache.  Its lookups one after the other
// (a ballot and a dozen steps a page, by one wavefront) are replaced by what
// they come to, see FifoLook; back-to-back calls, 10 entries: 24 B that are
// held 7.4 -> 4.8 us, 32 KiB held 11.4 -> 5.4, 100 KB 25.9 -> 9.0, 1 MiB 111.6
// -> 11.7, 4,147,200 B 377.7 -> 14.3, behind an EPT 396.9 -> 15.9.
template <bool FIFO>
__global__ void __launch_bounds__(64 * kPlainWaves) k_plain_walk(PlainArgs a) {
    __shared__ PlainShared sh;
    if (a.code0 || a.len == 0) {
        if (threadIdx.x == 0) {
            devirt_result r;
            r.bytes_done = 0;
            r.fault_gva = a.code0 ? a.gva : 0;
            r.code = a.code0;
            r.level = 0;
            r.pad = 0;
            *gp<DV_GLOBAL devirt_result>(a.res) = r;
        }
        if (!a.inline_copy && threadIdx.x < 2 * kQParts) a.ctr->q[threadIdx.x][0] = 0;
        return;
    }
    typedef DV_GLOBAL DSlot g_slot;
    const g_slot *row = gp<const g_slot>(a.v.slots) + (uint64_t)a.vm * kSlotRow;
    SlotLanes sl;
    sl.gpa = row[lane_id()].gpa;
    sl.end = row[lane_id()].end;
    sl.off = row[lane_id()].arena_off;
    const DVm vm = load_vm(a.v, a.vm, false);
    FifoLook fifo;
    if (FIFO) fifo_load(a, fifo);  // with the VM's record, not behind it
    if (threadIdx.x < kSlotRow) sh.slots[threadIdx.x] = DSlot{sl.gpa, sl.end, sl.off};
    if (threadIdx.x == 0) sh.ff = kNone;
    __syncthreads();
    if (a.levels == 5)
        plain_pages<5, FIFO>(a, vm, sl, fifo, sh);
    else if (a.levels == 4)
        plain_pages<4, FIFO>(a, vm, sl, fifo, sh);
    else
        plain_pages<3, FIFO>(a, vm, sl, fifo, sh);
}

// ------------------------------------------- small batches, one request a wave
// The pages [base, base + 64 * waves) of one request, 64 a wavefront (`part`:
// which 64 this wavefront takes): walk, the request's first fault, A/D bits,
// copy segments.  ff: shared by the wavefronts of a workgroup that walk one
// request together, null where a wavefront is alone.  Returns the first
// faulting page (kNone: none in these pages); its lane's outcome is left in f.
struct OneFault {
    uint32_t code, level;
    uint64_t lo;
};

template <int LEVELS>
__device__ uint32_t one_pages(const DBatch &b, const DVm &vm, const SlotLanes &sl, const DSlot *slots, uint64_t cr3,
                              uint64_t gva, uint64_t host, uint32_t len, bool dir, uint32_t req, uint32_t total,
                              uint32_t start, bool follows, uint32_t base, uint32_t part, uint32_t qpart, bool direct,
                              uint32_t *ff, OneFault *f) {
    const int lane = lane_id();
    const uint32_t c = base + 64 * part + (uint32_t)lane;
    const uint64_t end = gva + len;
    const uint64_t page = (gva & ~0xFFFull) + ((uint64_t)c << 12);
    const uint64_t lo = page > gva ? page : gva, hi = page + 4096 < end ? page + 4096 : end;
    const bool act = c < total;
    PageWalk<LEVELS> w;
    w.code = DEVIRT_OK;
    w.leaf = 0;
    if (base + 64 * part < total) page_walk<LEVELS>(vm, sl, slots, cr3, lo, dir, act, w);
    const uint64_t fm = __ballot(act && w.code != DEVIRT_OK);
    uint32_t first = fm ? base + 64 * part + (uint32_t)__ffsll((unsigned long long)fm) - 1 : kNone;
    if (ff) {
        if (fm && lane == 0) atomicMin(ff, first);
        __syncthreads();
        first = uniform_u32(*(volatile uint32_t *)ff);
    }
    if (act && c == first) *f = OneFault{w.code, w.level, lo};
    const bool copied = act && c < first;
    const uint64_t cm = __ballot(copied);
    if (!cm) return first;
    // copy segments: runs of pages that follow one another in guest memory
    const uint64_t gptr = (uint64_t)(uintptr_t)vm.arena + w.hpa, hptr = host + (lo - gva);
    uint32_t n = (uint32_t)(hi - lo);
    bool head = copied;
    if (b.seg_chunks > 1) {
        const int prev = lane > 0 ? lane - 1 : 0;
        const uint64_t p_end = shfl64(gptr, prev) + shfl32(n, prev);
        const bool cont = copied && lane > 0 && p_end == gptr && c % b.seg_chunks != 0;
        head = copied && !cont;
        const uint64_t ends = ~__ballot(cont) & ~mask_le(lane);
        const int last = ends ? __ffsll((unsigned long long)ends) - 2 : 63;  // the run's last page
        n = (uint32_t)(shfl64(hi, head ? last : lane) - lo);
    }
    const uint64_t src = dir ? hptr : gptr, dst = dir ? gptr : hptr;
    const bool small = head && !direct && n <= b.inline_bytes;
    const bool is_short = n <= kShortRun, queue = head && !direct && !small;
    const uint64_t lm = __ballot(queue && !is_short), sm = __ballot(queue && is_short);
    uint32_t lbase = 0, sbase = 0;
    if (lane == 0) {
        if (lm) lbase = atomicAdd(&b.ctr->q[qpart][0], (uint32_t)__popcll(lm));
        if (sm) sbase = atomicAdd(&b.ctr->q[kQParts + qpart][0], (uint32_t)__popcll(sm));
    }
    // A/D of the copied pages' paths, while the queue places are on their way:
    // an entry shared with the previous lane is left to that lane
    const bool lost = last_head_lost(gva, c, total, start, follows);
    const bool lost_before = ((__ballot(lost) << 1) >> lane) & 1;
#pragma unroll
    for (int i = 0; i < LEVELS; ++i) {
        const int lvl = LEVELS - i;
        const uint64_t po = shfl64(w.off[i], lane > 0 ? lane - 1 : 0);
        if (LEVELS == 3 && lvl == 3) continue;
        const uint32_t want = (uint32_t)kA | (w.leaf == (uint32_t)lvl && dir ? (uint32_t)kD : 0u);
        if (copied && lvl >= (int)w.leaf && (lane == 0 || po != w.off[i] || lost_before) && (w.lo[i] & want) != want &&
            !(lvl > 1 && lost))
            or_entry(vm.arena, w.off[i], want);
    }
    if (small) copy_lane((uint8_t *)dst, (const uint8_t *)src, n);
    bool full = head && direct;
    if (lm | sm) {
        lbase = uniform_u32(shfl32(lbase, 0));
        sbase = uniform_u32(shfl32(sbase, 0));
        if (queue) {
            const uint64_t pos = is_short ? (uint64_t)sbase + __popcll(sm & mask_lt(lane))
                                          : (uint64_t)lbase + __popcll(lm & mask_lt(lane));
            full = pos >= b.part_cap;
            if (!full) {
                DSeg sg;
                sg.src = src;
                sg.dst = dst;
                sg.len = n;
                sg.req = req;
                sg.pad = 0;
                gp<DV_GLOBAL DSeg>(is_short ? b.shorts : b.segs)[qpart * b.part_cap + pos] = sg;
            }
        }
    }
    for (uint64_t m = __ballot(full); m; m &= m - 1) {  // no queue, or it is full: the wavefront copies the run
        const int l = __ffsll((unsigned long long)m) - 1;
        copy_wave((uint8_t *)uniform_u64(shfl64(dst, l)), (const uint8_t *)uniform_u64(shfl64(src, l)),
                  uniform_u32(shfl32(n, l)), b.nontemporal != 0);
    }
    return first;
}

// A one-epoch batch so small that each request can have a wavefront to itself.
// Bound by the latency of one wavefront: its own instructions and cross-lane
// steps as much as its loads.  k_translate_groups spends about 1,200 vector
// instructions and 92 LDS operations on a wavefront's first pass, most of them
// to find which request a lane's page belongs to and to hand its fields round;
// here the request is the wavefront's, its fields are scalars, and the walk is
// that of the per-request copy.  A request of more than kOneAlone pages is
// walked by the workgroup's wavefronts together, 64 pages each a round.
// The rest of a request's group is looked at only for the accessed bits that
// it would have been left without there, see last_head_lost.  The kernel's
// time in us, k_translate_groups and this: 2,048 requests, one in a hundred of
// 4,147,200 bytes, 78.2 and 28.9; 8,191 of up to 64 KiB 15.3 and 17.1, which
// is why larger batches are not translated so.
constexpr uint32_t kOneAlone = 128;
struct OneShared {
    DSlot slots[4][kSlotRow];
    uint32_t big[4];   // the wavefront's request has more than kOneAlone pages
    uint32_t ff;
    OneFault f;
};

__device__ __forceinline__ void one_result(devirt_result *res, uint64_t i, uint64_t gva, uint32_t len, uint32_t code0,
                                           uint32_t ff, const OneFault &f) {
    devirt_result r;
    r.bytes_done = code0 ? 0 : ff == kNone ? len : f.lo - gva;
    r.fault_gva = code0 ? gva : ff == kNone ? 0 : f.lo;
    r.code = code0 ? code0 : ff == kNone ? (uint32_t)DEVIRT_OK : f.code;
    r.level = code0 || ff == kNone ? (uint16_t)0 : (uint16_t)f.level;
    r.pad = 0;
    gp<DV_GLOBAL devirt_result>(res)[i] = r;
}

// direct: the wavefront copies its request itself and nothing is queued.
__global__ void __launch_bounds__(256) k_translate_one(DView v, DBatch b, uint64_t n, int direct) {
    __shared__ OneShared sh;
    const int lane = lane_id();
    const uint32_t wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint64_t w0 = (uint64_t)blockIdx.x * waves;
    const uint32_t qpart = (uint32_t)((w0 + wave) % kQParts);
    if (threadIdx.x < 4) sh.big[threadIdx.x] = 0;
    __syncthreads();
    // one request: of this wavefront (team == 0), or of the workgroup
    const auto translate = [&](uint64_t i, uint32_t part, uint32_t team) {
        // the requests of its group, a lane each, for the places of its pages
        const int own = b.group == 1 ? 0 : (int)((uint32_t)i % b.group);
        const uint64_t g0 = i - (uint64_t)own;
        const uint32_t gn = n - g0 < b.group ? (uint32_t)(n - g0) : b.group;
        u32x4 qa{0, 0, 0, 0}, qb{0, 0, 0, 0};
        if ((uint32_t)lane < gn) {
            const g_u32x4 *p = gp<const g_u32x4>(b.reqs + g0) + 2 * lane;
            qa = p[0];
            qb = p[1];
        }
        const auto mine32 = [&](uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, own); };
        const uint64_t gva = ((uint64_t)mine32(qa.y) << 32) | mine32(qa.x);
        const uint64_t host = ((uint64_t)mine32(qa.w) << 32) | mine32(qa.z);
        const uint32_t len = mine32(qb.x), asid = mine32(qb.y);
        const bool dir = (mine32(qb.z) & 0xFF) != 0;
        uint32_t code0 = DEVIRT_OK, ff = kNone;
        OneFault f{0, 0, 0};
        if (asid >= v.nproc) {
            code0 = DEVIRT_INVALID;
        } else if (len) {
            const DV_GLOBAL DProc *pp = gp<const DV_GLOBAL DProc>(v.procs) + asid;
            const uint32_t levels = uniform_u32(pp->levels), vmi = uniform_u32(pp->vm);
            const uint64_t cr3 = uniform_u64(pp->cr3), lim = user_limit(levels);
            if (gva >= lim || (uint64_t)len > lim - gva) {
                code0 = DEVIRT_NONCANONICAL;
            } else {
                const uint32_t total = (uint32_t)(((gva + len - 1) >> 12) - (gva >> 12) + 1);
                uint32_t start = 0;
                bool follows = false;
                if (gn > 1) {
                    const uint64_t og = ((uint64_t)qa.y << 32) | qa.x;
                    uint32_t pages = 0;
                    if ((uint32_t)lane < gn && qb.y < v.nproc && qb.x) {
                        const uint64_t ol = user_limit(gp<const DV_GLOBAL DProc>(v.procs)[qb.y].levels);
                        if (og < ol && (uint64_t)qb.x <= ol - og)
                            pages = (uint32_t)(((og + qb.x - 1) >> 12) - (og >> 12) + 1);
                    }
                    for (int k = 0; k < own; ++k) start += (uint32_t)__builtin_amdgcn_readlane((int)pages, k);
                    follows = (__ballot(pages != 0) & ~mask_le(own)) != 0;
                }
                if (!team && waves > 1 && total > kOneAlone) {
                    if (lane == 0) sh.big[wave] = 1;
                    return;
                }
                const DV_GLOBAL DSlot *row = gp<const DV_GLOBAL DSlot>(v.slots) + (uint64_t)vmi * kSlotRow + lane;
                SlotLanes sl;
                sl.gpa = row->gpa;
                sl.end = row->end;
                sl.off = row->arena_off;
                const DVm vm = load_vm(v, vmi, false);
                DSlot *slots = sh.slots[wave];
                slots[lane] = DSlot{sl.gpa, sl.end, sl.off};
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                const uint32_t step = team ? 64 * waves : 64;
                OneFault *fo = team ? &sh.f : nullptr;
                OneFault mine{0, 0, 0};
                for (uint32_t base = 0; base < total && ff == kNone; base += step) {
                    uint32_t *sf = team ? &sh.ff : nullptr;
                    OneFault *out = team ? fo : &mine;
                    if (levels == 5)
                        ff = one_pages<5>(b, vm, sl, slots, cr3, gva, host, len, dir, (uint32_t)i, total, start,
                                          follows, base, part, qpart, direct != 0, sf, out);
                    else if (levels == 4)
                        ff = one_pages<4>(b, vm, sl, slots, cr3, gva, host, len, dir, (uint32_t)i, total, start,
                                          follows, base, part, qpart, direct != 0, sf, out);
                    else
                        ff = one_pages<3>(b, vm, sl, slots, cr3, gva, host, len, dir, (uint32_t)i, total, start,
                                          follows, base, part, qpart, direct != 0, sf, out);
                    if (team) __syncthreads();  // ff is read by every wavefront before the next round adds to it
                }
                if (ff != kNone) {
                    if (team) {
                        f = sh.f;
                    } else {  // the faulting page's lane has it
                        const int l = (int)(ff & 63);
                        f.code = shfl32(mine.code, l);
                        f.level = shfl32(mine.level, l);
                        f.lo = shfl64(mine.lo, l);
                    }
                }
            }
        }
        if (lane == 0 && part == 0) one_result(b.res, i, gva, len, code0, ff, f);
    };
    if (w0 + wave < n) translate(w0 + wave, 0, 0);
    __syncthreads();
    for (uint32_t k = 0; k < waves; ++k) {
        if (!*(volatile uint32_t *)&sh.big[k]) continue;  // uniform
        if (threadIdx.x == 0) sh.ff = kNone;
        __syncthreads();
        translate(w0 + k, wave, 1);
        __syncthreads();
    }
}

// ---------------------------------------------------------- translate only
// One process, one lane per address.  A workgroup keeps in LDS what every
// address of the process goes through: the VM's guest-physical space as one
// word per 2 MiB block, and the process's top-level table.  The words of a
// memslot VM come from the device table; those of a VM with an EPT are made
// here from its level-2 entries, so that both kinds of VM are looked up alike:
//   delta / 4 KiB << 2 | 2   the whole block lies at gpa + delta (EPT: readable
//                            and writable)
//   pt / 4 KiB << 2 | 3      EPT: a page table at arena offset pt maps the block
//   1                        search the slots, or walk the EPT
//   0                        no slot overlaps the block
//
// Large calls are bound by HBM (the addresses read and the records written),
// small ones by the chain of dependent loads.  What stood between a large call
// and HBM was instructions, about 450 per 64 addresses, half of them table
// lookups: a region now costs one 16-byte LDS load (its level-2 table already
// in arena offsets), a table or data page one LDS word, an address without a
// top-level entry no load at all; the depth and the accessed/dirty variant are
// template arguments.  4 Mi addresses, 4-level: 68.3 -> 33.7 us (2.5 -> 5.0
// TB/s of addresses and records); behind an EPT, where each lookup was a walk
// of four loads, 128.7 -> 39.0; 1000 addresses 6.4 -> 4.9.
//
// Accessed/dirty bits: every lane that found a shared entry clear used to
// issue its own atomic, on one address (a first pass of 4 Mi addresses took
// 5,960 us against 73 once the bits were set).  The LDS copies of the entries
// take the bit too, so that each workgroup sets it once: 317 us, then 40.6.
struct XlatShared {
    DSlot slots[kSlotRow];
    uint32_t words[kIndexWords];
    uint64_t top[512];
    uint32_t root_code;
    uint32_t pad[3];
};

// A 1 GiB region of the process, 16 bytes, read with one LDS load: what the
// levels above 2 gave.  info as in CEnt (code, level, leaf1g, u, w, abits of
// levels 4 and 3, dbit); pd: the level-2 table's arena offset, or a 1 GiB
// leaf's frame.
constexpr uint32_t kXlatWays = 32;  // regions kept per wavefront
constexpr uint32_t kXlatNone = 0xFFFFFFFFu;
struct XlatWave {
    u32x4 ent[kXlatWays];
    uint64_t path[2][kXlatWays];  // arena offsets of the level-4 (5-level paging) and level-3 entries
    uint32_t owner[kXlatWays];
    uint32_t stage[64 * 6];       // a round's records, written out as contiguous 16-byte chunks
};

__device__ __forceinline__ uint32_t block_word(int64_t delta) {
    const int64_t dp = delta >> 12;
    return dp < -(1ll << 29) || dp >= (1ll << 29) ? 1u : ((uint32_t)(int32_t)dp << 2) | 2u;
}

// Word of 2 MiB block b of a VM with an EPT (the walk's checks are those of
// ept_walk; anything but a plain readable and writable mapping is left to it).
__device__ uint32_t ept_block_word(const DVm &v, uint32_t b) {
    const auto table = [&](uint64_t e) {
        return (e & 3) == 3 && !(e & 0xF8) && (e & kAddrMask) < v.arena_bytes &&
               v.arena_bytes - (e & kAddrMask) >= 4096;
    };
    const auto leaf = [&](uint64_t e, uint32_t sh) {
        const uint64_t mt = (e >> 3) & 7;
        return (e & 3) == 3 && mt != 2 && mt != 3 && mt != 7 && !(e & ((1ull << sh) - 1) & ~0xFFFull);
    };
    const auto whole = [&](uint64_t h) {
        return h < v.arena_bytes && v.arena_bytes - h >= (1ull << 21) ? block_word((int64_t)(h - ((uint64_t)b << 21)))
                                                                      : 1u;
    };
    const uint64_t e4 = load_entry(v.arena, v.ept_root);
    if (!table(e4)) return 1;
    const uint64_t e3 = load_entry(v.arena, (e4 & kAddrMask) + 8 * (b >> 9));
    if (e3 & 0x80) return leaf(e3, 30) ? whole((e3 & kAddrMask) + ((uint64_t)(b & 511) << 21)) : 1u;
    if (!table(e3)) return 1;
    const uint64_t e2 = load_entry(v.arena, (e3 & kAddrMask) + 8 * (b & 511));
    if (e2 & 0x80) return leaf(e2, 21) ? whole(e2 & kAddrMask) : 1u;
    if (!table(e2) || (e2 & kAddrMask) >> 42) return 1;
    return (uint32_t)((e2 & kAddrMask) >> 12) << 2 | 3u;
}

// GPA -> arena offset as gpa_xlat, through the words in LDS.
__device__ __forceinline__ uint32_t block_xlat(const DVm &v, const XlatShared &sh, uint32_t nwords, uint64_t gpa,
                                               uint32_t need, uint64_t &hpa) {
    const uint64_t blk = gpa >> 21;
    const uint32_t w = blk < nwords ? sh.words[(uint32_t)blk] : 1u;
    if ((w & 3) == 2) {
        hpa = gpa + ((uint64_t)(int64_t)((int32_t)w >> 2) << 12);
        return DEVIRT_OK;
    }
    if (v.ept_root == kNoEpt) {
        if (w == 0 || (blk >= v.index_len && v.index_complete)) return DEVIRT_NO_MEMSLOT;
        uint32_t a = 0, b = v.nslots;
        while (a < b) {
            const uint32_t mid = (a + b) >> 1;
            if (sh.slots[mid].gpa <= gpa)
                a = mid + 1;
            else
                b = mid;
        }
        if (a == 0 || gpa >= sh.slots[a - 1].end) return DEVIRT_NO_MEMSLOT;
        hpa = sh.slots[a - 1].arena_off + (gpa - sh.slots[a - 1].gpa);
        return DEVIRT_OK;
    }
    if (w & 2) {  // the EPT's page table is known
        const uint64_t e = load_entry(v.arena, ((uint64_t)(w >> 2) << 12) + 8 * ((gpa >> 12) & 511));
        const uint64_t mt = (e >> 3) & 7, pg = e & kAddrMask;
        if (!(e & 7)) return DEVIRT_EPT_VIOLATION;
        if ((e & 3) == 2 || mt == 2 || mt == 3 || mt == 7 || pg >= v.arena_bytes || v.arena_bytes - pg < 4096)
            return DEVIRT_EPT_MISCONFIG;
        if (need & ~(uint32_t)e & 3) return DEVIRT_EPT_VIOLATION;
        hpa = pg | (gpa & 0xFFF);
        return DEVIRT_OK;
    }
    const XRes r = ept_walk(v.arena, v.arena_bytes, v.ept_root, gpa, need);
    if (r.code == DEVIRT_OK) hpa = r.hpa;
    return r.code;
}

__host__ __device__ constexpr size_t xlat_lds(uint32_t block) {
    return sizeof(XlatShared) + (size_t)(block / 64) * sizeof(XlatWave);
}

// The levels above 2 of one address (miss path), from the top entry in LDS.
template <int LEVELS>
__device__ __forceinline__ void xlat_upper(const XlatArgs &a, const DVm &vm, const XlatShared &sh, uint32_t nwords,
                                           uint64_t gva, uint32_t &info, uint64_t &pd, uint64_t (&path)[2]) {
    uint32_t u = 1, w = 1, abits = 0, dbit = 0, xc = sh.root_code;
    uint64_t e = LEVELS == 3 ? sh.top[(gva >> 30) & 3] : sh.top[(gva >> (12 + 9 * (LEVELS - 1))) & 511];
    pd = path[0] = path[1] = 0;
#pragma unroll
    for (int lvl = LEVELS; lvl >= 3; --lvl) {
        if (xc) {
            info = xc | ((uint32_t)lvl << 4);
            return;
        }
        if (lvl < LEVELS) {
            uint64_t th;
            xc = block_xlat(vm, sh, nwords, e & kAddrMask, kNeedTable, th);
            if (xc) {
                info = xc | ((uint32_t)lvl << 4);
                return;
            }
            path[4 - lvl] = th + 8 * ((gva >> (12 + 9 * (lvl - 1))) & 511);
            e = load_entry(vm.arena, path[4 - lvl]);
            if (e & kA) abits |= 1u << (4 - lvl);
        }
        if (!(e & kP)) {
            info = DEVIRT_NOT_PRESENT | ((uint32_t)lvl << 4);
            return;
        }
        if (LEVELS == 3) {
            if (e & kPaeRootRsvd) {
                info = DEVIRT_RESERVED | (3u << 4);
                return;
            }
        } else {
            u &= (uint32_t)(e >> 2) & 1u;
            w &= (uint32_t)(e >> 1) & 1u;
            if ((e & kPS) && (lvl >= 4 || (e & 0x3FFFE000ull))) {  // bits 29:13 of a 1 GiB leaf are reserved
                info = DEVIRT_RESERVED | ((uint32_t)lvl << 4);
                return;
            }
            if (lvl == 3 && (e & kPS)) {
                pd = e & kAddrMask & ~((1ull << 30) - 1);
                dbit = (e & kD) ? kCiDbit : 0u;
                info = (1u << 8) | (u << 9) | (w << 10) | (abits << 13) | dbit;
                return;
            }
        }
    }
    xc = block_xlat(vm, sh, nwords, e & kAddrMask, kNeedTable, pd);
    info = xc ? xc | (2u << 4) : (u << 9) | (w << 10) | (abits << 13);
}

template <int LEVELS, bool AD>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(AD ? 6 : 8))) k_xlat(XlatArgs a) {
    extern __shared__ __align__(16) uint8_t smem[];
    XlatShared &sh = *(XlatShared *)smem;
    const int lane = lane_id();
    XlatWave &wv = *(XlatWave *)(smem + sizeof(XlatShared) + (threadIdx.x >> 6) * sizeof(XlatWave));
    const bool write = (a.flags & DEVIRT_XLAT_WRITE) != 0;
    const DVm vm = load_vm(a.v, a.vm, false);
    typedef DV_GLOBAL DSlot g_slot;
    const g_slot *row = gp<const g_slot>(a.v.slots) + (uint64_t)a.vm * kSlotRow;
    if (threadIdx.x < kSlotRow) sh.slots[threadIdx.x] = row[threadIdx.x];
    uint32_t nwords = vm.nwords;
    if (vm.ept_root == kNoEpt) {
        for (uint32_t t = threadIdx.x; t < nwords; t += blockDim.x) sh.words[t] = gp<const g_u32>(vm.words)[t];
    } else {
        const uint64_t nb = (vm.arena_bytes + (1ull << 21) - 1) >> 21;
        nwords = nb < kIndexWords ? (uint32_t)nb : kIndexWords;
        for (uint32_t t = threadIdx.x; t < nwords; t += blockDim.x) sh.words[t] = ept_block_word(vm, t);
    }
    if (lane < (int)kXlatWays) wv.ent[lane] = (u32x4){kXlatNone, 0u, 0u, 0u};
    __syncthreads();
    uint64_t root = 0;  // the top-level table's arena offset
    const uint32_t root_code = block_xlat(vm, sh, nwords, LEVELS == 3 ? (a.cr3 & 0xFFFFFFE0ull) : (a.cr3 & kAddrMask),
                                          kNeedTable, root);
    if (threadIdx.x == 0) sh.root_code = root_code;
    if (!root_code)
        for (uint32_t t = threadIdx.x; t < (LEVELS == 3 ? 4u : 512u); t += blockDim.x)
            sh.top[t] = load_entry(vm.arena, root + 8 * t);
    __syncthreads();
    const uint64_t lim = user_limit(LEVELS);
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x >> 6);
    uint32_t hits = 0, misses = 0, atom = 0;
    // the next round's addresses are loaded at the top of this round
    const uint64_t first = ((uint64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 64;
    uint64_t gva_next = first + lane < a.n ? gp<const g_u64>(a.gva)[first + lane] : 0;
    for (uint64_t b0 = first; b0 < a.n; b0 += waves * 64) {
        const uint64_t gva = gva_next, i = b0 + lane;
        gva_next = i + waves * 64 < a.n ? gp<const g_u64>(a.gva)[i + waves * 64] : 0;
        const bool go = i < a.n && gva < lim;
        uint32_t code = DEVIRT_NONCANONICAL, level = 0, shift = 0, leaf = 0;
        uint64_t gpa = 0, hpa = 0, e2 = 0, e1 = 0, pde_off = 0, pte_off = 0;
        // ---- the levels above 2
        const uint32_t key = (uint32_t)(gva >> 30);
        const uint32_t slot = (key ^ (key >> 5) ^ (key >> 10)) & (kXlatWays - 1);
        const u32x4 ent = wv.ent[slot];
        uint32_t info = ent.y;
        uint64_t pd = ((uint64_t)ent.w << 32) | ent.z;
        const bool miss = go && ent.x != key;
        if (a.counters) {
            hits += go && !miss;
            misses += miss;
        }
        uint64_t path[2] = {0, 0};
        if (AD && LEVELS > 3) {
            path[0] = wv.path[0][slot];
            path[1] = wv.path[1][slot];
        }
        if (__ballot(miss)) {
            if (miss) xlat_upper<LEVELS>(a, vm, sh, nwords, gva, info, pd, path);
            // an address without a top-level entry leaves the region its slot holds alone
            const bool keep = miss && !(ci_code(info) && ci_level(info) == (uint32_t)LEVELS);
            if (keep) wv.owner[slot] = (uint32_t)lane;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (keep && wv.owner[slot] == (uint32_t)lane) {
                wv.ent[slot] = (u32x4){key, info, (uint32_t)pd, (uint32_t)(pd >> 32)};
                if (AD) {
                    wv.path[0][slot] = path[0];
                    wv.path[1][slot] = path[1];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        if (go) {
            uint32_t u = ci_u(info), w = ci_w(info);
            code = ci_code(info);
            level = ci_level(info);
            uint64_t frame = pd;
            if (code == 0) {
                leaf = 3;
                if (!ci_leaf(info)) {
                    pde_off = pd + 8 * ((gva >> 21) & 511);
                    e2 = load_entry(vm.arena, pde_off);
                    if (!(e2 & kP)) {
                        code = DEVIRT_NOT_PRESENT;
                        level = 2;
                    } else if ((LEVELS == 3 && (e2 & kPaeRsvd)) || ((e2 & kPS) && (e2 & 0x1FE000ull))) {
                        code = DEVIRT_RESERVED;  // bits 20:13 of a 2 MiB leaf
                        level = 2;
                    } else {
                        u &= (uint32_t)(e2 >> 2) & 1u;
                        w &= (uint32_t)(e2 >> 1) & 1u;
                        leaf = 2;
                        frame = e2 & kAddrMask & ~((1ull << 21) - 1);
                        if (!(e2 & kPS)) {
                            uint64_t pt;
                            code = block_xlat(vm, sh, nwords, e2 & kAddrMask, kNeedTable, pt);
                            level = 1;
                            if (!code) {
                                pte_off = pt + 8 * ((gva >> 12) & 511);
                                e1 = load_entry(vm.arena, pte_off);
                                if (!(e1 & kP)) {
                                    code = DEVIRT_NOT_PRESENT;
                                } else if (LEVELS == 3 && (e1 & kPaeRsvd)) {
                                    code = DEVIRT_RESERVED;
                                } else {
                                    u &= (uint32_t)(e1 >> 2) & 1u;
                                    w &= (uint32_t)(e1 >> 1) & 1u;
                                    leaf = 1;
                                    level = 0;
                                    frame = e1 & kAddrMask;
                                }
                            }
                        }
                    }
                }
            }
            if (code == 0) {
                shift = 3 + 9 * leaf;
                gpa = frame | (gva & ((1ull << shift) - 1));
                if (!u) {
                    code = DEVIRT_PROT_USER;
                    level = leaf;
                } else if (write && !w) {
                    code = DEVIRT_PROT_WRITE;
                    level = leaf;
                } else {
                    level = 0;
                    code = block_xlat(vm, sh, nwords, gpa, write ? kNeedW : kNeedR, hpa);
                    if (code) hpa = 0;
                }
            }
        }
        if (AD) {
            // A and D of the path.  The shared levels are set once: the LDS
            // copy of the entry takes the bit too, and only the lane that finds
            // it clear there goes to memory; of neighbouring lanes with one
            // level-2 entry the first sets it.
            const bool ok = go && code == 0;
            const uint64_t prev_off = shfl64(pde_off, lane > 0 ? lane - 1 : 0);
            const bool prev_ok = shfl32(ok ? 1u : 0u, lane > 0 ? lane - 1 : 0) != 0 && lane > 0;
            if (ok && LEVELS > 3) {
                const uint32_t ti = (uint32_t)(gva >> (12 + 9 * (LEVELS - 1))) & 511u;
                uint32_t *top = (uint32_t *)&sh.top[ti];
                if (!(*(volatile uint32_t *)top & (uint32_t)kA) && !(atomicOr(top, (uint32_t)kA) & (uint32_t)kA)) {
                    or_entry(vm.arena, root + 8 * ti, (uint32_t)kA);
                    atom++;
                }
                uint32_t *cached = (uint32_t *)&wv.ent[slot] + 1;
                const bool mine = ((uint32_t *)&wv.ent[slot])[0] == key;
#pragma unroll
                for (int lvl = LEVELS - 1; lvl >= 3; --lvl) {
                    uint32_t have = 1u << (17 - lvl), want = (uint32_t)kA;  // info bit of the level's accessed bit
                    if (lvl == 3 && leaf == 3 && write) {
                        have |= kCiDbit;
                        want |= (uint32_t)kD;
                    }
                    if ((info & have) != have && (!mine || (atomicOr(cached, have) & have) != have)) {
                        or_entry(vm.arena, path[4 - lvl], want);
                        atom++;
                    }
                }
            }
            if (ok && leaf <= 2) {
                const uint32_t want = (uint32_t)kA | ((leaf == 2 && write) ? (uint32_t)kD : 0u);
                if (((uint32_t)e2 & want) != want && !(prev_ok && prev_off == pde_off)) {
                    or_entry(vm.arena, pde_off, want);
                    atom++;
                }
            }
            if (ok && leaf == 1) {
                const uint32_t want = (uint32_t)kA | (write ? (uint32_t)kD : 0u);
                if (((uint32_t)e1 & want) != want) {
                    or_entry(vm.arena, pte_off, want);
                    atom++;
                }
            }
        }
        // every lane stages its record (an idle lane's is never written out)
        {
            uint32_t *r = wv.stage + 6 * lane;
            *(uint64_t *)r = gpa;
            *(uint64_t *)(r + 2) = hpa;
            r[4] = code;
            r[5] = level | (shift << 8) | (a.vm << 16);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        {
            const uint32_t valid = 24u * (uint32_t)(a.n - b0 < 64 ? a.n - b0 : 64);  // bytes of this round
            uint8_t *dst = (uint8_t *)a.out + 24 * b0;
#pragma unroll
            for (uint32_t k = 0; k < 2; ++k) {
                const uint32_t c = (uint32_t)lane + 64u * k;  // 16-byte chunk of the round
                if (16u * c + 16u <= valid)
                    __builtin_nontemporal_store(*(const u32x4 *)(wv.stage + 4 * c), gp<g_u32x4_w4>(dst + 16 * c));
                else if (16u * c < valid)  // the last 8 bytes of an odd count
                    __builtin_nontemporal_store(*(const uint64_t *)(wv.stage + 4 * c), gp<g_u64>(dst + 16 * c));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (a.counters) {
        GroupOut st = {0, hits, misses, 0, 0, atom, 0};
        flush_counters(a.counters, st);
    }
}

// The records of an unknown process.
__global__ void __launch_bounds__(256) k_xlat_unknown(XlatArgs a) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride)
        gp<DV_GLOBAL devirt_xlat>(a.out)[i] = devirt_xlat{0, 0, DEVIRT_INVALID, 0, 0, 0xFFFF};
}

// ------------------------------------------------------------ fault list
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t *lds, uint32_t &total) {
    const int lane = lane_id(), wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t t = shfl32(incl, lane >= d ? lane - d : lane);
        if (lane >= d) incl += t;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    uint32_t before = 0, tot = 0;
    for (int w = 0; w < nw; ++w) {
        uint32_t s = lds[w];
        if (w < wave) before += s;
        tot += s;
    }
    __syncthreads();
    total = tot;
    return before + incl - x;
}

__global__ void __launch_bounds__(256) k_fault_count(const devirt_result *res, uint64_t n, uint32_t *tile_cnt) {
    __shared__ uint32_t lds[16];
    const uint64_t t = blockIdx.x;
    uint32_t c = 0;
    for (int q = 0; q < 4; ++q) {
        uint64_t i = t * kFaultTile + (uint64_t)threadIdx.x * 4 + q;
        if (i < n && res[i].code != 0) c++;
    }
    uint32_t tot;
    block_exclusive_scan(c, lds, tot);
    if (threadIdx.x == 0) tile_cnt[t] = tot;
}

__global__ void __launch_bounds__(1024) k_fault_scan(uint32_t *tile_cnt, uint64_t ntiles, uint64_t *n_faults) {
    __shared__ uint32_t lds[16];
    uint64_t carry = 0;
    for (uint64_t b0 = 0; b0 < ntiles; b0 += blockDim.x) {
        const uint64_t i = b0 + threadIdx.x;
        const uint32_t x = i < ntiles ? tile_cnt[i] : 0u;
        uint32_t tot;
        const uint32_t ex = block_exclusive_scan(x, lds, tot);
        if (i < ntiles) tile_cnt[i] = (uint32_t)(carry + ex);
        carry += tot;
    }
    if (threadIdx.x == 0 && n_faults) *n_faults = carry;
}

__global__ void __launch_bounds__(256) k_fault_scatter(const devirt_result *res, uint64_t n, const uint32_t *tile_off,
                                                       devirt_fault *faults) {
    __shared__ uint32_t lds[16];
    const uint64_t t = blockIdx.x;
    uint32_t flags = 0, c = 0;
    for (int q = 0; q < 4; ++q) {
        uint64_t i = t * kFaultTile + (uint64_t)threadIdx.x * 4 + q;
        if (i < n && res[i].code != 0) {
            flags |= 1u << q;
            c++;
        }
    }
    uint32_t tot;
    uint32_t pos = tile_off[t] + block_exclusive_scan(c, lds, tot);
    for (int q = 0; q < 4; ++q) {
        if (flags & (1u << q)) {
            uint64_t i = t * kFaultTile + (uint64_t)threadIdx.x * 4 + q;
            devirt_result r = res[i];
            devirt_fault f;
            f.req_index = i;
            f.fault_gva = r.fault_gva;
            f.code = r.code;
            f.level = r.level;
            f.pad = 0;
            faults[pos++] = f;
        }
    }
}

// ---------------------------------------------------------------- launchers
static size_t wave_lds(int block) {
    return (size_t)(block / 64) * kCacheWays * (sizeof(CEnt) + sizeof(uint32_t));
}

hipError_t launch_reset(hipStream_t s, DBatch b, uint32_t n_epochs) {
    uint32_t blocks = (uint32_t)(((uint64_t)n_epochs * kCtrLines + 255) / 256);
    if (blocks == 0) blocks = 1;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_reset, dim3(blocks), dim3(256), 0, s, b, n_epochs);
    return hipGetLastError();
}

hipError_t launch_translate_groups(hipStream_t s, int grid, int block, DView v, DBatch b, uint64_t r0, uint64_t r1,
                                   uint32_t epoch, int direct) {
    hipLaunchKernelGGL(k_translate_groups, dim3(grid), dim3(block), wave_lds(block), s, v, b, r0, r1, epoch, direct);
    return hipGetLastError();
}

hipError_t launch_translate_one(hipStream_t s, int block, DView v, DBatch b, uint64_t n, int direct) {
    const uint64_t waves = (uint64_t)block / 64;
    hipLaunchKernelGGL(k_translate_one, dim3((unsigned)((n + waves - 1) / waves)), dim3(block), 0, s, v, b, n, direct);
    return hipGetLastError();
}

hipError_t launch_translate_large(hipStream_t s, int grid, int block, DView v, DBatch b, uint64_t r0,
                                  uint32_t epoch) {
    hipLaunchKernelGGL(k_translate_large, dim3(grid), dim3(block), wave_lds(block), s, v, b, r0, epoch);
    return hipGetLastError();
}

hipError_t launch_copy(hipStream_t s, int grid, int block, DBatch b, uint32_t epoch, const CopyTail &tail) {
    hipLaunchKernelGGL(k_copy, dim3(grid + (tail.n ? 1 : 0)), dim3(block), 0, s, b, epoch, tail);
    return hipGetLastError();
}

hipError_t launch_spill(hipStream_t s, int grid, int block, DView v, DBatch b, uint64_t r0, uint64_t r1,
                        uint32_t epoch) {
    hipLaunchKernelGGL(k_spill, dim3(grid), dim3(block), wave_lds(block), s, v, b, r0, r1, epoch);
    return hipGetLastError();
}

hipError_t launch_plain_walk(hipStream_t s, uint32_t waves, const PlainArgs &a) {
    hipLaunchKernelGGL(a.fifo_entries ? k_plain_walk<true> : k_plain_walk<false>, dim3(1), dim3(64 * waves), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_plain(hipStream_t s, DView v, DBatch b, devirt_request req, int inline_copy) {
    hipLaunchKernelGGL(k_plain, dim3(1), dim3(64), 0, s, v, b, req, inline_copy);
    return hipGetLastError();
}

hipError_t launch_xlat(hipStream_t s, int grid, int block, const XlatArgs &a) {
    void (*k)(XlatArgs) = k_xlat_unknown;
    const bool ad = (a.flags & DEVIRT_XLAT_SET_AD) != 0;
    if (a.levels == 5)
        k = ad ? k_xlat<5, true> : k_xlat<5, false>;
    else if (a.levels == 4)
        k = ad ? k_xlat<4, true> : k_xlat<4, false>;
    else if (a.levels == 3)
        k = ad ? k_xlat<3, true> : k_xlat<3, false>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(a.levels ? block : 256), a.levels ? xlat_lds(block) : 0, s, a);
    return hipGetLastError();
}

hipError_t launch_fault_count(hipStream_t s, const devirt_result *res, uint64_t n, uint32_t *tile_cnt) {
    uint64_t tiles = (n + kFaultTile - 1) / kFaultTile;
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fault_count, dim3((unsigned)tiles), dim3(256), 0, s, res, n, tile_cnt);
    return hipGetLastError();
}

hipError_t launch_fault_scan(hipStream_t s, uint32_t *tile_cnt, uint64_t ntiles, uint64_t *n_faults) {
    hipLaunchKernelGGL(k_fault_scan, dim3(1), dim3(1024), 0, s, tile_cnt, ntiles, n_faults);
    return hipGetLastError();
}

hipError_t launch_fault_scatter(hipStream_t s, const devirt_result *res, uint64_t n, const uint32_t *tile_off,
                                devirt_fault *faults) {
    uint64_t tiles = (n + kFaultTile - 1) / kFaultTile;
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fault_scatter, dim3((unsigned)tiles), dim3(256), 0, s, res, n, tile_off, faults);
    return hipGetLastError();
}


// ------------------------------------------------------------- map pages
// Mapping pages by writing the guest's own tables (section 4.2, the second
// kind of routine).  Keys name tables: (8 - level) in bits 63:56, the table's
// index (gva >> (12 + 9 level)) below, so ascending keys run from the top
// level down and by index within a level.
__device__ __forceinline__ uint64_t map_key(uint32_t level, uint64_t gva) {
    return ((uint64_t)(8 - level) << 56) | (gva >> (12 + 9 * level));
}

// Index of gva's entry in its table at `level` (a PAE root table has 4).
__device__ __forceinline__ uint64_t entry_index(uint32_t levels, uint32_t level, uint64_t gva) {
    return (levels == 3 && level == 3) ? ((gva >> 30) & 3) : ((gva >> (12 + 9 * (level - 1))) & 511);
}

__device__ __forceinline__ uint64_t root_table(const DProc &p) {
    return p.levels == 3 ? (p.cr3 & 0xFFFFFFE0ull) : (p.cr3 & kAddrMask);
}

__device__ __forceinline__ void store_entry(uint8_t *arena, uint64_t off, uint64_t v) { *gp<g_u64>(arena + off) = v; }

// Walk for a map on the tables as they are (no A/D).  On success `missing` is
// the highest level whose entry is not present (its child tables are lacking),
// 0 when the whole path exists.
__device__ uint32_t map_walk(const DVm &v, const DProc &p, uint64_t gva, uint32_t &level, uint32_t &missing) {
    const bool pae = p.levels == 3;
    uint64_t table = root_table(p);
    missing = 0;
    for (int lvl = (int)p.levels; lvl >= 2; --lvl) {
        uint64_t th;
        const uint32_t xc = gpa_xlat(v, table, kNeedTable, th);
        if (xc) {
            level = (uint32_t)lvl;
            return xc;
        }
        const uint64_t e = load_entry(v.arena, th + 8 * entry_index(p.levels, (uint32_t)lvl, gva));
        if (!(e & kP)) {
            missing = (uint32_t)lvl;
            return DEVIRT_OK;
        }
        const bool root = pae && lvl == 3;
        const bool rsvd = pae && (e & (root ? kPaeRootRsvd : kPaeRsvd)) != 0;
        if (rsvd || (!root && (e & kPS))) {  // reserved bits, or a large leaf on the path
            level = (uint32_t)lvl;
            return DEVIRT_RESERVED;
        }
        table = e & kAddrMask;
    }
    uint64_t th;
    const uint32_t xc = gpa_xlat(v, table, kNeedTable, th);  // the page table itself
    if (xc) {
        level = 1;
        return xc;
    }
    return DEVIRT_OK;
}

// Arena offset of the existing table at `level` on gva's path (the path to it
// is known to be present); level == top gives the root table.  False if a
// table on the way has no memslot (then nothing may be written).
__device__ bool existing_table(const DVm &v, const DProc &p, uint64_t gva, uint32_t level, uint64_t &th) {
    uint64_t table = root_table(p);
    for (int lvl = (int)p.levels; lvl > (int)level; --lvl) {
        if (gpa_xlat(v, table, kNeedTable, th)) return false;
        table = load_entry(v.arena, th + 8 * entry_index(p.levels, (uint32_t)lvl, gva)) & kAddrMask;
    }
    return gpa_xlat(v, table, kNeedTable, th) == DEVIRT_OK;
}

// ---- the EPT half of mapping a page (section 4.2: the backend creates the
// mapping in the guest tables and also in the EPT), devirt_ept_map_pages.
// The maps name guest-physical pages and the arena pages behind them; new EPT
// tables are linked with R, W and X, leaves carry the map's R/W/X bits and
// memory type WB.
constexpr uint64_t kEptRwx = 7ull, kEptWb = 6ull << 3;

__device__ __forceinline__ uint64_t ept_slot(uint64_t table, uint32_t level, uint64_t gpa) {
    return table + 8 * ((gpa >> (12 + 9 * (level - 1))) & 511);
}

// Walk of the EPT as it is, for a map of gpa.  On success `missing` is the
// highest level whose entry is not present (its child tables are lacking), 0
// when the EPT page table exists.  A present large leaf on the path fails the
// map (RESERVED: nothing is split), a misconfigured table entry or a table
// outside the arena fails it with EPT_MISCONFIG; `level` names the entry.
__device__ uint32_t ept_map_walk(const DVm &v, uint64_t gpa, uint32_t &level, uint32_t &missing) {
    uint64_t table = v.ept_root;
    missing = 0;
    for (uint32_t lvl = 4; lvl >= 2; --lvl) {
        const uint64_t e = load_entry(v.arena, ept_slot(table, lvl, gpa));
        if (!(e & 7)) {
            missing = lvl;
            level = 0;
            return DEVIRT_OK;
        }
        level = lvl;
        if ((e & 3) == 2) return DEVIRT_EPT_MISCONFIG;  // write without read
        if (lvl <= 3 && (e & 0x80)) return DEVIRT_RESERVED;
        if (e & 0xF8) return DEVIRT_EPT_MISCONFIG;  // bits 7:3 of a table entry
        table = e & kAddrMask;
        if (table >= v.arena_bytes || v.arena_bytes - table < 4096) return DEVIRT_EPT_MISCONFIG;
    }
    level = 0;
    return DEVIRT_OK;
}

// Arena offset of the existing EPT table at `level` on gpa's path (known present).
__device__ uint64_t existing_ept_table(const DVm &v, uint64_t gpa, uint32_t level) {
    uint64_t table = v.ept_root;
    for (uint32_t lvl = 4; lvl > level; --lvl) table = load_entry(v.arena, ept_slot(table, lvl, gpa)) & kAddrMask;
    return table;
}

// Position of key in the sorted keys[0, n), or -1.
__device__ __forceinline__ int64_t find_key(const uint64_t *keys, uint64_t n, uint64_t key) {
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (keys[mid] < key)
            lo = mid + 1;
        else
            hi = mid;
    }
    return (lo < n && keys[lo] == key) ? (int64_t)lo : -1;
}

// Fibonacci hashing (Knuth): the top log2 bits of key * 2^64/phi.
__device__ __forceinline__ uint64_t hash_slot(uint64_t key, uint32_t log2) {
    return (key * 0x9E3779B97F4A7C15ull) >> (64 - log2);
}

// Adds a table key to the set, probing from slot h (the key's probe number
// `probe` there); its first inserter also appends it to the list tkeys[0, m).
// sc[0] counts distinct keys.  A long probe chain gives up, with sc[3] set,
// once more than m distinct keys exist: the set holds at least twice m + 1
// slots, so chains grow long only then, and the count (an address every new
// key increments, so reads of it serialize) is read only on such chains.
// Every probe loop is bounded by the set's size.
constexpr uint64_t kLongChain = 8;
__device__ void tset_insert_from(const MapArgs &a, uint64_t key, uint64_t h, uint64_t probe) {
    const uint64_t mask = (1ull << a.tset_log2) - 1;
    for (; probe <= mask; ++probe) {
        const uint64_t cur = atomicCAS((unsigned long long *)&a.tset[h], ~0ull, (unsigned long long)key);
        if (cur == ~0ull) {
            const uint64_t idx = atomicAdd((unsigned long long *)&a.sc[0], 1ull);
            if (idx < a.m) a.tkeys[idx] = key;
            return;
        }
        if (cur == key) return;
        if (probe >= kLongChain && __hip_atomic_load(&a.sc[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > a.m)
            break;
        h = (h + 1) & mask;
    }
    __hip_atomic_store(&a.sc[3], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A lane's (up to four) table keys: the first probes are issued together, so
// the lane waits for one atomic round trip, not one per key; a key whose first
// slot holds another key continues in tset_insert_from.
__device__ void tset_insert4(const MapArgs &a, const uint64_t (&key)[4], const bool (&want)[4]) {
    const uint64_t mask = (1ull << a.tset_log2) - 1;
    uint64_t h[4], cur[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        h[j] = hash_slot(key[j], a.tset_log2);
        cur[j] = want[j] ? (uint64_t)atomicCAS((unsigned long long *)&a.tset[h[j]], ~0ull,
                                               (unsigned long long)key[j])
                         : key[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (!want[j] || cur[j] == key[j]) continue;
        if (cur[j] == ~0ull) {
            const uint64_t idx = atomicAdd((unsigned long long *)&a.sc[0], 1ull);
            if (idx < a.m) a.tkeys[idx] = key[j];
        } else {
            tset_insert_from(a, key[j], (h[j] + 1) & mask, 1);
        }
    }
}

// Records map i for its page: a slot holds (page << kMapIdxBits | index), and
// a later map of the same page raises it with atomicMax, so the slot ends up
// naming the page's last map.  A page seen once costs one atomic.  The set
// has at least twice as many slots as maps, so a free slot is always found.
__device__ void page_note(const MapArgs &a, uint64_t page, uint64_t i) {
    const uint64_t mask = (1ull << a.pset_log2) - 1;
    const uint64_t v = (page << kMapIdxBits) | i;
    uint64_t h = hash_slot(page, a.pset_log2);
    for (uint64_t probe = 0; probe <= mask; ++probe) {
        const uint64_t cur = atomicCAS((unsigned long long *)&a.pset[h], ~0ull, (unsigned long long)v);
        if (cur == ~0ull) return;
        if ((cur >> kMapIdxBits) == page) {
            atomicMax((unsigned long long *)&a.pset[h], (unsigned long long)v);
            return;
        }
        h = (h + 1) & mask;
    }
}

// Fill `ones` with ~0 (empty set slots, list padding) and `zeros` with 0, and
// fetch the pool from the host memory it is staged in: only the frames that
// the batch can use, and without a copy operation of their own (with one, and
// the wait for the one before, 16 maps took 42 us a call; now 20).
__global__ void __launch_bounds__(256) k_map_clear(uint64_t *ones, uint64_t n_ones, uint64_t *zeros, uint64_t n_zeros,
                                                   const uint64_t *staged, uint64_t *pool, uint64_t n_pool) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x, t0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (uint64_t t = t0; t < n_pool; t += stride) pool[t] = staged[t];
    for (uint64_t t = t0; t < n_ones / 2; t += stride) gp<g_u32x4>(ones)[t] = (u32x4){~0u, ~0u, ~0u, ~0u};
    if (t0 == 0 && (n_ones & 1)) ones[n_ones - 1] = ~0ull;
    if (t0 < n_zeros) zeros[t0] = 0;
}

// Whether map m is one that is walked (its addresses and flags are valid).
__device__ __forceinline__ bool map_valid(const MapArgs &a, const DVm &vm, uint32_t levels, const devirt_map &m) {
    if (a.ept_map) {  // gva: the guest-physical page; gpa: the arena page behind it
        const uint32_t perms = m.flags & 7u;
        return !((m.gva & 0xFFFull) || (m.gva >> 48) || (m.gpa & 0xFFFull) || m.gpa >= vm.arena_bytes ||
                 vm.arena_bytes - m.gpa < 4096 || (m.flags & ~7u) || perms == 0 || (perms & 3u) == 2u);
    }
    return !((m.gva & 0xFFFull) || m.gva >= user_limit(levels) || (m.gpa & 0xFFFull) || m.gpa >= (1ull << 52));
}

// A map's result, and the keys of the tables its path lacks (k, from the top
// level down, ~0 after the last).
__device__ __forceinline__ bool map_one(const MapArgs &a, const DVm &vm, const DProc &p, const devirt_map &m,
                                        devirt_result &r, uint64_t (&k)[4]) {
    r.bytes_done = 0;
    r.fault_gva = m.gva;
    r.code = DEVIRT_NONCANONICAL;
    r.level = 0;
    r.pad = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) k[j] = ~0ull;
    if (!map_valid(a, vm, p.levels, m)) return false;
    uint32_t level = 0, missing = 0;
    r.code = a.ept_map ? ept_map_walk(vm, m.gva, level, missing) : map_walk(vm, p, m.gva, level, missing);
    r.level = (uint16_t)level;
    if (r.code != DEVIRT_OK) return false;
    r.bytes_done = 4096;
    r.fault_gva = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j)
        if (missing > j + 1) k[j] = map_key(missing - 1 - j, m.gva);
    return true;
}

// One lane per map: its result; the tables its path lacks go into the set, a
// key that the map before it adds left to that map (a valid map that shares a
// lacking table with this one lacks all of the tables below the same entry).
// Maps whose pages do not ascend set sc[1]: only then can two name one page.
//
// Bound by device atomics.  On one address they take turns, 13 ns each, so a
// region's upper tables must not be added by every wavefront; and a page set
// costs an atomic per map, so maps in ascending order, which is how a region
// is mapped, do without one (and the others note their pages in the next
// launch).  131,072 maps of a fresh region: this launch 38.8 -> 10.1 us, the
// call 85.9 -> 38.5; 131,072 scattered remaps 51.5 -> 36.7 a call.
__global__ void __launch_bounds__(256) k_map_walk(MapArgs a) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int lane = lane_id();
    const bool live = i < a.n;
    const bool known = a.ept_map || a.asid < a.v.nproc;
    DProc p = {0, 0, 4};
    DVm vm = {};
    if (known) {
        if (!a.ept_map) p = a.v.procs[a.asid];
        vm = a.v.vms[a.ept_map ? a.vm : p.vm];
    }
    uint64_t k[4] = {~0ull, ~0ull, ~0ull, ~0ull};
    devirt_map m = {0, 0, 0, 0};
    if (live) {
        m = a.maps[i];
        devirt_result r;
        if (known) {
            map_one(a, vm, p, m, r, k);
        } else {
            r = devirt_result{0, m.gva, DEVIRT_INVALID, 0, 0};
        }
        a.res[i] = r;
    }
    // the map before, and whether it adds keys
    devirt_map q = {0, 0, 0, 0};
    q.gva = shfl64(m.gva, lane > 0 ? lane - 1 : 0);
    bool before = shfl32(live && known && map_valid(a, vm, p.levels, m) ? 1u : 0u, lane > 0 ? lane - 1 : 0) != 0;
    if (lane == 0 && live && i > 0) {
        q = a.maps[i - 1];
        before = known && map_valid(a, vm, p.levels, q);
    }
    if (i == 0) before = false;
    const bool descends = live && i > 0 && (q.gva >> 12) >= (m.gva >> 12);
    // by many wavefronts, the same value: an ordinary store, which stays in the
    // cache (an atomic or volatile one took turns on the line, 30 ns each)
    if (__ballot(descends) && lane == 0) gp<g_u64>(a.sc)[1] = 1;
    bool want[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t l = 8u - (uint32_t)(k[j] >> 56);  // the key's level
        want[j] = k[j] != ~0ull && !(before && map_key(l, q.gva) == k[j]);
    }
    tset_insert4(a, k, want);
}

// The page set, when the maps' pages do not ascend: each successful map is
// noted for its page.
__device__ __forceinline__ void note_pages(const MapArgs &a) {
    if (a.sc[1] == 0) return;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += stride)
        if (a.res[i].code == DEVIRT_OK) page_note(a, a.maps[i].gva >> 12, i);
}

// Whether successful map t is the last of its page.
__device__ __forceinline__ bool last_of_page(const MapArgs &a, uint64_t page, uint64_t t) {
    if (a.sc[1] == 0) return true;
    const uint64_t mask = (1ull << a.pset_log2) - 1;
    uint64_t h = hash_slot(page, a.pset_log2);
    for (uint64_t probe = 0; probe <= mask && (a.pset[h] >> kMapIdxBits) != page; ++probe) h = (h + 1) & mask;
    return a.pset[h] == ((page << kMapIdxBits) | t);
}

// A VM with an EPT: the pool frames the batch takes (the first sc[0]) are
// translated through the EPT, readable and writable like every table frame;
// one that is not makes the batch fail as a short pool does (sc[3]).
__global__ void __launch_bounds__(256) k_map_pool(const MapArgs a) {
    const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t nt = a.sc[0];
    if (a.sc[3] || nt > a.n_pool || k >= nt || a.asid >= a.v.nproc) return;
    const DVm vm = a.v.vms[a.v.procs[a.asid].vm];
    uint64_t h = 0;
    if (gpa_xlat(vm, a.pool_gpa[k], kNeedTable, h) == DEVIRT_OK)
        a.pool_hpa[k] = h;
    else
        __hip_atomic_store(&a.sc[3], 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The VM whose tables a map call writes (false: an unknown asid).
__device__ __forceinline__ bool map_vm(const MapArgs &a, DVm &vm) {
    if (a.ept_map) {
        vm = a.v.vms[a.vm];
        return true;
    }
    if (a.asid >= a.v.nproc) return false;
    vm = a.v.vms[a.v.procs[a.asid].vm];
    return true;
}

// Tables to create: 0 when the pool is too small (then nothing is written).
__device__ __forceinline__ uint64_t new_tables(const MapArgs &a) {
    const uint64_t u = a.sc[0];
    return (a.sc[3] != 0 || u > a.n_pool) ? 0 : u;
}
__device__ __forceinline__ bool pool_short(const MapArgs &a) { return a.sc[3] != 0 || a.sc[0] > a.n_pool; }

// The distinct keys are sorted by rank (the number of smaller keys; there are
// no ties), in LDS tiles: for lists of up to kMapRankMax keys.  The same
// launch zeroes the new tables, 16 bytes per lane, and notes the pages.
//
// Ranking is a chain of LDS reads, one per key in the list, so a workgroup
// ranks only 64 keys and its wavefronts share the chain; and it comes first,
// because the page notes of all the other workgroups keep the memory busy
// meanwhile.  524,288 maps of fresh regions in no order (2,149 new tables),
// 256 keys a workgroup behind the notes and so: 74.9 and 46.2 us; the notes
// alone take 34.
__global__ void __launch_bounds__(256) k_map_rank_zero(const MapArgs a) {
    __shared__ uint64_t tile[256];
    __shared__ uint32_t part[4][64];
    const uint64_t nt = new_tables(a);
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t k0 = (uint64_t)blockIdx.x * 64;
    if (a.rank && k0 < nt) {  // uniform per block
        const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const uint64_t key = k0 + lane < nt ? a.tkeys[k0 + lane] : ~0ull;
        uint32_t rank = 0;
        for (uint64_t base = 0; base < nt; base += 256) {
            __syncthreads();
            tile[threadIdx.x] = base + threadIdx.x < nt ? a.tkeys[base + threadIdx.x] : ~0ull;
            __syncthreads();
#pragma unroll 16
            for (uint32_t q = 0; q < 64; ++q) rank += tile[64 * wave + q] < key;
        }
        part[wave][lane] = rank;
        __syncthreads();
        if (wave == 0 && k0 + lane < nt)
            a.tkeys_sorted[part[0][lane] + part[1][lane] + part[2][lane] + part[3][lane]] = key;
    }
    DVm zvm;
    if (nt && map_vm(a, zvm)) {
        uint8_t *arena = zvm.arena;
        const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
        for (uint64_t z = t; z < nt * 256; z += stride)
            *gp<g_u32x4>(arena + a.pool_hpa[z >> 8] + 16 * (z & 255)) = (u32x4){0u, 0u, 0u, 0u};
    }
    note_pages(a);
}

// Longer key lists (more than kMapRankMax keys can exist) are sorted in two
// steps.  First tiles of kSortTile keys, each by rank in LDS; then rounds of
// pairwise merges of sorted runs, in which a key's place in the merged run is
// its place in its own run plus the number of smaller keys in the other run,
// found by a binary search of that run.  Only the list's first
// min(sc[0], m) entries are keys, all distinct, so there are no ties; the
// rest is never read.  The steps alternate between tkeys and tkeys_sorted.
// The first one, which few workgroups have tiles for, notes the pages too
// (with the zeroing, which fills the chip, the notes cost their full 34 us).
constexpr uint32_t kSortTile = 1024;

__device__ __forceinline__ uint64_t sort_count(const MapArgs &a) { return a.sc[0] < a.m ? a.sc[0] : a.m; }

__global__ void __launch_bounds__(256) k_map_tile_sort(const MapArgs a, const uint64_t *src, uint64_t *dst) {
    static_assert(kSortTile % 256 == 0, "a tile is a whole number of keys per lane");
    __shared__ uint64_t tile[kSortTile];
    const uint64_t cnt = sort_count(a);
    const uint64_t base = (uint64_t)blockIdx.x * kSortTile;
    if (base >= cnt) {  // uniform per block
        note_pages(a);
        return;
    }
    const uint32_t len = (uint32_t)std::min<uint64_t>(kSortTile, cnt - base);
    for (uint32_t i = threadIdx.x; i < len; i += blockDim.x) tile[i] = src[base + i];
    __syncthreads();  // src may be dst: every read of the tile is done
    // each lane ranks its kSortTile / 256 keys in one sweep of the tile; a
    // lane past the tile's end ranks the largest key, and its rank is not used
    constexpr uint32_t K = kSortTile / 256;
    uint64_t key[K];
    uint32_t rank[K];
#pragma unroll
    for (uint32_t j = 0; j < K; ++j) {
        key[j] = ~0ull;
        rank[j] = 0;
        if (threadIdx.x + 256 * j < len) key[j] = tile[threadIdx.x + 256 * j];
    }
    for (uint32_t q = 0; q < len; ++q) {
        const uint64_t t = tile[q];
#pragma unroll
        for (uint32_t j = 0; j < K; ++j) rank[j] += t < key[j];
    }
#pragma unroll
    for (uint32_t j = 0; j < K; ++j)
        if (threadIdx.x + 256 * j < len) dst[base + rank[j]] = key[j];
    note_pages(a);
}

// One merge round: runs of w keys (a power of two, at least kSortTile) are
// merged in pairs.
__global__ void __launch_bounds__(256) k_map_merge(const MapArgs a, const uint64_t *src, uint64_t *dst, uint64_t w) {
    const uint64_t cnt = sort_count(a);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += stride) {
        const uint64_t key = src[i];
        const uint64_t pair = i & ~(2 * w - 1);
        const bool second = (i & w) != 0;
        const uint64_t own = second ? pair + w : pair;
        const uint64_t other = second ? pair : pair + w;
        const uint64_t olen = other >= cnt ? 0 : std::min<uint64_t>(w, cnt - other);
        uint64_t lo = 0, hi = olen;  // smaller keys in the other run: [0, lo)
        while (lo < hi) {
            const uint64_t mid = (lo + hi) >> 1;
            if (src[other + mid] < key)
                lo = mid + 1;
            else
                hi = mid;
        }
        dst[pair + (i - own) + lo] = key;
    }
}

// Zero the new tables (after a long list's sort).
__global__ void __launch_bounds__(256) k_map_zero(const MapArgs a) {
    const uint64_t nt = new_tables(a);
    DVm zvm;
    if (!nt || !map_vm(a, zvm)) return;
    uint8_t *arena = zvm.arena;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nt * 256; t += stride)
        *gp<g_u32x4>(arena + a.pool_hpa[t >> 8] + 16 * (t & 255)) = (u32x4){0u, 0u, 0u, 0u};
}

// Lane t links new table t (sorted position t takes pool frame t) from its
// parent entry, in a new table or an existing one, and handles map t: NO_POOL
// when the pool is short, else the leaf if it is the last map of its page.
// Links and leaves touch disjoint entries: a leaf whose page table exists has
// a fully present path, and links write only not-present entries (in existing
// tables) or entries of new tables.
__global__ void __launch_bounds__(256) k_map_write(const MapArgs a) {
    const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool short_pool = pool_short(a);
    const uint64_t nt = short_pool ? 0 : a.sc[0];
    if (t == 0) *a.n_used = nt;
    const uint64_t *uniq = a.tkeys_sorted;
    if (a.ept_map) {
        const DVm vm = a.v.vms[a.vm];
        if (t < nt) {  // link new EPT table t from its parent (new, or existing above it)
            const uint64_t key = uniq[t];
            const uint32_t l = 8u - (uint32_t)(key >> 56);
            const uint64_t gpa = (key & ((1ull << 56) - 1)) << (12 + 9 * l);
            const int64_t j = l + 1 < 4 ? find_key(uniq, nt, map_key(l + 1, gpa)) : -1;
            const uint64_t parent = j >= 0 ? a.pool_hpa[j] : existing_ept_table(vm, gpa, l + 1);
            store_entry(vm.arena, ept_slot(parent, l + 1, gpa), a.pool_hpa[t] | kEptRwx);
        }
        if (t >= a.n || a.res[t].code != DEVIRT_OK) return;
        const devirt_map m = a.maps[t];
        if (short_pool) {
            a.res[t].code = DEVIRT_NO_POOL;
            a.res[t].bytes_done = 0;
            a.res[t].fault_gva = m.gva;
            return;
        }
        if (!last_of_page(a, m.gva >> 12, t)) return;
        const int64_t j = find_key(uniq, nt, map_key(1, m.gva));
        const uint64_t pt = j >= 0 ? a.pool_hpa[j] : existing_ept_table(vm, m.gva, 1);
        store_entry(vm.arena, ept_slot(pt, 1, m.gva), m.gpa | (m.flags & 7u) | kEptWb);
        return;
    }
    if (a.asid >= a.v.nproc) return;
    const DProc p = a.v.procs[a.asid];
    const DVm vm = a.v.vms[p.vm];
    if (t < nt) {
        const uint64_t key = uniq[t];
        const uint32_t l = 8u - (uint32_t)(key >> 56);
        const uint64_t id = key & ((1ull << 56) - 1);
        const uint64_t va = id << (12 + 9 * l);
        int64_t j = -1;
        if (l + 1 < p.levels) j = find_key(uniq, nt, map_key(l + 1, va));
        uint64_t phpa = 0;
        bool have = true;
        if (j >= 0)
            phpa = a.pool_hpa[j];
        else
            have = existing_table(vm, p, va, l + 1, phpa);
        if (have) {
            const bool root_pae = p.levels == 3 && l + 1 == 3;
            const uint64_t idx = root_pae ? ((va >> 30) & 3) : (id & 511);
            store_entry(vm.arena, phpa + 8 * idx, a.pool_gpa[t] | (root_pae ? kP : (kP | kRW | kUS)));
        }
    }
    if (t >= a.n || a.res[t].code != DEVIRT_OK) return;
    const devirt_map m = a.maps[t];
    if (short_pool) {
        a.res[t].code = DEVIRT_NO_POOL;
        a.res[t].bytes_done = 0;
        a.res[t].fault_gva = m.gva;
        return;
    }
    if (!last_of_page(a, m.gva >> 12, t)) return;
    const int64_t j = find_key(uniq, nt, map_key(1, m.gva));
    uint64_t pt = 0;
    if (j >= 0)
        pt = a.pool_hpa[j];
    else if (!existing_table(vm, p, m.gva, 1, pt))
        return;
    store_entry(vm.arena, pt + 8 * ((m.gva >> 12) & 511), m.gpa | kP | kUS | ((m.flags & DEVIRT_MAP_WRITE) ? kRW : 0ull));
}

static unsigned blocks_for(uint64_t n) { return (unsigned)((n + 255) / 256 ? (n + 255) / 256 : 1); }

hipError_t launch_map(hipStream_t s, const MapArgs &a) {
    hipError_t e;
    const uint64_t nset = (1ull << a.tset_log2), npset = (1ull << a.pset_log2);
    // tset, tkeys and pset are contiguous, then sc
    const uint64_t ones = nset + a.m + npset, zeros = 4;
    hipLaunchKernelGGL(k_map_clear, dim3(blocks_for(std::min<uint64_t>(std::max(ones / 2, 2 * a.m), 1ull << 18))),
                       dim3(256), 0, s, a.tset, ones, a.sc, zeros, a.staged, (uint64_t *)a.pool_gpa, 2 * a.m);
    hipLaunchKernelGGL(k_map_walk, dim3(blocks_for(a.n)), dim3(256), 0, s, a);
    if (a.ept_pool) hipLaunchKernelGGL(k_map_pool, dim3(blocks_for(a.m)), dim3(256), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.rank) {
        // lanes to zero the new tables 16 bytes each and to note the maps'
        // pages, at most 2^18 (four workgroups a CU: one without work still
        // has to be launched); 64 keys a workgroup need at most 2^16
        const uint64_t lanes = std::max(a.m, std::min<uint64_t>(std::max(a.m * 256, a.n), 1ull << 18));
        hipLaunchKernelGGL(k_map_rank_zero, dim3(blocks_for(lanes)), dim3(256), 0, s, a);
    } else {
        // merge rounds for m keys; the tile sort's output buffer is chosen so
        // that the last round writes tkeys_sorted
        uint32_t rounds = 0;
        for (uint64_t w = kSortTile; w < a.m; w *= 2) ++rounds;
        uint64_t *buf[2] = {a.tkeys, a.tkeys_sorted};
        uint32_t cur = (rounds & 1) ? 0 : 1;
        const uint64_t notes = std::min<uint64_t>(a.n, 1ull << 18);  // lanes
        const uint64_t tiles = (a.m + kSortTile - 1) / kSortTile;
        hipLaunchKernelGGL(k_map_tile_sort, dim3((unsigned)std::max<uint64_t>(tiles, blocks_for(notes))), dim3(256), 0,
                           s, a, a.tkeys, buf[cur]);
        const unsigned mblocks = blocks_for(std::min<uint64_t>(a.m, 1ull << 22));
        for (uint64_t w = kSortTile; w < a.m; w *= 2) {
            hipLaunchKernelGGL(k_map_merge, dim3(mblocks), dim3(256), 0, s, a, buf[cur], buf[cur ^ 1], w);
            cur ^= 1;
        }
        hipLaunchKernelGGL(k_map_zero, dim3(blocks_for(std::min<uint64_t>(a.m * 256, 1ull << 22))), dim3(256), 0, s, a);
    }
    hipLaunchKernelGGL(k_map_write, dim3(blocks_for(std::max(a.n, a.m))), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace dv
