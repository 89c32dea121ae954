// What the window search's sources share: constants, lane moves, keys,
// tickets, the launch parameters and the workspace's layout, and the rule that
// picks the search kernel.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include "coop.h"

// Nothing below is part of the exported ABI.
#pragma GCC visibility push(hidden)

namespace coop_win {

constexpr uint32_t kThreads = 512;
constexpr uint32_t kWaves = kThreads / 64;
constexpr uint32_t kItems = 8;
constexpr uint32_t kTileLog2 = 12;
constexpr uint32_t kTile = 1u << kTileLog2;
static_assert(kTile == kThreads * kItems, "tile = threads x items");
constexpr uint32_t kValBits = 50;
constexpr uint64_t kValMask = (1ull << kValBits) - 1;
// With every block below 2^37 bytes, any staged prefix (fewer than 2^13
// blocks) fits the 50-bit field, and no prefix wraps.  Keys then stay below
// 2^13 << 50 = 2^63, so the difference of two keys is exact as a
// signed 64-bit number (the merge relies on it).
constexpr uint32_t kBigHiLog2 = 37 - 32;
// The end key after a staged region: above every key and target, and
// positive as a signed number.
constexpr uint64_t kEndKey = (1ull << 63) - 1;
constexpr uint64_t kNone = ~0ull;
constexpr uint32_t kNone32 = ~0u;
constexpr uint32_t kWalkCap = 1024;              // blocks a wavefront walks past a staged region
constexpr uint32_t kEpochShift = 24;             // counter = epoch << 24 | tickets
// Call tags (40 bits).  An eager call takes the next value of a host counter
// (bit 39 clear); a call captured into a graph takes bit 39 and 39 bits that
// an odd multiplier maps one-to-one from a word in the workspace, which a
// one-thread kernel advances ahead of every replay.  The two kinds never
// meet, and no two replays on one workspace share a tag before 2^39 calls.
constexpr uint64_t kTagMask = (1ull << 39) - 1;
constexpr uint64_t kGraphTag = 1ull << 39;
constexpr uint64_t kTagOdd = 0x9e3779b97f4a7c15ull;
// The queue word's 32-bit tag: the call tag's low 31 bits, and bit 31 set
// for graph replays (call tag bit 39), so that an eager call and a replay
// never carry the same queue tag.
__host__ __device__ constexpr uint32_t queue_tag(uint64_t call_tag) {
    return static_cast<uint32_t>(call_tag & 0x7fffffffull) | ((call_tag & kGraphTag) ? 0x80000000u : 0u);
}
static_assert(queue_tag(kGraphTag) == 0x80000000u && queue_tag(kGraphTag - 1) == 0x7fffffffu,
              "graph and eager queue tags differ in bit 31");
// Queue word: call tag << 32 | chunks claimed.  A reserve chunk slot holds a
// chunk index, kQEmpty (nothing claimed yet) or kQDone (the queue ran dry).
constexpr uint64_t kQEmpty = ~0ull, kQDone = ~0ull - 1;

// DPP controls (GFX9 encoding).
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E;  // quad_perm [1,0,3,2] and [2,3,0,1]
constexpr int kRowHalfMirror = 0x141, kRowMirror = 0x140;

// Lane move within the wavefront; lanes whose source is outside the row, or
// whose row is masked off, get `old`.
template <int Ctrl, int RowMask = 0xf>
__device__ __forceinline__ uint32_t dpp32(uint32_t v, uint32_t old) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(
        static_cast<int>(old), static_cast<int>(v), Ctrl, RowMask, 0xf, false));
}

template <int Ctrl, int RowMask = 0xf>
__device__ __forceinline__ uint64_t dpp64(uint64_t v, uint64_t old) {
    const uint32_t lo = dpp32<Ctrl, RowMask>(static_cast<uint32_t>(v), static_cast<uint32_t>(old));
    const uint32_t hi = dpp32<Ctrl, RowMask>(static_cast<uint32_t>(v >> 32),
                                             static_cast<uint32_t>(old >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint32_t readlane32(uint32_t v, uint32_t lane) {
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), static_cast<int>(lane)));
}

__device__ __forceinline__ uint64_t readlane64(uint64_t v, uint32_t lane) {
    return (static_cast<uint64_t>(readlane32(static_cast<uint32_t>(v >> 32), lane)) << 32) |
           readlane32(static_cast<uint32_t>(v), lane);
}

__device__ __forceinline__ uint64_t shfl64(uint64_t v, uint32_t src) {
    const uint32_t lo = __shfl(static_cast<uint32_t>(v), static_cast<int>(src), 64);
    const uint32_t hi = __shfl(static_cast<uint32_t>(v >> 32), static_cast<int>(src), 64);
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    return (static_cast<uint64_t>(uniform(static_cast<uint32_t>(v >> 32))) << 32) | uniform(static_cast<uint32_t>(v));
}

// v += v of the lane Ctrl names (0 where that lane is outside the row; rows
// off in RowMask keep v), as one add and one add-with-carry whose first
// operand is the moved lane (DPP on the adds themselves).  The compiler
// moves each half with its own instruction and then adds, three times the
// instructions; these sums are most of the staging scans.  The s_nop gives
// the two wait states a DPP read needs after a VALU write of its source.
#define COOP_ADD_DPP64(lo, hi, ctrl, mask)                                                     \
    asm volatile("s_nop 1\n\t"                                                                \
                 "v_add_co_u32_dpp %0, vcc, %0, %0 " ctrl " row_mask:" mask                    \
                 " bank_mask:0xf bound_ctrl:1\n\t"                                             \
                 "v_addc_co_u32_dpp %1, vcc, %1, %1, vcc " ctrl " row_mask:" mask              \
                 " bank_mask:0xf bound_ctrl:1"                                                 \
                 : "+v"(lo), "+v"(hi)                                                          \
                 :                                                                             \
                 : "vcc")

template <int Ctrl, int RowMask>
__device__ __forceinline__ void add_dpp64(uint64_t& v) {
    uint32_t lo = static_cast<uint32_t>(v), hi = static_cast<uint32_t>(v >> 32);
    if constexpr (Ctrl == kRowShr1 && RowMask == 0xf) COOP_ADD_DPP64(lo, hi, "row_shr:1", "0xf");
    else if constexpr (Ctrl == kRowShr2 && RowMask == 0xf) COOP_ADD_DPP64(lo, hi, "row_shr:2", "0xf");
    else if constexpr (Ctrl == kRowShr4 && RowMask == 0xf) COOP_ADD_DPP64(lo, hi, "row_shr:4", "0xf");
    else if constexpr (Ctrl == kRowShr8 && RowMask == 0xf) COOP_ADD_DPP64(lo, hi, "row_shr:8", "0xf");
    else if constexpr (Ctrl == kRowBcast15 && RowMask == 0xa) COOP_ADD_DPP64(lo, hi, "row_bcast:15", "0xa");
    else if constexpr (Ctrl == kRowBcast31 && RowMask == 0xc) COOP_ADD_DPP64(lo, hi, "row_bcast:31", "0xc");
    else static_assert(Ctrl < 0, "a DPP control without an add form");
    v = (static_cast<uint64_t>(hi) << 32) | lo;
}

// Candidate window: ordered by (cost, bytes, start); `end` rides along.
// Start and end are snapshot-local.
struct Key {
    uint64_t cost, bytes, start, end;
};

__device__ __forceinline__ Key key_none() { return Key{kNone, kNone, kNone, kNone}; }

__device__ __forceinline__ bool key_less(const Key& a, const Key& b) {
    if (a.cost != b.cost) return a.cost < b.cost;
    if (a.bytes != b.bytes) return a.bytes < b.bytes;
    return a.start < b.start;
}

struct Params {
    const uint64_t* size;
    const uint64_t* cost;
    const uint8_t* kind;
    const uint64_t* seg;
    const uint64_t* req_size;
    const uint64_t* req_off;
    coop_window_t* out;
    Key* part;             // [num_requests][pc] partial keys
    uint64_t* counters;    // [slices][num_segments] arrival tickets
    uint64_t* queue;       // chunk queue word
    uint64_t* bounds;      // [num_requests] least costs found so far (subtiles), or null
    uint64_t* pick;        // whether the search on subtiles takes the batch (null: it does not)
    uint64_t num_blocks;
    uint64_t num_segments;
    uint64_t num_requests;
    // Counts of units and chunks are below 2^32 (units < 2^32 by the plan)
    // and held in 32 bits, which keeps the kernel's uniform state within the
    // scalar registers; products of them are formed in 64 bits.
    uint32_t num_virtual;  // tile ids per slice: floor(num_blocks / kTile) + num_segments
    uint32_t units;        // work units: slices * num_virtual (below 2^32)
    uint32_t grid;         // workgroups; chunk w < grid is workgroup w's first
    uint32_t c1, c2;       // units per chunk: first chunks [0, u1), queued chunks after
                           // (c2 is a lower bound from the host, set by the kernel)
    uint32_t u1;           // units in the first chunks
    uint64_t nchunks;      // chunks in all (set by the kernel when there is a queue)
    uint64_t c1_magic;     // ceil(2^64 / c1), for division by c1
    uint64_t c2_magic;     // ceil(2^64 / c2) (set by the kernel)
    uint64_t nv_magic;     // ceil(2^64 / num_virtual)
    uint32_t qtag;         // this call's queue tag
    uint32_t queue_on;     // units past u1 go through the queue
    uint32_t pc;           // partial slots per request (at most 2^23)
    uint64_t epoch;        // this call's tag on the arrival tickets
    const uint64_t* tag_word;  // captured calls: the workspace word the tags come from
    uint32_t defer_cap;    // deferred entries, at most (the arrays: see Ext)
    uint32_t slices_log2;  // request slices (a power of two): slice y takes y, y + slices, ...
    double inv_slope;      // guess of b per tile id, for the first snapshot lookup
};

// The workspace after the queue word, laid out the same way by the host
// (make_plan): the tag word, the deferred list's word (queue tag << 32 |
// entries), the word coop_window_long_kernel claims entries by (queue tag
// << 32 | claims), the deferred entries {first unit, end unit, g, G}
// (16-byte aligned), the tile records of tile p >= 1 of every snapshot at index
// (seg[b] >> kTileLog2) + p - 1 (bytes of all its blocks, cost of its
// evictable blocks, its pinned count; written by the search kernel, read by
// coop_window_long_kernel), and one deferral bit per partial slot (bit q * pc + g: request
// q left windows to coop_window_long_kernel in its chunk part g).  Derived
// where needed rather than passed, to keep the kernels' uniform state small.
struct Ext {
    uint64_t* defer_word;
    uint64_t* claim_word;
    uint4* entries;
    uint64_t* rec_p;
    uint64_t* rec_c;
    uint64_t* rec_r;
    uint32_t* bits;
};

__device__ __forceinline__ Ext ext_of(const Params& P) {
    Ext e;
    e.defer_word = P.queue + 2;
    e.claim_word = P.queue + 3;
    e.entries = reinterpret_cast<uint4*>((reinterpret_cast<uintptr_t>(P.queue + 4) + 15) & ~uintptr_t{15});
    e.rec_p = reinterpret_cast<uint64_t*>(e.entries + P.defer_cap);
    const uint64_t nrec = P.num_blocks >> kTileLog2;
    e.rec_c = e.rec_p + nrec;
    e.rec_r = e.rec_c + nrec;
    e.bits = reinterpret_cast<uint32_t*>(e.rec_r + nrec);
    return e;
}

// A read of an array the kernel never writes (offsets, request sizes)
// through the constant address space: uniform indices then become scalar
// loads, which do not queue behind the vector loads in flight.
typedef const __attribute__((address_space(4))) uint64_t* ConstU64;
__device__ __forceinline__ uint64_t ld_const(const uint64_t* p, uint64_t i) {
    return ((ConstU64)(p))[i];
}

// floor(n / d) for n < 2^32, with magic = ceil(2^64 / d) (0 for d = 1):
// the high word of n * magic (Lemire, Kaser and Kurz, "Faster remainder by
// direct computation", 2019).
__device__ __forceinline__ uint64_t div_magic(uint64_t n, uint64_t magic) {
    return magic ? __umul64hi(n, magic) : n;
}

__device__ __forceinline__ uint64_t first_id(uint64_t b, uint64_t seg_b) {
    return (seg_b >> kTileLog2) + b;
}

__device__ __forceinline__ coop_window_t to_window(const Key& k, uint64_t S) {
    if (S == 0) return coop_window_t{0, 0, 0};
    if (k.start == kNone) return coop_window_t{kNone, kNone, kNone};
    return coop_window_t{k.start, k.end, k.cost};
}

// Uniform lower bound: the first i in [lo, hi) with pred(i) (pred monotone),
// or hi.
template <typename Pred>
__device__ __forceinline__ uint32_t lower_bound(uint32_t lo, uint32_t hi, Pred pred) {
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (pred(mid)) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// The same search by a whole wavefront (every lane active, same arguments):
// 64 evenly spaced probes narrow [lo, hi) to one gap per round, so a tile
// takes two rounds of LDS reads instead of a dozen dependent ones.
template <typename Pred>
__device__ __forceinline__ uint32_t wave_lower_bound(uint32_t lo, uint32_t hi, uint32_t lane,
                                                     Pred pred) {
    while (hi - lo > 64) {
        const uint32_t step = (hi - lo + 63) >> 6;
        const uint32_t i = lo + lane * step;
        const uint64_t m = __ballot(i >= hi || pred(i));
        // pred false at every probe below lane f, true at f (or past hi)
        const uint32_t f = m ? static_cast<uint32_t>(__builtin_ctzll(m)) : 64u;
        const uint32_t nhi = f < 64 ? lo + f * step : hi;
        lo = f ? lo + (f - 1) * step + 1 : lo;
        hi = nhi < hi ? nhi : hi;
    }
    const uint64_t m = __ballot(lo + lane >= hi || pred(lo + lane));
    return m ? lo + static_cast<uint32_t>(__builtin_ctzll(m)) : hi;
}

// A ticket on a tagged counter (tag << shift | arrivals), which an earlier
// call may have left with its own tag: the first arrival of this call swaps
// in tag | 1; every later one, once it sees this call's tag, adds 1, so
// arrivals that come together queue at the atomic unit instead of retrying
// compare-and-swaps.  The count stays below 2^shift.  Returns the ticket,
// from 1.
__device__ inline uint64_t take_ticket(uint64_t* ctr, uint64_t tag, uint32_t shift) {
    uint64_t old = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    while ((old >> shift) != tag) {
        if (__hip_atomic_compare_exchange_strong(ctr, &old, (tag << shift) | 1ull, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return 1;
    }
    const uint64_t prev = __hip_atomic_fetch_add(ctr, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (prev & ((1ull << shift) - 1)) + 1;
}

// Words handed from one workgroup to another.
__device__ __forceinline__ void store_word_device(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_word_device(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Partial keys are read by whichever workgroup takes a snapshot's last
// ticket, possibly on another XCD, and the XCDs' L2 caches are not coherent
// with each other.  They are written and read with device-scope relaxed
// atomics, which act at the device-coherent level (stores written through,
// loads served from there): publishing them needs only the writes to have
// completed before the ticket is taken, and no L2 write-back, which a
// release on every writer would cost on every combine.  The reader issues
// its loads only after its ticket has come back, behind an acquire.
__device__ __forceinline__ void store_key_device(Key* p, const Key& k) {
    __hip_atomic_store(&p->cost, k.cost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p->bytes, k.bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p->start, k.start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&p->end, k.end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ Key load_key_device(Key* p) {
    return Key{__hip_atomic_load(&p->cost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
               __hip_atomic_load(&p->bytes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
               __hip_atomic_load(&p->start, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
               __hip_atomic_load(&p->end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)};
}

// Deferred entries, tile records and deferral bits are handed from one
// workgroup to another (of the same kernel or of the next one on the
// stream, possibly on another XCD) the same way: device-scope atomic
// stores and loads.  A plain load can return a copy of the line that a
// cache took before the writer's store (measured: entries of one call
// read back as zeros by the long kernel).
__device__ __forceinline__ void store_entry_device(uint4* p, const uint4& v) {
    uint64_t* w = reinterpret_cast<uint64_t*>(p);
    __hip_atomic_store(w, static_cast<uint64_t>(v.x) | (static_cast<uint64_t>(v.y) << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + 1, static_cast<uint64_t>(v.z) | (static_cast<uint64_t>(v.w) << 32), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint4 load_entry_device(uint4* p) {
    uint64_t* w = reinterpret_cast<uint64_t*>(p);
    const uint64_t a = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t b = __hip_atomic_load(w + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // every lane reads the same entry: taking the words from the first lane
    // keeps the control flow that depends on them scalar
    return make_uint4(uniform(static_cast<uint32_t>(a)), uniform(static_cast<uint32_t>(a >> 32)),
                      uniform(static_cast<uint32_t>(b)), uniform(static_cast<uint32_t>(b >> 32)));
}

__device__ __forceinline__ Key min_key(const Key& a, const Key& b) { return key_less(b, a) ? b : a; }

// ---------------------------------------------------------------------------
// The search on subtiles (coop_window_sub.hip)
// ---------------------------------------------------------------------------

constexpr uint32_t kSub = 512;     // starts a wavefront searches at a time
constexpr uint32_t kSubHalo = 64;  // blocks after them that it stages
// Blocks that it walks past them.  Longer windows have the second kernel
// search the chunk's tiles again, a workgroup alone: one run of 1100 blocks
// among 2^24 (4096 requests) took 31 ms there with a walk of 1024 blocks.  One
// run of 9500 blocks and a request of 9000: 76 ms in all (67 without it; 106 on
// tiles).  Where longer runs are common enough to be seen, the look at the
// batch leaves it to the search on tiles.
constexpr uint32_t kSubWalk = 8192;
// The fewest blocks of a snapshot whose windows the search on subtiles can
// leave to the second kernel: a walk stops before the snapshot end only if
// more than kSub + kSubWalk blocks follow the subtile start, which is at most
// 7 blocks before the snapshot start.  (A subtile next to a block of 2^37
// bytes is staged without the kSubHalo blocks, so they do not count.)
constexpr uint64_t kSubDeferMin = kSub + kSubWalk - 6;

// Batches that the search on subtiles may take: 16 tiles and more for every
// workgroup, so that most tiles meet bounds from earlier ones and the cold
// start of the longer code is paid back (8.5 tiles, 256 pools of 65536 blocks:
// 467 us on tiles, 507 on subtiles; 2 tiles, 1024 pools of 4096: 34 and 56),
// and snapshots of 8192 blocks and more on average (clustered pools, a request
// each: of 8192 blocks 251 us on tiles, 238 on subtiles; of 4096, 238 and 270).
constexpr uint64_t kSubUnits = 16, kSubBlocks = 8192;
inline bool subtiles_may_pay(uint64_t units, uint64_t grid, uint64_t num_blocks, uint64_t num_segments) {
    return units >= kSubUnits * grid && num_blocks / kSubBlocks >= num_segments;
}

// Enqueues the pick between the two search kernels (into *P.pick; 1: subtiles)
// and the search on subtiles; false when a launch failed.
bool launch_subtiles(const Params& P, hipStream_t s);

}  // namespace coop_win

#pragma GCC visibility pop
