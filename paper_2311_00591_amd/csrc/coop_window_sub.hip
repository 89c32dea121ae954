// The window search on subtiles: the search kernel of large batches whose
// windows are short or whose costs are uneven (coop_window.h says which sizes,
// subtiles_pay below which contents; planning, the second kernel and the C
// entry points are in coop_window_search.hip).
//
// A merge of all starts with all ends reads two records of LDS per start and
// request, whether or not the window can win: it was bound by LDS reads and
// the instructions around them.  Here a request looks at a start only if the
// start's first blocks do not already cost more than the best window known,
// which a comparison of one-byte codes tells, four starts to an instruction.
// Mixed batch of 66e6 blocks and 16384 requests: 709 -> 497 us; one pool of
// 2^24 blocks and 4096 requests: 98.3 -> 68.3 ms.  What is left (counted): of a
// request and a subtile's 512 starts, 4.8 are probed and 1.1 searched for in
// the mixed batch, so staging the subtiles leads there; in the huge pool 35 and
// 26 are, and these searches take the time (windows that leave the subtile are
// walked for in 0.6% of the pairs).

#include "coop_window.h"

using namespace coop_win;

namespace {

// The wavefront's least value, in every lane of it.
template <int Ctrl, int RowMask>
__device__ __forceinline__ void min64_step(uint64_t& v) {
    const uint64_t x = dpp64<Ctrl, RowMask>(v, kNone);
    v = x < v ? x : v;
}

__device__ __forceinline__ uint64_t wave_min64(uint64_t v) {
    min64_step<kQuadXor1, 0xf>(v);
    min64_step<kQuadXor2, 0xf>(v);
    min64_step<kRowHalfMirror, 0xf>(v);
    min64_step<kRowMirror, 0xf>(v);
    min64_step<kRowBcast15, 0xa>(v);
    min64_step<kRowBcast31, 0xc>(v);
    return readlane64(v, 63);
}

// What the wavefront's lanes stored in LDS before is what its lanes read after
// (no instruction: a wavefront's LDS operations complete in order).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The lane's place among the set lanes of m.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u));
}

// ---------------------------------------------------------------------------
// Keys, tickets, partial results
// ---------------------------------------------------------------------------

// The walk over the units and the snapshot list.  One wavefront of a workgroup
// at a time moves it, the first to end a job's last pass (a barrier follows
// before the next can), and its state waits in LDS in between: held
// in scalar registers by every wavefront, with the next job and the launch
// parameters, it had most of them spilled to vector lanes (a fifth of the
// search kernel's vector instructions moved such values).
constexpr uint32_t kCache = 16;  // offsets of consecutive snapshots kept at hand
struct Control {
    uint64_t epoch;             // this call's tags
    uint32_t qtag;
    uint32_t c2;                // units per queued chunk, once the kernel has seen the snapshots
    uint64_t c2_magic, nchunks; // ceil(2^64 / c2); chunks in all
    uint64_t chunk;             // the current chunk
    uint32_t queue_on;          // the queue may hold more
    uint32_t u, u_end, u_begin; // the next unit, and the current chunk's units
    uint32_t y, v;              // unit u as (slice, tile id)
    uint32_t b, b0;             // snapshot holding tile id v (kNone32: locate it); first one at hand
    uint64_t seg[kCache], req[kCache];  // seg[b0 + i], req_off[b0 + i]
};

// The chunk holding unit u, and the units of chunk c.
__device__ __forceinline__ uint64_t chunk_of(const Params& P, uint32_t u, uint64_t c2_magic) {
    return u < P.u1 ? div_magic(u, P.c1_magic) : P.grid + div_magic(u - P.u1, c2_magic);
}

__device__ __forceinline__ void chunk_range(const Params& P, uint64_t c, uint32_t c2, uint64_t& b, uint64_t& e) {
    if (c < P.grid) {
        b = c * P.c1;
        e = b + P.c1 < P.u1 ? b + P.c1 : P.u1;
    } else {
        b = P.u1 + (c - P.grid) * static_cast<uint64_t>(c2);
        e = b + c2 < P.units ? b + c2 : P.units;
    }
    if (b > e) b = e;
}

// A job: the tiles from p on of snapshot b that lie in the current chunk
// (units [lo, hi)), for the requests of slice y.  The chunks holding the tiles
// of (b, y) are G consecutive ones; the current chunk is the g-th.  Offsets
// are clamped to the array lengths: malformed offsets give wrong answers,
// never an out-of-bounds access.
struct Job {
    uint32_t y, b;     // slice, snapshot (b < num_segments <= 2^32)
    uint32_t lo, hi;
    uint64_t s0, s1, q0, K, tiles, p;
    uint32_t g, G;     // at most pc
    uint32_t direct;   // the chunk holds every tile (a truth value)
    uint32_t valid;    // there is such a job
};

// The snapshot holding tile id v: the largest b in [0, B) with f(b) =
// floor(seg[b] / kTile) + b <= v, by a whole wavefront (same arguments in
// every lane).  A guess from the average snapshot length is tried first, so
// uniform batches settle in one round of loads; otherwise 64 probes a round.
__device__ uint32_t locate(const Params& P, uint64_t v, uint32_t lane) {
    const uint64_t B = P.num_segments;
    uint64_t g = static_cast<uint64_t>(static_cast<double>(v) * P.inv_slope);
    if (g >= B) g = B - 1;
    uint64_t lo = 0, hi = B;  // f(lo) <= v < f(hi) (f(B) taken as infinite)
    const uint64_t sg = ld_const(P.seg, g), sg1 = ld_const(P.seg, g + 1);
    if (first_id(g, sg) > v) {
        hi = g;
    } else {
        lo = g;
        if (g + 1 < B && first_id(g + 1, sg1) > v) hi = g + 1;
    }
    while (hi - lo > 1) {
        const uint64_t step = (hi - lo + 63) >> 6;
        const uint64_t i = lo + (lane + 1) * step;
        const uint64_t m = __ballot(i >= hi || first_id(i, P.seg[i]) > v);
        const uint32_t f = m ? static_cast<uint32_t>(__builtin_ctzll(m)) : 63u;
        // f(lo + f * step) <= v < f(lo + (f + 1) * step)
        const uint64_t nhi = lo + (f + 1) * step;
        hi = m && nhi < hi ? nhi : hi;
        lo = lo + f * step;
    }
    return static_cast<uint32_t>(lo);
}

// Tile p of snapshot b (offsets s0, s1, q0, q1 clamped to the array lengths
// here) as a job of slice y; false if there is no such tile or the slice has
// no request.
__device__ __forceinline__ bool make_job(const Params& P, uint32_t y, uint32_t v, uint32_t b, uint64_t seg0,
                                         uint64_t seg1, uint64_t req0, uint64_t req1, Job& job) {
    const uint64_t s1 = seg1 < P.num_blocks ? seg1 : P.num_blocks;
    const uint64_t s0 = seg0 < s1 ? seg0 : s1;
    const uint64_t q1 = req1 < P.num_requests ? req1 : P.num_requests;
    const uint64_t q0 = req0 < q1 ? req0 : q1;
    const uint64_t R = q1 - q0, nb = s1 - s0;
    // tiles start at floor8(s0) + p * kTile
    const uint64_t tiles = nb ? (s1 - (s0 & ~7ull) + kTile - 1) >> kTileLog2 : 1;
    const uint64_t p = v - first_id(b, seg0);  // wraps (and is refused) if the offsets are malformed
    if (p >= tiles || y >= R) return false;
    job.y = y;
    job.b = b;
    job.s0 = s0;
    job.s1 = s1;
    job.q0 = q0;
    job.K = ((R - y - 1) >> P.slices_log2) + 1;
    job.tiles = tiles;
    job.p = p;
    job.valid = 1;
    return true;
}

// ---------------------------------------------------------------------------
// Filter codes
// ---------------------------------------------------------------------------
//
// A start i has a window inside the staged region only if its run still holds
// S bytes from there, and that window can win only if what it must hold costs
// no more than the best window found so far (the bound).  Both quantities are
// kept as 7-bit codes, monotone in the value, so that comparing codes never
// drops a start that the values would keep; four starts are compared by one
// 32-bit subtraction, whose bytes cannot borrow from each other because one
// operand has every byte's top bit set.

// The leading bits (exponent and the mantissa bits above `shift`) of the
// binary32 image of v.  Monotone: the sum of the halves rounds monotonically
// while v < 2^56, and larger values are cut to a place where all codes are
// the same.
__device__ __forceinline__ uint32_t code_image(uint64_t v, uint32_t shift) {
    const uint32_t hi = static_cast<uint32_t>(v >> 32);
    const float f = fmaf(static_cast<float>(hi < 0xfffffeu ? hi : 0xfffffeu), 4294967296.0f,
                         static_cast<float>(static_cast<uint32_t>(v)));
    return __float_as_uint(f) >> shift;
}

__device__ __forceinline__ uint32_t code_clamp(uint32_t image, uint32_t off) {
    const int c = static_cast<int>(image - off);
    return static_cast<uint32_t>(c < 1 ? 1 : c > 127 ? 127 : c);
}

// How a region's bytes and costs are coded: bytes floored by 2^ysh to below
// 2^31, two mantissa bits; costs by one or two
// mantissa bits by the region's total (31 or 63 octaves below it).
struct Coding {
    uint32_t ysh, aoff, cshift, coff;
};

__device__ __forceinline__ uint32_t bytes_image(uint32_t y) {
    return __float_as_uint(static_cast<float>(y)) >> 21;
}

__device__ __forceinline__ uint32_t cost_code(uint64_t c, const Coding& k) {
    return code_clamp(code_image(c, k.cshift), k.coff);
}

__device__ __forceinline__ Coding coding_of(uint64_t bytes, uint64_t cost) {
    Coding k;
    const uint32_t top = static_cast<uint32_t>(bytes >> 31);
    k.ysh = uniform(top ? 32u - static_cast<uint32_t>(__builtin_clz(top)) : 0u);
    k.aoff = uniform(bytes_image(static_cast<uint32_t>(bytes >> k.ysh))) - 127u;
    k.cshift = uniform(cost >> 40 ? 22u : 21u);
    k.coff = uniform(code_image(cost, k.cshift)) - 127u;
    return k;
}

// ---------------------------------------------------------------------------
// The search of a tile: eight wavefronts, each on its own eighth
// ---------------------------------------------------------------------------
//
// Each wavefront stages kSub starts and kSubHalo blocks after them into LDS of
// its own and answers every request of the job on them, with no barrier: the
// wavefronts of a workgroup meet only where a snapshot (in the current chunk)
// ends.  A workgroup that staged a tile together had its wavefronts waiting
// at the tile's three barriers, and for the slowest request, for a third of
// the time.

constexpr uint32_t kSubStage = kSub + kSubHalo;
static_assert(kSub == 64 * kItems && kSub * kWaves == kTile, "eight blocks a lane, eight wavefronts a tile");
constexpr uint32_t kProbe = 4;  // boundaries a start's first probes read past it
constexpr uint32_t kSubN = (kSubStage + 2 + kProbe + 7) / 8 * 8;
static_assert(kSubStage + 2 < (1u << (63 - kValBits)), "keys stay below 2^63");
static_assert(kSubStage < (1u << (kValBits - 37)), "staged prefixes fit the key field");
constexpr uint32_t kGroup = 64;  // requests answered in one pass over a job, one per lane
constexpr uint32_t kStartMask = kSub - 1;
static_assert(kGroup * kSub <= 65536, "a start and a request fit a queue entry");
// Starts that wait for their first probes (from the bottom) and for their
// search (from the top): fewer than 64 of each, and 64 more of one.
constexpr uint32_t kQueue = 192;
constexpr uint32_t kRecRing = 16;  // tiles of a job whose records are being summed

// Staged boundaries: the key (R << 50 | P, or plain P beside a huge block) and
// the cost prefix C, one 16-byte record where the cost has 64 bits.  Within
// each eight boundaries the places are permuted by the number of the eight, so
// that the lanes of a wavefront, each storing one of its own eight, spread over
// the LDS banks (rotating the values in registers instead took a hundred
// vector instructions a subtile and spilled).
__device__ __forceinline__ uint32_t place(uint32_t i) { return i ^ ((i >> 3) & 7u); }

struct Bounds {
    __attribute__((aligned(16))) uint64_t kv[2 * kSubN];
    __device__ __forceinline__ uint64_t K(uint32_t i) const { return kv[2 * place(i)]; }
    __device__ __forceinline__ uint64_t C(uint32_t i) const { return kv[2 * place(i) + 1]; }
    __device__ __forceinline__ void get(uint32_t i, uint64_t& k, uint64_t& c) const {
        const ulonglong2 r = *reinterpret_cast<const ulonglong2*>(&kv[2 * place(i)]);
        k = r.x;
        c = r.y;
    }
    __device__ __forceinline__ void put(uint32_t i, uint64_t k, uint64_t c) {
        *reinterpret_cast<ulonglong2*>(&kv[2 * place(i)]) = ulonglong2{k, c};
    }
    __device__ __forceinline__ void put_key(uint32_t i, uint64_t k) { kv[2 * place(i)] = k; }
    __device__ __forceinline__ char* spare(uint32_t i) { return reinterpret_cast<char*>(&kv[2 * i]); }
};

struct Sub {
    Bounds bd;
    uint16_t queue[kQueue];
};
static_assert(sizeof(Key) * kGroup <= sizeof(Bounds), "a wavefront's answers take its boundaries' place");

// The record of a tile being summed: its wavefronts add their shares; the
// last of them publishes it and clears the place.
struct RecSum {
    uint64_t q, r;
    uint64_t c;
    uint32_t n;
};

struct SearchSmem {
    Sub sub[kWaves];
    RecSum rec[kRecRing];
    uint64_t bound[kGroup];  // the group's requests: least cost found so far, packed
    Control ctl;
    Job job[3];              // the job at hand, and the next two
    uint64_t deferred;       // requests of the group with windows left to the second kernel
    uint32_t arrived;        // wavefronts that have ended the pass
    uint32_t rec_done;       // tiles of the job whose records are out
    uint32_t last_flag;
    uint64_t tmax[kWaves];
};

// A subtile's blocks as loaded, one lane's share: kItems blocks and one halo
// block.
struct SubRegs {
    uint64_t sz[kItems], ct[kItems];
    uint32_t kd[2];  // kind of block j in byte j & 3 of kd[j / 4]
    uint64_t hq, hc;
    uint32_t hk;
};

struct SubGeom {
    uint64_t t0;    // global index of the first block (a multiple of 8)
    uint32_t nt;    // blocks, counting the lead (0: the snapshot ends before)
    uint32_t hm;    // halo blocks
    uint32_t lead;  // blocks before the snapshot start: pinned phantoms
};

// Wavefront w's part of tile p of a snapshot: tiles start on multiples of 8
// (tile p at floor8(s0) + p * kTile).
__device__ __forceinline__ SubGeom sub_geom(uint64_t s0, uint64_t s1, uint64_t p, uint32_t w) {
    SubGeom t;
    t.t0 = (s0 & ~7ull) + (p << kTileLog2) + w * kSub;
    const uint64_t left = s1 > t.t0 ? s1 - t.t0 : 0;
    t.nt = static_cast<uint32_t>(left < kSub ? left : kSub);
    const uint64_t after = left - t.nt;
    t.hm = static_cast<uint32_t>(after < kSubHalo ? after : kSubHalo);
    t.lead = t.t0 < s0 ? static_cast<uint32_t>(s0 - t.t0) : 0u;  // below 8: only where p and w are 0
    return t;
}

// Issues every load of a subtile; nothing waits for them here.  16-byte loads
// of size and cost pairs and one 8-byte load of the kinds, at indices clamped
// to the subtile (blocks past nt are masked when staged), when every such
// load stays inside the arrays; else one load per block.
__device__ __forceinline__ void sub_loads(const Params& P, const SubGeom& t, uint32_t lane, SubRegs& r) {
    r.hq = 0;
    r.hc = 0;
    r.hk = COOP_FREE;
    if (t.nt == 0) return;
    const uint32_t i0 = lane * kItems;
    const bool aligned = ((reinterpret_cast<uintptr_t>(P.size) | reinterpret_cast<uintptr_t>(P.cost)) &
                          15u) == 0 &&
                         (reinterpret_cast<uintptr_t>(P.kind) & 7u) == 0;
    if (aligned && t.t0 + ((t.nt + 7u) & ~7u) <= P.num_blocks) {
        const uint32_t last2 = (t.nt - 1) & ~1u, last8 = (t.nt - 1) & ~7u;
#pragma unroll
        for (uint32_t j = 0; j < kItems / 2; ++j) {
            const uint32_t i = i0 + 2 * j < last2 ? i0 + 2 * j : last2;
            const ulonglong2 a = *reinterpret_cast<const ulonglong2*>(P.size + t.t0 + i);
            const ulonglong2 b = *reinterpret_cast<const ulonglong2*>(P.cost + t.t0 + i);
            r.sz[2 * j] = a.x;
            r.sz[2 * j + 1] = a.y;
            r.ct[2 * j] = b.x;
            r.ct[2 * j + 1] = b.y;
        }
        const uint2 k2 = *reinterpret_cast<const uint2*>(P.kind + t.t0 + (i0 < last8 ? i0 : last8));
        r.kd[0] = k2.x;
        r.kd[1] = k2.y;
    } else {
        r.kd[0] = 0;
        r.kd[1] = 0;
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) {
            const uint32_t i = i0 + j < t.nt ? i0 + j : t.nt - 1;
            r.sz[j] = P.size[t.t0 + i];
            r.ct[j] = P.cost[t.t0 + i];
            r.kd[j >> 2] |= static_cast<uint32_t>(P.kind[t.t0 + i]) << (8 * (j & 3));
        }
    }
    if (lane < t.hm) {
        const uint64_t gp = t.t0 + t.nt + lane;
        r.hk = P.kind[gp];
        r.hq = P.size[gp];
        r.hc = P.cost[gp];
    }
}

// What staging left behind: uniform values, and this lane's filter codes
// (starts 8 lane .. 8 lane + 7; the bytes' codes with 128 added).
struct SubState {
    bool packed;      // keys R << 50 | P; otherwise plain P with R in the spare place
    uint32_t end;     // staged boundaries [0, end]
    uint32_t endrun;  // R at the region end
    uint64_t xend;    // key at the region end
    uint64_t xcend;          // C at the region end
    uint64_t tq, tr;  // the starts' blocks: bytes, pinned blocks
    uint64_t tc;             // and cost
    Coding code;
    uint32_t av[2], cc[2];
};

struct SumOf {
    uint64_t q;
    uint64_t c;
};

template <int Ctrl, int RowMask>
__device__ __forceinline__ void sum_step(SumOf& s) {
    add_dpp64<Ctrl, RowMask>(s.q);
    add_dpp64<Ctrl, RowMask>(s.c);
}

// Inclusive sums over the wavefront: rows of 16 lanes, then row 0 into row 1
// and row 2 into row 3, then row 1 into rows 2 and 3.
__device__ __forceinline__ void wave_inclusive_sum(SumOf& s) {
    sum_step<kRowShr1, 0xf>(s);
    sum_step<kRowShr2, 0xf>(s);
    sum_step<kRowShr4, 0xf>(s);
    sum_step<kRowShr8, 0xf>(s);
    sum_step<kRowBcast15, 0xa>(s);
    sum_step<kRowBcast31, 0xc>(s);
}

// Run ids of a plain subtile (no halo), in the place of the halo's boundaries.
__device__ __forceinline__ uint16_t* plain_runs(Bounds& bd) {
    return reinterpret_cast<uint16_t*>(bd.spare(kSub + 1));
}
static_assert((kSub + 1) * sizeof(uint16_t) <= (kSubN - kSub - 1) * 16, "the run ids fit there");

// Stages a subtile and its halo.  One pass of prefix sums: the key itself, X =
// sum of (size + 2^50 per pinned block), which is R << 50 | P exactly while P
// stays below 2^50 (every block below 2^37 bytes), and the cost prefix C.  A
// subtile holding a block of 2^37 bytes or more is staged plain instead: P =
// X - 2^50 R (exact modulo 2^64), R beside it, no halo, no codes.
// least: the least request.
__device__ __forceinline__ SubState sub_stage(Bounds& bd, const SubGeom& tg, uint32_t lane, SubRegs& r,
                                                 uint64_t least) {
    constexpr uint64_t kRunOne = 1ull << kValBits;
    const uint32_t nt = tg.nt, hm = tg.hm;
    const uint32_t i0 = lane * kItems;
    uint64_t hx = 0;
    uint64_t hcost = 0;
    if (lane < hm) {
        hx = r.hq + (r.hk >= COOP_PINNED ? kRunOne : 0);
        if (r.hk == COOP_EVICTABLE) hcost = r.hc;
    }
    const bool hbig = lane < hm && ((r.hq >> 32) >> kBigHiLog2) != 0;
    // this lane's exclusive sums (blocks past nt: empty free blocks; blocks
    // before the lead: empty pinned blocks)
    SumOf t{0, 0};
    uint64_t sx[kItems];
    uint64_t sc[kItems];
    uint32_t pinned = 0;  // bit j: block j pinned
    uint32_t hi_or = 0;
    auto item = [&](uint32_t j, bool in) {
        const uint64_t s_j = in ? r.sz[j] : 0;
        const uint32_t raw = (r.kd[j >> 2] >> (8 * (j & 3))) & 0xffu;
        const uint32_t k_j = in ? raw
                                : (i0 + j < tg.lead ? static_cast<uint32_t>(COOP_PINNED)
                                                    : static_cast<uint32_t>(COOP_FREE));
        const uint32_t p_j = k_j >= COOP_PINNED ? 1u : 0u;
        pinned |= p_j << j;
        sx[j] = t.q;
        sc[j] = t.c;
        t.q += s_j + (static_cast<uint64_t>(p_j) << kValBits);
        const uint64_t c_j = r.ct[j];
        t.c = t.c + (k_j == COOP_EVICTABLE ? c_j : 0);
        hi_or |= static_cast<uint32_t>(s_j >> 32);
    };
    if (nt == kSub && tg.lead == 0) {
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) item(j, true);
    } else {
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) item(j, i0 + j < nt && i0 + j >= tg.lead);
    }
    SumOf wi = t;
    wave_inclusive_sum(wi);
    const uint64_t base_x = wi.q - t.q;
    const uint64_t base_c = wi.c - t.c;
    SubState ts;
    ts.tq = readlane64(wi.q, 63);
    ts.tc = readlane64(wi.c, 63);
    ts.packed = !__ballot((hi_or >> kBigHiLog2) != 0);
    ts.end = nt;
    ts.xend = ts.tq;
    ts.xcend = ts.tc;
    ts.av[0] = ts.av[1] = 0x80808080u;
    ts.cc[0] = ts.cc[1] = 0;
    if (ts.packed) {
        ts.tr = ts.tq >> kValBits;
        uint64_t hwall = kNone;  // key before the halo's first pinned block
        if (hm && !__ballot(hbig)) {
            SumOf hs{hx, hcost};
            wave_inclusive_sum(hs);
            const uint64_t hpins = __ballot(hx >= kRunOne);
            const uint64_t k = ts.tq + hs.q - hx;
            if (lane < hm) bd.put(nt + lane, k, ts.tc + hs.c - hcost);
            if (hpins) hwall = readlane64(k, static_cast<uint32_t>(__builtin_ctzll(hpins)));
            ts.end = nt + hm;
            ts.xend = ts.tq + readlane64(hs.q, 63);
            ts.xcend = ts.tc + readlane64(hs.c, 63);
        }
        ts.endrun = static_cast<uint32_t>(ts.xend >> kValBits);
        // wall: the key before the first pinned block after this lane's blocks
        // (the region end's when there is none)
        uint64_t fx = 0;
#pragma unroll
        for (uint32_t j = kItems; j-- > 0;) fx = (pinned >> j) & 1u ? sx[j] : fx;
        fx += base_x;
        const uint64_t pins = __ballot(pinned != 0);
        const uint64_t later = pins & (~1ull << lane);
        const uint64_t nx = shfl64(fx, later ? static_cast<uint32_t>(__builtin_ctzll(later)) : lane);
        uint64_t wall = later ? nx : hwall != kNone ? hwall : ts.xend;
        ts.code = coding_of(ts.xend & kValMask, ts.xcend);
        // A window of any of the job's requests from block j costs at least
        // as much as block j and as many of the next kAhead - 1 as are needed
        // to reach the least request (within this lane's blocks).  Bytes are
        // compared in 32 bits: y floors them by 2^ysh, so a difference below
        // floor(least / 2^ysh) is one below the least request (a pinned block
        // between changes it, but no window crosses one).
        constexpr uint32_t kAhead = 4;
        const uint64_t lf = least >> ts.code.ysh;
        const uint32_t least32 = uniform(lf < 0x7fffffffull ? static_cast<uint32_t>(lf) : 0x7fffffffu);
        uint32_t y[kItems];
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) y[j] = static_cast<uint32_t>(sx[j] >> ts.code.ysh);
        uint32_t ac[2] = {0, 0}, cc[2] = {0, 0};
#pragma unroll
        for (uint32_t j = kItems; j-- > 0;) {
            const uint64_t x = base_x + sx[j];
            const bool stop = (pinned >> j) & 1u;
            wall = stop ? x : wall;
            const bool in = !stop && (nt == kSub || i0 + j < nt);
            uint64_t ce = j + 1 < kItems ? sc[j + 1] : t.c;
            bool more = true;
#pragma unroll
            for (uint32_t k = j + 2; k <= kItems && k <= j + kAhead; ++k) {
                more = more && y[k - 1] - y[j] < least32;
                const uint64_t ck = k < kItems ? sc[k] : t.c;
                ce = more ? ck : ce;
            }
            const uint32_t left = static_cast<uint32_t>((wall - x) >> ts.code.ysh);
            const uint32_t a = in ? code_clamp(bytes_image(left), ts.code.aoff) : 0u;
            const uint32_t c = cost_code(ce - sc[j], ts.code);
            ac[j >> 2] |= (a | 0x80u) << (8 * (j & 3));
            cc[j >> 2] |= c << (8 * (j & 3));
        }
        ts.av[0] = ac[0];
        ts.av[1] = ac[1];
        ts.cc[0] = cc[0];
        ts.cc[1] = cc[1];
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j)
            if (nt == kSub || i0 + j < nt) bd.put(i0 + j, base_x + sx[j], base_c + sc[j]);
        if (lane == 0) bd.put(ts.end, ts.xend, ts.xcend);
        if (lane <= kProbe) bd.put_key(ts.end + 1 + lane, kEndKey);
    } else {
        // pinned blocks before this lane's first block, and in all
        uint32_t before = 0, all = 0;
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) {
            const uint64_t m = __ballot((pinned >> j) & 1u);
            before += lanes_below(m);
            all += static_cast<uint32_t>(__builtin_popcountll(m));
        }
        uint16_t* run = plain_runs(bd);
        ts.tr = all;
        ts.tq -= static_cast<uint64_t>(all) << kValBits;
        ts.endrun = all;
        ts.xend = ts.tq;
        uint32_t rr = before;
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) {
            if (i0 + j < nt) {
                bd.put(i0 + j, base_x + sx[j] - (static_cast<uint64_t>(rr) << kValBits), base_c + sc[j]);
                run[i0 + j] = static_cast<uint16_t>(rr);
            }
            rr += (pinned >> j) & 1u;
        }
        if (lane == 0) {
            bd.put(nt, ts.xend, ts.xcend);
            run[nt] = static_cast<uint16_t>(all);
        }
    }
    if (ts.packed) ts.tq &= kValMask;
    wave_sync();
    return ts;
}

// A group's state in a wavefront: lane n holds request n's size, and the least
// window this wavefront has found for it.
struct Group {
    uint64_t S;
    Key acc;
    uint64_t live;  // requests to search for (uniform)
};

// Folds the lanes' windows (valid where ok; lane's request rq, snapshot-local
// start and end) into the requests' least ones and lowers their bounds.
__device__ __forceinline__ void fold(Group& g, uint64_t* bounds, uint32_t lane, bool ok, uint32_t rq, uint64_t cost,
                                     uint64_t bytes, uint64_t start, uint64_t end) {
    for (uint64_t todo; (todo = __ballot(ok)) != 0;) {
        // the least window of one request among the lanes
        uint32_t l = static_cast<uint32_t>(__builtin_ctzll(todo));
        const uint32_t n = readlane32(rq, l);
        const bool same = ok && rq == n;
        Key best;
        for (;;) {
            best = Key{readlane64(cost, l), readlane64(bytes, l), readlane64(start, l), 0};
            const uint64_t m = __ballot(same && key_less(Key{cost, bytes, start, 0}, best));
            if (!m) break;
            l = static_cast<uint32_t>(__builtin_ctzll(m));
        }
        best.end = readlane64(end, l);
        if (lane == n && key_less(best, g.acc)) {
            g.acc = best;
            __hip_atomic_fetch_min(&bounds[n], best.cost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        ok = ok && rq != n;
    }
}

// Whether a lane's window, of a cost at most its request's bound, can take
// the place of the least one this wavefront holds: equal costs decide by
// bytes and start.
__device__ __forceinline__ bool beats(const Group& g, bool ok, uint32_t rq, uint64_t cost, uint64_t bound,
                                      uint64_t bytes, uint64_t start) {
    ok = ok && cost <= bound;
    if (__ballot(ok && cost == bound)) {
        const Key a{shfl64(g.acc.cost, rq), shfl64(g.acc.bytes, rq), shfl64(g.acc.start, rq), 0};
        ok = ok && key_less(Key{cost, bytes, start, 0}, a);
    }
    return ok;
}

// First probes of up to 64 queued starts (from the queue's bottom): windows
// of one or two blocks are scored; longer ones join the search queue unless
// their first two blocks (four, when the window is longer still) already
// cost more than the bound.
__device__ __forceinline__ void probe_starts(Sub& sub, Group& g, uint64_t* bounds, uint32_t lane, uint64_t tl,
                                             uint32_t n, uint32_t& n0, uint32_t& n1) {
    wave_sync();
    n0 -= n;
    const bool act = lane < n;
    const uint32_t e = act ? sub.queue[n0 + lane] : 0u;
    const uint32_t i = e & kStartMask, rq = e / kSub;
    const uint64_t S = shfl64(g.S, rq);
    const uint64_t bound = bounds[rq];
    const uint64_t Sc = S < (1ull << kValBits) ? S : (1ull << kValBits);
    uint64_t x0, x1, x2, x4;
    uint64_t c0, c1, c2, c4;
    sub.bd.get(i, x0, c0);
    sub.bd.get(i + 1, x1, c1);
    sub.bd.get(i + 2, x2, c2);
    sub.bd.get(i + 4, x4, c4);
    const bool one = x1 - x0 >= Sc, two = x2 - x0 >= Sc, four = x4 - x0 >= Sc;
    const uint64_t d = one ? x1 - x0 : x2 - x0;
    const uint64_t c = (one ? c1 : c2) - c0;
    const bool ok = beats(g, act && two && d < (1ull << kValBits), rq, c, bound, d, tl + i);
    const bool more = act && !two && (four ? c2 : c4) - c0 <= bound;
    const uint64_t m = __ballot(more);
    if (more) sub.queue[kQueue - 1 - n1 - lanes_below(m)] = static_cast<uint16_t>(e);
    n1 += static_cast<uint32_t>(__builtin_popcountll(m));
    if (__ballot(ok)) fold(g, bounds, lane, ok, rq, c, d, tl + i, tl + i + (one ? 1u : 2u));
}

// The search of up to 64 queued starts (from the queue's top) whose windows
// hold three blocks or more: probes at doubling distances until S bytes are
// reached, then a bisection.  A lane stops once the blocks known to be in its
// window cost more than the bound.
__device__ __forceinline__ void search_starts(Sub& sub, Group& g, uint64_t* bounds, uint32_t lane, uint64_t tl,
                                              uint32_t end, uint32_t n, uint32_t& n1) {
    wave_sync();
    n1 -= n;
    const uint32_t e = lane < n ? sub.queue[kQueue - 1 - n1 - lane] : 0u;
    const uint32_t i = e & kStartMask, rq = e / kSub;
    const uint64_t S = shfl64(g.S, rq);
    const uint64_t bound = bounds[rq];
    const uint64_t Sc = S < (1ull << kValBits) ? S : (1ull << kValBits);
    uint64_t x0;
    uint64_t c0;
    sub.bd.get(i, x0, c0);
    uint32_t lo = i + 2, hi = i + 2, step = 4;
    uint64_t dh = 0;
    uint64_t ch = 0;  // of boundary hi
    bool act = lane < n;
    while (__ballot(act)) {
        if (act) {
            const uint32_t k = i + step < end + 1 ? i + step : end + 1;
            uint64_t x;
            uint64_t c;
            sub.bd.get(k, x, c);
            const uint64_t d = x - x0;
            c = c - c0;
            if (d >= Sc || k > end) {  // (the key past the region end is above every target)
                hi = k;
                dh = d;
                ch = c;
                act = false;
            } else {
                lo = k;
                act = c <= bound;
                step <<= 1;
            }
        }
    }
    // a window ends in (lo, hi] for the lanes that got there
    bool live = lane < n && hi > lo;
    act = live && hi - lo > 1;
    while (__ballot(act)) {
        if (act) {
            const uint32_t mid = (lo + hi) >> 1;
            uint64_t x;
            uint64_t c;
            sub.bd.get(mid, x, c);
            const uint64_t d = x - x0;
            c = c - c0;
            if (d >= Sc) {
                hi = mid;
                dh = d;
                ch = c;
            } else {
                lo = mid;
                live = c <= bound;
            }
            act = live && hi - lo > 1;
        }
    }
    const bool ok = beats(g, live && dh < (1ull << kValBits), rq, ch, bound, dh, tl + i);
    if (__ballot(ok)) fold(g, bounds, lane, ok, rq, ch, dh, tl + i, tl + hi);
}

// The in-region windows of the group's live requests in a packed subtile.
__device__ __forceinline__ void sub_requests(Sub& sub, Group& g, uint64_t* bounds, const SubState& ts,
                                             uint32_t lane, uint64_t tl) {
    // lane n: request n's codes, in every byte (a request that is not
    // searched for, or needs more bytes than the region holds, passes no start)
    const uint64_t bytes = ts.xend & kValMask;
    const bool on = ((g.live >> lane) & 1u) != 0 && g.S <= bytes;
    const uint32_t s4 =
        (on ? code_clamp(bytes_image(static_cast<uint32_t>(g.S >> ts.code.ysh)), ts.code.aoff) : 0u) * 0x01010101u;
    uint32_t n0 = 0, n1 = 0, n = 0, mask = 0;
    // Requests without a bound yet look at the most promising starts first
    // (half of the lanes' least codes and those below), which finds them one:
    // the windows of every other start would be searched for otherwise.
    uint64_t first = __ballot(on && bounds[lane] == kNone);
    uint64_t todo = first ? first : __ballot(on);
    uint32_t b4 = 0;
    if (first) {
        uint32_t least = 127;
#pragma unroll
        for (uint32_t j = 0; j < kItems; ++j) {
            const uint32_t c = (ts.cc[j >> 2] >> (8 * (j & 3))) & 0xffu;
            const bool in = ((ts.av[j >> 2] >> (8 * (j & 3))) & 0x7fu) != 0;
            least = in && c < least ? c : least;
        }
        uint32_t lo = 1, hi = 127;  // the least code that half of the lanes reach
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (__builtin_popcountll(__ballot(least <= mid)) >= 32) hi = mid;
            else lo = mid + 1;
        }
        b4 = lo * 0x01010101u | 0x80808080u;
    } else {
        b4 = cost_code(bounds[lane], ts.code) * 0x01010101u | 0x80808080u;
    }
    for (;;) {
        const uint64_t any = __ballot(mask != 0);
        if (any) {
            // each lane's next start
            const uint32_t bit = static_cast<uint32_t>(__builtin_ctz(mask | 0x80000000u));
            const uint32_t e = n * kSub + lane * kItems + (bit & 1u) * 4u + (bit >> 3);
            if (mask) sub.queue[n0 + lanes_below(any)] = static_cast<uint16_t>(e);
            mask &= mask - 1;
            n0 += static_cast<uint32_t>(__builtin_popcountll(any));
            if (n0 < 64) continue;
        } else if (todo) {
            // the next request: bit 8 b + h of mask for start 4 h + b of this
            // lane, set where it survives
            n = static_cast<uint32_t>(__builtin_ctzll(todo));
            todo &= todo - 1;
            const uint32_t sn = readlane32(s4, n), bn = readlane32(b4, n);
            mask = (((ts.av[0] - sn) & (bn - ts.cc[0])) >> 7) & 0x01010101u;
            mask |= (((ts.av[1] - sn) & (bn - ts.cc[1])) >> 6) & 0x02020202u;
            continue;
        }
        if (n0) probe_starts(sub, g, bounds, lane, tl, n0 < 64 ? n0 : 64u, n0, n1);
        if (n1 >= 64 || (!any && n1)) search_starts(sub, g, bounds, lane, tl, ts.end, n1 < 64 ? n1 : 64u, n1);
        if (!any && !n0 && !n1) {
            if (!first) break;
            first = 0;
            todo = __ballot(on);
            b4 = cost_code(bounds[lane], ts.code) * 0x01010101u | 0x80808080u;
        }
    }
}

// The same in a plain subtile: each start by two bisections, the end of its
// run, then its first end with at least S bytes.
__device__ void plain_requests(Sub& sub, Group& g, uint64_t* bounds, const SubState& ts, uint32_t nt,
                               uint32_t lane, uint64_t tl) {
    const uint16_t* run = plain_runs(sub.bd);
    for (uint64_t todo = g.live; todo; todo &= todo - 1) {
        const uint32_t n = static_cast<uint32_t>(__builtin_ctzll(todo));
        const uint64_t S = readlane64(g.S, n);
        Key best = key_none();
        for (uint32_t i = lane; i < nt; i += 64) {
            const uint32_t r = run[i];
            const uint64_t base = sub.bd.K(i);
            const uint32_t rend = lower_bound(i, ts.end, [&](uint32_t k) { return run[k + 1] != r; });
            const uint32_t e = lower_bound(i, rend, [&](uint32_t k) { return sub.bd.K(k + 1) - base >= S; });
            if (e < rend) {
                const Key k{sub.bd.C(e + 1) - sub.bd.C(i), sub.bd.K(e + 1) - base, tl + i, tl + e + 1};
                if (key_less(k, best)) best = k;
            }
        }
        fold(g, bounds, lane, best.start != kNone, n, best.cost, best.bytes, best.start, best.end);
    }
}

// The windows of request n (size S) that leave the staged region, whose last
// run goes on past it: the starts [cur, nt) of that run.  The wavefront walks
// the run 64 blocks at a time (one per lane, wavefront prefix sums) up to
// block lim; each chunk resolves a prefix of the pending starts, 64 at a
// time, since their shortest ends are monotone.  Ends early once every window
// still pending costs more than the bound.  Returns false when starts are
// still pending at lim.
__device__ bool walk_starts(const Params& P, Sub& sub, Group& g, uint64_t* bounds, const SubState& ts,
                            uint32_t lane, uint32_t n, uint32_t cur, uint32_t nt, uint64_t pos, uint64_t lim,
                            uint64_t s0, uint64_t s1, uint64_t tl, uint64_t S) {
    const uint64_t vmask = ts.packed ? kValMask : kNone;
    uint64_t cq = ts.xend & vmask;
    uint64_t cc = ts.xcend;
    const uint64_t clast = sub.bd.C(nt - 1);
    Key best = key_none();
    bool resolved = false;
    auto load = [&](uint64_t at, uint32_t& kd, uint64_t& sz, uint64_t& ct) {
        kd = COOP_PINNED;
        sz = 0;
        ct = 0;
        if (at + lane < lim) {
            kd = P.kind[at + lane];
            sz = P.size[at + lane];
            ct = P.cost[at + lane];
        }
    };
    uint32_t kd;
    uint64_t sz, ct;
    load(pos, kd, sz, ct);
    while (cur < nt && pos < lim) {
        const uint32_t m = lim - pos < 64 ? static_cast<uint32_t>(lim - pos) : 64u;
        uint32_t nkd;
        uint64_t nsz, nct;
        load(pos + 64, nkd, nsz, nct);
        const uint64_t pinned = __ballot(kd >= COOP_PINNED);
        uint32_t fp = pinned ? static_cast<uint32_t>(__builtin_ctzll(pinned)) : 64u;
        fp = fp < m ? fp : m;
        const bool in = lane < fp;
        SumOf s{in ? sz : 0, 0};
        if (in && kd == COOP_EVICTABLE) s.c = ct;
        wave_inclusive_sum(s);
        const uint64_t q = cq + s.q;  // prefixes after this lane's block
        const uint64_t c = cc + s.c;
        const uint32_t lastl = fp ? fp - 1 : 0;
        const uint64_t lastq = fp ? readlane64(q, lastl) : cq;
        const uint64_t lastc = fp ? readlane64(c, lastl) : cc;
        // (no window from the first pending start ends in this chunk: none
        // from a later one does either)
        if (fp && lastq - (sub.bd.K(cur) & vmask) >= S) {
            for (;;) {
                const uint32_t i = cur + lane;
                const uint32_t ii = i < nt ? i : nt - 1;
                const uint64_t base = sub.bd.K(ii) & vmask;
                const bool ok = i < nt && lastq - base >= S;
                // the first chunk lane k < fp with q_k - base >= S
                uint32_t lo = 0, hi = lastl;
#pragma unroll
                for (int st = 0; st < 6; ++st) {
                    const uint32_t mid = (lo + hi) >> 1;
                    const bool ge = shfl64(q, mid) - base >= S;
                    const bool more = lo < hi;
                    hi = more && ge ? mid : hi;
                    lo = more && !ge ? mid + 1 : lo;
                }
                const uint64_t qe = shfl64(q, lo);
                const uint64_t ce = shfl64(c, lo);
                if (ok) {
                    const Key k{ce - sub.bd.C(ii), qe - base, tl + i, pos - s0 + lo + 1};
                    if (key_less(k, best)) best = k;
                }
                const uint64_t res = __ballot(ok);
                const uint32_t done = ~res ? static_cast<uint32_t>(__builtin_ctzll(~res)) : 64u;
                cur += done;
                if (done < 64 || cur >= nt) break;
            }
        }
        if (fp < m) {  // the run closes inside this chunk
            resolved = true;
            break;
        }
        cq = lastq;
        cc = lastc;
        pos += m;
        kd = nkd;
        sz = nsz;
        ct = nct;
        // what every pending window holds: the blocks from the last start on
        const uint64_t bound = uniform64(bounds[n]);
        if (__ballot(bound < cc - clast)) {
            resolved = true;
            break;
        }
    }
    const bool done = resolved || cur >= nt || pos >= s1;
    fold(g, bounds, lane, best.start != kNone, n, best.cost, best.bytes, best.start, best.end);
    return done;
}

// The windows of the group's requests that leave the staged region (its last
// run may go on).  Returns the requests with windows that end more than
// kSubWalk blocks past it (left to the second kernel).
__device__ uint64_t sub_pending(const Params& P, Sub& sub, Group& g, uint64_t* bounds, const SubState& ts,
                                const SubGeom& tg, uint32_t lane, uint64_t s0, uint64_t s1, uint64_t tl) {
    const uint32_t nt = tg.nt;
    const uint64_t vmask = ts.packed ? kValMask : kNone;
    const uint64_t pos = tg.t0 + ts.end;
    const uint64_t lim = pos + kSubWalk < s1 ? pos + kSubWalk : s1;
    const uint64_t S = g.S;
    const uint64_t xlast = sub.bd.K(nt - 1);
    const uint16_t* run = plain_runs(sub.bd);
    // lane n: request n's first pending start (run endrun, fewer than S bytes
    // to the region end) that does not cost more than the bound up to there
    bool pend = ((g.live >> lane) & 1u) != 0;
    if (ts.packed) pend = pend && (xlast >> kValBits) == ts.endrun && ((ts.xend - xlast) & vmask) < S;
    else pend = pend && run[nt - 1] == ts.endrun && ts.xend - xlast < S;
    if (!__ballot(pend)) return 0;
    uint32_t cur = nt;
    uint64_t need = 0;  // bytes a window from there needs past the region
    if (pend) {
        const uint64_t bound = bounds[lane];
        cur = lower_bound(0, nt - 1, [&](uint32_t i) {
            const uint64_t x = sub.bd.K(i);
            return (ts.packed ? (x >> kValBits) == ts.endrun : run[i] == ts.endrun) && ((ts.xend - x) & vmask) < S;
        });
        cur = lower_bound(cur, nt, [&](uint32_t i) { return ts.xcend - sub.bd.C(i) <= bound; });
        if (cur < nt) need = S - ((ts.xend - sub.bd.K(cur)) & vmask);
    }
    uint64_t todo = __ballot(cur < nt);
    if (!todo) return 0;
    // how far the run goes on, for all of them: bytes to its end, or to lim
    uint64_t ext = 0;
    bool closed = false;
    for (uint64_t at = pos; at < lim && !closed; at += 256) {
        uint64_t sum = 0;
        uint32_t first = 256;  // the first pinned block
        uint32_t kd[4];
        uint64_t sz[4];
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
            const uint64_t k = at + j * 64 + lane;
            kd[j] = k < lim ? P.kind[k] : static_cast<uint32_t>(COOP_FREE);
            sz[j] = k < lim ? P.size[k] : 0;
        }
#pragma unroll
        for (uint32_t j = 4; j-- > 0;) {
            const uint64_t m = __ballot(kd[j] >= COOP_PINNED);
            first = m ? j * 64 + static_cast<uint32_t>(__builtin_ctzll(m)) : first;
        }
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) sum += j * 64 + lane < first ? sz[j] : 0;
        add_dpp64<kRowShr1, 0xf>(sum);
        add_dpp64<kRowShr2, 0xf>(sum);
        add_dpp64<kRowShr4, 0xf>(sum);
        add_dpp64<kRowShr8, 0xf>(sum);
        add_dpp64<kRowBcast15, 0xa>(sum);
        add_dpp64<kRowBcast31, 0xc>(sum);
        ext += readlane64(sum, 63);
        closed = first < 256;
    }
    closed = closed || lim == s1;
    // beyond that a window ends past lim, or nowhere
    const uint64_t beyond = __ballot(cur < nt && need > ext);
    uint64_t deferred = closed ? 0 : beyond;
    for (todo &= ~beyond; todo; todo &= todo - 1) {
        const uint32_t n = static_cast<uint32_t>(__builtin_ctzll(todo));
        if (!walk_starts(P, sub, g, bounds, ts, lane, n, readlane32(cur, n), nt, pos, lim, s0, s1, tl,
                         readlane64(S, n)))
            deferred |= 1ull << n;
    }
    return deferred;
}

// The most tiles of any snapshot (as sub_geom cuts them), over the
// workgroup: queued chunks must be long enough that no snapshot spans more
// than pc - 2 of them.  Offsets are clamped as in make_job.
__device__ uint64_t max_tiles(const Params& P, SearchSmem& sm, uint32_t tid) {
    uint64_t m = 1;
    for (uint64_t b = tid; b < P.num_segments; b += kThreads) {
        const uint64_t s1 = P.seg[b + 1] < P.num_blocks ? P.seg[b + 1] : P.num_blocks;
        const uint64_t s0 = P.seg[b] < s1 ? P.seg[b] : s1;
        const uint64_t t = (s1 - (s0 & ~7ull) + kTile - 1) >> kTileLog2;
        m = t > m ? t : m;
    }
    for (int o = 32; o >= 1; o >>= 1) {
        const uint64_t x = __shfl_xor(m, o, 64);
        m = x > m ? x : m;
    }
    if ((tid & 63u) == 0) sm.tmax[tid >> 6] = m;
    __syncthreads();
    m = sm.tmax[0];
    for (uint32_t i = 1; i < kWaves; ++i) m = sm.tmax[i] > m ? sm.tmax[i] : m;
    return uniform64(m);
}

// Claims the next queued chunk (one wavefront).  Returns a chunk index, kQDone
// once the queue has run dry, or kQEmpty if the queue word still holds an
// earlier call's tag (this call's reset has not landed yet).
__device__ uint64_t claim_chunk(const Params& P, const Control& ctl, uint32_t lane) {
    uint64_t old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(P.queue, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    old = uniform64(old);
    if ((old >> 32) != uniform(ctl.qtag)) {
        __builtin_amdgcn_s_sleep(16);
        return kQEmpty;
    }
    const uint64_t c = P.grid + (old & 0xffffffffull);
    return c < uniform64(ctl.nchunks) ? c : kQDone;
}

// Moves the walk to the next job and writes it to `out` (its `valid` is 0 when
// there is none): in the current chunk, else in chunks claimed from the queue
// until it runs dry.  One wavefront at a time, every lane active.
__device__ __forceinline__ void find_next(const Params& P, Control& ctl, uint32_t lane, Job& out) {
    uint32_t u = uniform(ctl.u), u_begin = uniform(ctl.u_begin), u_end = uniform(ctl.u_end);
    uint32_t y = uniform(ctl.y), v = uniform(ctl.v), b = uniform(ctl.b), b0 = uniform(ctl.b0);
    uint64_t chunk = uniform64(ctl.chunk);
    bool more = uniform(ctl.queue_on) != 0;
    Job job;
    job.valid = 0;
    // snapshots [b, b + kCache - 1) at hand
    auto fill = [&]() {
        b0 = b;
        const uint64_t i = b + static_cast<uint64_t>(lane) < P.num_segments ? b + static_cast<uint64_t>(lane)
                                                                            : P.num_segments;
        wave_sync();  // earlier reads are done
        if (lane < kCache) {
            ctl.seg[lane] = P.seg[i];
            ctl.req[lane] = P.req_off[i];
        }
        wave_sync();
    };
    for (;;) {
        bool found = false;
        for (; u < u_end; ++u, ++v) {
            if (v == P.num_virtual) {
                v = 0;
                ++y;
                b = kNone32;
            }
            if (b == kNone32) {
                b = locate(P, v, lane);
                fill();
            } else {
                while (b + 1ull < P.num_segments && v >= first_id(b + 1ull, uniform64(ctl.seg[b + 1 - b0]))) {
                    ++b;
                    if (b + 1 - b0 >= kCache) fill();
                }
            }
            found = make_job(P, y, v, b, uniform64(ctl.seg[b - b0]), uniform64(ctl.seg[b + 1 - b0]),
                             uniform64(ctl.req[b - b0]), uniform64(ctl.req[b + 1 - b0]), job);
            if (found) break;
        }
        if (found || !more) break;
        const uint64_t c = claim_chunk(P, ctl, lane);
        if (c == kQEmpty) continue;
        if (c == kQDone) {
            more = false;
            continue;
        }
        chunk = c;
        uint64_t cb, ce;
        chunk_range(P, chunk, uniform(ctl.c2), cb, ce);
        u = u_begin = static_cast<uint32_t>(cb);
        u_end = static_cast<uint32_t>(ce);
        y = static_cast<uint32_t>(div_magic(u, P.nv_magic));
        v = u - y * P.num_virtual;
        b = kNone32;  // located from scratch
    }
    if (job.valid) {
        // the units of (b, y), those left in this chunk, and the chunks that hold them
        const uint64_t c2_magic = uniform64(ctl.c2_magic);
        const uint64_t ub = static_cast<uint64_t>(y) * P.num_virtual + (v - job.p);  // unit of tile 0
        const uint64_t hi = ub + job.tiles < u_end ? ub + job.tiles : u_end;
        job.lo = u;
        job.hi = static_cast<uint32_t>(hi);
        const uint64_t ue = ub + job.tiles - 1 < P.units ? ub + job.tiles - 1 : P.units - 1;
        const uint64_t i_lo = chunk_of(P, static_cast<uint32_t>(ub), c2_magic);
        const uint64_t i_hi = chunk_of(P, static_cast<uint32_t>(ue), c2_magic);
        const uint64_t G = i_hi - i_lo + 1;
        job.G = static_cast<uint32_t>(G > P.pc ? P.pc : G);  // P.pc only with malformed offsets
        const uint64_t g = chunk - i_lo;
        job.g = g >= job.G ? job.G - 1 : static_cast<uint32_t>(g);  // likewise
        job.direct = job.G == 1;
        v += job.hi - u;
        u = job.hi;
    }
    if (lane == 0) {
        out = job;
        ctl.u = u;
        ctl.u_begin = u_begin;
        ctl.u_end = u_end;
        ctl.y = y;
        ctl.v = v;
        ctl.b = b;
        ctl.b0 = b0;
        ctl.chunk = chunk;
        ctl.queue_on = more;
    }
}

// A job read back from LDS, in scalar registers.
__device__ __forceinline__ Job uniform_job(const Job& j) {
    Job r;
    r.y = uniform(j.y);
    r.b = uniform(j.b);
    r.lo = uniform(j.lo);
    r.hi = uniform(j.hi);
    r.s0 = uniform64(j.s0);
    r.s1 = uniform64(j.s1);
    r.q0 = uniform64(j.q0);
    r.K = uniform64(j.K);
    r.tiles = uniform64(j.tiles);
    r.p = uniform64(j.p);
    r.g = uniform(j.g);
    r.G = uniform(j.G);
    r.direct = uniform(j.direct);
    r.valid = uniform(j.valid);
    return r;
}

// The call's tags into LDS (one thread).  A call replayed from a graph takes
// them from the tag word, advanced by the kernel before the search on the
// stream, so every workgroup (of both search kernels) reads the same value;
// P.epoch then holds a per-process salt.
__device__ __forceinline__ void call_tags(const Params& P, Control& ctl) {
    uint64_t epoch = P.epoch;
    if (P.tag_word) {
        const uint64_t t = load_word_device(P.tag_word);
        epoch = kGraphTag | ((t * kTagOdd + epoch) & kTagMask);
    }
    ctl.epoch = epoch;
    ctl.qtag = queue_tag(epoch);
}

// After the last tile of (b, y) in the current chunk, when other chunks
// hold tiles of it too: a ticket on the (b, y) counter; the last of the G
// arrivals reduces the G partial keys of every request of the slice.  The
// partial keys are device-scope atomics (store_key_device), so the ticket
// only has to follow the completion of this workgroup's writes.
__device__ void combine_partials(const Params& P, uint64_t epoch, const Job& job, uint32_t tid, uint32_t& last_flag) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);  // every write of this thread has completed
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __syncthreads();
    if (tid == 0) {
        uint64_t* ctr = P.counters + static_cast<uint64_t>(job.y) * P.num_segments + job.b;
        last_flag = take_ticket(ctr, epoch, kEpochShift) == job.G;
    }
    __syncthreads();
    if (!uniform(last_flag)) return;
    // The last arrival reads what the others published: an agent-scope
    // acquire, so that no line its CU cached earlier is read (the partial
    // keys are read with device-scope atomics anyway).
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    // tpr threads per request (a power of two within a wavefront), each
    // taking every tpr-th slot; then a shuffle reduction inside the group
    uint32_t tpr = 64;
    while (tpr > 1 && static_cast<uint64_t>(tpr) * job.K > kThreads) tpr >>= 1;
    const uint32_t groups = kThreads / tpr, sub = tid % tpr;
    for (uint64_t k0 = 0; k0 < job.K; k0 += groups) {
        const uint64_t k = k0 + tid / tpr;
        const bool act = k < job.K;
        const uint64_t q = job.q0 + job.y + ((act ? k : 0) << P.slices_log2);
        Key best = key_none();
        if (act) {
            for (uint64_t gg = sub; gg < job.G; gg += tpr) {
                const Key o = load_key_device(P.part + q * P.pc + gg);
                if (key_less(o, best)) best = o;
            }
        }
        const uint32_t lane = tid & 63u;
        for (uint32_t m = tpr >> 1; m >= 1; m >>= 1) {
            Key o;
            o.cost = shfl64(best.cost, lane ^ m);
            o.bytes = shfl64(best.bytes, lane ^ m);
            o.start = shfl64(best.start, lane ^ m);
            o.end = shfl64(best.end, lane ^ m);
            if (key_less(o, best)) best = o;
        }
        if (act && sub == 0) P.out[q] = to_window(best, P.req_size[q]);
    }
}

// Appends the job's part of the chunk (its units, g and G) to the deferred
// list (one thread).  The list's word carries the call's queue tag, so the
// first append of a call restarts the count.
__device__ void defer_job(const Params& P, uint32_t qtag, const Job& job) {
    const Ext e = ext_of(P);
    const uint64_t idx = take_ticket(e.defer_word, qtag, 32) - 1;
    if (idx < P.defer_cap) store_entry_device(e.entries + idx, make_uint4(job.lo, job.hi, job.g, job.G));
}

// Adds a wavefront's share (uniform) to the record of tile p of the job, in
// its place of the ring; the tile's last wavefront publishes the record (of
// tiles p >= 1: bytes of all the blocks, cost of the evictable ones, pinned
// count) and clears the place.  Every unit of the tile writes the same
// values; the second kernel, next on the stream, reads them.
__device__ __forceinline__ void add_record(const Params& P, RecSum& rec, uint32_t& done, const SubState& ts,
                                           uint64_t s0, uint64_t p, uint32_t lane) {
    if (lane == 0) {
        __hip_atomic_fetch_add(&rec.q, ts.tq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add(&rec.r, ts.tr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_fetch_add(&rec.c, ts.tc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // (a wavefront's LDS operations complete in the order they are issued
        // in, which the fences keep the compiler from changing: the sums, then
        // the count; the last one's reads and clears after its count, and
        // before the place is given to a later tile)
        __atomic_signal_fence(__ATOMIC_ACQ_REL);
        const uint32_t n = __hip_atomic_fetch_add(&rec.n, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __atomic_signal_fence(__ATOMIC_ACQ_REL);
        if (n == kWaves - 1) {
            const uint64_t idx = (s0 >> kTileLog2) + p - 1;
            if (p != 0 && idx < (P.num_blocks >> kTileLog2)) {
                const Ext e = ext_of(P);
                store_word_device(e.rec_p + idx, rec.q);
                store_word_device(e.rec_c + idx, rec.c);
                store_word_device(e.rec_r + idx, rec.r);
            }
            rec.q = 0;
            rec.r = 0;
            rec.c = 0;
            rec.n = 0;
            __atomic_signal_fence(__ATOMIC_ACQ_REL);
            __hip_atomic_fetch_add(&done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
}

// The search of every unit the workgroup gets: its first chunk, then chunks
// from the queue.
__device__ __forceinline__ void search_units(const Params& P, SearchSmem& sm) {
    const uint32_t tid = threadIdx.x;
    const uint32_t w = uniform(tid >> 6);
    Key* const part = P.part;
    // The queue, when there is one: workgroup 0 stamps this call's tag; claims
    // that reach the word before the stamp see an old tag and try again.
    // Queued chunks are sized from the snapshots' tile counts, the same in
    // every workgroup.
    const uint64_t tmax = P.queue_on ? max_tiles(P, sm, tid) : 1;
    if (tid < kRecRing) sm.rec[tid] = RecSum{};
    if (tid < kGroup) sm.bound[tid] = kNone;
    if (w == 0) {
        if (tid == 0) {
            Control& ctl = sm.ctl;
            call_tags(P, ctl);
            ctl.c2 = P.c2;
            ctl.nchunks = P.grid;
            ctl.queue_on = P.queue_on;
            if (P.queue_on) {
                if (blockIdx.x == 0) store_word_device(P.queue, static_cast<uint64_t>(ctl.qtag) << 32);
                const uint64_t need = (tmax + P.pc - 3) / (P.pc - 2);
                ctl.c2 = static_cast<uint32_t>(need > P.c2 ? need : P.c2);
                ctl.nchunks = P.grid + (static_cast<uint64_t>(P.units) - P.u1 + ctl.c2 - 1) / ctl.c2;
            }
            ctl.c2_magic = ctl.c2 == 1 ? 0 : ~0ull / ctl.c2 + 1;
            uint64_t cb, ce;
            chunk_range(P, blockIdx.x, ctl.c2, cb, ce);
            ctl.chunk = blockIdx.x;
            ctl.u = ctl.u_begin = static_cast<uint32_t>(cb);
            ctl.u_end = static_cast<uint32_t>(ce);
            ctl.y = static_cast<uint32_t>(div_magic(cb, P.nv_magic));
            ctl.v = ctl.u - ctl.y * P.num_virtual;
            ctl.b = kNone32;
            ctl.b0 = 0;
            sm.deferred = 0;
            sm.arrived = 0;
            sm.rec_done = 0;
        }
        wave_sync();
        find_next(P, sm.ctl, tid, sm.job[0]);
        wave_sync();
        if (uniform(sm.job[0].valid)) find_next(P, sm.ctl, tid, sm.job[1]);
    }
    __syncthreads();
    Job job = uniform_job(sm.job[0]);
    if (!job.valid) return;
    uint32_t slot = 0;
    Sub& sub = sm.sub[w];
    const uint32_t qtag = uniform(sm.ctl.qtag);
    bool any_deferred = false;
    for (uint64_t base = 0;;) {
        // The lane, opaque to the compiler: values derived from it are
        // recomputed in every pass, and for every tile, instead of being kept
        // live (and spilled) across the loops.
        uint32_t lane = threadIdx.x & 63u;
        asm volatile("" : "+v"(lane));
        const uint32_t kg = job.K - base < kGroup ? static_cast<uint32_t>(job.K - base) : kGroup;
        const bool last_group = base + kGroup >= job.K;
        // lane n: request n of the group
        const uint64_t q = job.q0 + job.y + ((base + lane) << P.slices_log2);
        Group g{0, key_none(), 0};
        if (lane < kg) {
            g.S = P.req_size[q];
            if (P.bounds && !job.direct) {
                // (the window of that cost is in some partial slot by the end)
                __hip_atomic_fetch_min(&sm.bound[lane], load_word_device(P.bounds + q), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
        const uint64_t wanted = __ballot(g.S != 0);
        const uint64_t least = wave_min64(g.S ? g.S : kNone);
        const uint32_t np = job.hi - job.lo;
        for (uint32_t k = 0; k < np; ++k) {
            asm volatile("" : "+v"(lane));
            const uint64_t p = job.p + k;
            const SubGeom now = sub_geom(job.s0, job.s1, p, w);
            const uint64_t tl = now.t0 - job.s0;
            SubState ts;
            if (now.nt) {
                SubRegs regs;
                sub_loads(P, now, lane, regs);
                ts = sub_stage(sub.bd, now, lane, regs, least);
            } else {
                ts.tq = 0;
                ts.tr = 0;
                ts.tc = 0;
            }
            // a place of the ring is free once its earlier tile's record is out
            // (wavefronts are seldom that far apart; the slowest never waits)
            while (k >= kRecRing && base == 0 &&
                   uniform(__hip_atomic_load(&sm.rec_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) + kRecRing <= k)
                __builtin_amdgcn_s_sleep(1);
            __atomic_signal_fence(__ATOMIC_ACQUIRE);  // (no add to the place before that)
            if (base == 0) add_record(P, sm.rec[k % kRecRing], sm.rec_done, ts, job.s0, p, lane);
            if (now.nt == 0) continue;
            g.live = wanted & ~uniform64(__hip_atomic_load(&sm.deferred, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            if (!g.live) continue;
            if (ts.packed) sub_requests(sub, g, sm.bound, ts, lane, tl);
            else plain_requests(sub, g, sm.bound, ts, now.nt, lane, tl);
            if (now.t0 + ts.end < job.s1) {
                const uint64_t d = sub_pending(P, sub, g, sm.bound, ts, now, lane, job.s0, job.s1, tl);
                if (d && lane == 0)
                    __hip_atomic_fetch_or(&sm.deferred, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            wave_sync();  // LDS is restaged next
        }
        // ---- the pass has ended: this wavefront's answers into LDS
        Key* const mine = reinterpret_cast<Key*>(sub.bd.spare(0));
        if (lane < kg) mine[lane] = g.acc;
        // the first wavefront here looks up the job after the next one
        uint32_t turn = 0;
        if (lane == 0) turn = __hip_atomic_fetch_add(&sm.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (uniform(turn) == 0 && last_group && uniform(sm.job[slot == 2 ? 0 : slot + 1].valid))
            find_next(P, sm.ctl, lane, sm.job[slot == 0 ? 2 : slot - 1]);
        __syncthreads();
        const uint64_t deferred = uniform64(sm.deferred);
        any_deferred = any_deferred || deferred != 0;
        if (w == 0) {
            if (lane < kg) {
                Key best = g.acc;
                for (uint32_t i = 1; i < kWaves; ++i)
                    best = min_key(best, reinterpret_cast<const Key*>(sm.sub[i].bd.spare(0))[lane]);
                const bool put_off = ((deferred >> lane) & 1u) != 0;
                if (job.direct && !put_off) P.out[q] = to_window(best, g.S);
                if (!job.direct || put_off) store_key_device(part + q * P.pc + job.g, best);
                if (P.bounds && !job.direct && best.start != kNone && best.cost < load_word_device(P.bounds + q))
                    __hip_atomic_fetch_min(P.bounds + q, best.cost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // Set or cleared where the job can be deferred: a bit that an
                // earlier use of the memory left set would have the second
                // kernel take the request's slot for a key of this call.
                if (job.s1 - job.s0 >= kSubDeferMin) {
                    const uint64_t bit = q * P.pc + job.g;
                    uint32_t* const word = ext_of(P).bits + (bit >> 5);
                    const uint32_t m = 1u << (bit & 31u);
                    const bool set = (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & m) != 0;
                    if (put_off && !set) __hip_atomic_fetch_or(word, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (!put_off && set) __hip_atomic_fetch_and(word, ~m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            sm.bound[lane] = kNone;
            if (lane == 0) {
                sm.arrived = 0;
                sm.rec_done = 0;
            }
        }
        __syncthreads();
        if (tid == 0) sm.deferred = 0;  // (every wavefront has read it)
        if (!last_group) {
            base += kGroup;
            __syncthreads();
            continue;
        }
        if (any_deferred) {
            if (tid == 0) defer_job(P, qtag, job);
        } else if (!job.direct) {
            combine_partials(P, uniform64(sm.ctl.epoch), job, tid, sm.last_flag);
        }
        __syncthreads();
        any_deferred = false;
        base = 0;
        slot = slot == 2 ? 0 : slot + 1;
        job = uniform_job(sm.job[slot]);
        if (!job.valid) break;
    }
}

__global__ __launch_bounds__(kThreads, 4) void coop_window_sub_kernel(Params P) {
    __shared__ SearchSmem sm;
    if (!uniform64(load_word_device(P.pick))) return;  // coop_window_search_kernel, next, takes the batch
    search_units(P, sm);
}

// Whether this kernel pays, from kLook stretches of blocks, one a thread of a
// workgroup: of 64 blocks each, 1024 where many requests share a snapshot (the
// search then takes milliseconds).  The stretches lie at multiples of the
// golden ratio of the batch, so that no period of the snapshots' lengths can
// put them all at the same place of a pool (evenly spaced over 512 pools of
// 65536 blocks, they met nothing but the pinned block at each pool's start:
// 354 us on tiles, 685 on subtiles).  It pays when:
// - No more than three fifths of the open blocks are free or cost nothing:
//   among windows of cost 0 nothing is passed over, and each is searched for
//   (clustered pools, 4 requests: 709 us on tiles and 645 on subtiles with 0.57
//   of them at no cost, 710 and 813 with 0.74; 64 requests: 61 and 52 ms, 61
//   and 84).
// - Few requests a snapshot: two of the 512 stretches at most hold no pinned
//   block.  Runs are then short throughout, few windows leave a subtile, and
//   its least bytes and costs tell starts apart.  Pools of 30% pinned blocks, 4
//   requests each: 708 us on tiles, 490 on subtiles; 8% or 10% scattered over
//   1024 pools of 65536, 4 requests: 661 and 480, 467; 16 requests: 1746 and
//   840, 760.  The few open stretches are for batches that hold long runs too:
//   one pool in 64 without a pinned block, requests of 100 to 9000 blocks
//   there: 1112 and 1220 us; every other pool: 961 and 1350; a sixth of each
//   pool pinned, at its two ends: 1479 and 1935.  (Scattered pinned blocks
//   alone would do with fewer: 5%, 4 requests: 664 and 554.  One such pool in
//   4096 is not seen: 1064 and 1157.)
// - 64 requests a snapshot or more share the staging, one of the longer
//   stretches at most is open (one run of 100,000 blocks among 2^24, a request
//   of 20,000: 128 ms on tiles, 165 on subtiles), and either an eighth of the
//   short ones at most are (costs of one magnitude, 64 requests, 2, 3 and 4%
//   pinned: 17.4 ms on tiles, 19.2, 14.1 and 11.3 on subtiles), or five eighths
//   at most are and most costs are far below the average, so that the few
//   large ones rule most windows out (costs over twelve decades, 4096
//   requests, 1% pinned: 98.3 and 67.0 ms; 0.5%: 106 and 105; 0.2%: 134 and
//   164).
// Otherwise the windows that leave a subtile cost more than the starts passed
// over save: 1% pinned, costs of one magnitude, 8 requests: 514 and 1022 us;
// 4096 requests: 26.0 and 35.2 ms; 3%, 4 requests: 576 and 618 us.
constexpr uint32_t kLook = kThreads;
constexpr uint32_t kLookShort = 64, kLookLong = 1024;
static_assert(kSubBlocks > kLookLong + 15, "the smallest batch holds a stretch at any alignment");

// A wavefront's counts over its stretches.
struct Look {
    uint32_t closed_short, closed_long;   // stretches with a pinned block
    uint32_t open, costless, evictable;   // of the stretches' first blocks
    uint32_t below;
    float sum;                            // the evictable ones' costs
};

__device__ __forceinline__ uint32_t lanes_where(bool is) {
    return static_cast<uint32_t>(__builtin_popcountll(__ballot(is)));
}

// (the first workgroup, every thread; every thread gets the answer, the same
// from call to call: the sums are added in the same order)
__device__ bool subtiles_pay(const Params& P, Look* looks, uint32_t tid) {
    const bool many = P.num_requests / 64 >= P.num_segments;
    const uint32_t span = many ? kLookLong : kLookShort;
    // from the first 16-byte boundary at or after the place
    const uint64_t at = __umul64hi((tid + 1) * 0x9e3779b97f4a7c15ull, P.num_blocks - span - 15);
    const uint64_t first = at + ((0 - (reinterpret_cast<uintptr_t>(P.kind) + at)) & 15u);
    const ulonglong2* const kinds = reinterpret_cast<const ulonglong2*>(P.kind + first);
    const uint32_t kind = P.kind[first];
    const uint64_t cost = P.cost[first];
    uint64_t any = 0;
    auto look = [&](uint32_t j) {
#pragma unroll
        for (uint32_t k = 0; k < kLookShort / 16; ++k) any |= kinds[j + k].x | kinds[j + k].y;
    };
    look(0);
    constexpr uint64_t kPinnedBits = 0xfefefefefefefefeull;  // set in pinned kinds (2 and more) only
    const bool closed_short = (any & kPinnedBits) != 0;
    for (uint32_t j = kLookShort / 16; j < span / 16; j += kLookShort / 16) look(j);
    const bool evictable = kind == COOP_EVICTABLE;
    float sum = evictable ? static_cast<float>(cost) : 0.0f;
    if (many)
        for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
    const Look mine{lanes_where(closed_short), lanes_where((any & kPinnedBits) != 0),
                    lanes_where(kind < COOP_PINNED),
                    lanes_where(kind < COOP_PINNED && !(evictable && cost != 0)), lanes_where(evictable), 0, sum};
    if ((tid & 63u) == 0) looks[tid >> 6] = mine;
    __syncthreads();
    Look all{};
    for (uint32_t w = 0; w < kWaves; ++w) {
        all.closed_short += looks[w].closed_short;
        all.closed_long += looks[w].closed_long;
        all.open += looks[w].open;
        all.costless += looks[w].costless;
        all.evictable += looks[w].evictable;
        all.sum += looks[w].sum;
    }
    if (5 * all.costless > 3 * all.open) return false;
    if (!many) return all.closed_short >= kLook - kLook / 256;
    if (all.closed_long < kLook - 1) return false;
    if (all.closed_short >= kLook - kLook / 8) return true;
    if (all.closed_short < kLook - kLook * 5 / 8 || all.evictable == 0) return false;
    const uint32_t below =
        lanes_where(evictable && static_cast<float>(cost) * (8.0f * static_cast<float>(all.evictable)) < all.sum);
    if ((tid & 63u) == 0) looks[tid >> 6].below = below;
    __syncthreads();
    for (uint32_t w = 0; w < kWaves; ++w) all.below += looks[w].below;
    return 2 * all.below >= all.evictable;
}

// Ahead of the searches on the stream: picks the kernel, and clears the shared
// bounds.
__global__ __launch_bounds__(kThreads) void coop_window_pick_kernel(Params P) {
    __shared__ Look looks[kWaves];
    const uint64_t i = blockIdx.x * static_cast<uint64_t>(kThreads) + threadIdx.x;
    if (P.bounds && i < P.num_requests) P.bounds[i] = kNone;
    if (blockIdx.x == 0) {
        const bool pay = subtiles_pay(P, looks, threadIdx.x);
        if (threadIdx.x == 0) *P.pick = pay;
    }
}

}  // namespace

bool coop_win::launch_subtiles(const Params& P, hipStream_t s) {
    const uint64_t n = P.bounds ? P.num_requests : 1;
    hipLaunchKernelGGL(coop_window_pick_kernel, dim3(static_cast<uint32_t>((n + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, P);
    if (hipGetLastError() != hipSuccess) return false;
    hipLaunchKernelGGL(coop_window_sub_kernel, dim3(P.grid), dim3(kThreads), 0, s, P);
    return hipGetLastError() == hipSuccess;
}
