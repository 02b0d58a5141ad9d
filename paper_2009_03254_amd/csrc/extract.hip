// Extraction kernels for gfx950 (paper Sec. 4): active-block culling (4.1),
// the GPU-driven LRU cache update (4.2, Alg. 1), and block-wise marching cubes
// (4.3-4.5).  Every count the host does not know is read from device memory,
// so the whole sequence is enqueued without host round-trips.
//
// Shared idioms:
//   * wave64 primitives: ballot / mbcnt compaction, shuffle scans;
//   * no launch for a prefix sum that is short: the counts of one kernel are
//     added up by every workgroup of the next that needs a prefix of them
//     (a launch costs 4-6 us of a small call, a few KB of counts 1-2 us);
//   * what a call counts from zero is kept twice: a call counts in one copy
//     and clears the other for the next call, so no launch resets them;
//   * device-scope atomics on one address serialise (~14 ns each), so work
//     is spread statically (workgroup w takes items w, w + G, ...) and counts
//     go to arrays, not one counter.
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "mc_device.h"
#include "mc_ntri.h"

namespace bcmc {
namespace {
// ---------------------------------------------------------------------------
// Sec. 4.1: active blocks.  Block b is active when its range, or its range
// united with the range of one of its 26 neighbours, contains iso
// (lo < iso <= hi).  With LO / HI the min / max over the 3x3x3 neighbourhood
// that is:  (lo_b < iso <= HI)  or  (LO < iso <= hi_b).
// ---------------------------------------------------------------------------
// Tiled: a workgroup culls a CULL_TX x CULL_TY x CULL_TZ box of blocks.  The
// box's ranges with a one-block halo (+inf / -inf outside the volume) are
// staged in LDS with all loads in flight at once; the 3x3 in-plane min / max
// and the 2x2 positive-quadrant min / max are then combined across z in
// registers, so every range is read about 1.6 times and no load waits inside
// the sweep.
constexpr int CULL_TX = 32, CULL_TY = 8, CULL_TZ = 8;
// Layers of blocks per workgroup of the direct cull: it is a latency chain over
// its layers on a chip that few tiles leave half empty.  2 layers: 6.1 us for
// 3060 blocks' rows (10.3 with all 8), 9.5 us at 3.7 M blocks (11.8), 21 at 512^3
// (21; 4 layers 19, but 7.2 us instead of 6.1 for the 3060).
constexpr int CULL_LAYERS = 2;

// Hull of the ranges over a tile's box with its one-block halo (clipped to
// the volume), one workgroup per tile, at load.  When the hull does not
// straddle iso, no block of the tile can be active: every block's
// neighbourhood range lies inside it.
__global__ __launch_bounds__(256) void k_tile_ranges(Geom g, const float2 *__restrict__ ranges,
                                                    float2 *__restrict__ tile_ranges) {
    constexpr int RX = CULL_TX + 2, RY = CULL_TY + 2, RZ = CULL_TZ + 2;
    const uint32_t ntx = (g.nbx + CULL_TX - 1) / CULL_TX, nty = (g.nby + CULL_TY - 1) / CULL_TY;
    uint32_t t = blockIdx.x;
    const uint32_t tx = t % ntx;
    t /= ntx;
    const uint32_t ty = t % nty, tz = t / nty;
    float lo = INFINITY, hi = -INFINITY;
    for (int i = threadIdx.x; i < RX * RY * RZ; i += 256) {
        const int hz = i / (RX * RY), r = i - hz * RX * RY, hy = r / RX, hx = r - hy * RX;
        const int x = (int)(tx * CULL_TX) + hx - 1, y = (int)(ty * CULL_TY) + hy - 1,
                  z = (int)(tz * CULL_TZ) + hz - 1;
        if (x >= 0 && x < (int)g.nbx && y >= 0 && y < (int)g.nby && z >= 0 && z < (int)g.nbz) {
            const float2 q = ranges[((uint64_t)z * g.nby + (uint32_t)y) * g.nbx + (uint32_t)x];
            lo = fminf(lo, q.x);
            hi = fmaxf(hi, q.y);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, d, 64));
        hi = fmaxf(hi, __shfl_xor(hi, d, 64));
    }
    __shared__ float2 s_h[4];
    if (lane() == 0) s_h[threadIdx.x >> 6] = make_float2(lo, hi);
    __syncthreads();
    if (threadIdx.x == 0)
        tile_ranges[blockIdx.x] = make_float2(fminf(fminf(s_h[0].x, s_h[1].x), fminf(s_h[2].x, s_h[3].x)),
                                              fmaxf(fmaxf(s_h[0].y, s_h[1].y), fmaxf(s_h[2].y, s_h[3].y)));
}

// A tile is live when its hull straddles iso (culled block by block), stale
// when it is not and may hold flags (its hull straddled the previous call's
// isovalue, or `rewrite`: nothing is known of them): they are cleared.
__device__ __forceinline__ void tile_state(float2 hull, float iso, float prev_iso, int rewrite, bool &live,
                                           bool &stale) {
    live = hull.x < iso && iso <= hull.y;
    stale = !live && (rewrite || (hull.x < prev_iso && prev_iso <= hull.y));
}

// Tile queue of a large volume's cull, one tile per thread, appended with
// one atomic per wave.  live: n_tiles entries, stale: the n_tiles after.
__global__ __launch_bounds__(256) void k_cull_scan(const float2 *__restrict__ tile_ranges, uint64_t n_tiles,
                                                  float iso, float prev_iso, int rewrite,
                                                  uint32_t *__restrict__ list, Counters *ctr) {
    const uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    bool live = false, stale = false;
    if (t < n_tiles) tile_state(tile_ranges[t], iso, prev_iso, rewrite, live, stale);
    const uint64_t lm = __ballot(live), sm = __ballot(stale);
    uint32_t lb = 0, sb = 0;
    if (lane() == 0) {
        if (lm) lb = atomicAdd(&ctr->cull_live, (uint32_t)__popcll(lm));
        if (sm) sb = atomicAdd(&ctr->cull_stale, (uint32_t)__popcll(sm));
    }
    lb = __shfl(lb, 0, 64);
    sb = __shfl(sb, 0, 64);
    if (live) list[lb + mbcnt(lm)] = (uint32_t)t;
    if (stale) list[n_tiles + sb + mbcnt(sm)] = (uint32_t)t;
}

// A round's counts of active, new and may-emit blocks (at most 4096 each).
__device__ __forceinline__ unsigned long long round_pack(uint32_t act, uint32_t fresh, uint32_t can) {
    return (unsigned long long)__popc(act) | (unsigned long long)__popc(fresh) << 21 |
           (unsigned long long)__popc(can) << 42;
}
constexpr unsigned long long ROUND_M = (1ull << 21) - 1;
// ... as (active << 32 | new), for sums over rounds.
__device__ __forceinline__ uint64_t round_lists(uint64_t c) { return (c & ROUND_M) << 32 | ((c >> 21) & ROUND_M); }

// Flags per block: bit 0 active, bit 1 may emit, bit 2 active without a
// slot (new, Alg. 1 MarkNewBlocks; never set for an identity cache); the
// slots of the active blocks that have one are stamped with the call's number
// (Alg. 1 IncrementSlotAge: a slot's age is the calls since its stamp).
// The flags are zero outside the tiles the previous call culled, so a tile
// live then and dead now (stale) is cleared here, a live tile is rewritten
// in full, and no other flag is touched.  The active, new and may-emit blocks
// of each 4096-block round are counted in round_cnt (round_pack) for the
// compaction: a tile adds up its rows that lie in one round first (an atomic
// per row of 32 blocks, all on few cache lines: a 512^3 cull of 53 us instead
// of 21).
// QUEUE (many tiles): persistent, workgroup w takes entries w, w + G, ... of
// k_cull_scan's queue (stale tiles first), so that a surface's live tiles
// spread evenly over the workgroups whatever their layout.  Otherwise one
// workgroup per tile, which looks at the tile's hull itself: no launch for the
// queue (up to CULL_DIRECT tiles, where dead workgroups cost less than that).
// A workgroup culls LAYERS of the tile's CULL_TZ layers of blocks (direct:
// CULL_TZ / LAYERS workgroups per tile, a chain of LAYERS + 2 layers each).
template <bool QUEUE, int LAYERS>
__global__ __launch_bounds__(256) void k_cull(Geom g, const float2 *__restrict__ ranges, float iso, float prev_iso,
                                             int rewrite, const float2 *__restrict__ tile_ranges,
                                             const uint32_t *__restrict__ list, uint64_t n_tiles,
                                             const int32_t *__restrict__ I_slot, int identity,
                                             uint32_t *__restrict__ S_stamp, uint32_t now,
                                             uint8_t *__restrict__ active, const Counters *ctr,
                                             unsigned long long *__restrict__ round_cnt) {
    constexpr int NL = LAYERS + 2, RX = CULL_TX + 2, RY = CULL_TY + 2, SLOTS = RX * RY;
    constexpr uint32_t PARTS = CULL_TZ / LAYERS;
    __shared__ float2 sh[NL][RY][RX];
    __shared__ unsigned long long s_cnt[LAYERS * CULL_TY];   // per row (z, y) of the box: its counts
    const uint32_t the_tile = blockIdx.x / PARTS, part = blockIdx.x % PARTS;   // (direct)
    const uint32_t ntx = (g.nbx + CULL_TX - 1) / CULL_TX, nty = (g.nby + CULL_TY - 1) / CULL_TY;
    uint32_t n_live, n_stale;
    if constexpr (QUEUE) {
        n_live = ctr->cull_live;
        n_stale = ctr->cull_stale;
    } else {   // a queue of this tile alone
        bool live, stale;
        tile_state(tile_ranges[the_tile], iso, prev_iso, rewrite, live, stale);
        n_live = live;
        n_stale = stale;
    }
    const uint32_t n_q = n_stale + n_live, step = QUEUE ? gridDim.x : 1u;
    auto live_tile = [&](uint32_t i) { return QUEUE ? list[i] : the_tile; };
    auto first_layer = [&](uint32_t tz) { return (int)(tz * CULL_TZ + (QUEUE ? 0u : part * LAYERS)); };
    const int lx = threadIdx.x % CULL_TX, ly = threadIdx.x / CULL_TX;
    auto tile_of = [&](uint32_t t, uint32_t &tx, uint32_t &ty, uint32_t &tz) {
        tx = t % ntx;
        t /= ntx;
        ty = t % nty;
        tz = t / nty;
    };
    uint32_t q = QUEUE ? blockIdx.x : 0u;
    for (; q < n_stale; q += step) {   // culled last time only: flags cleared
        uint32_t tx, ty, tz;
        tile_of(QUEUE ? list[n_tiles + q] : the_tile, tx, ty, tz);
        const int z0 = first_layer(tz), z1 = min(z0 + LAYERS, (int)g.nbz);
        const uint32_t bx = tx * CULL_TX + lx, by = ty * CULL_TY + ly;
        if (bx < g.nbx && by < g.nby)
            for (int z = z0; z < z1; z++) active[((uint64_t)z * g.nby + by) * g.nbx + bx] = 0;
    }
    // live tiles: a box's ranges with their halo, all loads in flight
    // together; the next box's are loaded while this one is culled
    constexpr int PER = (NL * SLOTS + 255) / 256;
    auto load_box = [&](uint32_t qq, float2 (&v)[PER]) {
        uint32_t tx, ty, tz;
        tile_of(live_tile(qq - n_stale), tx, ty, tz);
        const int z0 = first_layer(tz), z1 = min(z0 + LAYERS, (int)g.nbz);
        // the places in the box are worked out for each tile: kept over the queue
        // for every load they take 42 registers (135 and 3 waves per SIMD instead
        // of 85 and 5: 59 against 56.5 us at 236 M blocks)
        int t = (int)threadIdx.x;
        if constexpr (QUEUE) asm volatile("" : "+v"(t));
#pragma unroll
        for (int k = 0; k < PER; k++) {
            const int i = t + 256 * k;
            const int li = i / SLOTS, r = i - li * SLOTS;
            const int hy = r / RX, hx = r - hy * RX;
            const int zl = z0 - 1 + li;
            const int x = (int)(tx * CULL_TX) + hx - 1, y = (int)(ty * CULL_TY) + hy - 1;
            v[k] = make_float2(INFINITY, -INFINITY);
            if (i < NL * SLOTS && zl >= 0 && zl < (int)g.nbz && zl <= z1 && x >= 0 && x < (int)g.nbx &&
                y >= 0 && y < (int)g.nby)
                v[k] = ranges[((uint64_t)zl * g.nby + (uint32_t)y) * g.nbx + (uint32_t)x];
        }
    };
    float2 v[PER];
    if (q < n_q) load_box(q, v);
    for (; q < n_q; q += step) {
        uint32_t tx, ty, tz;
        tile_of(live_tile(q - n_stale), tx, ty, tz);
        const int z0 = first_layer(tz), z1 = min(z0 + LAYERS, (int)g.nbz);
        const uint32_t bx = tx * CULL_TX + lx, by = ty * CULL_TY + ly;
#pragma unroll
        for (int k = 0; k < PER; k++) {
            const int i = (int)threadIdx.x + 256 * k;
            if (i < NL * SLOTS) (&sh[0][0][0])[i] = v[k];
        }
        __syncthreads();
        if (QUEUE && q + step < n_q) load_box(q + step, v);
        uint32_t act = 0, can = 0, fresh = 0;   // bit z - z0: block (bx, by, z) is active, may emit, is new
        if (bx < g.nbx && by < g.nby) {
            // per layer: 3x3 min / max, 2x2 positive min / max, own range
            float l3a = INFINITY, h3a = -INFINITY;                       // layer zl - 2
            float l3b = INFINITY, h3b = -INFINITY, p2lb = INFINITY, p2hb = -INFINITY;
            float2 ownb = make_float2(INFINITY, -INFINITY);             // layer zl - 1
#pragma unroll
            for (int li = 0; li < NL; li++) {
                float l3 = INFINITY, h3 = -INFINITY, p2l = INFINITY, p2h = -INFINITY;
#pragma unroll
                for (int dy = -1; dy <= 1; dy++)
#pragma unroll
                    for (int dx = -1; dx <= 1; dx++) {
                        const float2 q2 = sh[li][ly + 1 + dy][lx + 1 + dx];
                        l3 = fminf(l3, q2.x);
                        h3 = fmaxf(h3, q2.y);
                        if (dx >= 0 && dy >= 0) {
                            p2l = fminf(p2l, q2.x);
                            p2h = fmaxf(p2h, q2.y);
                        }
                    }
                const float2 own = sh[li][ly + 1][lx + 1];
                if (li >= 2 && z0 - 2 + li < z1) {   // layer z0 - 2 + li has both z neighbours now
                    const float LO = fminf(l3a, fminf(l3b, l3)), HI = fmaxf(h3a, fmaxf(h3b, h3));
                    const float PLO = fminf(p2lb, p2l), PHI = fmaxf(p2hb, p2h);
                    // "can emit": the hull of the 2x2x2 group headed by the block
                    // contains iso (implies act, as that group contains the block)
                    if ((ownb.x < iso && iso <= HI) || (LO < iso && iso <= ownb.y)) act |= 1u << (li - 2);
                    if (PLO < iso && iso <= PHI) can |= 1u << (li - 2);
                }
                l3a = l3b;
                h3a = h3b;
                l3b = l3;
                h3b = h3;
                p2lb = p2l;
                p2hb = p2h;
                ownb = own;
            }
            // the slots of the active blocks (new: none), their loads in flight together
            int32_t sl[LAYERS];
#pragma unroll
            for (int z = 0; z < LAYERS; z++) {
                sl[z] = 0;
                if (!identity && ((act >> z) & 1u))
                    sl[z] = I_slot[((uint64_t)(z0 + z) * g.nby + by) * g.nbx + bx];
            }
#pragma unroll
            for (int z = 0; z < LAYERS; z++) {
                if (z0 + z >= z1) break;
                const bool a = (act >> z) & 1u;
                const uint64_t b = ((uint64_t)(z0 + z) * g.nby + by) * g.nbx + bx;
                const bool nw = a && sl[z] < 0;
                fresh |= (nw ? 1u : 0u) << z;
                active[b] = (a ? 1u : 0u) | (((can >> z) & 1u) ? 2u : 0u) | (nw ? 4u : 0u);
                if (!identity && a && sl[z] >= 0) S_stamp[sl[z]] = now;
            }
        }
        // the rounds' counts: each half-wave is 32 consecutive blocks of one
        // row, which lie in one round or in two
        const int half = lane() & 32;
#pragma unroll
        for (int z = 0; z < LAYERS; z++) {
            const uint32_t am = (uint32_t)(__ballot((act >> z) & 1u) >> half);
            const uint32_t cm = (uint32_t)(__ballot((can >> z) & 1u) >> half);
            const uint32_t nm = (uint32_t)(__ballot((fresh >> z) & 1u) >> half);
            if (lane() == half) {
                // the part of a row beyond its first block's round goes there directly
                const uint64_t b0 = ((uint64_t)(z0 + z) * g.nby + by) * g.nbx + bx;
                const uint32_t room = BLK_TILE - (uint32_t)(b0 % BLK_TILE);
                const uint32_t m = room >= 32 ? ~0u : (1u << room) - 1u;
                s_cnt[z * CULL_TY + ly] = round_pack(am & m, nm & m, cm & m);
                if (am & ~m) atomicAdd(&round_cnt[b0 / BLK_TILE + 1], round_pack(am & ~m, nm & ~m, cm & ~m));
            }
        }
        __syncthreads();
        if (threadIdx.x < 64) {   // the rows' rounds ascend: one atomic per run of rows in one round
            const int z = threadIdx.x / CULL_TY, y = threadIdx.x % CULL_TY;
            const uint64_t b0 = ((uint64_t)(z0 + z) * g.nby + ty * CULL_TY + y) * g.nbx + tx * CULL_TX;
            const uint32_t r = (uint32_t)(b0 / BLK_TILE);
            const uint64_t sum = wave_incl_scan((uint64_t)(threadIdx.x < LAYERS * CULL_TY ? s_cnt[threadIdx.x] : 0ull));
            const uint32_t after = (uint32_t)__shfl_down((int)r, 1, 64);
            const uint64_t ends = __ballot(threadIdx.x == 63 || after != r);
            const uint64_t mine = ends & ((1ull << threadIdx.x) - 1);
            const int prev = mine ? 63 - __builtin_clzll(mine) : 0;
            const uint64_t base = ((uint64_t)(uint32_t)__shfl((int)(sum >> 32), prev, 64) << 32) |
                                  (uint32_t)__shfl((int)(uint32_t)sum, prev, 64);
            const uint64_t c = sum - (mine ? base : 0ull);
            if (((ends >> threadIdx.x) & 1u) && c) atomicAdd(&round_cnt[r], (unsigned long long)c);
        }
        __syncthreads();   // sh is restaged for the next live tile
    }
}

// I_active (StreamCompactIDs of M_active) and I_new (active blocks without a
// slot, Alg. 1 MarkNewBlocks, flagged by the cull).  The blocks are cut into
// rounds of 4096 consecutive blocks, whose counts the cull has formed; the
// flags of a round without active blocks are not looked at.  Each live round
// is one workgroup's, with no waiting between workgroups: a round's place
// in the lists is the sum of the counts before it, which its workgroup adds up
// itself (up to ROUNDS_DIRECT rounds, 16 KB of counts; larger volumes: of
// the sums that k_round_sums forms of 256 rounds each, then of rounds).
// Bit 0 of each byte of w, gathered into bits 0..3: the four bits land on
// bits 21..24 of the product with no carries between them.
__device__ __forceinline__ uint32_t byte_bits(uint32_t w) {
    return (((w & 0x01010101u) * 0x00204081u) >> 21) & 0xFu;
}

__device__ __forceinline__ void flag_bits(uint4 q, uint32_t &actb, uint32_t &newb) {
    actb = newb = 0;
    if ((q.x | q.y | q.z | q.w) == 0) return;   // the common case of a sparse volume
    const uint32_t wds[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {   // flags use bits 0..2 of each byte
        const uint32_t w = wds[i];
        actb |= byte_bits(w | (w >> 1) | (w >> 2)) << (4 * i);
        newb |= byte_bits(w >> 2) << (4 * i);
    }
}

__device__ __forceinline__ uint4 load_flags16(const uint8_t *__restrict__ active, uint64_t base,
                                              uint64_t nb) {
    if (base + 16 <= nb) return *reinterpret_cast<const uint4 *>(active + base);
    uint32_t wd[4] = {0, 0, 0, 0};
    for (int j = 0; j < 16; j++)
        if (base + j < nb) wd[j >> 2] |= (uint32_t)active[base + j] << (8 * (j & 3));
    return make_uint4(wd[0], wd[1], wd[2], wd[3]);
}


// Alg. 1's early exit (nothing new), growth and supply of slots, from the
// call's counts.  Every active block that is not new holds one slot, so
// n_slots - (n_act - n_new) slots are available, and growth (more new blocks
// than that) needs no pass over the slots.  Slots are taken into use in
// ascending order before any used one is evicted, so the unused ones are
// always [n_used, n_slots): the new blocks take those first, then the oldest
// n_evict of the used available ones.
struct SlotPlan {
    uint64_t grow, n_slots, n_used, n_evicted;
    bool fits;
};
__device__ __forceinline__ SlotPlan plan_slots(uint64_t n_act, uint64_t n_new, const SlotState &ss) {
    SlotPlan p{0, ss.n_slots, ss.n_used, 0, true};
    if (ss.identity || n_new == 0) return p;
    const uint64_t avail = ss.n_slots - (n_act - n_new);
    if (n_new > avail) {
        p.grow = n_new - avail;
        const uint64_t half = (ss.n_slots + 1) / 2;
        if (half > p.grow) p.grow = half;
        if (ss.n_slots + p.grow > ss.max_slots) p.grow = ss.max_slots - ss.n_slots;
    }
    if (avail + p.grow < n_new) {
        p.fits = false;
        return p;
    }
    p.n_slots += p.grow;
    const uint64_t unused = p.n_slots - ss.n_used;
    p.n_evicted = n_new > unused ? n_new - unused : 0;
    p.n_used += n_new < unused ? n_new : unused;
    return p;
}
// ... published for the call's later kernels and the host, and the next
// call's counters cleared (one workgroup).
__device__ __forceinline__ void publish_plan(Counters *ctr, Counters *next, uint64_t n_act, uint64_t n_new,
                                             uint64_t n_cand, const SlotState &ss) {
    for (unsigned i = threadIdx.x; i < sizeof(Counters) / 4; i += 256) reinterpret_cast<uint32_t *>(next)[i] = 0;
    if (threadIdx.x != 0) return;
    const SlotPlan p = plan_slots(n_act, n_new, ss);
    ctr->n_act = n_act;
    ctr->n_new = n_new;
    ctr->n_cand = n_cand;
    ctr->n_slots = p.n_slots;
    ctr->n_used = p.n_used;
    ctr->n_evicted = p.n_evicted;
    if (!p.fits) ctr->err |= ERR_CACHE_CAP;
}

// Large volumes: the sums of 256 rounds each as (active << 32 | new), their
// may-emit blocks, and the next call's counts cleared.
__global__ __launch_bounds__(256) void k_round_sums(const uint64_t *__restrict__ round_cnt, uint64_t n,
                                                   uint64_t *__restrict__ sums, uint64_t *__restrict__ round_next) {
    __shared__ uint64_t s_l[4], s_c[4];
    const uint64_t i = blockIdx.x * 256ull + threadIdx.x;
    const uint64_t c = i < n ? round_cnt[i] : 0ull;
    if (i < n) round_next[i] = 0;
    const uint64_t lists = wave_sum(round_lists(c)), cand = wave_sum(c >> 42);
    if (lane() == 0) {
        s_l[threadIdx.x >> 6] = lists;
        s_c[threadIdx.x >> 6] = cand;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sums[2 * blockIdx.x] = s_l[0] + s_l[1] + s_l[2] + s_l[3];
        sums[2 * blockIdx.x + 1] = s_c[0] + s_c[1] + s_c[2] + s_c[3];
    }
}

// Sums over the workgroup (256 threads), returned to every thread; s has 12
// entries and may be reused after a barrier.
__device__ __forceinline__ void wg_sum3(uint64_t &a, uint64_t &b, uint64_t &c, uint64_t *s) {
    a = wave_sum(a);
    b = wave_sum(b);
    c = wave_sum(c);
    const int w = threadIdx.x >> 6;
    if (lane() == 0) {
        s[w] = a;
        s[4 + w] = b;
        s[8 + w] = c;
    }
    __syncthreads();
    a = s[0] + s[1] + s[2] + s[3];
    b = s[4] + s[5] + s[6] + s[7];
    c = s[8] + s[9] + s[10] + s[11];
}
// One round's place in the lists (before), and the call's totals: both as
// (active << 32 | new), cand the may-emit blocks of all rounds.
__device__ __forceinline__ void round_sums_direct(const uint64_t *__restrict__ round_cnt, uint64_t n, uint64_t r,
                                                  uint64_t &before, uint64_t &total, uint64_t &cand, uint64_t *s) {
    before = total = cand = 0;
    for (uint64_t i0 = threadIdx.x; i0 < n; i0 += 1024) {   // 4 loads in flight
        uint64_t c[4];
#pragma unroll
        for (int j = 0; j < 4; j++) c[j] = i0 + 256 * j < n ? round_cnt[i0 + 256 * j] : 0ull;
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint64_t v = round_lists(c[j]);
            total += v;
            before += i0 + 256 * j < r ? v : 0ull;
            cand += c[j] >> 42;
        }
    }
    wg_sum3(before, total, cand, s);
}

// ---------------------------------------------------------------------------
// Alg. 1 SortByKey, as a selection: the n_evicted oldest used slots that hold
// no active block, oldest first and by ascending slot among equals (the first
// entries of the stable sort of all available slots by age; the unused slots,
// older than every used one, precede them and need no list).  A slot's key is
// the call that last used it less `base`, a call no used slot is older than.
// Per pass the keys' digits are counted per tile of slots (with the
// compaction in the first pass, whose kernel waits on memory), and k_evict_list
// finds the digit up to which slots are taken and ranks the tile's slots below
// it.  The keys span the calls since the oldest slot's use (few, since a cache
// that must evict drops the oldest), so one pass covers spans of 1023 calls;
// longer spans take stable passes over 10-bit digits, the last of which stops
// at n_evicted.  Latency bound: tiles of 1024 slots, every load of a tile in
// flight at once.  At 1.5e5 slots the list takes 7 us and the counts under 1 of
// the compaction (tiles of 4096, counted by a launch: 15 and 12 us; a radix sort
// of all available slots after a pass that aged them: 31-42 us in five launches).
// ---------------------------------------------------------------------------
struct EvictPass {
    uint32_t base, now;      // keys: stamps in [base, now)
    int shift, bits;         // the pass's digit
    int first, last;         // first: slots in slot order; else `in`
    const uint32_t *in;      // the previous pass's list
    uint32_t *out;           // this pass's list (last: n_evicted entries)
    uint32_t n_used;         // used slots (first)
    uint32_t tiles;          // stride of the histogram's rows
    int scanned;             // the histogram rows hold prefixes (k_evict_scan ran)
    int refresh;             // look for the oldest used slot's stamp, for the next calls' base
};
constexpr int EVICT_PER = EVICT_TILE / 256;   // elements per lane: wave w has [256 w, 256 w + 256) of the tile

// The lane's elements of the tile: slots and stamps, all loads in flight;
// bit r of the result: element r is there and available.
__device__ __forceinline__ uint32_t evict_load(const EvictPass &p, const uint32_t *__restrict__ S_stamp, uint32_t n,
                                               uint32_t tile, uint32_t (&slot)[EVICT_PER],
                                               uint32_t (&stamp)[EVICT_PER]) {
    const uint32_t i0 = tile * EVICT_TILE + (threadIdx.x >> 6) * (EVICT_TILE / 4) + lane();
#pragma unroll
    for (int r = 0; r < EVICT_PER; r++) {
        const uint32_t i = i0 + 64 * r;
        slot[r] = p.first ? i : (i < n ? p.in[i] : 0u);
    }
    uint32_t there = 0;
#pragma unroll
    for (int r = 0; r < EVICT_PER; r++) {
        const bool in = i0 + 64 * r < n;
        stamp[r] = in ? S_stamp[slot[r]] : ~0u;
        there |= (in && (!p.first || stamp[r] < p.now) ? 1u : 0u) << r;
    }
    return there;
}
__device__ __forceinline__ uint32_t evict_digit(const EvictPass &p, uint32_t stamp) {
    return ((stamp - p.base) >> p.shift) & ((1u << p.bits) - 1u);
}

// Adds the wave's digits to h, one lane per distinct digit: neighbouring
// slots were mostly last used by the same call.
__device__ __forceinline__ void wave_digit_count(uint32_t *h, bool valid, uint32_t d) {
    uint64_t left = __ballot(valid);
    while (left) {
        const int leader = (int)__builtin_ctzll(left);
        const uint32_t ld = (uint32_t)__builtin_amdgcn_readlane((int)d, leader);
        const uint64_t same = __ballot(valid && d == ld) & left;
        if (lane() == leader) atomicAdd(&h[ld], (uint32_t)__popcll(same));
        left &= ~same;
    }
}

// hist[digit][tile] of one tile (by a workgroup; h: EVICT_BINS words of LDS),
// if slots have to be evicted.
__device__ __forceinline__ void evict_count_tile(const EvictPass &p, const uint32_t *__restrict__ S_stamp,
                                                 uint32_t n, uint32_t tile, const uint32_t (&stamp)[EVICT_PER],
                                                 uint32_t there, bool need, uint32_t *h,
                                                 uint32_t *__restrict__ hist, Counters *ctr) {
    if (p.refresh) {
        uint32_t oldest = ~0u;
#pragma unroll
        for (int r = 0; r < EVICT_PER; r++) oldest = min(oldest, stamp[r]);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) oldest = min(oldest, (uint32_t)__shfl_xor((int)oldest, d, 64));
        if (lane() == 0) atomicMax(&ctr->span, p.now - min(oldest, p.now) + 1u);
    }
    if (!need) return;
    for (int d = threadIdx.x; d < 1 << p.bits; d += 256) h[d] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < EVICT_PER; r++) wave_digit_count(h, (there >> r) & 1u, evict_digit(p, stamp[r]));
    __syncthreads();
    for (int d = threadIdx.x; d < 1 << p.bits; d += 256) hist[(uint64_t)d * p.tiles + tile] = h[d];
}

// Each live round's active and new block ids, from its offsets on.  A wave
// takes 1024 consecutive flags of the round (16 per lane, one 16-byte load),
// puts them in LDS and writes the ids 64 blocks at a time: lane l takes block
// 64 j + l, a ballot orders the wave's ids, and each store covers one
// contiguous run of the lists.  LARGE: rounds blockIdx.x, + G, ... with
// k_round_sums' sums; otherwise workgroup r has round r, and the workgroups
// after the rounds' count tiles of slots for the eviction.  Workgroup 0
// publishes the slots' plan.
template <bool LARGE>
__global__ __launch_bounds__(256) void k_compact_blocks(Geom g, const uint8_t *__restrict__ active,
                                                       const uint64_t *__restrict__ round_cnt, uint64_t n_rounds,
                                                       const uint64_t *__restrict__ sums,
                                                       uint64_t *__restrict__ round_next,
                                                       uint32_t *__restrict__ I_active,
                                                       uint32_t *__restrict__ I_new, Counters *ctr,
                                                       Counters *next, SlotState ss, EvictPass ev,
                                                       const uint32_t *__restrict__ S_stamp,
                                                       uint32_t *__restrict__ evict_hist) {
    __shared__ uint32_t s_w[4];
    __shared__ uint4 s_fl[4][64];   // per wave: its 1024 flags in block order
    static_assert(sizeof(s_fl) >= EVICT_BINS * sizeof(uint32_t), "a tile's digit counts take the flags' place");
    __shared__ uint64_t s_sum[12];
    const int w = threadIdx.x >> 6, l = lane();
    uint64_t off = 0, total = 0, cand = 0;
    if constexpr (LARGE) {
        if (blockIdx.x == 0) {
            for (uint64_t i = threadIdx.x; i < (n_rounds + 255) / 256; i += 256) {
                total += sums[2 * i];
                cand += sums[2 * i + 1];
            }
            wg_sum3(off, total, cand, s_sum);
        }
    } else {
        if (blockIdx.x >= n_rounds) {
            const uint32_t tile = blockIdx.x - (uint32_t)n_rounds;
            uint32_t slot[EVICT_PER], stamp[EVICT_PER];
            const uint32_t there = evict_load(ev, S_stamp, ev.n_used, tile, slot, stamp);
            round_sums_direct(round_cnt, n_rounds, 0, off, total, cand, s_sum);
            const SlotPlan p = plan_slots(total >> 32, total & 0xFFFFFFFFull, ss);
            evict_count_tile(ev, S_stamp, ev.n_used, tile, stamp, there, p.fits && p.n_evicted,
                             reinterpret_cast<uint32_t *>(s_fl), evict_hist, ctr);
            return;
        }
        if (threadIdx.x == 0) round_next[blockIdx.x] = 0;
        if (blockIdx.x != 0 && round_cnt[blockIdx.x] == 0) return;
        round_sums_direct(round_cnt, n_rounds, blockIdx.x, off, total, cand, s_sum);
    }
    if (blockIdx.x == 0)
        publish_plan(ctr, next, total >> 32, total & 0xFFFFFFFFull, cand, ss);
    for (uint64_t k = blockIdx.x; k < n_rounds; k += gridDim.x) {
        if (round_cnt[k] == 0) continue;
        const uint64_t wbase = k * BLK_TILE + 1024u * w;
        const uint4 q = load_flags16(active, wbase + 16u * l, g.nb);
        if constexpr (LARGE) {
            const uint64_t big = k / 256;
            off = 256 * big + threadIdx.x < k ? round_lists(round_cnt[256 * big + threadIdx.x]) : 0ull;
            for (uint64_t i = threadIdx.x; i < big; i += 256) off += sums[2 * i];
            uint64_t none = 0, unused = 0;
            __syncthreads();   // s_sum is rewritten
            wg_sum3(off, none, unused, s_sum);
        }
        uint32_t actb, newb;
        flag_bits(q, actb, newb);
        const uint32_t tot = wave_sum(((uint32_t)__popc(actb) << 16) | (uint32_t)__popc(newb));   // < 2^11 each
        if (l == 0) s_w[w] = tot;
        s_fl[w][l] = q;
        __syncthreads();
        uint32_t ex = 0;
#pragma unroll
        for (int i = 0; i < 4; i++)
            if (i < w) ex += s_w[i];
        uint64_t pa = (off >> 32) + (ex >> 16), pn = (off & 0xFFFFFFFFull) + (ex & 0xFFFFu);
        if (tot) {
            const uint8_t *fl = reinterpret_cast<const uint8_t *>(s_fl[w]);
#pragma unroll 4
            for (int j = 0; j < 16; j++) {
                const uint32_t f = fl[64 * j + l];
                const bool a = (f & 7u) != 0, nw = (f & 4u) != 0;   // any flag bit marks an active block
                const uint64_t am = __ballot(a), nm = __ballot(nw);
                const uint32_t blk = (uint32_t)(wbase + 64u * j + (uint32_t)l);
                if (a) I_active[pa + mbcnt(am)] = blk;
                if (nw) I_new[pn + mbcnt(nm)] = blk;
                pa += (uint64_t)__popcll(am);
                pn += (uint64_t)__popcll(nm);
            }
        }
        __syncthreads();   // s_w and s_fl are rewritten by the next round
    }
}

// The digits of a pass, a tile per workgroup (the first pass of a volume of
// up to ROUNDS_DIRECT rounds is counted by the compaction).
__global__ __launch_bounds__(256) void k_evict_count(EvictPass p, const uint32_t *__restrict__ S_stamp,
                                                    uint32_t *__restrict__ hist, Counters *ctr) {
    __shared__ uint32_t h[EVICT_BINS];
    if (ctr->err) return;
    const bool need = ctr->n_evicted != 0;
    if (!need && !p.refresh) return;
    const uint32_t n = p.first ? p.n_used : ctr->n_sort;
    uint32_t slot[EVICT_PER], stamp[EVICT_PER];
    const uint32_t there = evict_load(p, S_stamp, n, blockIdx.x, slot, stamp);
    evict_count_tile(p, S_stamp, n, blockIdx.x, stamp, there, need, h, hist, ctr);
}

// Many tiles: each digit's row of the histogram into its exclusive prefix,
// the row's total to totals[digit]; one workgroup per digit.
__global__ __launch_bounds__(256) void k_evict_scan(uint32_t tiles, uint32_t *__restrict__ hist,
                                                   uint32_t *__restrict__ totals, const Counters *ctr) {
    __shared__ uint32_t s_w[4];
    if (ctr->err || !ctr->n_evicted) return;
    uint32_t *row = hist + (uint64_t)blockIdx.x * tiles;
    uint32_t carry = 0;
    for (uint32_t t0 = 0; t0 < tiles; t0 += 256) {
        const uint32_t t = t0 + threadIdx.x;
        const uint32_t x = t < tiles ? row[t] : 0u;
        const uint32_t incl = wave_incl_scan(x);
        if (lane() == 63) s_w[threadIdx.x >> 6] = incl;
        __syncthreads();
        uint32_t o = carry + incl - x;
        for (int i = 0; i < 4; i++) {
            if (i < (int)(threadIdx.x >> 6)) o += s_w[i];
            carry += s_w[i];
        }
        if (t < tiles) row[t] = o;
        __syncthreads();   // s_w is rewritten next step
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// The pass's list.  Each workgroup forms the digits' offsets (totals over
// all tiles, then the tile's own) and ranks its tile in order: each wave
// owns 256 consecutive elements and its own running counts.
__global__ __launch_bounds__(256) void k_evict_list(EvictPass p, const uint32_t *__restrict__ S_stamp,
                                                   const uint32_t *__restrict__ hist,
                                                   const uint32_t *__restrict__ totals, Counters *ctr) {
    __shared__ uint32_t off[EVICT_BINS];       // first position of the tile's elements, per digit
    __shared__ uint32_t run[4][EVICT_BINS];    // per wave: elements of its share, then its next position
    __shared__ uint32_t s_w[4], s_thr;
    if (ctr->err || !ctr->n_evicted) return;
    const uint32_t bins = 1u << p.bits, n = p.first ? p.n_used : ctr->n_sort, tile = blockIdx.x;
    const uint32_t want = p.last ? (uint32_t)ctr->n_evicted : ~0u;   // positions past it are dropped
    const int w = threadIdx.x >> 6, l = lane();
    uint32_t slot[EVICT_PER], stamp[EVICT_PER], dig[EVICT_PER];
    const uint32_t there = evict_load(p, S_stamp, n, tile, slot, stamp);
    for (uint32_t d = threadIdx.x; d < bins; d += 256) run[0][d] = off[d] = 0;
    if (threadIdx.x == 0) s_thr = bins;
    __syncthreads();
    // per digit: elements in all tiles (run[0]) and in the tiles before this
    // one (off); few digits: several threads per row
    if (p.scanned) {
        for (uint32_t d = threadIdx.x; d < bins; d += 256) {
            run[0][d] = totals[d];
            off[d] = hist[(uint64_t)d * p.tiles + tile];
        }
    } else {
        const uint32_t per = bins < 256 ? 256 / bins : 1u, part = threadIdx.x % per;
        for (uint32_t d = threadIdx.x / per; d < bins; d += 256 / per) {
            const uint32_t *row = hist + (uint64_t)d * p.tiles;
            uint32_t all = 0, before = 0;
#pragma unroll 8
            for (uint32_t t = part; t < p.tiles; t += per) {
                const uint32_t x = row[t];
                all += x;
                before += t < tile ? x : 0u;
            }
            if (all) atomicAdd(&run[0][d], all);
            if (before) atomicAdd(&off[d], before);
        }
    }
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t d0 = 0; d0 < bins; d0 += 256) {   // exclusive prefix over the digits
        const uint32_t d = d0 + threadIdx.x;
        const uint32_t x = d < bins ? run[0][d] : 0u;
        const uint32_t incl = wave_incl_scan(x);
        if (l == 63) s_w[w] = incl;
        __syncthreads();
        uint32_t o = carry + incl - x;
        for (int i = 0; i < 4; i++) {
            if (i < w) o += s_w[i];
            carry += s_w[i];
        }
        if (d < bins) {
            off[d] += o;
            run[0][d] = run[1][d] = run[2][d] = run[3][d] = 0;
            if (o < want && want - o <= x) s_thr = d;   // the digit the list ends in
        }
        __syncthreads();
    }
    const uint32_t thr = s_thr;
    if (tile == 0 && threadIdx.x == 0) {
        if (p.first) ctr->n_sort = carry;
        if (p.last) {
            if (carry < want) atomicOr(&ctr->err, ERR_INTERNAL);
            ctr->span = p.now - (p.base + (thr << p.shift)) + 1u;   // what stays is no older
        }
    }
    if (carry < want && p.last) return;
    uint32_t take = 0;
#pragma unroll
    for (int r = 0; r < EVICT_PER; r++) {
        dig[r] = evict_digit(p, stamp[r]);
        const bool v = ((there >> r) & 1u) && dig[r] <= thr;
        take |= (v ? 1u : 0u) << r;
        wave_digit_count(run[w], v, dig[r]);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < bins; d += 256) {   // counts -> each wave's first position
        uint32_t o = off[d];
        for (int i = 0; i < 4; i++) {
            const uint32_t x = run[i][d];
            run[i][d] = o;
            o += x;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < EVICT_PER; r++) {
        const bool v = (take >> r) & 1u;
        uint64_t left = __ballot(v);
        while (left) {
            const int leader = (int)__builtin_ctzll(left);
            const uint32_t ld = (uint32_t)__builtin_amdgcn_readlane((int)dig[r], leader);
            const uint64_t same = __ballot(v && dig[r] == ld) & left;
            const uint32_t o = run[w][ld];
            wave_lds_sync();
            if ((same >> l) & 1u) {
                const uint32_t pos = o + mbcnt(same);
                if (pos < (p.last ? want : n)) p.out[pos] = slot[r];
            }
            if (l == leader) run[w][ld] = o + (uint32_t)__popcll(same);
            wave_lds_sync();
            left &= ~same;
        }
    }
}

// Empties the cache: the used slots lose their blocks (the others hold none).
__global__ __launch_bounds__(256) void k_cache_empty(uint64_t n_used, int32_t *__restrict__ S_block,
                                                    uint32_t *__restrict__ S_stamp,
                                                    int32_t *__restrict__ I_slot) {
    for (uint64_t s = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; s < n_used;
         s += (uint64_t)gridDim.x * blockDim.x) {
        const int32_t b = S_block[s];
        if (b >= 0) I_slot[b] = -1;
        S_block[s] = -1;
        S_stamp[s] = 0;
    }
}

// Sign masks (Sec. 4.4's per-cell classification, one bit per sample) of the
// active blocks of a volume whose blocks are all resident: bit i of masks[b]
// is set when sample i of block b (x fastest) is below iso.  One lane per
// block: its 16 float4 loads are all in flight before the first compare.
// (Cached volumes build theirs with the decode.)
__global__ __launch_bounds__(256) void k_masks(const uint32_t *__restrict__ I_active,
                                              const float *__restrict__ blocks, float iso,
                                              uint64_t *__restrict__ masks, const Counters *ctr) {
    if (ctr->err) return;
    const uint64_t n_act = ctr->n_act;
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n_act;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t b = I_active[i];
        const float4 *src = reinterpret_cast<const float4 *>(blocks) + (uint64_t)b * 16;
        float4 v[16];
#pragma unroll
        for (int q = 0; q < 16; q++) v[q] = src[q];
        uint64_t m = 0;
#pragma unroll
        for (int q = 0; q < 16; q++) {
            const uint64_t nib = (v[q].x < iso ? 1u : 0u) | (v[q].y < iso ? 2u : 0u) |
                                 (v[q].z < iso ? 4u : 0u) | (v[q].w < iso ? 8u : 0u);
            m |= nib << (4 * q);
        }
        masks[b] = m;
    }
}

// Count pass (Sec. 4.4): vertex count of every active block (0 unless it can
// emit), one lane per block, over the chunks of xcd_chunks (mc_chunk_size
// blocks each); each chunk's total goes to chunk_tot, and the vertices and
// occupied blocks of each XCD eighth (the split of xcd_chunks) are added up in
// the counters, one atomic per workgroup on the eighth's own cache line.  The
// cases of all 64 cells are evaluated at once on the corner masks, and the
// triangle count per case by the bit-sliced diagram of the marching-cubes
// table (mc_ntri_bits, generated at build time).
__global__ __launch_bounds__(256) void k_mc_count(Geom g, const uint32_t *__restrict__ I_active,
                                                 const uint8_t *__restrict__ active,
                                                 const int32_t *__restrict__ I_slot, int identity,
                                                 const uint64_t *__restrict__ masks,
                                                 uint32_t *__restrict__ blk_cnt,
                                                 uint32_t *__restrict__ chunk_tot, uint32_t emit_waves,
                                                 Counters *ctr) {
    __shared__ uint64_t s_v[MC_WAVES];
    __shared__ uint32_t s_o[MC_WAVES];
    if (ctr->err) return;
    const uint64_t n_act = ctr->n_act;
    const uint32_t cs = mc_chunk_size(n_act, emit_waves);   // the emission's chunks
    const ChunkRange cr = xcd_chunks((n_act + cs - 1) / cs);
    uint32_t wocc = 0;
    uint64_t wverts = 0;
    for (uint64_t c = cr.first; c < cr.end; c += cr.stride) {
        const uint64_t i = c * cs + lane();
        const bool in = lane() < (int)cs && i < n_act;
        uint32_t cnt = 0;
        const uint32_t b = in ? I_active[i] : 0u;
        if (in && (active[b] & 2u)) {
            uint32_t so[8], bx, by, bz;
            if (!octet(g, b, I_slot, identity, so, bx, by, bz)) {
                atomicOr(&ctr->err, ERR_INTERNAL);
            } else {
                uint64_t M[8], cm[8];
#pragma unroll
                for (int m = 0; m < 8; m++) M[m] = masks[so[m]];
                corner_masks(M, cm);
                uint64_t n0, n1, n2;
                mc_ntri_bits(cm, n0, n1, n2);
                const uint64_t V = valid_cells(g, bx, by, bz);
                const uint32_t tris = (uint32_t)__popcll(n0 & V) + 2u * (uint32_t)__popcll(n1 & V) +
                                      4u * (uint32_t)__popcll(n2 & V);
                cnt = 3u * tris;
            }
        }
        if (in) blk_cnt[i] = cnt;
        const uint32_t tot = wave_sum(cnt);
        if (lane() == 0) chunk_tot[c] = tot;
        wverts += tot;
        wocc += cnt ? 1u : 0u;
    }
    wocc = wave_sum(wocc);
    if (lane() == 0) {
        s_v[threadIdx.x >> 6] = wverts;
        s_o[threadIdx.x >> 6] = wocc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t v = 0;
        uint32_t o = 0;
        for (int k = 0; k < MC_WAVES; k++) {
            v += s_v[k];
            o += s_o[k];
        }
        if (o) {
            atomicAdd(&ctr->xcd[blockIdx.x % 8u].verts, (unsigned long long)v);
            atomicAdd(&ctr->xcd[blockIdx.x % 8u].occ, (unsigned long long)o);
        }
    }
}

// Emission pass (Sec. 4.5), over the chunks of xcd_chunks (the count pass's
// schedule).  A wave's first chunk follows the eighths before its own and the
// chunks of its eighth before it (fewer than the eighth's waves: 3.5 KB of
// totals at most), each next one the chunks between: the wave adds them up
// itself, which a launch scanning the totals (4.5-5 us of every call) does not
// pay for.  Within a chunk: the block offsets by a wave scan of the counts, then the occupied blocks restaged a few at a time;
// each block's in-block prefix of its per-cell triangle counts, the
// triangles of the staged blocks listed together and written lane per vertex
// from the first block's offset, in canonical order (block, cell, triangle,
// vertex).  Bound by memory and VALU issue together (70 % busy at 512^3): with
// the place of a block's cells looked at only at the volume's far faces, one LDS
// address for a cell's corners and the list's length a scalar, a wave's blocks
// take 153 VALU instructions each instead of 170 (edge records 166 -> 158 us,
// 16 calls of a 1280 x 960 sheet 410 -> 391).
template <int FMT>
__global__ __launch_bounds__(256, FMT == VFMT_GRAD ? 5 : 7) void k_mc_emit(Geom g, const uint32_t *__restrict__ I_active,
                                                const int32_t *__restrict__ I_slot, int identity,
                                                const float *__restrict__ slots,
                                                const uint64_t *__restrict__ mc_table, float iso,
                                                const uint32_t *__restrict__ blk_cnt,
                                                uint64_t *__restrict__ blk_off,
                                                void *__restrict__ out, uint64_t cap,
                                                const uint32_t *__restrict__ chunk_tot,
                                                uint32_t chunk_waves, Counters *ctr,
                                                const float *__restrict__ gV = nullptr,
                                                float *__restrict__ dfield = nullptr,
                                                float *__restrict__ part_giso = nullptr) {
    __shared__ std::conditional_t<FMT == VFMT_GRAD, EmitSharedGrad, EmitSharedPlain> sh;
    if (ctr->err) return;
    for (int i = threadIdx.x; i < 256; i += blockDim.x) sh.tab[i] = mc_table[i];
    if (threadIdx.x < 16) sh.edge[threadIdx.x] = edge_entry((int)threadIdx.x);
    if constexpr (FMT == VFMT_GRAD) {
        for (int i = threadIdx.x; i < MC_WAVES * EMIT_SB * 128; i += blockDim.x) (&sh.acc[0][0][0])[i] = 0.0f;
    }
    __syncthreads();
    const uint64_t n_act = uniform64(ctr->n_act);
    const int w = (int)wave_id(), l = lane();
    const uint32_t cs = mc_chunk_size(n_act, chunk_waves);   // the count pass's chunks
    const ChunkRange cr = xcd_chunks((n_act + cs - 1) / cs);
    GradCtx gc;
    if constexpr (FMT == VFMT_GRAD) {
        gc.gV = gV;
        gc.dfield = dfield;
        gc.err = &ctr->err;
        gc.nbx = g.nbx;
        gc.nbxy = g.nbx * g.nby;
        gc.giso = 0.0f;
    }
    // the vertices of the XCD eighths before this workgroup's; workgroup 0
    // forms the call's totals
    uint64_t base = 0, all = 0, occ = 0;
    for (uint32_t x = 0; x < 8; x++) {
        const uint64_t tx = ctr->xcd[x].verts;
        base += x < blockIdx.x % 8u ? tx : 0ull;
        all += tx;
        occ += ctr->xcd[x].occ;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctr->total_verts = all;
        ctr->n_occ = occ;
    }
    base = uniform64(base);
    if (cr.first < cr.end) base += chunks_sum(chunk_tot, cr.lo, cr.first);
    const LaneGeom q = lane_geom();
    for (uint64_t c = cr.first; c < cr.end; c += cr.stride) {
        const uint64_t idx = c * cs + l;
        const bool valid = l < (int)cs && idx < n_act;
        const uint32_t cnt = valid ? blk_cnt[idx] : 0u;
        const uint32_t incl = wave_incl_scan(cnt);
        const uint64_t off = base + (incl - cnt);
        if (valid) blk_off[idx] = off;
        const uint32_t b = cnt ? I_active[idx] : 0u;
        const uint64_t boff = off;
        uint32_t so[8], lbx, lby, lbz;
        octet(g, b, I_slot, identity, so, lbx, lby, lbz);
        uint64_t todo = __ballot(cnt != 0);
        while (todo) {
            const uint64_t left = todo;
            int jl[EMIT_SB], nsb = 0;
#pragma unroll
            for (int k = 0; k < EMIT_SB; k++) {
                jl[k] = k ? jl[0] : 0;
                if (todo) {
                    jl[k] = (int)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    nsb++;
                }
            }
            // the triangle list area is empty between batches (emit_batch flushes)
            static_assert(8 * EMIT_SB <= EMIT_TRIS, "slot table fits the triangle list");
            stage_batch_tab<EMIT_SB>(q, slots, so, left & ~todo, nsb, sh.tri[w], sh.tiles[w]);
            wave_lds_sync();
            // the staged blocks are consecutive occupied blocks: their vertex
            // ranges follow each other from the first one's offset, so their
            // triangles are listed together and written by one lane-per-vertex
            // loop (a block's last partial pass of 64 lanes is shared)
            const uint64_t ob = ((uint64_t)bcast((uint32_t)(boff >> 32), jl[0]) << 32) |
                                bcast((uint32_t)boff, jl[0]);
            auto info = [&](int k, Geom &gk, uint32_t &bk, uint32_t &bx, uint32_t &by, uint32_t &bz,
                            float &isok) {
                gk = g;
                bk = bcast(b, jl[k]);
                bx = bcast(lbx, jl[k]);
                by = bcast(lby, jl[k]);
                bz = bcast(lbz, jl[k]);
                isok = iso;
            };
            if constexpr (FMT == VFMT_GRAD) {
#pragma unroll
                for (int k = 0; k < EMIT_SB; k++) gc.expect[k] = bcast(cnt, jl[k]);
            }
            emit_batch<FMT>(nsb, info, sh.tiles[w], sh.tab, sh, w, ob, out, cap, &gc);
        }
        if (c + cr.stride < cr.end) base += chunks_sum(chunk_tot, c, c + cr.stride);
    }
    if constexpr (FMT == VFMT_GRAD) {   // the wave's share of dL/diso (summed by k_sum_f32: no
                                        // same-address atomics, a fixed order)
        const float gi = wave_sum(gc.giso);
        if (l == 0) part_giso[blockIdx.x * MC_WAVES + w] = gi;
    }
}

// out = sum of p[0..n) in a fixed order (one workgroup of 1024 threads).
__global__ __launch_bounds__(1024) void k_sum_f32(const float *__restrict__ p, uint32_t n,
                                                 float *__restrict__ out) {
    __shared__ float s_w[16];
    float v = 0.0f;
    for (uint32_t i = threadIdx.x; i < n; i += 1024) v += p[i];
    v = wave_sum(v);
    if (lane() == 0) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int k = 0; k < 16; k++) t += s_w[k];
        *out = t;
    }
}

// Cases of every cell of every active block (0 for cells outside the volume
// or in blocks that cannot emit), [n_act][64].
__global__ __launch_bounds__(256) void k_debug_cases(Geom g, const uint32_t *__restrict__ I_active,
                                                    const uint8_t *__restrict__ active,
                                                    const int32_t *__restrict__ I_slot, int identity,
                                                    const float *__restrict__ slots, float iso,
                                                    uint8_t *__restrict__ cases,
                                                    const Counters *ctr) {
    __shared__ float tiles[MC_WAVES][128];
    if (ctr->err) return;
    const uint64_t n_act = ctr->n_act;
    const int w = threadIdx.x >> 6;
    const uint64_t waves = (uint64_t)gridDim.x * MC_WAVES;
    for (uint64_t i = (uint64_t)blockIdx.x * MC_WAVES + w; i < n_act; i += waves) {
        const uint32_t b = I_active[i];
        int cs = -1;
        if (active[b] & 2u) {
            Halo h;
            halo_setup(g, b, I_slot, identity, h);
            if (!h.bad) {
                stage_tile(g, h, slots, tiles[w]);
                wave_lds_sync();
                cs = cell_case(g, h, tiles[w], iso);
                wave_lds_sync();
            }
        }
        cases[i * 64 + lane()] = (uint8_t)(cs < 0 ? 0 : cs);
    }
}

// The call's counters to the host's copy (pinned memory), then the call's
// number behind them: the host polls it.  As a kernel of its own it starts when
// the emission has ended, so the number means that the soup is whole.
__global__ __launch_bounds__(64) void k_publish(const uint32_t *__restrict__ ctr, uint32_t *__restrict__ host,
                                               uint32_t *seq, uint32_t value) {
    if (threadIdx.x < CTR_READ / 4) host[threadIdx.x] = ctr[threadIdx.x];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(seq, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Plain streaming copy (16 B per lane per iteration): a known-size reference
// for reading memory-traffic counters.
__global__ __launch_bounds__(256) void k_copy_calibration(uint4 *__restrict__ dst,
                                                         const uint4 *__restrict__ src, uint64_t n) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, uint64_t n) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// The backward's outputs before it adds to them: the field's gradient zero
// (16 bytes per lane where it is so aligned) and the call's error bits clear.
// One launch for what were three memory commands, 6 us each of a 256^3 pass.
__global__ __launch_bounds__(256) void k_clear_gradient(float *__restrict__ dfield, uint64_t n, int wide, Counters *ctr) {
    const uint64_t i0 = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x, step = (uint64_t)gridDim.x * blockDim.x;
    if (i0 == 0) ctr->err = 0;
    if (wide) {
        for (uint64_t i = i0; i < n / 4; i += step)
            reinterpret_cast<float4 *>(dfield)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    } else {
        for (uint64_t i = i0; i < n; i += step) dfield[i] = 0.0f;
    }
}

__global__ void k_iota_i32(int32_t *p, uint64_t n) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = (int32_t)i;
}

unsigned grid_cap(uint64_t n_threads, unsigned cap) {
    uint64_t gsz = (n_threads + 255) / 256;
    if (gsz < 1) gsz = 1;
    return (unsigned)(gsz < cap ? gsz : cap);
}

}  // namespace

static unsigned mc_grid(uint64_t max_blocks) {
    uint64_t g = (max_blocks + MC_WAVES - 1) / MC_WAVES;
    g = g < MC_MAX_GRID ? g : MC_MAX_GRID;
    return (unsigned)((g + 7) / 8 * 8);   // whole XCD rounds
}

void launch_cull(const Geom &g, const DevState &d, float iso, float prev_iso, int rewrite, int identity_cache,
                 uint32_t now, hipStream_t s) {
    const uint64_t nt = cull_tiles(g);
    unsigned long long *cnt = reinterpret_cast<unsigned long long *>(d.round_cnt);
    if (nt <= CULL_DIRECT) {
        k_cull<false, CULL_LAYERS><<<(unsigned)nt * (CULL_TZ / CULL_LAYERS), 256, 0, s>>>(
            g, d.ranges, iso, prev_iso, rewrite, d.tile_ranges, nullptr, nt, d.I_slot, identity_cache, d.S_stamp,
            now, d.active, d.ctr, cnt);
        return;
    }
    static unsigned rgrid = 0;
    if (!rgrid) rgrid = resident_grid(k_cull<true, CULL_TZ>);
    k_cull_scan<<<(unsigned)((nt + 255) / 256), 256, 0, s>>>(d.tile_ranges, nt, iso, prev_iso, rewrite,
                                                             d.cull_list, d.ctr);
    k_cull<true, CULL_TZ><<<(unsigned)std::min<uint64_t>(nt, rgrid), 256, 0, s>>>(
        g, d.ranges, iso, prev_iso, rewrite, d.tile_ranges, d.cull_list, nt, d.I_slot, identity_cache, d.S_stamp,
        now, d.active, d.ctr, cnt);
}

uint64_t cull_tiles(const Geom &g) {
    return (uint64_t)((g.nbx + CULL_TX - 1) / CULL_TX) * ((g.nby + CULL_TY - 1) / CULL_TY) *
           ((g.nbz + CULL_TZ - 1) / CULL_TZ);
}

void launch_tile_ranges(const Geom &g, const float2 *ranges, float2 *tile_ranges, hipStream_t s) {
    k_tile_ranges<<<(unsigned)cull_tiles(g), 256, 0, s>>>(g, ranges, tile_ranges);
}

// Pass k of the eviction's selection (k_evict_count, k_evict_list).
static EvictPass evict_pass(const DevState &d, uint32_t n_used, uint32_t base, uint32_t now, int k) {
    const int key_bits = 32 - __builtin_clz((now - base) | 1u);
    EvictPass p;
    p.base = base;
    p.now = now;
    p.shift = k * EVICT_BITS;
    p.bits = std::min(EVICT_BITS, key_bits - p.shift);
    p.first = k == 0;
    p.last = p.shift + p.bits == key_bits;
    p.in = d.evict[(k & 1) ^ 1];
    p.out = d.evict[k & 1];
    p.n_used = n_used;
    p.tiles = (n_used + EVICT_TILE - 1) / EVICT_TILE;
    // up to 32 K counts every workgroup of k_evict_list adds up the rows
    // itself (128 loads a thread at most); beyond, a launch scans them
    p.scanned = ((uint64_t)p.tiles << p.bits) > 32768;
    p.refresh = k == 0 && now - base > EVICT_REFRESH;
    return p;
}

void launch_compact_blocks(const Geom &g, const DevState &d, const SlotState &ss, uint32_t base, uint32_t now,
                           hipStream_t s) {
    const uint64_t n = block_rounds(g.nb);
    const EvictPass ev = evict_pass(d, (uint32_t)ss.n_used, base, now, 0);
    if (n <= ROUNDS_DIRECT) {
        k_compact_blocks<false><<<(unsigned)n + ev.tiles, 256, 0, s>>>(
            g, d.active, d.round_cnt, n, nullptr, d.round_next, d.I_active, d.I_new, d.ctr, d.ctr_next, ss, ev,
            d.S_stamp, d.evict_hist);
        return;
    }
    static unsigned wgrid = 0;
    if (!wgrid) wgrid = resident_grid(k_compact_blocks<true>);
    k_round_sums<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(d.round_cnt, n, d.round_sums, d.round_next);
    k_compact_blocks<true><<<(unsigned)std::min<uint64_t>(n, wgrid), 256, 0, s>>>(
        g, d.active, d.round_cnt, n, d.round_sums, d.round_next, d.I_active, d.I_new, d.ctr, d.ctr_next, ss, ev,
        d.S_stamp, d.evict_hist);
}

uint32_t *launch_evict(const Geom &g, const DevState &d, uint32_t n_used, uint32_t base, uint32_t now,
                       hipStream_t s) {
    if (n_used == 0) return d.evict[0];   // nothing to evict
    for (int k = 0;; k++) {
        const EvictPass p = evict_pass(d, n_used, base, now, k);
        if (k > 0 || block_rounds(g.nb) > ROUNDS_DIRECT)
            k_evict_count<<<p.tiles, 256, 0, s>>>(p, d.S_stamp, d.evict_hist, d.ctr);
        if (p.scanned) k_evict_scan<<<1u << p.bits, 256, 0, s>>>(p.tiles, d.evict_hist, d.evict_tot, d.ctr);
        k_evict_list<<<p.tiles, 256, 0, s>>>(p, d.S_stamp, d.evict_hist, d.evict_tot, d.ctr);
        if (p.last) return p.out;
    }
}

void launch_cache_empty(const DevState &d, uint64_t n_used, hipStream_t s) {
    if (n_used)
        k_cache_empty<<<grid_cap(n_used, 8192), 256, 0, s>>>(n_used, d.S_block, d.S_stamp, d.I_slot);
}


// Grid of the emission: as many workgroups as are resident at once (their
// waves sweep the chunks of the active list as one window), in whole XCD
// rounds.  Its wave count also sets the chunk size (mc_chunk_size).  One
// workgroup per CU fewer than fit (8: 64 VGPRs, 19.8 KB of LDS): the eighth
// measured slower, its waves being more than the memory serves (a call on 512^3
// turbulence 553 against 530 us, with edge records 284 against 267).
constexpr int EMIT_PER_CU = 7;
static unsigned emit_grid(const Geom &g, int fmt) {
    static unsigned grid[3] = {0, 0, 0};
    if (!grid[0]) grid[0] = resident_grid(k_mc_emit<VFMT_F32>, EMIT_PER_CU);
    if (!grid[1]) grid[1] = resident_grid(k_mc_emit<VFMT_EDGE8>, EMIT_PER_CU);
    if (!grid[2]) grid[2] = resident_grid(k_mc_emit<VFMT_Q10>, EMIT_PER_CU);
    return std::min<unsigned>(grid[fmt >= 0 && fmt < 3 ? fmt : 0], mc_grid(g.nb));
}

void launch_mc_count(const Geom &g, const DevState &d, const float *slots, const int32_t *I_slot,
                     int identity_cache, float iso, int fmt, hipStream_t s) {
    if (identity_cache) {
        static unsigned mgrid = 0;
        if (!mgrid) mgrid = resident_grid(k_masks);
        k_masks<<<std::min<unsigned>(mgrid, mc_grid(g.nb / 16 + 1)), 256, 0, s>>>(d.I_active, slots, iso, d.masks,
                                                                                 d.ctr);
    }
    // the count pass takes the emission's chunks on a grid of its own (all
    // of it resident)
    static unsigned cres = 0;
    if (!cres) cres = std::min<unsigned>(resident_grid(k_mc_count), MC_MAX_GRID);
    const unsigned egrid = emit_grid(g, fmt), cgrid = std::min<unsigned>(cres, mc_grid(g.nb));
    k_mc_count<<<cgrid, 256, 0, s>>>(g, d.I_active, d.active, I_slot, identity_cache, d.masks,
                                     d.blk_cnt, d.chunk_tot, egrid * MC_WAVES, d.ctr);
}

void launch_mc_emit(const Geom &g, const DevState &d, const float *slots, const int32_t *I_slot,
                    int identity_cache, float iso, void *out, uint64_t cap_verts, int fmt,
                    hipStream_t s) {
    const unsigned n = emit_grid(g, fmt);
#define BCMC_EMIT(F)                                                                          \
    k_mc_emit<F><<<n, 256, 0, s>>>(g, d.I_active, I_slot, identity_cache, slots, d.mc_table, iso, \
                                   d.blk_cnt, d.blk_off, out, cap_verts, d.chunk_tot, n * MC_WAVES, d.ctr)
    if (fmt == VFMT_EDGE8) BCMC_EMIT(VFMT_EDGE8);
    else if (fmt == VFMT_Q10) BCMC_EMIT(VFMT_Q10);
    else BCMC_EMIT(VFMT_F32);
#undef BCMC_EMIT
}

// 16-byte vertices -> Sec. 4.5's 8-byte records (q10_code | block << 32),
// two vertices per lane per iteration.
__global__ __launch_bounds__(256) void k_vertices_q10(const uint4 *__restrict__ in, uint64_t n,
                                                     uint64_t *__restrict__ out) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint4 v = in[i];
        const uint32_t q = q10_code(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z));
        __builtin_nontemporal_store((uint64_t)q | ((uint64_t)v.w << 32), out + i);
    }
}

void launch_vertices_q10(const void *in, uint64_t n, void *out, hipStream_t s) {
    if (n) k_vertices_q10<<<grid_cap(n, 8192), 256, 0, s>>>(reinterpret_cast<const uint4 *>(in), n,
                                                            reinterpret_cast<uint64_t *>(out));
}

void launch_debug_cases(const Geom &g, const DevState &d, const float *slots,
                        const int32_t *I_slot, int identity_cache, float iso, uint8_t *cases,
                        uint64_t max_act, hipStream_t s) {
    k_debug_cases<<<mc_grid(max_act), 256, 0, s>>>(g, d.I_active, d.active, I_slot, identity_cache,
                                                    slots, iso, cases, d.ctr);
}

// Backward of the vertex positions through t = (iso - a)/(b - a), topology
// fixed: the emission's pass over the last extract's soup (same chunks and
// offsets) in VFMT_GRAD mode, which for a vertex on an edge along axis e
// with g = dL/dv[e] adds g (t - 1)/(b - a) to dL/da, -g t/(b - a) to dL/db
// and g/(b - a) to dL/diso (float atomics into the field through per-block
// LDS sums; dL/diso by per-wave partial sums).  Both outputs are written in
// full.  fmt: the extract's vertex
// format (its grid set the chunks).
void launch_backward(const Geom &g, const DevState &d, const float *slots, float iso,
                     const float *gV, uint64_t n_verts, float *dfield, float *diso, int fmt,
                     hipStream_t s) {
    static unsigned grid = 0;
    if (!grid) grid = resident_grid(k_mc_emit<VFMT_GRAD>);
    const unsigned n = std::min<unsigned>(grid, mc_grid(g.nb));
    const uint64_t nf = g.nb * 64;
    k_clear_gradient<<<grid_cap(nf / 4, 4096), 256, 0, s>>>(dfield, nf, reinterpret_cast<uintptr_t>(dfield) % 16 == 0,
                                                            d.ctr);
    k_mc_emit<VFMT_GRAD><<<n, 256, 0, s>>>(g, d.I_active, nullptr, 1, slots, d.mc_table, iso, d.blk_cnt,
                                          d.blk_off, nullptr, n_verts, d.chunk_tot,
                                          emit_grid(g, fmt) * MC_WAVES, d.ctr, gV, dfield, d.part_giso);
    k_sum_f32<<<1, 1024, 0, s>>>(d.part_giso, n * MC_WAVES, diso);
}

void launch_copy_calibration(void *dst, const void *src, uint64_t n16, hipStream_t s) {
    if (n16) k_copy_calibration<<<grid_cap(n16, 16384), 256, 0, s>>>(
        reinterpret_cast<uint4 *>(dst), reinterpret_cast<const uint4 *>(src), n16);
}

void launch_publish(const void *ctr, HostCounters *host, uint32_t value, hipStream_t s) {
    static_assert(CTR_READ / 4 <= 64, "one lane per word");
    k_publish<<<1, 64, 0, s>>>(reinterpret_cast<const uint32_t *>(ctr), reinterpret_cast<uint32_t *>(host->c),
                               &host->seq, value);
}

void launch_fill_u32(uint32_t *p, uint32_t v, uint64_t n, hipStream_t s) {
    if (n) k_fill_u32<<<grid_cap(n, 8192), 256, 0, s>>>(p, v, n);
}

void launch_iota_i32(int32_t *p, uint64_t n, hipStream_t s) {
    if (n) k_iota_i32<<<grid_cap(n, 8192), 256, 0, s>>>(p, n);
}

}  // namespace bcmc
