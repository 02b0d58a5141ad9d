// Batched extraction: many volumes of uneven size, several isovalues each,
// in six launches, replayable from a hipGraph.
//
// Each job j = (volume v_j, isovalue iso_j) produces exactly the triangle soup
// a single-volume extract of v_j at iso_j produces (same arithmetic, same
// canonical order); the jobs' soups are concatenated in job order.
//
// The batch keeps its own decoded-block store: a block needed by any job of
// its volume (the union over the volume's isovalues, Sec. 4.1 rule per job)
// is decoded once, into the next free slot, and stays resident (an
// unbounded cache: nothing is evicted, so later runs decode only blocks no
// earlier run needed).
//
//   flags   per block, in units of BATCH_UNIT consecutive blocks of one volume:
//           used by some job of its volume (new or resident) and, per job,
//           whether it may emit (2x2x2 hull rule), as bits, with counts per
//           unit and totals per group of a volume's or a job's units
//   lists   the new blocks, the resident used ones, and the list L of
//           (job, block) pairs in job-major, block-ascending order (= the
//           concatenated canonical orders): a wave per unit and list, whose
//           place is the sum of the totals and counts before it
//   decode  the new blocks into slots slot_base + rank; sign masks of every
//           used block for every job of its volume
//   count   count pass over L from the sign masks (Sec. 4.4), in the chunks of
//           xcd_chunks; totals per chunk and per XCD eighth
//   back    the emission over L (Sec. 4.5), chunk by chunk: a wave adds up the
//           totals before each of its chunks, a wave scan of the chunk's counts
//           gives its entries' offsets; per-job output offsets
//   done    the run's results to the host's copies
#include <stdint.h>

#include "batch.h"
#include "common.h"
#include "mc_device.h"
#include "mc_ntri.h"
#include "zfp_device.h"

namespace bcmc {
namespace {

constexpr int BT = 256;  // threads per workgroup

// Which volume / job an index belongs to: largest i with base[i] <= x.
__device__ __forceinline__ uint32_t find_base(const uint64_t *base, uint32_t n, uint64_t x) {
    uint32_t lo = 0, hi = n;  // base[lo] <= x < base[hi]
    while (hi - lo > 1) {
        uint32_t mid = (lo + hi) >> 1;
        if (base[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Sign mask of a decoded block for one isovalue: bit i = (sample i < iso),
// the inside test of the per-cell classification (Sec. 4.4).
__device__ __forceinline__ uint64_t sign_mask(const float *v, float iso) {
    uint64_t m = 0;
#pragma unroll
    for (int i = 0; i < 64; i++) m |= (uint64_t)(v[i] < iso ? 1u : 0u) << i;
    return m;
}

// Jobs per volume whose masks the decoder builds in registers.
constexpr int MASK_JOBS = 4;

// The masks of global block gb (block b of volume vol) for every job of its
// volume.
__device__ __forceinline__ void store_masks(const BatchParams &p, const BatchVol &vol, uint32_t b,
                                            const float *v) {
    for (uint32_t k = vol.job_lo; k < vol.job_hi; k++) {
        const uint32_t j = p.vol_jobs[k];
        p.jmask[p.job_jbase[j] + b] = sign_mask(v, p.job_iso[j]);
    }
}

// Clock stamp k, at the start of a phase (by workgroup 0).
__device__ __forceinline__ void stamp(const BatchParams &p, int k) {
    if (blockIdx.x == 0 && threadIdx.x == 0) p.phase_ts[k] = wall_clock64();
}

// ---- flags -------------------------------------------------------------------
// Per block, with its volume uniform over the workgroup's unit: the ranges of
// its 3x3x3 neighbourhood (indices clamped into the volume: a clamped
// neighbour is one already in the neighbourhood, so no load is conditional),
// whether some job of the volume uses it (Sec. 4.1 rule) and, per job, whether
// it may emit (2x2x2 hull of its octet).  A bit per block and per pair (word w
// of a unit from wave w), and the number of bits per unit.  Latency bound: a
// block per thread, 27 loads in flight each, and no workgroup waits for another
// (as phases of one persistent kernel between grid barriers, with a byte per
// pair, flags and lists took 300 us of the batch of 48 volumes x 4 isovalues,
// 2.7 M blocks; as two launches 98 + 18; units of 512 or 256 blocks: 101 + 29,
// 126 + 48).
constexpr int UNIT_WAVES = BATCH_UNIT / 64;
__global__ __launch_bounds__(BATCH_UNIT) void k_batch_flags(BatchParams p) {
    constexpr int JOBS = 32;   // jobs between two barriers
    __shared__ uint32_t s_n[JOBS][UNIT_WAVES], s_u[UNIT_WAVES];
    stamp(p, 0);
    stamp(p, 1);
    if (blockIdx.x == 0 && threadIdx.x == 0) p.ctr->grid_front = gridDim.x;
    if (blockIdx.x == 0 && threadIdx.x < 8) p.ctr->xcd[threadIdx.x].verts = 0;   // for the count pass
    const int w = (int)wave_id(), l = lane();
    for (uint32_t u = blockIdx.x; u < p.n_units; u += gridDim.x) {
        const uint32_t vi = find_base(p.vol_unit, p.n_vols, u);
        const BatchVol &vol = p.vols[vi];
        const Geom g = vol.g;
        const uint32_t k = u - (uint32_t)p.vol_unit[vi];   // the volume's k-th unit
        const uint32_t b0 = k * BATCH_UNIT + threadIdx.x, b = b0 < g.nb ? b0 : (uint32_t)g.nb - 1;
        const uint32_t r = b / g.nbx, bx = b - r * g.nbx, by = r % g.nby, bz = r / g.nby;
        uint32_t xs[3], ys[3], zs[3];
        xs[0] = bx ? bx - 1 : 0; xs[1] = bx; xs[2] = bx + 1 < g.nbx ? bx + 1 : bx;
        ys[0] = by ? by - 1 : 0; ys[1] = by; ys[2] = by + 1 < g.nby ? by + 1 : by;
        zs[0] = bz ? bz - 1 : 0; zs[1] = bz; zs[2] = bz + 1 < g.nbz ? bz + 1 : bz;
        float2 q[27];
#pragma unroll
        for (int t = 0; t < 27; t++)
            q[t] = vol.ranges[xs[t % 3] + g.nbx * ((uint64_t)ys[(t / 3) % 3] + (uint64_t)g.nby * zs[t / 9])];
        float LO = q[0].x, HI = q[0].y, PLO = q[13].x, PHI = q[13].y;
#pragma unroll
        for (int t = 1; t < 27; t++) {
            LO = fminf(LO, q[t].x);
            HI = fmaxf(HI, q[t].y);
        }
#pragma unroll
        for (int t = 14; t < 27; t++)
            if (t % 3 != 0 && (t / 3) % 3 != 0) {   // offsets in {0, 1}^3
                PLO = fminf(PLO, q[t].x);
                PHI = fmaxf(PHI, q[t].y);
            }
        float2 own = q[13];
        if (b0 >= g.nb) {   // past the volume: no isovalue lies in an empty range
            own = make_float2(INFINITY, -INFINITY);
            PLO = LO = INFINITY;
        }
        bool used = false;
        for (uint32_t t0 = vol.job_lo; t0 < vol.job_hi; t0 += JOBS) {
            const uint32_t nt = min((uint32_t)JOBS, vol.job_hi - t0);
            for (uint32_t t = 0; t < nt; t++) {
                const uint32_t j = p.vol_jobs[t0 + t];
                const float iso = p.job_iso[j];
                used = used || (own.x < iso && iso <= HI) || (LO < iso && iso <= own.y);
                const uint64_t m = __ballot(PLO < iso && iso <= PHI);
                if (l == 0) {
                    p.pair_bits[(p.job_unit[j] + k) * UNIT_WAVES + w] = m;
                    s_n[t][w] = (uint32_t)__popcll(m);
                }
            }
            __syncthreads();
            if (threadIdx.x < nt) {   // one atomic per unit and job
                const uint32_t j = p.vol_jobs[t0 + threadIdx.x];
                uint32_t n = 0;
                for (int i = 0; i < UNIT_WAVES; i++) n += s_n[threadIdx.x][i];
                p.pair_cnt[p.job_unit[j] + k] = n;
                if (n) atomicAdd(&p.job_tot[p.job_group[j] + k / BATCH_GROUP], (unsigned long long)n);
            }
            __syncthreads();   // s_n is rewritten
        }
        const int32_t sl = used ? p.I_slot[vol.gbase + b] : 0;
        const uint64_t nm = __ballot(used && sl < 0), rm = __ballot(used && sl >= 0);
        if (l == 0) {
            p.new_bits[(uint64_t)u * UNIT_WAVES + w] = nm;
            p.res_bits[(uint64_t)u * UNIT_WAVES + w] = rm;
            s_u[w] = (uint32_t)__popcll(nm) | (uint32_t)__popcll(rm) << 16;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t n = 0;
            for (int i = 0; i < UNIT_WAVES; i++) n += s_u[i];
            p.unit_cnt[u] = n;
            if (n)
                atomicAdd(&p.vol_tot[p.vol_group[vi] + k / BATCH_GROUP],
                          (unsigned long long)(n & 0xFFFFu) << 32 | (n >> 16));
        }
        __syncthreads();   // s_u is rewritten
    }
}

// ---- lists -------------------------------------------------------------------
// The bits of one unit as list entries first + bit, from list[o] on.
template <class Put>
__device__ __forceinline__ void list_unit(const uint64_t *__restrict__ words, uint64_t o, const Put &put) {
    constexpr int W = UNIT_WAVES;
    const uint64_t mine = lane() < W ? words[lane()] : 0ull;
#pragma unroll
    for (int i = 0; i < W; i++) {
        const uint64_t m = ((uint64_t)bcast((uint32_t)(mine >> 32), i) << 32) | bcast((uint32_t)mine, i);
        if ((m >> lane()) & 1u) put(o + mbcnt(m), 64u * i + (uint32_t)lane());
        o += (uint64_t)__popcll(m);
    }
}
// Sum of a[lo..hi) over the wave.
template <typename T, class Get>
__device__ __forceinline__ uint64_t wave_range_sum(const T *__restrict__ a, uint64_t lo, uint64_t hi, const Get &get) {
    uint64_t v = 0;
#pragma unroll 4
    for (uint64_t i = lo + lane(); i < hi; i += 64) v += get(a[i]);
    return wave_sum(v);
}

__global__ __launch_bounds__(BT) void k_batch_lists(BatchParams p) {
    stamp(p, 2);
    constexpr int W = UNIT_WAVES;
    auto all = [](uint64_t x) { return x; };
    if (blockIdx.x == 0 && wave_id() == 0) {   // the run's totals; the new blocks' slots
        const uint64_t tv = wave_range_sum(p.vol_tot, 0, p.n_groups, all),
                       tl = wave_range_sum(p.job_tot, 0, p.n_jgroups, all);
        if (lane() == 0) {
            const uint64_t n0 = p.ctr->n_slots, tn = tv >> 32;
            p.ctr->slot_base = n0;
            p.ctr->n_slots = n0 + tn;
            p.ctr->n_new = tn;
            p.ctr->n_res = tv & 0xFFFFFFFFull;
            p.ctr->n_list = tl;
        }
    }
    stamp(p, 3);
    const uint64_t waves = (uint64_t)gridDim.x * (BT / 64);
    for (uint64_t t = (uint64_t)blockIdx.x * (BT / 64) + wave_id(); t < p.n_units + p.n_junits; t += waves) {
        if (t < p.n_units) {
            const uint32_t n = p.unit_cnt[t];
            if (!n) continue;
            const uint32_t vi = find_base(p.vol_unit, p.n_vols, t);
            const uint64_t k = t - p.vol_unit[vi];   // the volume's k-th unit
            auto parts = [](uint32_t x) { return (uint64_t)(x & 0xFFFFu) << 32 | (x >> 16); };
            const uint64_t o = wave_range_sum(p.vol_tot, 0, p.vol_group[vi] + k / BATCH_GROUP, all) +
                               wave_range_sum(p.unit_cnt, t - k % BATCH_GROUP, t, parts);
            const uint32_t gb0 = (uint32_t)(p.vols[vi].gbase + k * BATCH_UNIT);
            if (n & 0xFFFFu)
                list_unit(p.new_bits + t * W, o >> 32, [&](uint64_t at, uint32_t i) { p.new_list[at] = gb0 + i; });
            if (n >> 16)
                list_unit(p.res_bits + t * W, o & 0xFFFFFFFFull, [&](uint64_t at, uint32_t i) { p.res_list[at] = gb0 + i; });
        } else {
            const uint64_t ju = t - p.n_units;
            if (!p.pair_cnt[ju]) continue;
            const uint32_t j = find_base(p.job_unit, p.n_jobs, ju);
            const uint64_t k = ju - p.job_unit[j];
            const uint64_t o = wave_range_sum(p.job_tot, 0, p.job_group[j] + k / BATCH_GROUP, all) +
                               wave_range_sum(p.pair_cnt, ju - k % BATCH_GROUP, ju, all);
            const uint32_t e0 = (uint32_t)(p.job_jbase[j] + k * BATCH_UNIT);
            list_unit(p.pair_bits + ju * W, o, [&](uint64_t at, uint32_t i) {
                p.list[at] = e0 + i;
                p.list_job[at] = j;
            });
        }
    }
}

// ---- decode kernel: phase 4 ---------------------------------------------------
// STAGED: every volume has rate p.uniform_rate <= STAGE_MAX_RATE and each
// wave stages its blocks' words in LDS before decoding (whole waves iterate
// together: the staging is a wave-wide copy).  Single precision is held to 4
// waves per SIMD (127 VGPRs): left to itself the compiler takes 136 and 3
// waves, 480 us against 437 for 48 volumes of 32^3..256^3.
template <bool F64, bool STAGED>
__global__ __launch_bounds__(BT, F64 ? 1 : 4) void k_batch_decode(BatchParams p) {
    stamp(p, 4);
    if (p.ctr->err) return;   // an earlier run failed: nothing to do
    const uint64_t gtid = blockIdx.x * (uint64_t)BT + threadIdx.x;
    if (gtid == 0) p.ctr->grid_decode = gridDim.x;
    const uint64_t gstride = (uint64_t)gridDim.x * BT;
    const uint64_t n_slots0 = p.ctr->slot_base;
    const uint64_t n_new = p.ctr->n_new;
    extern __shared__ uint64_t stage_lds[];
    const int urate = (int)p.uniform_rate;
    uint64_t *st = stage_lds + (threadIdx.x >> 6) * (STAGED ? stage_wave_words(urate, F64) : 0u);
    for (uint64_t i0 = gtid & ~63ull; i0 < n_new; i0 += gstride) {
        const uint64_t i = i0 + lane();
        bool valid = i < n_new;
        const uint32_t gb = valid ? p.new_list[i] : 0u;
        const BatchVol &vol = p.vols[find_base(p.vol_gbase, p.n_vols, gb)];
        const uint64_t slot = n_slots0 + i;
        if (valid && slot >= p.max_slots) {   // never expected: report, do not touch memory
            atomicOr(&p.ctr->err, ERR_INTERNAL);
            valid = false;
        }
        const uint32_t b = (uint32_t)(gb - vol.gbase);
        float v[64];
        if (STAGED) {
            stage_words_at(vol.stream + (uint64_t)b * urate, urate, valid, st);
            if (valid) decode_block_staged<F64>(st, urate, v);
            __builtin_amdgcn_wave_barrier();   // st is rewritten by the next round
        } else if (valid) {
            decode_block<F64>(vol.stream + (uint64_t)b * vol.rate, (int)vol.rate, v);
        }
        if (!valid) continue;
        // store the block, building the masks of the volume's first
        // MASK_JOBS jobs on the way
        const uint32_t nj = vol.job_hi - vol.job_lo;
        float iso[MASK_JOBS];
        uint32_t mw[MASK_JOBS][2];
#pragma unroll
        for (int t = 0; t < MASK_JOBS; t++) {
            iso[t] = (uint32_t)t < nj ? p.job_iso[p.vol_jobs[vol.job_lo + t]] : -INFINITY;
            mw[t][0] = mw[t][1] = 0u;
        }
        float4 *dst = reinterpret_cast<float4 *>(p.slots + slot * 64);
#pragma unroll
        for (int q = 0; q < 16; q++) {
            const float4 f = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
            dst[q] = f;
#pragma unroll
            for (int t = 0; t < MASK_JOBS; t++)
                mw[t][q >> 3] |= ((f.x < iso[t] ? 1u : 0u) | (f.y < iso[t] ? 2u : 0u) |
                                  (f.z < iso[t] ? 4u : 0u) | (f.w < iso[t] ? 8u : 0u)) << (4 * (q & 7));
        }
        p.I_slot[gb] = (int32_t)slot;
#pragma unroll
        for (int t = 0; t < MASK_JOBS; t++)
            if ((uint32_t)t < nj)
                p.jmask[p.job_jbase[p.vol_jobs[vol.job_lo + t]] + b] = (uint64_t)mw[t][1] << 32 | mw[t][0];
    }
    if (p.max_vol_jobs > MASK_JOBS) {
        // the remaining jobs' masks; lane i reads back the block it stored above
        for (uint64_t i = gtid; i < n_new; i += gstride) {
            const uint32_t gb = p.new_list[i];
            const BatchVol &vol = p.vols[find_base(p.vol_gbase, p.n_vols, gb)];
            const uint64_t slot = n_slots0 + i;
            if (vol.job_hi - vol.job_lo <= MASK_JOBS || slot >= p.max_slots) continue;
            const float4 *src = reinterpret_cast<const float4 *>(p.slots + slot * 64);
            float w[64];
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const float4 t4 = src[q];
                w[4 * q] = t4.x;
                w[4 * q + 1] = t4.y;
                w[4 * q + 2] = t4.z;
                w[4 * q + 3] = t4.w;
            }
            const uint32_t b = (uint32_t)(gb - vol.gbase);
            for (uint32_t k = vol.job_lo + MASK_JOBS; k < vol.job_hi; k++) {
                const uint32_t j = p.vol_jobs[k];
                p.jmask[p.job_jbase[j] + b] = sign_mask(w, p.job_iso[j]);
            }
        }
    }
    const uint64_t n_res = p.ctr->n_res;
    for (uint64_t i = gtid; i < n_res; i += gstride) {
        const uint32_t gb = p.res_list[i];
        const BatchVol &vol = p.vols[find_base(p.vol_gbase, p.n_vols, gb)];
        const float4 *src = reinterpret_cast<const float4 *>(p.slots) + (uint64_t)p.I_slot[gb] * 16;
        float v[64];
#pragma unroll
        for (int q = 0; q < 16; q++) {
            const float4 t = src[q];
            v[4 * q] = t.x;
            v[4 * q + 1] = t.y;
            v[4 * q + 2] = t.z;
            v[4 * q + 3] = t.w;
        }
        store_masks(p, vol, (uint32_t)(gb - vol.gbase), v);
    }
}

// ---- count kernel ---------------------------------------------------------------
// One lane per (job, block) pair of L, over the chunks that the emission uses:
// the cases of the block's 64 cells from the sign masks of its octet, the
// triangle count per case by the bit-sliced table circuit (Sec. 4.4).
__global__ __launch_bounds__(BT) void k_batch_count(BatchParams p) {
    __shared__ uint64_t s_v[MC_WAVES];
    const int l = lane();
    stamp(p, 5);
    // the totals have been read (lists): cleared for the next run
    if (blockIdx.x == 0) {
        for (uint64_t i = threadIdx.x; i < p.n_groups; i += BT) p.vol_tot[i] = 0;
        for (uint64_t i = threadIdx.x; i < p.n_jgroups; i += BT) p.job_tot[i] = 0;
    }
    if (p.ctr->err) return;   // an earlier kernel failed: nothing to do
    const uint64_t n_list = uniform64(p.ctr->n_list);
    const uint32_t cs = mc_chunk_size(n_list, gridDim.x * MC_WAVES);
    const ChunkRange cr = xcd_chunks((n_list + cs - 1) / cs);
    uint64_t verts = 0;
    for (uint64_t k = cr.first; k < cr.end; k += cr.stride) {
        const uint64_t idx = k * cs + l;
        uint32_t c = 0;
        if (l < (int)cs && idx < n_list) {
            const uint32_t j = p.list_job[idx];
            const uint64_t jb = p.job_jbase[j];
            const BatchVol &vol = p.vols[p.job_vol[j]];
            const uint32_t b = (uint32_t)(p.list[idx] - jb);
            uint32_t so[8], bx, by, bz;
            octet(vol.g, b, nullptr, 1, so, bx, by, bz);
            uint64_t M[8], cm[8];
#pragma unroll
            for (int m = 0; m < 8; m++) M[m] = p.jmask[jb + so[m]];
            corner_masks(M, cm);
            uint64_t n0, n1, n2;
            mc_ntri_bits(cm, n0, n1, n2);
            const uint64_t V = valid_cells(vol.g, bx, by, bz);
            c = 3u * ((uint32_t)__popcll(n0 & V) + 2u * (uint32_t)__popcll(n1 & V) +
                      4u * (uint32_t)__popcll(n2 & V));
            p.cnt[idx] = c;
        }
        c = wave_sum(c);
        if (l == 0) p.chunk_tot[k] = c;
        verts += c;
    }
    if (l == 0) s_v[wave_id()] = verts;
    __syncthreads();
    if (threadIdx.x == 0) {
        verts = 0;
        for (int k = 0; k < MC_WAVES; k++) verts += s_v[k];
        if (verts) atomicAdd(&p.ctr->xcd[blockIdx.x % 8u].verts, (unsigned long long)verts);
    }
}

// ---- back kernel ----------------------------------------------------
struct BackShared {
    EmitShared emit;
    uint64_t tab[256];   // the triangle table (per-lane lookups at LDS latency)
};

template <int SB>
__global__ __launch_bounds__(BT) void k_batch_back(BatchParams p) {
    __shared__ BackShared sh;
    const int l = lane(), w = (int)wave_id();
    stamp(p, 6);
    if (p.ctr->err) return;   // an earlier kernel failed: nothing to do
    const uint64_t n_list = uniform64(p.ctr->n_list);
    const uint32_t cs = mc_chunk_size(n_list, gridDim.x * MC_WAVES);   // the count pass's chunks
    const ChunkRange cr = xcd_chunks((n_list + cs - 1) / cs);
    for (int i = threadIdx.x; i < 256; i += BT) sh.tab[i] = p.mc_table[i];
    if (threadIdx.x < 16) sh.emit.edge[threadIdx.x] = edge_entry((int)threadIdx.x);
    __syncthreads();
    uint64_t base = 0, total = 0;
    for (uint32_t x = 0; x < 8; x++) {
        const uint64_t tx = p.ctr->xcd[x].verts;
        base += x < blockIdx.x % 8u ? tx : 0ull;
        total += tx;
    }
    base = uniform64(base);
    total = uniform64(total);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        p.ctr->total_verts = total;
        p.ctr->grid_back = gridDim.x;
    }
    if (cr.first < cr.end) base += chunks_sum(p.chunk_tot, cr.lo, cr.first);
    stamp(p, 7);

    // emission (Sec. 4.5) and the jobs' output offsets
    if (n_list == 0 && blockIdx.x == 0)
        for (uint32_t j = threadIdx.x; j <= p.n_jobs; j += BT) p.job_off[j] = 0;
    const LaneGeom q = lane_geom();
    for (uint64_t k = cr.first; k < cr.end; k += cr.stride) {
        const uint64_t idx = k * cs + l;
        const bool valid = l < (int)cs && idx < n_list;
        const uint32_t c = valid ? p.cnt[idx] : 0u;
        const uint32_t incl = wave_incl_scan(c);
        const uint64_t off = base + incl - c;
        uint32_t j = 0;
        if (valid) {
            j = p.list_job[idx];
            // first entry of its job: it starts the soups of the jobs since the
            // previous entry's job (jobs with no entry have empty soups)
            const uint32_t jp = idx ? p.list_job[idx - 1] : 0u;
            if (idx == 0 || jp != j)
                for (uint32_t k = idx ? jp + 1 : 0u; k <= j; k++) p.job_off[k] = off;
            if (idx + 1 == n_list)
                for (uint32_t k = j + 1; k <= p.n_jobs; k++) p.job_off[k] = total;
        }
        const BatchVol &vol = p.vols[p.job_vol[j]];
        const float liso = p.job_iso[j];
        const uint32_t b = c ? (uint32_t)(p.list[idx] - p.job_jbase[j]) : 0u;
        uint32_t so[8], lbx, lby, lbz;
        octet(vol.g, b, p.I_slot + vol.gbase, 0, so, lbx, lby, lbz);
        uint64_t todo = __ballot(c != 0);
        while (todo) {
            const uint64_t left = todo;
            int jl[SB], nsb = 0;
#pragma unroll
            for (int k = 0; k < SB; k++) {
                jl[k] = k ? jl[0] : 0;
                if (todo) {
                    jl[k] = (int)__builtin_ctzll(todo);
                    todo &= todo - 1;
                    nsb++;
                }
            }
            // the triangle list area is empty between batches (emit_batch flushes)
            static_assert(8 * SB <= EMIT_TRIS, "slot table fits the triangle list");
            stage_batch_tab<SB>(q, p.slots, so, left & ~todo, nsb, sh.emit.tri[w], sh.emit.tiles[w]);
            wave_lds_sync();
            // consecutive entries of L with triangles: adjacent vertex ranges
            const uint64_t ob = ((uint64_t)bcast((uint32_t)(off >> 32), jl[0]) << 32) |
                                bcast((uint32_t)off, jl[0]);
            auto info = [&](int k, Geom &gk, uint32_t &bk, uint32_t &bx, uint32_t &by, uint32_t &bz,
                            float &isok) {
                gk.nx = bcast(vol.g.nx, jl[k]);
                gk.ny = bcast(vol.g.ny, jl[k]);
                gk.nz = bcast(vol.g.nz, jl[k]);
                bk = bcast(b, jl[k]);
                bx = bcast(lbx, jl[k]);
                by = bcast(lby, jl[k]);
                bz = bcast(lbz, jl[k]);
                isok = __uint_as_float(bcast(__float_as_uint(liso), jl[k]));
            };
            emit_batch<VFMT_F32>(nsb, info, sh.emit.tiles[w], sh.tab, sh.emit, w, ob, p.out, p.cap);
        }
        if (k + cr.stride < cr.end) base += chunks_sum(p.chunk_tot, k, k + cr.stride);
    }
}

// The run's results into the host's copies (pinned memory).
__global__ __launch_bounds__(BT) void k_batch_done(BatchParams p) {
    const uint64_t now = wall_clock64();
    const uint32_t *c = reinterpret_cast<const uint32_t *>(p.ctr);
    for (uint32_t i = threadIdx.x; i < sizeof(BatchCounters) / 4; i += BT) reinterpret_cast<uint32_t *>(p.h_ctr)[i] = c[i];
    for (uint32_t i = threadIdx.x; i <= p.n_jobs; i += BT) p.h_job_off[i] = p.job_off[i];
    if (threadIdx.x < 8) p.h_ts[threadIdx.x] = p.phase_ts[threadIdx.x];
    if (threadIdx.x == 8) p.h_ts[8] = now;
}

const void *decode_kernel(int is_f64, int staged) {
    if (is_f64)
        return staged ? (const void *)k_batch_decode<true, true> : (const void *)k_batch_decode<true, false>;
    return staged ? (const void *)k_batch_decode<false, true> : (const void *)k_batch_decode<false, false>;
}

unsigned decode_lds(const BatchParams &p, int is_f64) {
    return p.uniform_rate ? stage_lds_bytes((int)p.uniform_rate, is_f64 != 0) : 0u;
}

}  // namespace

int batch_front_per_cu(int *per_cu) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_lists, BT, 0) != hipSuccess) return -1;
    *per_cu = n;
    return 0;
}


int batch_decode_per_cu(const BatchParams &p, int is_f64, int *per_cu) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, decode_kernel(is_f64, p.uniform_rate != 0), BT,
                                                     decode_lds(p, is_f64)) != hipSuccess)
        return -1;
    *per_cu = n;
    return 0;
}

int batch_back_per_cu(int sb, int *per_cu) {
    int n = 0;
    hipError_t e = sb == 4 ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_back<4>, BT, 0)
                           : hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_back<8>, BT, 0);
    if (e != hipSuccess) return -1;
    *per_cu = n;
    return 0;
}

hipError_t launch_batch(const BatchParams &p, int is_f64, int sb, const unsigned grids[3], hipStream_t s) {
    void *args[] = {const_cast<BatchParams *>(&p)};
    const void *back = sb == 4 ? (const void *)k_batch_back<4> : (const void *)k_batch_back<8>;
    // count and back share one grid: they partition L the same way
    const struct {
        const void *kernel;
        unsigned grid, threads, lds;
    } steps[] = {{(const void *)k_batch_flags, grids[0], BATCH_UNIT, 0},
                 {(const void *)k_batch_lists, grids[0], BT, 0},
                 {decode_kernel(is_f64, p.uniform_rate != 0), grids[1], BT, decode_lds(p, is_f64)},
                 {(const void *)k_batch_count, grids[2], BT, 0},
                 {back, grids[2], BT, 0},
                 {(const void *)k_batch_done, 1, BT, 0}};
    for (const auto &k : steps)
        if (hipError_t e = hipLaunchKernel(k.kernel, dim3(k.grid), dim3(k.threads), args, k.lds, s)) return e;
    return hipSuccess;
}

}  // namespace bcmc
