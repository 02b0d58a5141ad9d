// Internal definitions shared by the HIP sources of libbcmc (not part of the
// C ABI).  gfx950 only: wave64, one process per GPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <string>

namespace bcmc {

// ---- constants ----------------------------------------------------------
constexpr uint32_t HIGH_AGE = 0x80000000u;  // age of a slot created empty
// Tag of a sign mask built for no isovalue: a NaN pattern (isovalues are
// never NaN, so no call's tag equals it).
constexpr uint32_t MASK_NONE = 0x7FC00001u;
constexpr int BLK_TILE = 4096;               // blocks per round of the compaction
// Volumes of more than 2048 rounds (8.4 M blocks) have the rounds' counts
// summed in two levels, the first by a launch of its own (4.5 us, where every
// workgroup would read up to 460 KB of counts at 236 M blocks); below, each
// workgroup's own sum takes 1-2 us.
constexpr uint64_t ROUNDS_DIRECT = 2048;
// Tiles from which the cull takes the live ones from a queue: at 1800 (3.7 M
// blocks) the cull alone takes less than the queue's launch more, while the
// 115,200 of 236 M blocks, a tenth of them live, would mostly be dead workgroups.
constexpr uint64_t CULL_DIRECT = 4096;
constexpr int EVICT_TILE = 1024;             // slots per tile of the eviction's selection (256 per wave)
constexpr int EVICT_BITS = 10;               // key bits per pass of it
constexpr int EVICT_BINS = 1 << EVICT_BITS;
constexpr uint32_t EVICT_REFRESH = 512;      // key span from which its base is looked for again
constexpr int MC_MAX_GRID = 2048;           // workgroups of the count / emission grid at most
constexpr int MC_WAVES = 4;                  // blocks (one per wave) per MC tile

enum : uint32_t { ERR_CACHE_CAP = 1u, ERR_NONFINITE = 2u, ERR_INTERNAL = 4u };

// Device-resident scalars of one extract call.  Written only by kernels of
// that call (zeroed by the call before), read back once by the host at its
// end.
struct Counters {
    unsigned long long n_act;        // active blocks
    unsigned long long n_new;        // active blocks not in the cache
    unsigned long long n_slots;      // slots of the cache (after growth)
    unsigned long long n_used;       // slots taken into use: [0, n_used) (after this call)
    unsigned long long n_evicted;    // blocks evicted this call
    unsigned long long n_occ;        // active blocks that emit triangles
    unsigned long long n_cand;       // active blocks that may emit (staged by the count pass)
    unsigned long long total_verts;  // 3 * triangles
    unsigned int err;                // ERR_* bits
    unsigned int span;               // 1 + calls since the oldest used slot's last use, at most (0: not looked for)
    unsigned int n_sort;             // available used slots (with n_evicted)
    unsigned int n_retry;            // blocks the low-rate decoder handed back
    unsigned int cull_live, cull_stale;  // the cull's queued tiles
    unsigned int pad;
    // per XCD eighth of the chunks (xcd_chunks), a cache line each: vertices
    // and occupied blocks.  Not read back.
    struct alignas(128) Xcd {
        unsigned long long verts, occ;
    } xcd[8];
};
constexpr size_t CTR_READ = offsetof(Counters, xcd);   // what the host reads
// The host's copy of a call's counters (pinned memory the device writes):
// valid for the call whose number seq holds.
struct HostCounters {
    unsigned char c[CTR_READ];
    uint32_t seq;
};
// Double-precision streams up to this rate decode with the low-rate decoder
// (and a general pass over the blocks it hands back).
constexpr uint32_t LOW_RATE_MAX = 4;


// The cache as a call finds it (host mirror).
struct SlotState {
    uint64_t n_slots, n_used, max_slots;
    int identity;   // every block resident, no slots
};

// Geometry of a volume in blocks.
struct Geom {
    uint32_t nx, ny, nz;
    uint32_t nbx, nby, nbz;
    uint64_t nb;
};

// Device buffers of a volume (all owned by the volume).
struct DevState {
    uint64_t *stream = nullptr;     // fixed-rate ZFP words, block b at b*rate
    float2 *ranges = nullptr;       // per block (min, max) of decoded valid samples
    float2 *tile_ranges = nullptr;  // per cull tile: hull of its blocks' and halo's ranges
    uint32_t *cull_list = nullptr;  // 2 x cull tiles: the call's live tiles, then its stale ones
    uint8_t *active = nullptr;      // M_active
    uint32_t *I_active = nullptr;   // ascending active block ids
    uint32_t *I_new = nullptr;      // ascending new block ids
    uint32_t *retry = nullptr;      // low-rate f64 decode: indices into I_new handed back
    int32_t *I_slot = nullptr;      // per block: slot or -1
    // cache (max_slots entries)
    int32_t *S_block = nullptr;
    uint32_t *S_stamp = nullptr;    // call that last used the slot (unused: that created it), 0: the reset
    float *slots = nullptr;         // [max_slots][64] decoded blocks
    uint64_t *masks = nullptr;      // [max_slots] per slot: bit i = sample i below iso
    uint32_t *mask_iso = nullptr;   // [max_slots] bits of the isovalue masks[] was built for
                                    // (MASK_NONE: none)
    uint32_t *evict[2] = {nullptr, nullptr};     // slots to evict, oldest first (two for passes)
    uint32_t *evict_hist = nullptr;              // EVICT_BINS per EVICT_TILE slots
    uint32_t *evict_tot = nullptr;               // EVICT_BINS
    // MC
    uint32_t *blk_cnt = nullptr;    // per active block vertex count
    uint64_t *blk_off = nullptr;    // per active block first vertex
    uint64_t *round_cnt = nullptr;  // per 4096-block round: counts of its blocks (round_pack)
    uint64_t *round_next = nullptr; // the next call's, zeroed by this one
    uint64_t *round_sums = nullptr; // more than ROUNDS_DIRECT rounds: sums of 256 of them
    uint32_t *chunk_tot = nullptr;  // vertices of each chunk of the active list (mc_chunk_slots entries)
    float *part_giso = nullptr;     // [4 * max MC grid] per-wave dL/diso of the backward
    Counters *ctr = nullptr;
    Counters *ctr_next = nullptr;   // the next call's, zeroed by this one
    uint64_t *mc_table = nullptr;   // 256 packed cases
};

// ---- launchers (extract.hip) -------------------------------------------
// prev_iso: the previous cull's isovalue; rewrite: the flags hold anything
// (new ranges).  now: the call's number since the cache was reset (slots'
// stamps).
void launch_cull(const Geom &g, const DevState &d, float iso, float prev_iso, int rewrite, int identity_cache,
                 uint32_t now, hipStream_t s);
// base, now: the stamps' range, as launch_evict.
void launch_compact_blocks(const Geom &g, const DevState &d, const SlotState &ss, uint32_t base, uint32_t now,
                           hipStream_t s);
inline uint64_t block_rounds(uint64_t nb) { return (nb + BLK_TILE - 1) / BLK_TILE; }
// Entries of the count pass's chunk totals: a call
// with n_act active blocks on W waves has ceil(n_act / cs) chunks of
// cs = min(64, ceil(n_act / W)) blocks (mc_chunk_size), at most
// max(ceil(nb / 64), W).
inline uint64_t mc_chunk_slots(uint64_t nb) {
    const uint64_t a = (nb + 63) / 64, b = 4ull * MC_MAX_GRID;
    return a > b ? a : b;
}
// The slots to evict, oldest first (n_evicted entries of the returned list),
// among [0, n_used); base: a call number no used slot's stamp is below.
// After launch_compact_blocks, which counts for the first pass.
uint32_t *launch_evict(const Geom &g, const DevState &d, uint32_t n_used, uint32_t base, uint32_t now,
                       hipStream_t s);
// Every block out of the cache; the slots from n_used on hold none.
void launch_cache_empty(const DevState &d, uint64_t n_used, hipStream_t s);
void launch_mc_count(const Geom &g, const DevState &d, const float *slots, const int32_t *I_slot,
                     int identity_cache, float iso, int fmt, hipStream_t s);

void launch_mc_emit(const Geom &g, const DevState &d, const float *slots, const int32_t *I_slot,
                    int identity_cache, float iso, void *out, uint64_t cap_verts, int fmt,
                    hipStream_t s);
// fmt: the bcmc_vertex_format codes (0 = 16-byte vertex, 1 = edge record,
// 2 = 10-bit quantised vertex).
void launch_vertices_q10(const void *in, uint64_t n, void *out, hipStream_t s);
void launch_debug_cases(const Geom &g, const DevState &d, const float *slots,
                        const int32_t *I_slot, int identity_cache, float iso, uint8_t *cases,
                        uint64_t max_act, hipStream_t s);
void launch_backward(const Geom &g, const DevState &d, const float *slots, float iso,
                     const float *gV, uint64_t n_verts, float *dfield, float *diso, int fmt,
                     hipStream_t s);
// Writes the counters, then value as host->seq, when s gets there.
void launch_publish(const void *ctr, HostCounters *host, uint32_t value, hipStream_t s);
void launch_fill_u32(uint32_t *p, uint32_t v, uint64_t n, hipStream_t s);
void launch_copy_calibration(void *dst, const void *src, uint64_t n16, hipStream_t s);
void launch_iota_i32(int32_t *p, uint64_t n, hipStream_t s);

// ---- launchers (dense.hip): dense marching cubes baseline ---------------
struct DenseCounters {
    unsigned long long n_active, n_verts;
    struct alignas(128) Xcd {   // per XCD eighth of the chunks, a cache line each
        unsigned long long verts, cells;
    } xcd[8];
};
static_assert(sizeof(DenseCounters) >= CTR_READ, "read back like an extract's counters");
uint64_t dense_sign_words(uint32_t nx, uint32_t ny, uint32_t nz);
uint64_t dense_chunk_words(uint32_t nx, uint32_t ny, uint32_t nz);
void launch_dense(uint32_t nx, uint32_t ny, uint32_t nz, const float *field, float iso, uint64_t *bits,
                  uint32_t *chunk_tot, DenseCounters *ctr, const uint64_t *mc_table, void *out, uint64_t cap,
                  hipStream_t s);

// ---- launchers (zfp.hip) -----------------------------------------------
void launch_decode_ranges(const Geom &g, const uint64_t *stream, int is_f64, uint32_t rate,
                          float2 *ranges, float *blocks_out, unsigned int *err, hipStream_t s);
// Hull of the ranges over each cull tile and its one-block halo (after every
// change of the ranges).
uint64_t cull_tiles(const Geom &g);
void launch_tile_ranges(const Geom &g, const float2 *ranges, float2 *tile_ranges, hipStream_t s);
void launch_ranges_from_blocks(const Geom &g, const float *blocks, float2 *ranges,
                               unsigned int *err, hipStream_t s);
// evict: launch_evict's list; ss, now: as the call began.
void launch_assign_decode(const DevState &d, int is_f64, uint32_t rate, uint64_t max_new, float iso,
                          const uint32_t *evict, const SlotState &ss, uint32_t now, hipStream_t s);
void launch_encode(const Geom &g, const void *field, int is_f64, uint32_t rate,
                   uint64_t *stream, unsigned int *err, hipStream_t s);

// ---- host-side tables (tables.cpp) --------------------------------------
// Packed marching cubes table: bits 4k..4k+3 = k-th edge id (15 = unused),
// bits 60..63 = number of triangles.
const uint64_t *mc_table_host();
int mc_table_status();  // 0 when the generator succeeded

// ---- error reporting (capi.cpp) -----------------------------------------
void set_error(const std::string &msg);

}  // namespace bcmc

#define BCMC_HIP_TRY(expr)                                                  \
    do {                                                                    \
        hipError_t e_ = (expr);                                             \
        if (e_ != hipSuccess) {                                             \
            bcmc::set_error(std::string(#expr) + ": " + hipGetErrorString(e_)); \
            return BCMC_E_HIP;                                              \
        }                                                                   \
    } while (0)
