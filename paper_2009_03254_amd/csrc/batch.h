// Device-side description of a batch (volumes x isovalues) for the batched
// extraction kernels.
#pragma once

#include <stdint.h>

#include "common.h"

namespace bcmc {

struct BatchVol {
    Geom g;
    const uint64_t *stream;   // fixed-rate ZFP words of the volume
    const float2 *ranges;     // its block ranges
    uint32_t rate;
    uint32_t job_lo, job_hi;  // its jobs: vol_jobs[job_lo .. job_hi)
    uint64_t gbase;           // first global block id of the volume
};

struct BatchCounters {
    unsigned long long n_slots;      // decoded blocks resident (persists across runs)
    unsigned long long n_new;        // blocks decoded by this run
    unsigned long long n_res;        // used blocks that were resident
    unsigned long long n_list;       // (job, block) pairs that may emit
    unsigned long long total_verts;
    unsigned long long slot_base;    // first slot of this run's new blocks
    unsigned int err;
    unsigned int grid_front, grid_decode, grid_back;   // grids the kernels ran with
    unsigned int pad[2];
    struct alignas(128) Xcd {        // vertices per XCD eighth of the chunks, a cache line each
        unsigned long long verts;
    } xcd[8];
};

// Blocks of one volume that a workgroup of the flags kernel takes at a time.
constexpr int BATCH_UNIT = 1024;
// Units of one volume whose counts have a total: a unit's place in the lists is
// the sum of the totals before its group and of the counts before it in the
// group.  With one total per volume every unit's wave added up all the volume's
// units before it: 0.89 ms of lists for 59 M blocks and 2 isovalues (57,600
// units), growing with the square of the volume, against 0.20 with groups; one
// group holds volumes of up to 524,288 blocks, whose lists take what they took.
constexpr int BATCH_GROUP = 512;

struct BatchParams {
    const BatchVol *vols;
    uint32_t n_vols, n_jobs;
    const uint64_t *vol_gbase;   // [n_vols]
    const uint32_t *vol_jobs;    // jobs grouped by volume
    const uint32_t *job_vol;     // [n_jobs]
    const uint64_t *job_jbase;   // [n_jobs] first (job, block) index of each job
    const float *job_iso;        // [n_jobs] (device, so a captured graph follows updates)
    uint64_t n_gblocks, n_jblocks, max_slots;
    uint32_t uniform_rate;       // the rate of every volume when they share one <= 16, else 0
    uint32_t max_vol_jobs;       // most jobs of one volume
    uint64_t n_units, n_junits;  // units of all volumes, of all jobs' volumes
    const uint64_t *vol_unit;    // [n_vols] first unit of each volume
    const uint64_t *job_unit;    // [n_jobs] first unit of each job among the jobs' units
    uint64_t n_groups, n_jgroups;  // groups of units of all volumes, of all jobs' volumes
    const uint64_t *vol_group;   // [n_vols] first group of each volume
    const uint64_t *job_group;   // [n_jobs] first group of each job among the jobs' groups
    int32_t *I_slot;             // [n_gblocks] slot of each global block or -1
    float *slots;                // [max_slots][64]
    uint64_t *new_bits;          // [n_units][BATCH_UNIT / 64] used and new
    uint64_t *res_bits;          // [n_units][BATCH_UNIT / 64] used and resident
    uint64_t *pair_bits;         // [n_junits][BATCH_UNIT / 64] may emit
    uint32_t *unit_cnt;          // [n_units] new | resident << 16
    uint32_t *pair_cnt;          // [n_junits] may emit
    unsigned long long *vol_tot; // [n_groups] new << 32 | resident (zero between runs)
    unsigned long long *job_tot; // [n_jgroups] may emit (zero between runs)
    uint64_t *jmask;             // [n_jblocks] sign masks of the used blocks per job
    uint32_t *new_list;          // [n_gblocks]
    uint32_t *res_list;          // [n_gblocks]
    uint32_t *list;              // [n_jblocks] (job-major, block-ascending)
    uint32_t *list_job;          // [n_jblocks] job of each list entry
    uint32_t *cnt;               // [n_jblocks] vertex count of each list entry
    uint32_t *chunk_tot;         // [mc_chunk_slots(n_jblocks)] vertices of each chunk of the list
    uint64_t *job_off;           // [n_jobs + 1] vertex offsets of the jobs' soups
    const uint64_t *mc_table;
    void *out;
    uint64_t cap;
    BatchCounters *ctr;
    unsigned long long *phase_ts;  // [8] real-time clock at the phases' starts
    // the host's copies (pinned)
    BatchCounters *h_ctr;
    uint64_t *h_job_off;
    unsigned long long *h_ts;      // [9]
};

// Resident workgroups per CU of the lists kernel, the decode kernel (decode
// and sign masks) and the back kernel (`sb` blocks staged per wave round trip).
int batch_front_per_cu(int *per_cu);
int batch_decode_per_cu(const BatchParams &p, int is_f64, int *per_cu);
int batch_back_per_cu(int sb, int *per_cu);
// Launches the run's kernels: flags and lists on grids[0] workgroups, decode
// on grids[1], count and back on grids[2].
hipError_t launch_batch(const BatchParams &p, int is_f64, int sb, const unsigned grids[3], hipStream_t s);

}  // namespace bcmc
