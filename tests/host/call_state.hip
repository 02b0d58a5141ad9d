// The host side of the calls (capi.cpp, batch_api.cpp) on a pretended device:
// device memory is host memory, the launchers below do with it what the kernels
// do (one slot per new block, counts from zero), and the HIP calls can be made
// to fail.  Checks what the next calls find after one that failed.  Prints a
// line and exits 1 at the first thing that does not hold.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <string>
#include <vector>

#include "../../include/bcmc.h"
#include "../../paper_2009_03254_amd/csrc/batch.h"
#include "../../paper_2009_03254_amd/csrc/common.h"

#define CHECK(x)                                                        \
    do {                                                                \
        if (!(x)) {                                                     \
            printf("line %d: %s does not hold\n", __LINE__, #x);        \
            exit(1);                                                    \
        }                                                               \
    } while (0)

// ---- what is made to fail -------------------------------------------------
static bool lost = false;            // kernels are enqueued but never run, waits fail
static bool readback_fails = false;  // kernels run, the wait for the counters fails
static bool launch_fails = false;    // hipGetLastError after the launches
static bool capturing = false;       // the stream records: kernels do not run, waits fail
static size_t malloc_limit = ~(size_t)0;
static int launches = 0;             // kernels enqueued
static int unwaited = 0;             // ... since the last synchronisation
static std::vector<uint32_t> active_now;   // the blocks the next call finds active

// ---- HIP --------------------------------------------------------------------
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    *p = n > malloc_limit ? nullptr : calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = aligned_alloc(128, (n + 127) / 128 * 128); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) {
    *c = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return lost || readback_fails || capturing ? hipErrorLaunchFailure : hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { unwaited = 0; return lost || readback_fails || capturing ? hipErrorLaunchFailure : hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return launch_fails ? hipErrorLaunchFailure : hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 8; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return capturing ? hipErrorCapturedEvent : hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

// ---- the kernels --------------------------------------------------------------
namespace bcmc {
template <typename T>
static bool all_zero(const T *p, uint64_t n) {
    for (uint64_t i = 0; i < n * sizeof(T); i++)
        if (reinterpret_cast<const unsigned char *>(p)[i]) return false;
    return true;
}
static bool enqueue() { launches++, unwaited++; return !lost && !capturing; }   // does the kernel run?

uint64_t cull_tiles(const Geom &) { return 1; }
static int last_rewrite = -1;
static float last_prev = 0;
void launch_cull(const Geom &g, const DevState &d, float, float prev_iso, int rewrite, int identity, uint32_t now,
                 hipStream_t) {
    last_rewrite = rewrite;
    last_prev = prev_iso;
    if (!enqueue()) return;
    CHECK(all_zero(d.ctr, 1));                              // a call counts from zero
    CHECK(all_zero(d.round_cnt, block_rounds(g.nb)));
    for (uint32_t b : active_now) {
        d.round_cnt[b / BLK_TILE]++;
        if (!identity && d.I_slot[b] >= 0) d.S_stamp[d.I_slot[b]] = now;
    }
}
void launch_compact_blocks(const Geom &g, const DevState &d, const SlotState &ss, uint32_t, uint32_t, hipStream_t) {
    if (!enqueue()) return;
    memset(d.ctr_next, 0, sizeof(Counters));
    memset(d.round_next, 0, 8 * block_rounds(g.nb));
    uint64_t n_new = 0;
    for (uint32_t b : active_now)
        if (!ss.identity && d.I_slot[b] < 0) d.I_new[n_new++] = b;
    d.ctr->n_act = active_now.size();
    d.ctr->n_new = n_new;
    d.ctr->n_used = ss.n_used + n_new;
    d.ctr->n_slots = std::max(ss.n_slots, ss.n_used + n_new);
    if (!ss.identity && d.ctr->n_slots > ss.max_slots) d.ctr->err |= ERR_CACHE_CAP;
}
uint32_t *launch_evict(const Geom &, const DevState &d, uint32_t, uint32_t, uint32_t, hipStream_t) {
    enqueue();
    return d.evict[0];
}
void launch_assign_decode(const DevState &d, int, uint32_t, uint64_t, float, const uint32_t *, const SlotState &ss,
                          uint32_t now, hipStream_t) {
    if (!enqueue() || d.ctr->err) return;
    for (uint64_t i = 0; i < d.ctr->n_new; i++) {
        const uint64_t s = ss.n_used + i;
        CHECK(d.S_block[s] < 0);   // the slots past the used ones hold no block
        d.S_block[s] = (int32_t)d.I_new[i];
        d.I_slot[d.I_new[i]] = (int32_t)s;
        d.S_stamp[s] = now;
    }
}
void launch_mc_count(const Geom &, const DevState &d, const float *, const int32_t *, int, float, int, hipStream_t) {
    if (enqueue() && !d.ctr->err) d.ctr->xcd[0].verts += 3 * d.ctr->n_act;
}
void launch_mc_emit(const Geom &, const DevState &d, const float *, const int32_t *, int, float, void *, uint64_t, int,
                    hipStream_t) {
    if (enqueue() && !d.ctr->err) d.ctr->total_verts = d.ctr->xcd[0].verts;
}
void launch_publish(const void *ctr, HostCounters *host, uint32_t value, hipStream_t) {
    if (!enqueue() || readback_fails) return;
    memcpy(host->c, ctr, CTR_READ);
    host->seq = value;
}
void launch_cache_empty(const DevState &d, uint64_t n_used, hipStream_t) {
    if (!enqueue()) return;
    for (uint64_t s = 0; s < n_used; s++) {
        CHECK(d.S_block);
        if (d.S_block[s] >= 0) d.I_slot[d.S_block[s]] = -1;
        d.S_block[s] = -1;
        d.S_stamp[s] = 0;
    }
}
void launch_fill_u32(uint32_t *p, uint32_t v, uint64_t n, hipStream_t) {
    if (!enqueue()) return;
    CHECK(p || !n);
    for (uint64_t i = 0; i < n; i++) p[i] = v;
}
void launch_backward(const Geom &, const DevState &d, const float *, float, const float *, uint64_t, float *, float *,
                     int, hipStream_t) {
    if (enqueue()) d.ctr->err = 0;
}
void launch_decode_ranges(const Geom &, const uint64_t *, int, uint32_t, float2 *, float *, unsigned int *, hipStream_t) { enqueue(); }
void launch_tile_ranges(const Geom &, const float2 *, float2 *, hipStream_t) { enqueue(); }
void launch_ranges_from_blocks(const Geom &, const float *, float2 *, unsigned int *, hipStream_t) { enqueue(); }
void launch_encode(const Geom &, const void *, int, uint32_t, uint64_t *, unsigned int *, hipStream_t) { enqueue(); }
void launch_vertices_q10(const void *, uint64_t, void *, hipStream_t) { enqueue(); }
void launch_debug_cases(const Geom &, const DevState &, const float *, const int32_t *, int, float, uint8_t *, uint64_t,
                        hipStream_t) { enqueue(); }
void launch_copy_calibration(void *, const void *, uint64_t, hipStream_t) { enqueue(); }
uint64_t dense_sign_words(uint32_t, uint32_t, uint32_t) { return 1; }
uint64_t dense_chunk_words(uint32_t, uint32_t, uint32_t) { return 1; }
void launch_dense(uint32_t, uint32_t, uint32_t, const float *, float, uint64_t *, uint32_t *, DenseCounters *,
                  const uint64_t *, void *, uint64_t, hipStream_t) { enqueue(); }
int batch_front_per_cu(int *n) { return *n = 1, 0; }
int batch_decode_per_cu(const BatchParams &, int, int *n) { return *n = 1, 0; }
int batch_back_per_cu(int, int *n) { return *n = 1, 0; }
// A run whose launches end after the flags (batch_fails), or one in full.
static bool batch_fails = false;
hipError_t launch_batch(const BatchParams &p, int, int, const unsigned *, hipStream_t) {
    if (!enqueue()) return hipSuccess;
    CHECK(all_zero(p.vol_tot, p.n_groups));   // the flags add to them
    CHECK(all_zero(p.job_tot, p.n_jgroups));
    for (uint64_t v = 0; v < p.n_groups; v++) p.vol_tot[v] = 7ull << 32;
    for (uint64_t j = 0; j < p.n_jgroups; j++) p.job_tot[j] = 5;
    if (batch_fails) return hipErrorLaunchFailure;
    memset(p.vol_tot, 0, 8 * p.n_groups);
    memset(p.job_tot, 0, 8 * p.n_jgroups);
    p.ctr->n_slots += 7;
    *p.h_ctr = *p.ctr;
    return hipSuccess;
}
}  // namespace bcmc
using namespace bcmc;

// ---- the scenarios --------------------------------------------------------------
static const uint32_t NX = 40, NB = 1000;

static bcmc_volume *load() {
    static std::vector<uint64_t> words(NB);
    bcmc_volume *v = nullptr;
    CHECK(bcmc_load_compressed(words.data(), 8 * NB, 0, NX, NX, NX, BCMC_F32, 1, nullptr, &v) == BCMC_OK);
    return v;
}
static int extract(bcmc_volume *v, float iso, std::vector<uint32_t> blocks, uint64_t *T = nullptr) {
    uint64_t t = 0;
    active_now = blocks;
    const int rc = bcmc_extract(v, iso, nullptr, 0, &t, nullptr);
    if (T) *T = t;
    return rc;
}
// The call's triangles, and a cache in which every block's slot holds it.
static void good_call(bcmc_volume *v, float iso, std::vector<uint32_t> blocks) {
    uint64_t T = 0;
    CHECK(extract(v, iso, blocks, &T) == BCMC_E_CAPACITY && T == blocks.size());
    std::vector<int32_t> I_slot(NB), S_block(NB);
    uint64_t n = 0;
    CHECK(bcmc_debug_cache_state(v, I_slot.data(), S_block.data(), nullptr, &n) == BCMC_OK);
    for (uint32_t b : blocks) CHECK(I_slot[b] >= 0);
    for (uint32_t b = 0; b < NB; b++)
        if (I_slot[b] >= 0) CHECK((uint64_t)I_slot[b] < n && S_block[I_slot[b]] == (int32_t)b);
}

// A call whose kernels never run, then one whose counters do not arrive: the
// next ones count from zero and rewrite the flags.
static void counts() {
    bcmc_volume *v = load();
    good_call(v, 0.5f, {1, 2, 3});
    good_call(v, 0.25f, {2, 3, 4});
    CHECK(last_rewrite == 0 && last_prev == 0.5f);
    lost = true;
    CHECK(extract(v, 0.75f, {9}) == BCMC_E_HIP);
    lost = false;
    good_call(v, 0.5f, {1, 2, 7});
    CHECK(last_rewrite == 1);
    good_call(v, 0.25f, {2, 3, 4});
    CHECK(last_rewrite == 0);
    // caller-owned blocks: the failed call's volume holds no extract to look at
    std::vector<float> blocks(64 * NB);
    float g = 0;
    uint64_t T = 0;
    std::vector<float> field(64 * NB);
    CHECK(bcmc_volume_from_blocks(blocks.data(), NX, NX, NX, nullptr, &v) == BCMC_OK);
    CHECK(extract(v, 0.5f, {1, 2, 3}, &T) == BCMC_E_CAPACITY && T == 3);
    std::vector<float> gV(9 * 3);
    CHECK(bcmc_backward(v, 0.5f, gV.data(), 9, field.data(), &g, nullptr) == BCMC_OK);
    lost = true;
    CHECK(extract(v, 0.75f, {9}) == BCMC_E_HIP);
    lost = false;
    CHECK(bcmc_backward(v, 0.5f, gV.data(), 9, field.data(), &g, nullptr) == BCMC_E_INVALID);
    CHECK(extract(v, 0.5f, {1, 2, 3, 4}, &T) == BCMC_E_CAPACITY && T == 4);
}

// A call that assigns slots and whose counters do not arrive: the next call
// takes no slot that a block holds, and an emptied cache is empty.
static void cache() {
    for (int how = 0; how < 2; how++) {
        bcmc_volume *v = load();
        good_call(v, 0.5f, {1, 2, 3});
        (how ? launch_fails : readback_fails) = true;
        CHECK(extract(v, 0.75f, {3, 4, 5, 6}) == BCMC_E_HIP);
        readback_fails = launch_fails = false;
        good_call(v, 0.25f, {3, 6, 7});
        good_call(v, 0.5f, {1, 2, 3, 4, 5, 6});
        (how ? launch_fails : readback_fails) = true;
        CHECK(extract(v, 0.75f, {11, 12}) == BCMC_E_HIP);
        readback_fails = launch_fails = false;
        CHECK(bcmc_reset_cache(v, nullptr) == BCMC_OK);
        std::vector<int32_t> I_slot(NB);
        CHECK(bcmc_debug_cache_state(v, I_slot.data(), nullptr, nullptr, nullptr) == BCMC_OK);
        for (uint32_t b = 0; b < NB; b++) CHECK(I_slot[b] == -1);
        good_call(v, 0.5f, {1, 2, 3});
    }
}

// On a capturing stream the calls that wait for their counters fail without a
// launch (what a replay would run), and leave the handle as it was.
static void capture() {
    bcmc_volume *v = load();
    good_call(v, 0.5f, {1, 2, 3});
    capturing = true;
    int before = launches;
    CHECK(extract(v, 0.75f, {9}) == BCMC_E_HIP && launches == before);
    capturing = false;
    good_call(v, 0.25f, {2, 3, 4});
    CHECK(last_rewrite == 0 && last_prev == 0.5f);
    std::vector<float> blocks(64 * NB), field(64 * NB), gV(27);
    float g = 0;
    uint64_t T = 0;
    CHECK(bcmc_volume_from_blocks(blocks.data(), NX, NX, NX, nullptr, &v) == BCMC_OK);
    CHECK(extract(v, 0.5f, {1, 2, 3}, &T) == BCMC_E_CAPACITY && T == 3);
    bcmc_dense *h = nullptr;
    CHECK(bcmc_dense_create(NX, NX, NX, &h) == BCMC_OK);
    capturing = true;
    before = launches;
    CHECK(extract(v, 0.75f, {9}) == BCMC_E_HIP);
    CHECK(bcmc_backward(v, 0.5f, gV.data(), 9, field.data(), &g, nullptr) == BCMC_E_HIP);
    CHECK(bcmc_dense_extract(h, blocks.data(), 0.5f, nullptr, 0, &T, nullptr) == BCMC_E_HIP);
    CHECK(launches == before);
    capturing = false;
    CHECK(bcmc_backward(v, 0.5f, gV.data(), 9, field.data(), &g, nullptr) == BCMC_OK);
}

// A batch on a capturing stream, and one whose launches end half-way: the next
// run starts from zero totals.
static void batch() {
    bcmc_volume *v = load();
    const uint32_t job_vol[2] = {0, 0};
    const float iso[2] = {0.5f, 0.25f};
    bcmc_batch *b = nullptr;
    uint64_t off[3];
    CHECK(bcmc_batch_create(&v, 1, job_vol, iso, 2, nullptr, &b) == BCMC_OK);
    CHECK(bcmc_batch_set_graph(b, 0) == BCMC_OK);
    auto resident = [&] {
        bcmc_batch_info i;
        CHECK(bcmc_batch_get_info(b, &i) == BCMC_OK);
        return i.n_resident;
    };
    for (uint64_t k = 1; k <= 2; k++) {
        CHECK(bcmc_batch_run(b, nullptr, 0, off, nullptr) == BCMC_OK);
        CHECK(resident() == 7 * k);   // the store carries over
    }
    capturing = true;   // refused: the store stays
    const int before = launches;
    CHECK(bcmc_batch_run(b, nullptr, 0, off, nullptr) == BCMC_E_HIP && launches == before);
    capturing = false;
    CHECK(bcmc_batch_run(b, nullptr, 0, off, nullptr) == BCMC_OK && resident() == 21);
    batch_fails = true;
    CHECK(bcmc_batch_run(b, nullptr, 0, off, nullptr) == BCMC_E_HIP);
    batch_fails = false;
    for (uint64_t k = 1; k <= 2; k++) {
        CHECK(bcmc_batch_run(b, nullptr, 0, off, nullptr) == BCMC_OK);
        CHECK(resident() == 7 * k);   // started over
    }
}

// A budget that does not fit the memory: no slots, and no array that is not
// there is touched; the next budget that fits works.
static void budget() {
    bcmc_volume *v = load();
    good_call(v, 0.5f, {1, 2, 3});
    for (size_t limit : {(size_t)2000, (size_t)1 << 17}) {   // the first array fails, the slots fail
        malloc_limit = limit;
        CHECK(bcmc_set_cache_budget(v, 256 * 100, 256 * 1000) == BCMC_E_NOMEM);
        malloc_limit = ~(size_t)0;
        CHECK(extract(v, 0.5f, {1, 2, 3}) == BCMC_E_CACHE_CAP);
        CHECK(bcmc_reset_cache(v, nullptr) == BCMC_OK);
        CHECK(extract(v, 0.5f, {2, 3, 4}) == BCMC_E_CACHE_CAP);
        uint64_t n = 1;
        CHECK(bcmc_debug_cache_state(v, nullptr, nullptr, nullptr, &n) == BCMC_OK && n == 0);
        CHECK(bcmc_set_cache_budget(v, 256 * 100, 256 * 1000) == BCMC_OK);
        good_call(v, 0.5f, {1, 2, 3});
    }
}

// A handle and a budget may be used on any stream afterwards: the budget takes
// none that a caller could order, so neither leaves work behind.
static void ready() {
    bcmc_volume *v = load();
    CHECK(unwaited == 0);
    good_call(v, 0.5f, {1, 2, 3});
    CHECK(bcmc_set_cache_budget(v, 256 * 100, 256 * 1000) == BCMC_OK && unwaited == 0);
}

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "counts") counts();
    else if (what == "cache") cache();
    else if (what == "capture") capture();
    else if (what == "batch") batch();
    else if (what == "budget") budget();
    else if (what == "ready") ready();
    else return 2;
    printf("%s ok\n", what.c_str());
    return 0;
}
