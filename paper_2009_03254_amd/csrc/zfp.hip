// Fixed-rate ZFP codec for gfx950 (Sec. 3.3.4; on-demand block decode into
// cache slots, Sec. 4.2.1).  One lane owns one 4x4x4 block: the per-block
// bit-plane loop is serial, so 64 blocks per wave keep the SIMDs busy.
//
// Codec (Lindstrom, "Fixed-Rate Compressed Floating-Point Arrays", TVCG 2014,
// as realised by this project):
//   header   1 bit (0 = all-zero block) then emax+bias in 8 (f32) / 11 (f64)
//            bits; emax = largest frexp exponent, clamped so that
//            2^(emax-(P-2)) is a normal number;
//   values   i = trunc(x * 2^(P-2-emax)) as P-bit integers (P = 32 / 64);
//   lifting  separable 4-point decorrelating transform along x, y, z;
//   order    coefficients by ascending i+j+k, ties by ascending index;
//   negabinary, then embedded bit-plane coding with group tests, cut at
//            64*rate bits; bits are LSB-first in little-endian u64 words.
#include <stdint.h>

#include <algorithm>

#include "common.h"
#include "zfp_device.h"

namespace bcmc {
namespace {
// ---- kernels ---------------------------------------------------------------

__device__ __forceinline__ void block_xyz(const Geom &g, uint64_t b, uint32_t &bx, uint32_t &by,
                                          uint32_t &bz) {
    bx = (uint32_t)(b % g.nbx);
    uint64_t r = b / g.nbx;
    by = (uint32_t)(r % g.nby);
    bz = (uint32_t)(r / g.nby);
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Decode every block once: value range over the valid samples (Sec. 4.1),
// non-finite detection, and optionally the decoded blocks themselves.  Bound
// by VALU issue (about 90 % busy): 512^3 float32 at rate 4 takes 275 us (311-317
// with the longer parse step, 64-bit addresses for each plane's word and a
// predicate per sample in the range; the bytes moved need 127).
template <bool F64, bool STAGED>
__global__ __launch_bounds__(256) void k_decode_ranges(Geom g, const uint64_t *__restrict__ stream,
                                                      int rate, float2 *__restrict__ ranges,
                                                      float *__restrict__ blocks,
                                                      unsigned int *err) {
    extern __shared__ uint64_t stage_lds[];
    constexpr bool staged = STAGED;
    uint64_t *st = stage_lds + (threadIdx.x >> 6) * (STAGED ? stage_wave_words(rate, F64) : 0u);
    // whole waves iterate together (the staging is a wave-wide copy)
    for (uint64_t b0 = blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~63u); b0 < g.nb;
         b0 += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t b = b0 + __lane_id();
        const bool valid = b < g.nb;
        float v[64];
        if (staged) {
            stage_words(stream, rate, b, valid, st);
            if (valid) decode_block_staged<F64>(st, rate, v);
        } else if (valid) {
            decode_block<F64>(stream + b * rate, rate, v);
        }
        if (staged) __builtin_amdgcn_wave_barrier();   // st is rewritten by the next round
        if (!valid) continue;
        uint32_t bx, by, bz;
        block_xyz(g, b, bx, by, bz);
        // the range over the valid samples: a decoded value is an integer times a
        // power of two, infinite or finite but never NaN, so the range tells
        const uint32_t vx = min(4u, g.nx - 4 * bx), vy = min(4u, g.ny - 4 * by), vz = min(4u, g.nz - 4 * bz);
        float lo = v[0], hi = v[0];
        if (__ballot(vx + vy + vz != 12) == 0) {
#pragma unroll
            for (int i = 1; i < 64; i++) {
                lo = fminf(lo, v[i]);
                hi = fmaxf(hi, v[i]);
            }
        } else {
#pragma unroll
            for (int i = 1; i < 64; i++) {   // samples past the volume replaced by sample 0 (always valid)
                const bool in = (uint32_t)(i & 3) < vx && (uint32_t)((i >> 2) & 3) < vy && (uint32_t)(i >> 4) < vz;
                const float x = in ? v[i] : v[0];
                lo = fminf(lo, x);
                hi = fmaxf(hi, x);
            }
        }
        ranges[b] = make_float2(lo, hi);
        if (!isfinite(lo) || !isfinite(hi)) atomicOr(err, ERR_NONFINITE);
        if (blocks) {
            float4 *o = reinterpret_cast<float4 *>(blocks + b * 64);
#pragma unroll
            for (int q = 0; q < 16; q++) o[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        }
    }
}

__global__ __launch_bounds__(256) void k_ranges_from_blocks(Geom g, const float *__restrict__ blocks,
                                                           float2 *__restrict__ ranges,
                                                           unsigned int *err) {
    // a wave takes 64 consecutive blocks at a time, lane l the l-th (its
    // valid extent); the blocks' 16 KB are read 1 KB per load (in step q,
    // lanes 16 m .. 16 m + 15 hold the 16 float4 of block 4 q + m) and
    // reduced over each row of 16 lanes; the rows' results meet in LDS
    __shared__ float2 s_r[4][64];
    const int l = (int)__lane_id(), w = threadIdx.x >> 6;
    const uint64_t waves = (uint64_t)gridDim.x * 4;
    bool finite = true;
    for (uint64_t b0 = (blockIdx.x * 4ull + w) * 64; b0 < g.nb; b0 += waves * 64) {
        uint32_t ext = 0x040404u;   // the lane's block: valid samples per axis, as bytes
        if (b0 + l < g.nb) {
            uint32_t bx, by, bz;
            block_xyz(g, b0 + l, bx, by, bz);
            ext = min(4u, g.nx - 4 * bx) | min(4u, g.ny - 4 * by) << 8 | min(4u, g.nz - 4 * bz) << 16;
        }
        const int part = l & 15;   // float4 part: samples 4 part .. 4 part + 3 (y = part & 3, z = part >> 2)
#pragma unroll 4
        for (int q = 0; q < 16; q++) {
            const int m = l >> 4;
            const uint64_t blk = b0 + 4 * q + m;
            const uint32_t e = (uint32_t)__shfl((int)ext, 4 * q + m, 64);
            float lo = INFINITY, hi = -INFINITY;
            if (blk < g.nb) {
                const float4 f = reinterpret_cast<const float4 *>(blocks + blk * 64)[part];
                const float v[4] = {f.x, f.y, f.z, f.w};
                const bool rowok = (uint32_t)(part & 3) < ((e >> 8) & 0xFFu) && (uint32_t)(part >> 2) < (e >> 16);
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    if (rowok && (uint32_t)j < (e & 0xFFu)) {
                        lo = fminf(lo, v[j]);
                        hi = fmaxf(hi, v[j]);
                        finite = finite && isfinite(v[j]);
                    }
                }
            }
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) {
                lo = fminf(lo, __shfl_xor(lo, d, 64));
                hi = fmaxf(hi, __shfl_xor(hi, d, 64));
            }
            if (part == 0) s_r[w][4 * q + m] = make_float2(lo, hi);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (b0 + l < g.nb) ranges[b0 + l] = s_r[w][l];
        // s_r is rewritten next step
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (__ballot(!finite) && l == 0) atomicOr(err, ERR_NONFINITE);
}

// Set bits of m below the calling lane.
__device__ __forceinline__ uint32_t mbcnt_lo_hi(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Sign mask of a block: bit i = sample i below iso.
__device__ __forceinline__ uint64_t sign_mask_of(const float4 (&f)[16], float iso) {
    uint32_t mw[2] = {0u, 0u};
#pragma unroll
    for (int q = 0; q < 16; q++)
        mw[q >> 3] |= ((f[q].x < iso ? 1u : 0u) | (f[q].y < iso ? 2u : 0u) | (f[q].z < iso ? 4u : 0u) |
                       (f[q].w < iso ? 8u : 0u)) << (4 * (q & 7));
    return (uint64_t)mw[1] << 32 | mw[0];
}

// Store a decoded block into its slot, with its sign mask for this call's
// isovalue (so the freshly decoded slot need not be read back for it).
__device__ __forceinline__ void store_slot(const float *v, uint64_t s, float iso, float *__restrict__ slots,
                                           uint64_t *__restrict__ masks, uint32_t *__restrict__ mask_iso) {
    float4 *o = reinterpret_cast<float4 *>(slots + s * 64);
    float4 f[16];
#pragma unroll
    for (int q = 0; q < 16; q++) o[q] = f[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    masks[s] = sign_mask_of(f, iso);
    mask_iso[s] = __float_as_uint(iso);
}

// Sign masks for iso of the active blocks that were resident before the call
// (not flagged new) and hold none for it, one lane per block, its 16 float4
// loads all in flight before the first compare; the last waves first.
__device__ __forceinline__ void resident_masks(const Counters *ctr, const uint32_t *__restrict__ I_active,
                                               const uint8_t *__restrict__ active,
                                               const int32_t *__restrict__ I_slot, const float *__restrict__ slots,
                                               float iso, uint64_t *__restrict__ masks,
                                               uint32_t *__restrict__ mask_iso) {
    const uint64_t n_act = ctr->n_act;
    if (ctr->n_new == n_act) return;
    const uint32_t tag = __float_as_uint(iso);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t wave0 = (blockIdx.x * (uint64_t)blockDim.x + threadIdx.x) & ~63ull;
    for (uint64_t i = stride - 64 - wave0 + __lane_id(); i < n_act; i += stride) {
        const uint32_t b = I_active[i];
        if (active[b] & 4u) continue;
        const int32_t s = I_slot[b];
        if (s < 0 || mask_iso[s] == tag) continue;
        const float4 *src = reinterpret_cast<const float4 *>(slots) + (uint64_t)s * 16;
        float4 f[16];
#pragma unroll
        for (int q = 0; q < 16; q++) f[q] = src[q];
        masks[s] = sign_mask_of(f, iso);
        mask_iso[s] = tag;
    }
}

// Alg. 1 AssignSlots: the slots of the call's new blocks, in their order:
// the unused ones from n_used on, then the list of those to evict.
struct SlotSource {
    const uint32_t *evict;
    uint64_t n_used, n_unused;   // before the call; unused ones after its growth
    __device__ __forceinline__ uint64_t slot(uint64_t i) const {
        return i < n_unused ? n_used + i : evict[i - n_unused];
    }
};

// AssignSlots fused with DecompressBlocks: new block I_new[i] takes its
// slot, evicting the previous owner, and is decoded straight into it.
// The sign masks of the active blocks that were resident already, for calls
// at an isovalue other than the one their masks were built for, go with the
// decode: the waves that have no block to decode start on them (a launch of
// their own took 4.5-5 us of every call, whether there was anything to build
// or not).
// LOW (double precision, staged, low rates): the decode is
// decode_block_staged_low, which holds the kernel to the registers of the
// low-rate decoder (4 waves per SIMD; 5 spills registers and is slower); the
// blocks it hands back (their indices into I_new) are listed in `retry` for
// k_masks_retry, which builds the masks too.
template <bool F64, bool STAGED, bool LOW = false>
__global__ __launch_bounds__(256, LOW ? 4 : (F64 ? 1 : 4)) void k_assign_decode(Counters *ctr, const uint32_t *__restrict__ I_new,
                                                      const uint32_t *__restrict__ evict,
                                                      SlotState ss, uint32_t now,
                                                      int32_t *S_block, int32_t *I_slot,
                                                      uint32_t *S_stamp, const uint64_t *__restrict__ stream,
                                                      int rate, float *__restrict__ slots,
                                                      uint64_t n_blocks, float iso,
                                                      uint64_t *__restrict__ masks,
                                                      uint32_t *__restrict__ mask_iso,
                                                      const uint32_t *__restrict__ I_active,
                                                      const uint8_t *__restrict__ active,
                                                      uint32_t *__restrict__ retry = nullptr) {
    if (ctr->err) return;
    const uint64_t n_slots = ctr->n_slots;
    const uint64_t n_new = ctr->n_new;
    const SlotSource src{evict, ss.n_used, n_slots - ss.n_used};
    // slots this call created and leaves unused: their age counts from here
    const uint64_t created = ctr->n_used > ss.n_slots ? ctr->n_used : ss.n_slots;
    for (uint64_t i = created + blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n_slots;
         i += (uint64_t)gridDim.x * blockDim.x)
        S_stamp[i] = now;
    extern __shared__ uint64_t stage_lds[];
    constexpr bool staged = STAGED;
    uint64_t *st = stage_lds + (threadIdx.x >> 6) * (STAGED ? stage_wave_words(rate, F64) : 0u);
    // whole waves iterate together (the staging is a wave-wide copy)
    for (uint64_t i0 = blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~63u); i0 < n_new;
         i0 += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = i0 + __lane_id();
        bool valid = i < n_new;
        const uint32_t b = valid ? I_new[i] : 0u;
        const uint64_t s = valid ? src.slot(i) : 0u;
        if (valid && (b >= n_blocks || s >= n_slots)) {  // never expected: report, do not touch memory
            atomicOr(&ctr->err, ERR_INTERNAL);
            valid = false;
        }
        if (valid) {
            if (i >= src.n_unused) {
                const int32_t old = S_block[s];
                if (old >= 0) I_slot[old] = -1;
            }
            S_block[s] = (int32_t)b;
            I_slot[b] = (int32_t)s;
            S_stamp[s] = now;
        }
        float v[64];
        bool done = true;
        if (staged) {
            stage_words(stream, rate, b, valid, st);
            if constexpr (LOW) {
                if (valid) done = decode_block_staged_low(st, rate, v);
            } else {
                if (valid) decode_block_staged<F64>(st, rate, v);
            }
            __builtin_amdgcn_wave_barrier();   // st is rewritten by the next round
        } else if (valid) {
            decode_block<F64>(stream + (uint64_t)b * rate, rate, v);
        }
        if (valid && done) store_slot(v, s, iso, slots, masks, mask_iso);
        if constexpr (LOW) {   // one atomic per wave for the blocks handed back
            const uint64_t back = __ballot(valid && !done);
            if (back) {
                const int first = (int)__builtin_ctzll(back);
                uint32_t base = 0;
                if (__lane_id() == (unsigned)first)
                    base = atomicAdd(&ctr->n_retry, (uint32_t)__popcll(back));
                base = __shfl(base, first, 64);
                if (valid && !done) retry[base + mbcnt_lo_hi(back)] = (uint32_t)i;
            }
        }
    }
    if constexpr (!LOW) resident_masks(ctr, I_active, active, I_slot, slots, iso, masks, mask_iso);
}

// The 64 samples of block (bx, by, bz), partial blocks replicating the last
// valid sample along each axis.  quad (wave-uniform): every lane's block is
// whole and its rows of 4 samples are 16-byte aligned.
template <typename T>
__device__ __forceinline__ void load_block(const Geom &g, const T *__restrict__ f, uint32_t bx, uint32_t by,
                                           uint32_t bz, bool quad, T *x) {
    if (quad) {
        const T *p = f + 4 * bx + (uint64_t)g.nx * (4 * by + (uint64_t)g.ny * (4 * bz));
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const T *row = p + (uint64_t)g.nx * ((r & 3) + (uint64_t)g.ny * (r >> 2));
            if constexpr (sizeof(T) == 4) {
                const float4 q = *reinterpret_cast<const float4 *>(row);
                x[4 * r] = q.x, x[4 * r + 1] = q.y, x[4 * r + 2] = q.z, x[4 * r + 3] = q.w;
            } else {
                const double2 q = reinterpret_cast<const double2 *>(row)[0], h = reinterpret_cast<const double2 *>(row)[1];
                x[4 * r] = q.x, x[4 * r + 1] = q.y, x[4 * r + 2] = h.x, x[4 * r + 3] = h.y;
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 64; i++) {
        const uint32_t gx = min(4 * bx + (i & 3), g.nx - 1);
        const uint32_t gy = min(4 * by + ((i >> 2) & 3), g.ny - 1);
        const uint32_t gz = min(4 * bz + (i >> 4), g.nz - 1);
        x[i] = f[gx + (uint64_t)g.nx * (gy + (uint64_t)g.ny * gz)];
    }
}

// One lane per block, 64 consecutive blocks per wave.  STAGED: the words go
// through the wave's LDS (word w of lane l at st[w * STAGE_STRIDE + l]) and out
// in one contiguous run.  VALU bound: the planes are formed by bit transposes of
// the coefficients (a bit extract per plane and coefficient took 6,000
// instructions of a wave's single-precision blocks), and the coder forms the
// group tests of 16 coefficients at a time from a table of 256 bytes'
// (encode_planes32).  512^3 float32 at rate 8: 255 us (964 with the planes
// extracted bit by bit; 362 with a step per run, 328 with the runs placed by
// one shift), at 3 waves per SIMD (4 spill).
template <bool F64, bool STAGED>
__global__ __launch_bounds__(256, F64 ? 2 : 3) void k_encode(Geom g, const void *__restrict__ field, int aligned,
                                                            int rate, uint64_t *__restrict__ stream,
                                                            unsigned int *err) {
    using T = std::conditional_t<F64, double, float>;
    extern __shared__ uint64_t stage_lds[];
    __shared__ uint16_t group[256];
    group[threadIdx.x] = (uint16_t)group_bits(threadIdx.x);
    __syncthreads();
    uint64_t *st = stage_lds + (threadIdx.x >> 6) * (STAGED ? STAGE_STRIDE * rate : 0);
    const T *f = static_cast<const T *>(field);
    const uint32_t l = __lane_id();
    bool finite = true;
    // whole waves iterate together (the words leave by a wave-wide copy)
    for (uint64_t b0 = blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~63u); b0 < g.nb;
         b0 += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t b = b0 + l;
        const bool valid = b < g.nb;
        uint32_t bx, by, bz;
        block_xyz(g, valid ? b : b0, bx, by, bz);
        const bool whole = 4 * bx + 3 < g.nx && 4 * by + 3 < g.ny && 4 * bz + 3 < g.nz;
        T x[64];
        load_block(g, f, bx, by, bz, aligned && !__ballot(!whole), x);
        if constexpr (STAGED) {
            finite &= encode_block<F64, STAGE_STRIDE>(x, rate, (lds_group)group, (lds_out)st + l) || !valid;
            wave_sync();
            const uint32_t total = (uint32_t)(g.nb - b0 < 64 ? g.nb - b0 : 64) * (uint32_t)rate;
            const uint64_t magic = ((1ull << 32) + (uint64_t)rate - 1) / (uint64_t)rate;   // i / rate, i < 2^32 / rate
            uint64_t *dst = stream + b0 * rate;
            for (uint32_t i = l; i < total; i += 64) {
                const uint32_t ln = (uint32_t)((i * magic) >> 32);
                dst[i] = st[(i - ln * rate) * STAGE_STRIDE + ln];
            }
            wave_sync();   // st is rewritten by the next round
        } else if (valid) {
            finite &= encode_block<F64, 1>(x, rate, (lds_group)group, stream + b * rate);
        }
    }
    if (__ballot(!finite) && l == 0) atomicOr(err, ERR_NONFINITE);
}

// The blocks the low-rate decoder handed back, decoded with the general
// decoder from global memory into the slots the assignment gave them, and the
// resident blocks' masks.
__global__ __launch_bounds__(256) void k_masks_retry(const Counters *ctr, const uint32_t *__restrict__ I_new,
                                                     const uint32_t *__restrict__ evict, SlotState ss,
                                                     const uint64_t *__restrict__ stream, int rate,
                                                     float *__restrict__ slots, float iso,
                                                     uint64_t *__restrict__ masks,
                                                     uint32_t *__restrict__ mask_iso,
                                                     const uint32_t *__restrict__ retry,
                                                     const uint32_t *__restrict__ I_active,
                                                     const uint8_t *__restrict__ active,
                                                     const int32_t *__restrict__ I_slot) {
    if (ctr->err) return;
    const uint32_t n = ctr->n_retry;
    const SlotSource src{evict, ss.n_used, ctr->n_slots - ss.n_used};
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        const uint32_t i = retry[j];
        const uint32_t b = I_new[i];
        const uint64_t s = src.slot(i);
        float v[64];
        decode_block<true>(stream + (uint64_t)b * rate, rate, v);
        store_slot(v, s, iso, slots, masks, mask_iso);
    }
    resident_masks(ctr, I_active, active, I_slot, slots, iso, masks, mask_iso);
}

unsigned grid_for(uint64_t n, unsigned cap) {
    uint64_t gsz = (n + 255) / 256;
    if (gsz < 1) gsz = 1;
    return (unsigned)(gsz < cap ? gsz : cap);
}

}  // namespace

// Instantiates a decode kernel for (type, staged) and launches it with the
// staging LDS the rate needs.
#define BCMC_DECODE_LAUNCH(KERNEL, grid, rate, s, ...)                                      \
    do {                                                                                    \
        const unsigned lds_ = stage_lds_bytes((int)(rate), is_f64 != 0);                                 \
        if (is_f64 && lds_) KERNEL<true, true><<<grid, 256, lds_, s>>>(__VA_ARGS__);         \
        else if (is_f64) KERNEL<true, false><<<grid, 256, 0, s>>>(__VA_ARGS__);              \
        else if (lds_) KERNEL<false, true><<<grid, 256, lds_, s>>>(__VA_ARGS__);             \
        else KERNEL<false, false><<<grid, 256, 0, s>>>(__VA_ARGS__);                         \
    } while (0)

void launch_decode_ranges(const Geom &g, const uint64_t *stream, int is_f64, uint32_t rate,
                          float2 *ranges, float *blocks_out, unsigned int *err, hipStream_t s) {
    unsigned grid = grid_for(g.nb, 8192);
    BCMC_DECODE_LAUNCH(k_decode_ranges, grid, rate, s, g, stream, (int)rate, ranges, blocks_out, err);
}

void launch_ranges_from_blocks(const Geom &g, const float *blocks, float2 *ranges,
                               unsigned int *err, hipStream_t s) {
    k_ranges_from_blocks<<<grid_for(g.nb, 8192), 256, 0, s>>>(g, blocks, ranges, err);
}

void launch_assign_decode(const DevState &d, int is_f64, uint32_t rate, uint64_t max_new, float iso,
                          const uint32_t *evict, const SlotState &ss, uint32_t now, hipStream_t s) {
    unsigned grid = grid_for(max_new, 2048);
    const unsigned lds = stage_lds_bytes((int)rate, is_f64 != 0);
    if (is_f64 && lds && rate <= LOW_RATE_MAX && d.retry) {
        k_assign_decode<true, true, true><<<grid, 256, lds, s>>>(
            d.ctr, d.I_new, evict, ss, now, d.S_block, d.I_slot, d.S_stamp, d.stream, (int)rate, d.slots,
            max_new, iso, d.masks, d.mask_iso, d.I_active, d.active, d.retry);
        k_masks_retry<<<std::min(grid, 1024u), 256, 0, s>>>(d.ctr, d.I_new, evict, ss, d.stream, (int)rate, d.slots,
                                                           iso, d.masks, d.mask_iso, d.retry, d.I_active, d.active,
                                                           d.I_slot);
        return;
    }
    BCMC_DECODE_LAUNCH(k_assign_decode, grid, rate, s, d.ctr, d.I_new, evict, ss, now, d.S_block, d.I_slot,
                       d.S_stamp, d.stream, (int)rate, d.slots, max_new, iso, d.masks, d.mask_iso, d.I_active,
                       d.active);
}

void launch_encode(const Geom &g, const void *field, int is_f64, uint32_t rate, uint64_t *stream,
                   unsigned int *err, hipStream_t s) {
    const unsigned grid = grid_for(g.nb, 8192);
    // rows of 4 samples 16-byte aligned (doubles: 32 bytes in two loads)
    const int aligned = g.nx % 4 == 0 && reinterpret_cast<uintptr_t>(field) % 16 == 0;
    const unsigned lds = rate <= STAGE_MAX_RATE ? 4u * STAGE_STRIDE * rate * 8u : 0u;
    if (is_f64 && lds) k_encode<true, true><<<grid, 256, lds, s>>>(g, field, aligned, (int)rate, stream, err);
    else if (is_f64) k_encode<true, false><<<grid, 256, 0, s>>>(g, field, aligned, (int)rate, stream, err);
    else if (lds) k_encode<false, true><<<grid, 256, lds, s>>>(g, field, aligned, (int)rate, stream, err);
    else k_encode<false, false><<<grid, 256, 0, s>>>(g, field, aligned, (int)rate, stream, err);
}

}  // namespace bcmc
