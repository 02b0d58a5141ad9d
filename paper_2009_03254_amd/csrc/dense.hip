// Dense data-parallel marching cubes over an uncompressed field resident in
// device memory: the standard GPU formulation the paper measures as its
// baseline (Sec. 3.3.3, tab:mc_naive_parallel_perf): every cell of the volume
// classified and counted, prefix sums over the counts, and a pass that writes
// the soup of the cells that hold the surface.  No blocks, culling or cache:
// it measures what the block-compressed path's culling buys.
//
// Records are the 16-byte vertices of the block path (block-relative float32
// position + block id), computed with the same operations, so the soup is
// the block path's soup with the cells in global row-major order (x fastest)
// instead of block order.
//
// Cells are handled 64 at a time as bits of a word (a word: 64 cells of one
// row, x fastest), in three launches.  k_dense_signs reads the field once and
// keeps one bit per sample (below iso); k_dense_count gets the triangle counts
// of 64 cells at once from the four rows' bits by the bit-sliced diagram of
// the case table; k_dense_emit forms the words' bits again, lists their cells
// and triangles in LDS and writes one vertex per lane.  Bound by memory: the
// field read once for the signs and, where the surface lies, again for the
// vertices, and the soup written.  512^3 turbulence at its median (14.5 M
// triangles): 109 + 26 + 306 us, the signs at 5.0 TB/s (before, with each
// cell's case and offset kept in memory: 985 for a classification whose lanes
// read 64 bytes apart and 1433 for an emission whose lanes wrote 48 bytes
// apart, 2.6 ms in all).  More waves (7 or 8 per SIMD, spilling) or two vertices
// per lane in flight gained nothing (376-385 us against 378, before
// dense_chunk_size).
#include <stdint.h>

#include <algorithm>

#include "common.h"
#include "mc_device.h"
#include "mc_ntri.h"

namespace bcmc {
namespace {

struct DenseGeom {
    uint32_t nx, ny, nz;
    uint32_t swords;      // words per row of samples
    uint32_t cwords;      // words per row of cells
    uint32_t n_swords;    // swords * ny * nz (at most 2^32 - 1 samples)
    uint32_t n_cwords;    // cwords * (ny - 1) * (nz - 1)
    uint32_t nbx, nby;    // blocks per row / per layer (for the block ids of the records)
};

// bits[row][w]: bit i = sample 64 w + i of the row is below iso (0 past its
// end).  One lane per sample, 8 words in flight per wave.  Also clears the
// counters of the passes that follow.
__global__ __launch_bounds__(256) void k_dense_signs(DenseGeom g, const float *__restrict__ f, float iso,
                                                    uint64_t *__restrict__ bits, DenseCounters *ctr) {
    constexpr int J = 8;
    if (blockIdx.x == 0)
        for (unsigned i = threadIdx.x; i < sizeof(DenseCounters) / 4; i += 256) reinterpret_cast<uint32_t *>(ctr)[i] = 0;
    const uint64_t waves = (uint64_t)gridDim.x * 4;
    for (uint64_t w0 = ((uint64_t)blockIdx.x * 4 + wave_id()) * J; w0 < g.n_swords; w0 += waves * J) {
        uint32_t row = (uint32_t)w0 / g.swords, wx = (uint32_t)w0 - row * g.swords;
        float v[J];
        bool in[J];
#pragma unroll
        for (int j = 0; j < J; j++) {
            const uint32_t x = 64 * wx + (uint32_t)lane();
            in[j] = w0 + j < g.n_swords && x < g.nx;
            v[j] = in[j] ? f[(uint64_t)row * g.nx + x] : 0.0f;
            if (++wx == g.swords) {
                wx = 0;
                row++;
            }
        }
        uint64_t mine = 0;
#pragma unroll
        for (int j = 0; j < J; j++) {
            const uint64_t b = __ballot(in[j] && v[j] < iso);
            if (lane() == j) mine = b;
        }
        if (lane() < J && w0 + lane() < g.n_swords) bits[w0 + lane()] = mine;
    }
}

// Word i of the cells: the corner bits of its 64 cells (corner k at
// +(k&1, k>>1&1, k>>2&1)), which of them are in the volume, and where it lies.
struct CellWord {
    uint64_t c[8], valid;
    uint32_t x0, y, z;
};
__device__ __forceinline__ CellWord load_word(const DenseGeom &g, const uint64_t *__restrict__ bits, uint32_t i) {
    CellWord q;
    const uint32_t r = i / g.cwords, wx = i - r * g.cwords;
    q.y = r % (g.ny - 1);
    q.z = r / (g.ny - 1);
    q.x0 = 64 * wx;
    const bool more = wx + 1 < g.swords;
    uint64_t a[4], b[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const uint64_t at = ((uint64_t)(q.z + (k >> 1)) * g.ny + q.y + (k & 1)) * g.swords + wx;
        a[k] = bits[at];
        b[k] = more ? bits[at + 1] : 0ull;
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        q.c[2 * k] = a[k];
        q.c[2 * k + 1] = a[k] >> 1 | b[k] << 63;
    }
    const uint32_t n = min(64u, g.nx - 1 - q.x0);
    q.valid = n == 64 ? ~0ull : (1ull << n) - 1;
    return q;
}

// Vertices of the word's cells; act: the cells that have triangles.
__device__ __forceinline__ uint32_t count_word(const CellWord &q, uint64_t &act) {
    uint64_t n0, n1, n2;
    mc_ntri_bits(q.c, n0, n1, n2);
    n0 &= q.valid;
    n1 &= q.valid;
    n2 &= q.valid;
    act = n0 | n1 | n2;
    return 3u * ((uint32_t)__popcll(n0) + 2u * (uint32_t)__popcll(n1) + 4u * (uint32_t)__popcll(n2));
}

// Vertices per chunk of words (the emission's chunks: xcd_chunks), and the
// vertices and active cells of each XCD eighth of them.
__global__ __launch_bounds__(256) void k_dense_count(DenseGeom g, const uint64_t *__restrict__ bits,
                                                    uint32_t cs, uint32_t *__restrict__ chunk_tot,
                                                    DenseCounters *ctr) {
    __shared__ uint64_t s_v[MC_WAVES], s_a[MC_WAVES];
    const ChunkRange cr = xcd_chunks((g.n_cwords + (uint64_t)cs - 1) / cs);
    uint64_t verts = 0, cells = 0;
    for (uint64_t c = cr.first; c < cr.end; c += cr.stride) {
        const uint64_t i = c * cs + lane();
        uint32_t n = 0;
        if (lane() < (int)cs && i < g.n_cwords) {
            uint64_t act;
            n = count_word(load_word(g, bits, (uint32_t)i), act);
            cells += (uint64_t)__popcll(act);
        }
        n = wave_sum(n);
        if (lane() == 0) chunk_tot[c] = n;
        verts += n;
    }
    cells = wave_sum(cells);
    if (lane() == 0) {
        s_v[wave_id()] = verts;
        s_a[wave_id()] = cells;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < MC_WAVES; k++) {
            verts += s_v[k];
            cells += s_a[k];
        }
        if (cells) {
            atomicAdd(&ctr->xcd[blockIdx.x % 8u].verts, (unsigned long long)verts);
            atomicAdd(&ctr->xcd[blockIdx.x % 8u].cells, (unsigned long long)cells);
        }
    }
}

// Per-wave LDS of the emission: up to 64 active cells and their triangles.
struct DenseShared {
    uint64_t tab[256];                // the case table
    uint2 edge[12];                   // per edge: sample offsets of its two corners from the cell's lowest
    uint32_t egeo[12];                // first corner as bytes x | y << 8 | z << 16, axis in byte 3
    uint32_t at[MC_WAVES][64];        // per cell: index of its lowest sample
    uint32_t geo[MC_WAVES][64];       // its place in its block as bytes x | y << 8 | z << 16, case in byte 3
    uint32_t blk[MC_WAVES][64];       // its block
    uint32_t tri[MC_WAVES][64 * 5];   // per triangle: cell | 3 edge ids << 20
};

__global__ __launch_bounds__(256, 6) void k_dense_emit(DenseGeom g, const float *__restrict__ f, float iso,
                                                   const uint64_t *__restrict__ bits, uint32_t cs,
                                                   const uint32_t *__restrict__ chunk_tot,
                                                   const uint64_t *__restrict__ mc_table,
                                                   void *__restrict__ out, uint64_t cap, DenseCounters *ctr) {
    __shared__ DenseShared sh;
    sh.tab[threadIdx.x] = mc_table[threadIdx.x];
    if (threadIdx.x < 12) {
        const uint32_t d = (uint32_t)(kEdgeGeom >> (5 * threadIdx.x)) & 31u;   // ox | oy << 1 | oz << 2 | axis << 3
        const uint32_t ox = d & 1u, oy = (d >> 1) & 1u, oz = (d >> 2) & 1u, axis = d >> 3;
        const uint32_t d0 = ox + g.nx * (oy + g.ny * oz);
        sh.edge[threadIdx.x] = make_uint2(d0, d0 + (axis == 0 ? 1u : (axis == 1 ? g.nx : g.nx * g.ny)));
        sh.egeo[threadIdx.x] = ox | oy << 8 | oz << 16 | axis << 24;
    }
    __syncthreads();
    const int w = (int)wave_id(), l = lane();
    const ChunkRange cr = xcd_chunks((g.n_cwords + (uint64_t)cs - 1) / cs);
    uint64_t base = 0, all = 0, cells = 0;
    for (uint32_t x = 0; x < 8; x++) {
        const uint64_t tx = ctr->xcd[x].verts;
        base += x < blockIdx.x % 8u ? tx : 0ull;
        all += tx;
        cells += ctr->xcd[x].cells;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctr->n_verts = all;
        ctr->n_active = cells;
    }
    base = uniform64(base);
    if (cr.first < cr.end) base += chunks_sum(chunk_tot, cr.lo, cr.first);
    for (uint64_t c = cr.first; c < cr.end; c += cr.stride) {
        const uint64_t i = c * cs + l;
        CellWord q;
        uint64_t act = 0;
        uint32_t n = 0;
        if (l < (int)cs && i < g.n_cwords) {
            q = load_word(g, bits, (uint32_t)i);
            n = count_word(q, act);
        }
        const uint32_t na = (uint32_t)__popcll(act);
        const uint32_t incl = wave_incl_scan(na), vincl = wave_incl_scan(n);
        const uint32_t total = bcast(incl, 63);
        // the words in order, as many at a time as have 64 active cells
        for (uint32_t done = 0; done < total;) {
            const bool in = na && incl - na >= done && incl <= done + 64;
            const uint64_t m = __ballot(in);
            const int first = (int)__builtin_ctzll(m), last = 63 - (int)__builtin_clzll(m);
            const uint32_t ncell = bcast(incl, last) - done;
            const uint64_t o0 = base + bcast(vincl - n, first);
            if (in) {
                uint32_t slot = incl - na - done;
                const uint32_t row = (q.z * g.ny + q.y) * g.nx + q.x0;
                const uint32_t brow = (q.x0 >> 2) + g.nbx * ((q.y >> 2) + g.nby * (q.z >> 2));
                const uint32_t geo = (q.y & 3u) << 8 | (q.z & 3u) << 16;
                for (uint64_t a = act; a; a &= a - 1, slot++) {
                    const uint32_t x = (uint32_t)__builtin_ctzll(a);
                    uint32_t cse = 0;
#pragma unroll
                    for (int k = 0; k < 8; k++) cse |= (uint32_t)(q.c[k] >> x & 1u) << k;
                    sh.at[w][slot] = row + x;
                    sh.geo[w][slot] = geo | (x & 3u) | cse << 24;
                    sh.blk[w][slot] = brow + (x >> 2);
                }
            }
            wave_lds_sync();
            const uint64_t tb = l < (int)ncell ? sh.tab[sh.geo[w][l] >> 24] : 0ull;
            const uint32_t nt = (uint32_t)(tb >> 60);
            const uint32_t tincl = wave_incl_scan(nt);
            const int nv = 3 * (int)bcast(tincl, 63);
            for (uint32_t t = 0; t < nt; t++)
                sh.tri[w][tincl - nt + t] = (uint32_t)l | (uint32_t)(tb >> (12 * t)) << 20;
            wave_lds_sync();
            for (int j = l; j < nv; j += 64) {
                const int t = (j * 43691) >> 17;   // j / 3 for j < 960
                const uint32_t rec = sh.tri[w][t];
                const uint32_t e = (rec >> (20 + 4 * (j - 3 * t))) & 15u, k = rec & 63u;
                const uint2 d = sh.edge[e];
                const uint32_t at = sh.at[w][k];
                const float a = f[at + d.x], bv = f[at + d.y];
                const uint32_t eg = sh.egeo[e], axis = eg >> 24;
                const uint32_t p = (sh.geo[w][k] & 0x030303u) + (eg & 0x010101u);   // the edge's first corner
                const float tt = (iso - a) / (bv - a);
                const float px = (float)(p & 0xFFu) + (axis == 0 ? tt : 0.0f);
                const float py = (float)((p >> 8) & 0xFFu) + (axis == 1 ? tt : 0.0f);
                const float pz = (float)(p >> 16) + (axis == 2 ? tt : 0.0f);
                const uint64_t o = o0 + (uint64_t)j;
                if (o < cap) store_record(out, o, px, py, pz, sh.blk[w][k]);
            }
            wave_lds_sync();   // the lists are rewritten next
            done += ncell;
        }
        if (c + cr.stride < cr.end) base += chunks_sum(chunk_tot, c, c + cr.stride);
    }
}

DenseGeom dense_geom(uint32_t nx, uint32_t ny, uint32_t nz) {
    DenseGeom g;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.swords = (nx + 63) / 64;
    g.cwords = (nx - 2) / 64 + 1;
    g.n_swords = g.swords * ny * nz;
    g.n_cwords = g.cwords * (ny - 1) * (nz - 1);
    g.nbx = (nx + 3) / 4;
    g.nby = (ny + 3) / 4;
    return g;
}

// Words per chunk: mc_chunk_size's, but not whole rows a multiple of 4 KB
// apart.  The waves would then start every chunk at the same x of such rows
// and gather through the same few L2 channels: a call on 512^3 turbulence takes
// 533..547 us with chunks of 64 words (8 rows of 2 KB) and 473..486 with 61 (three
// fields; 60 and 62 as 61, 63 4 % and 56 5 % slower); 256 x 256 x 256 121 with 64,
// 103 with 61.  Where the rows differ, 61 measured from 4 % faster (384^3, 300^3)
// to 4 % slower (640 x 512 x 512): those keep 64.
constexpr uint32_t DENSE_ODD_CHUNK = 61;
uint32_t dense_chunk_size(const DenseGeom &g, uint32_t waves) {
    const uint32_t cs = mc_chunk_size(g.n_cwords, waves);
    if (cs % g.cwords || (uint64_t)(cs / g.cwords) * g.nx % 1024) return cs;
    return cs > DENSE_ODD_CHUNK ? DENSE_ODD_CHUNK : cs + 1;
}

}  // namespace

uint64_t dense_sign_words(uint32_t nx, uint32_t ny, uint32_t nz) { return dense_geom(nx, ny, nz).n_swords; }

uint64_t dense_chunk_words(uint32_t nx, uint32_t ny, uint32_t nz) {
    return std::max<uint64_t>(mc_chunk_slots(dense_geom(nx, ny, nz).n_cwords),
                              dense_geom(nx, ny, nz).n_cwords / DENSE_ODD_CHUNK + 1);
}

// bits: dense_sign_words, chunk_tot: dense_chunk_words entries; ctr holds the
// call's n_active and n_verts when the stream reaches the end.
void launch_dense(uint32_t nx, uint32_t ny, uint32_t nz, const float *field, float iso, uint64_t *bits,
                  uint32_t *chunk_tot, DenseCounters *ctr, const uint64_t *mc_table, void *out, uint64_t cap,
                  hipStream_t s) {
    const DenseGeom g = dense_geom(nx, ny, nz);
    static unsigned sgrid = 0, cgrid = 0, egrid = 0;
    if (!sgrid) sgrid = resident_grid(k_dense_signs);
    if (!cgrid) cgrid = resident_grid(k_dense_count);
    if (!egrid) egrid = std::min<unsigned>(resident_grid(k_dense_emit), MC_MAX_GRID);
    const unsigned words = (unsigned)std::min<uint64_t>(((uint64_t)g.n_swords + 31) / 32, 1u << 20);
    const unsigned need = ((unsigned)std::min<uint64_t>(g.n_cwords, 4u * MC_MAX_GRID) + 3) / 4;
    const unsigned eg = std::min(egrid, (need + 7) / 8 * 8), cg = std::min(cgrid, (need + 7) / 8 * 8);
    const uint32_t cs = dense_chunk_size(g, eg * MC_WAVES);
    k_dense_signs<<<std::min(words, sgrid), 256, 0, s>>>(g, field, iso, bits, ctr);
    k_dense_count<<<cg, 256, 0, s>>>(g, bits, cs, chunk_tot, ctr);
    k_dense_emit<<<eg, 256, 0, s>>>(g, field, iso, bits, cs, chunk_tot, mc_table, out, cap, ctr);
}

}  // namespace bcmc
