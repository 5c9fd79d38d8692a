// Stable cell-tile sort for gfx950.
//
// key(p) = tile of the particle's cell, or tile * cells_per_tile + cell in
// tile, or (rank-interleaved) tile, rank of the particle among the particles
// of its cell, cell in tile.  The permutation is the stable one (ties keep
// their order), built by least-significant-digit radix sort on (key, source
// index) pairs with 8-bit digits: per pass a digit histogram per block, an
// exclusive scan in digit-major order (of few blocks: by the scatter itself),
// and a scatter in which every wave ranks its 64 elements by digit with ballots
// (so equal digits keep their order) and the block's waves take consecutive
// sub-ranges.  The final index list moves every SoA array into the alternate
// buffer set, and a boundary pass writes the first-particle offset of every
// tile.
//
// Several items of a call are sorted together where the scratch holds their
// particles (SortGroup): item i's keys start after the keys of the items before
// it, so one sort of the concatenated particles leaves every item in its own
// range, in its own stable order.  A sort's launches cost about 5 us each
// whatever they do, and a call over eleven items took 220 of them.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "pl_device.h"
#include "sort_groups.h"

namespace pl {

constexpr int kSortWaves = 8;
constexpr int kSortThreads = kSortWaves * 64;
// Elements per thread of a block: 16, or 4 where 16 would leave most CUs without
// a block (262107 particles: 32 blocks or 128).
constexpr int kPerThread = 16, kPerThreadSmall = 4;
constexpr int kSmallSort = 1 << 19;
constexpr int kPerBlock = kSortThreads * kPerThread;
// Digit counts of one pass over up to np elements (the smaller blocks' at most).
constexpr int64_t kSortHist(int64_t np)
{
    const int64_t small = np < kSmallSort ? np : kSmallSort, s = kSortThreads * kPerThreadSmall;
    const int64_t a = (np + kPerBlock - 1) / kPerBlock, b = (small + s - 1) / s;
    return ((a > b ? a : b) << kMaxDigitBits) + 1024;
}
__host__ inline int sort_per(int np) { return np > kSmallSort ? kPerThread : kPerThreadSmall; }
__host__ inline int sort_blocks(int np) { return (np + kSortThreads * sort_per(np) - 1) / (kSortThreads * sort_per(np)); }
constexpr int kScanBlocks = 512;

// Digit count of one key per lane (v: the lane has one, the lanes with one
// come first, the first nv of the lanes) added to cnt: the first lane of every run of equal
// digits adds the run's length.  All lanes of the wave take part.
__device__ __forceinline__ void count_runs(uint32_t key, bool v, int nv, int shift, uint32_t mask, uint32_t *cnt)
{
    const int lane = threadIdx.x & 63;
    const uint32_t d = v ? (key >> shift) & mask : ~0u;
    const uint32_t prev = __shfl_up(d, 1, 64);
    const bool head = v && (lane == 0 || prev != d);
    const uint64_t hm = __ballot(head);
    if (head) {
        const uint64_t later = hm & ~((2ull << lane) - 1ull);     // heads after this lane
        const int stop = later ? __builtin_ctzll(later) : min(64, nv);
        atomicAdd(&cnt[d], (uint32_t)(stop - lane));
    }
}

// Items sorted together: their particles one after another (item i's at
// [base[i], base[i + 1])) and their keys (item i's from kbase[i]).  tbase: tiles
// before item i.  Passed to the kernels by value.
struct SortItem {
    int n[3], tile[3];
    int np, ntiles;
    const uint32_t *cell;            // F32_OFFSET
    const double *x[3];              // F64
    int32_t *tile_start;
    int32_t *runs;
};
struct SortGroup {
    int count, total, prec, ndim, key_mode;
    int base[kGroup + 1], tbase[kGroup + 1];
    uint32_t kbase[kGroup];
    SortItem it[kGroup];
};
static_assert(sizeof(SortGroup) <= 3072, "kernel arguments");

// Key of particle p of an item.
__device__ __forceinline__ uint32_t sort_key(const SortGroup &g, const SortItem &a, int p)
{
    const int tx = a.tile[0], ty = a.tile[1], tz = a.tile[2];
    const int ntx = (a.n[0] + tx - 1) / tx, nty = (a.n[1] + ty - 1) / ty;     // (the plain algorithm's may not divide)
    const int per_tile = tx * ty * tz;
    const bool p2 = ((tx & (tx - 1)) | (ty & (ty - 1)) | (tz & (tz - 1))) == 0;
    int c[3] = {0, 0, 0};
    if (g.prec == PL_F32_OFFSET) {
        unpack_cell(a.cell[p], c[0], c[1], c[2]);
        for (int d = 0; d < 3; ++d)
            if (c[d] >= a.n[d]) c[d] %= a.n[d];
    } else {
        for (int d = 0; d < g.ndim; ++d) {
            double v = a.x[d][p];
            double nn = (double)a.n[d];
            if (!(v >= 0.0 && v < nn)) {
                if (!isfinite(v)) v = 0.0;
                v = v - nn * floor(v / nn);
                if (v >= nn || v < 0.0) v = 0.0;
            }
            c[d] = (int)floor(v);
        }
    }
    // power-of-two tile sides (the usual case) divide by shifts
    int q[3], r[3];
    const int td[3] = {tx, ty, tz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        if (p2) {
            const int lg = __builtin_ctz((unsigned)td[d]);
            q[d] = c[d] >> lg;
            r[d] = c[d] & (td[d] - 1);
        } else {
            q[d] = c[d] / td[d];
            r[d] = c[d] % td[d];
        }
    }
    int t = q[0] + ntx * (q[1] + nty * q[2]);
    uint32_t key = (uint32_t)t;
    if (g.key_mode == PL_KEY_TILE_CELL || g.key_mode == PL_KEY_TILE_RUN) {
        int yy = r[1];
        // run order: rows taken as 0, 2, 4, 6, 1, 3, 5, 7 within every group
        // of eight (0, 2, 1, 3 within groups of four), so that the lanes
        // served together by one LDS access hold rows of one parity and
        // their records and deposit cells fall on distinct banks
        if (g.key_mode == PL_KEY_TILE_RUN && (ty & 7) == 0)
            yy = (yy & ~7) | ((yy & 1) << 2) | ((yy >> 1) & 3);
        else if (g.key_mode == PL_KEY_TILE_RUN && (ty & 3) == 0)
            yy = (yy & ~3) | ((yy & 1) << 1) | ((yy >> 1) & 1);
        int loc = r[0] + tx * (yy + ty * r[2]);
        key = (uint32_t)t * (uint32_t)per_tile + (uint32_t)loc;
    }
    return key;
}

// Keys of every particle, and the digit histogram of the first pass (low
// dbits bits) of each block's keys, stored digit-major: hist[d *
// nblocks + b].
template <int PT>
__global__ __launch_bounds__(kSortThreads) void k_keys(SortGroup g, uint32_t *keys, int dbits, int nblocks, uint32_t *hist)
{
    constexpr int kBlock = PT * kSortThreads;
    __shared__ uint32_t h[1 << kMaxDigitBits];
    const int nd = 1 << dbits;
    for (int d = threadIdx.x; d < nd; d += blockDim.x) h[d] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int beg = blockIdx.x * kBlock, end = min(g.total, beg + kBlock);
    constexpr int PER = 4;                            // a thread's keys in flight
    for (int b0 = beg; b0 < end; b0 += PER * kSortThreads) {
        uint32_t k[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) k[q] = 0;
        for (int i = 0; i < g.count; ++i) {           // uniform
            if (g.base[i] >= b0 + PER * kSortThreads || g.base[i + 1] <= b0) continue;
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int e = b0 + q * kSortThreads + (int)threadIdx.x;
                if (e < end && e >= g.base[i] && e < g.base[i + 1])
                    k[q] = g.kbase[i] + sort_key(g, g.it[i], e - g.base[i]);
            }
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = b0 + q * kSortThreads + (int)threadIdx.x;
            if (e < end) keys[e] = k[q];
            if (e - lane < end) count_runs(k[q], e < end, end - (e - lane), 0, (uint32_t)nd - 1u, h);     // uniform per wave
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += blockDim.x) hist[(size_t)d * nblocks + blockIdx.x] = h[d];
}

// Per-block digit histogram of dbits-bit digits, stored digit-major:
// hist[d * nblocks + b].  Equal digits in consecutive lanes (the keys are
// mostly in order after the first sort) count with one LDS atomic per run.
template <int PT>
__global__ __launch_bounds__(kSortThreads) void k_hist(const uint32_t *keys, int np, int shift, int dbits,
                                                       int nblocks, uint32_t *hist)
{
    __shared__ uint32_t h[1 << kMaxDigitBits];
    const int nd = 1 << dbits;
    const uint32_t mask = (uint32_t)nd - 1u;
    for (int d = threadIdx.x; d < nd; d += blockDim.x) h[d] = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int beg = blockIdx.x * (PT * kSortThreads);
    const int end = min(np, beg + PT * kSortThreads);
    constexpr int PER = PT;                           // a thread's keys, all in flight
    uint32_t k[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = beg + q * kSortThreads + (int)threadIdx.x;
        k[q] = e < end ? keys[e] : 0u;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e0 = beg + q * kSortThreads + (int)threadIdx.x - lane;
        if (e0 < end) count_runs(k[q], e0 + lane < end, end - e0, shift, mask, h);     // uniform per wave
    }
    __syncthreads();
    for (int d = threadIdx.x; d < nd; d += blockDim.x) hist[(size_t)d * nblocks + blockIdx.x] = h[d];
}

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t &total)
{
    // sh: blockDim.x/64 entries
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) sh[wv] = x;
    __syncthreads();
    int nw = blockDim.x >> 6;
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int k = 0; k < nw; ++k) {
            uint32_t t = sh[k];
            sh[k] = run;
            run += t;
        }
        sh[nw] = run;
    }
    __syncthreads();
    uint32_t r = x - v + sh[wv];
    total = sh[nw];
    __syncthreads();
    return r;
}

// Three-kernel exclusive scan of hist[0..m): segment sums, scan of the sums,
// segment scan with offsets.
__global__ __launch_bounds__(256) void k_scan_reduce(const uint32_t *in, long m, long seg, uint32_t *part)
{
    long beg = blockIdx.x * seg, end = min(m, beg + seg);
    uint32_t s = 0;
    for (long i = beg + threadIdx.x; i < end; i += blockDim.x) s += in[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    __shared__ uint32_t w[4];
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = w[0] + w[1] + w[2] + w[3];
}

__global__ __launch_bounds__(kScanBlocks) void k_scan_parts(uint32_t *part, int nparts)
{
    __shared__ uint32_t sh[kScanBlocks / 64 + 1];
    uint32_t v = threadIdx.x < nparts ? part[threadIdx.x] : 0u;
    uint32_t total;
    uint32_t r = block_exclusive_scan(v, sh, total);
    if (threadIdx.x < nparts) part[threadIdx.x] = r;
}

__global__ __launch_bounds__(256) void k_scan_apply(const uint32_t *in, long m, long seg, const uint32_t *part,
                                                    uint32_t *out)
{
    __shared__ uint32_t sh[256 / 64 + 1];
    long beg = blockIdx.x * seg, end = min(m, beg + seg);
    uint32_t run = part[blockIdx.x];
    for (long base = beg; base < end; base += blockDim.x) {
        long i = base + threadIdx.x;
        uint32_t v = i < end ? in[i] : 0u;
        uint32_t total;
        uint32_t r = block_exclusive_scan(v, sh, total);
        if (i < end) out[i] = run + r;
        run += total;
    }
}

// Stable scatter of one radix pass of dbits-bit digits (per-wave digit
// cursors in dynamic LDS: kSortWaves << dbits words).  idx_in == nullptr
// means identity (first pass).  A wave holds its keys and indices in registers:
// one read of each, all of them in flight (the keys were read twice, 64 at a
// time: 179 to 132 us per pass over 2^24 pairs).  offs: the scanned histogram, or (raw) the histogram
// itself, which few enough blocks sum up for themselves.
template <int PT>
__global__ __launch_bounds__(kSortThreads) void k_scatter(const uint32_t *keys_in, const uint32_t *idx_in,
                                                          uint32_t *keys_out, uint32_t *idx_out, int np,
                                                          int shift, int dbits, int nblocks, const uint32_t *offs,
                                                          bool raw)
{
    extern __shared__ uint32_t wcs[];
    __shared__ uint32_t sh[kSortWaves + 1];
    constexpr int PER = PT, kPerWave = 64 * PT;
    const int nd = 1 << dbits;
    const uint32_t mask = (uint32_t)nd - 1u;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t *wc = wcs + wv * nd;                     // this wave's cursors
    const int wbeg = (int)blockIdx.x * (PT * kSortThreads) + wv * kPerWave;
    const int wend = min(np, wbeg + kPerWave);
    uint32_t kr[PER], ir[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = wbeg + 64 * i + lane;
        kr[i] = e < wend ? keys_in[e] : 0u;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = wbeg + 64 * i + lane;
        ir[i] = idx_in ? (e < wend ? idx_in[e] : 0u) : (uint32_t)e;
    }
    for (int e = threadIdx.x; e < kSortWaves * nd; e += blockDim.x) wcs[e] = 0;
    // first position of digit d of this block, thread d
    uint32_t first = 0;
    if (raw) {
        uint32_t all = 0;
        if ((int)threadIdx.x < nd)
#pragma unroll 8
            for (int b = 0; b < nblocks; ++b) {
                const uint32_t v = offs[(size_t)threadIdx.x * nblocks + b];
                first += b < (int)blockIdx.x ? v : 0u;
                all += v;
            }
        uint32_t total;
        first += block_exclusive_scan(all, sh, total);
    } else if ((int)threadIdx.x < nd) {
        first = offs[(size_t)threadIdx.x * nblocks + blockIdx.x];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e0 = wbeg + 64 * i;
        if (e0 < wend) count_runs(kr[i], e0 + lane < wend, wend - e0, shift, mask, wc);      // uniform per wave
    }
    __syncthreads();
    if ((int)threadIdx.x < nd) {
        uint32_t run = first;
        for (int w = 0; w < kSortWaves; ++w) {
            uint32_t t = wcs[w * nd + threadIdx.x];
            wcs[w * nd + threadIdx.x] = run;
            run += t;
        }
    }
    __syncthreads();
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (wbeg + 64 * i >= wend) break;             // uniform per wave
        const bool valid = wbeg + 64 * i + lane < wend;
        const uint32_t k = kr[i];
        uint32_t d = (k >> shift) & mask;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < dbits; ++b) {
            uint64_t m = __ballot(valid && ((d >> b) & 1u));
            peers &= ((d >> b) & 1u) ? m : ~m;
        }
        if (valid) {
            uint32_t rank = (uint32_t)__popcll(peers & lt);
            uint32_t dst = wc[d] + rank;
            keys_out[dst] = k;
            idx_out[dst] = ir[i];
        }
        // make every lane's read of wc[d] happen before the update
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        if (valid) {
            // highest lane of each peer group advances its digit's cursor
            uint64_t higher = peers & ~(lt | (1ull << lane));
            if (higher == 0) wc[d] += (uint32_t)__popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Every SoA array of an item moved by one permutation in one pass: the
// permutation is read once, and all of a position's loads are in flight
// before its stores.  With perm2 the source of position r is
// perm2[perm[r]] (run order: new position -> sorted position -> source).
// Positions and sources count from the group's first particle; items share a
// launch where they have the same arrays.  With run tables the first blocks list
// the work units, which nothing else in the launch waits for.
struct PermArrays {
    int first[kGroup + 1];   // positions of the launch's items, counted from the group's first particle
    const void *src[kGroup][SortArgs::kMaxArrays];
    void *dst[kGroup][SortArgs::kMaxArrays];
    int wide;                // bit k: array k has 8-byte elements
    int n, count;
};
struct UnitLists {
    int count;
    int32_t *runs[kGroup];
    int np[kGroup], ntiles[kGroup];
};
constexpr int kPermThreads = 256;
__device__ __forceinline__ void unit_list(int32_t *runs, int np, int ntiles);

__global__ __launch_bounds__(kPermThreads) void k_permute_all(const uint32_t *__restrict__ perm,
                                                              const uint32_t *__restrict__ perm2, PermArrays pa,
                                                              UnitLists ul)
{
    if ((int)blockIdx.x < ul.count) {                // uniform
        unit_list(ul.runs[blockIdx.x], ul.np[blockIdx.x], ul.ntiles[blockIdx.x]);
        return;
    }
    // two positions per iteration, every load of both issued before any store
    const int stride = ((int)gridDim.x - ul.count) * kPermThreads;
    const int b0 = ((int)blockIdx.x - ul.count) * kPermThreads + (int)threadIdx.x;
    for (int it = 0; it < pa.count; ++it) {
        const int base = pa.first[it], end = pa.first[it + 1];
        for (int r0 = base + b0; r0 < end; r0 += 2 * stride) {
            const int r1 = r0 + stride;
            const bool two = r1 < end;
            uint32_t q0 = perm[r0], q1 = two ? perm[r1] : q0;
            if (perm2) {
                q0 = perm2[q0];
                q1 = perm2[q1];
            }
            q0 -= (uint32_t)base;
            q1 -= (uint32_t)base;
            unsigned long long v0[SortArgs::kMaxArrays], v1[SortArgs::kMaxArrays];
#pragma unroll
            for (int k = 0; k < SortArgs::kMaxArrays; ++k) {
                if (k < pa.n) {
                    if ((pa.wide >> k) & 1) {
                        v0[k] = ((const unsigned long long *)pa.src[it][k])[q0];
                        v1[k] = ((const unsigned long long *)pa.src[it][k])[q1];
                    } else {
                        v0[k] = ((const uint32_t *)pa.src[it][k])[q0];
                        v1[k] = ((const uint32_t *)pa.src[it][k])[q1];
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < SortArgs::kMaxArrays; ++k) {
                if (k < pa.n) {
                    if ((pa.wide >> k) & 1) {
                        ((unsigned long long *)pa.dst[it][k])[r0 - base] = v0[k];
                        if (two) ((unsigned long long *)pa.dst[it][k])[r1 - base] = v1[k];
                    } else {
                        ((uint32_t *)pa.dst[it][k])[r0 - base] = (uint32_t)v0[k];
                        if (two) ((uint32_t *)pa.dst[it][k])[r1 - base] = (uint32_t)v1[k];
                    }
                }
            }
        }
    }
}

// Spectral rows (nb float64 per particle, particle-major): destination row r
// takes source row perm[r] (perm2[perm[r]] with perm2); one wave per row.
__global__ __launch_bounds__(256) void k_permute_rows(const uint32_t *perm, const uint32_t *perm2, int base, int np, int nb,
                                                      const double *src0, double *dst0, const double *src1,
                                                      double *dst1)
{
    const int lane = threadIdx.x & 63;
    for (int r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6; r < np; r += (gridDim.x * blockDim.x) >> 6) {
        const uint32_t q = (perm2 ? perm2[perm[base + r]] : perm[base + r]) - (uint32_t)base;
        const long s = (long)q * nb, d = (long)r * nb;
        for (int i = lane; i < nb; i += 64) {
            dst0[d + i] = src0[s + i];
            dst1[d + i] = src1[s + i];
        }
    }
}

// Every array of the items args[0 .. g.count) moved by the group's
// permutation, and (lists) their work units listed.
static void permute_arrays(Ctx *c, const SortGroup &g, const SortArgs *args, const uint32_t *perm, const uint32_t *perm2,
                           bool lists)
{
    for (int i = 0; i < g.count; ++i) {
        const SortArgs &a = args[i];
        if (a.nb <= 0) continue;
        const int grid = std::max(1, std::min((a.np + 3) / 4, 64 * c->num_cu));
        hipLaunchKernelGGL(k_permute_rows, dim3(grid), dim3(256), 0, c->stream, perm, perm2, g.base[i], a.np, a.nb,
                           a.rsrc[0], a.rdst[0], a.rsrc[1], a.rdst[1]);
        c->stats[0]++;
    }
    for (int i0 = 0, i1 = 0; i0 < g.count; i0 = i1) {
        PermArrays pa;
        UnitLists ul;
        memset(&pa, 0, sizeof(pa));
        memset(&ul, 0, sizeof(ul));
        pa.n = args[i0].narrays;
        for (int k = 0; k < pa.n; ++k)
            if (args[i0].esize[k] == 8) pa.wide |= 1 << k;
        for (i1 = i0; i1 < g.count; ++i1) {
            const SortArgs &a = args[i1];
            int wide = 0;
            for (int k = 0; k < a.narrays; ++k)
                if (a.esize[k] == 8) wide |= 1 << k;
            if (a.narrays != pa.n || wide != pa.wide) break;
            const int m = i1 - i0;
            pa.first[m] = g.base[i1];
            pa.first[m + 1] = g.base[i1 + 1];
            for (int k = 0; k < a.narrays; ++k) {
                pa.src[m][k] = a.src[k];
                pa.dst[m][k] = a.dst[k];
            }
            if (lists) {
                ul.runs[ul.count] = a.runs;
                ul.np[ul.count] = a.np;
                ul.ntiles[ul.count++] = a.ntiles;
            }
        }
        pa.count = i1 - i0;
        const int np = g.base[i1] - g.base[i0];
        const int grid = std::min((np + kPermThreads - 1) / kPermThreads, 16 * c->num_cu) + ul.count;
        hipLaunchKernelGGL(k_permute_all, dim3(grid), dim3(kPermThreads), 0, c->stream, perm, perm2, pa, ul);
        c->stats[0]++;
    }
}

// First particle of every tile of every item (offsets within the item).
__global__ void k_tile_start(SortGroup g, const uint32_t *keys, int shift, int key_mode)
{
    for (int i = 0; i < g.count; ++i) {
        const SortItem &a = g.it[i];
        const uint32_t per = key_mode == PL_KEY_TILE || shift > 0 ? 1u : (uint32_t)(a.tile[0] * a.tile[1] * a.tile[2]);
        const uint32_t kb = g.kbase[i];
        const uint32_t *k = keys + g.base[i];
        for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < a.np; q += gridDim.x * blockDim.x) {
            const int t = (int)(((k[q] - kb) >> shift) / per);
            const int prev = q > 0 ? (int)(((k[q - 1] - kb) >> shift) / per) : -1;
            for (int m = prev + 1; m <= t; ++m) a.tile_start[m] = q;
            if (q == a.np - 1)
                for (int m = t + 1; m <= a.ntiles; ++m) a.tile_start[m] = a.np;
        }
    }
}

// First sorted position of every cell (keys sorted by tile * cells_per_tile +
// cell in tile); cells without particles are never read.
__global__ void k_cell_start(const uint32_t *keys, int np, int32_t *cs)
{
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < np; r += gridDim.x * blockDim.x)
        if (r == 0 || keys[r] != keys[r - 1]) cs[keys[r]] = r;
}

// Rank-interleaved key of sorted position r: its rank among the particles of
// its cell (positions are in stable order, so this is the number of earlier
// particles of the same cell), capped at 2^rank_bits - 1, between tile and cell.
// The input key is tile * per_tile + cell in tile; per_tile <= 2^cell_bits.
__global__ void k_rank_keys(uint32_t *keys, int np, const int32_t *cs, int per_tile, int cell_bits, int rank_bits)
{
    const uint32_t rmax = (1u << rank_bits) - 1u, pt = (uint32_t)per_tile;
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < np; r += gridDim.x * blockDim.x) {
        uint32_t k = keys[r];
        uint32_t rank = min((uint32_t)(r - cs[k]), rmax);
        uint32_t tile = k / pt, local = k - tile * pt;
        keys[r] = (tile << (rank_bits + cell_bits)) | (rank << cell_bits) | local;
    }
}

// Run table of one tile per block (keys sorted by tile * cells_per_tile + cell
// in tile): the particles of every cell are cut into runs of up to kRunLen
// consecutive positions, and the runs are listed by (index of the run inside
// its cell, cell), so consecutive runs belong to distinct cells.  Entry:
// (first position << 2) | (length - 1), stored from runs[tile_start[t]];
// the tile's run count goes to runs[np + t].  With perm_out (run order) the
// runs are laid out one after another in table order from tile_start[t]: the
// entries hold those positions, and perm_out[new position] = sorted position
// (the permute pass composes it with the sort's permutation).  The first
// kRunsDense rounds (run index inside the cell) take one block scan each; the
// cells with more runs (crowded cells of clumped particles, up to hundreds of
// rounds) are then listed in cell order and the block's waves take the
// remaining rounds in turn, each dropping a cell from its own list after the
// cell's last run in that wave's rounds.
constexpr int kRunsBuildThreads = 256;
constexpr int kRunsDense = 8;
static_assert(kRunLen == 4, "the crowded rounds' ballot prefix sums take run shortfalls of two bits");
__global__ __launch_bounds__(kRunsBuildThreads) void k_runs_build(SortGroup g, const uint32_t *all_keys,
                                                                  uint32_t *all_perm)
{
    // this block's item (its tiles are the blocks from tbase), keys and permutation
    int im = 0;
    while (im + 1 < g.count && (int)blockIdx.x >= g.tbase[im + 1]) ++im;
    const SortItem &a = g.it[im];
    const int np = a.np, per_tile = a.tile[0] * a.tile[1] * a.tile[2];
    const int32_t *ts = a.tile_start;
    int32_t *runs = a.runs;
    const uint32_t *keys = all_keys + g.base[im];
    uint32_t *perm_out = all_perm ? all_perm + g.base[im] : nullptr;
    const uint32_t pbase = (uint32_t)g.base[im];

    __shared__ int cnt[kRunsMaxTileCells];
    __shared__ int first[kRunsMaxTileCells];
    __shared__ int4 crowd[kRunsMaxTileCells];
    __shared__ int wl[(kRunsBuildThreads / 64) * kRunsMaxTileCells];
    __shared__ uint32_t sh[kRunsBuildThreads / 64 + 1];
    __shared__ int s_max;
    const int cpt = (per_tile + kRunsBuildThreads - 1) / kRunsBuildThreads;   // cells per thread
    const int c0 = threadIdx.x * cpt, c1 = min(per_tile, c0 + cpt);
    {
        const int t = (int)blockIdx.x - g.tbase[im];
        const int beg = ts[t], end = ts[t + 1];
        for (int c = threadIdx.x; c < per_tile; c += blockDim.x) cnt[c] = 0;
        if (threadIdx.x == 0) s_max = 0;
        __syncthreads();
        // first sorted position and end of every cell from the key boundaries
        // (the keys are sorted: no atomics, crowded cells included).  Each
        // thread takes four consecutive keys per 16-byte load and issues the
        // loads of KB such groups before using any.
        const uint32_t kb = g.kbase[im] + (uint32_t)t * (uint32_t)per_tile;
        {
            typedef uint32_t U4 __attribute__((ext_vector_type(4), aligned(4)));
            constexpr int KB = 8;
            const int bd = (int)blockDim.x;
            for (int p0 = beg + 4 * (int)threadIdx.x; p0 < end; p0 += 4 * KB * bd) {
                uint32_t kc[KB][4], kp[KB], kn[KB];
#pragma unroll
                for (int i = 0; i < KB; ++i) {
                    const int p = p0 + 4 * i * bd;
                    if (p + 4 <= end) {
                        const U4 v = *reinterpret_cast<const U4 *>(keys + p);
                        kc[i][0] = v[0];
                        kc[i][1] = v[1];
                        kc[i][2] = v[2];
                        kc[i][3] = v[3];
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; ++q) kc[i][q] = p + q < end ? keys[p + q] : ~0u;
                    }
                    kp[i] = p < end && p > beg ? keys[p - 1] : ~0u;
                    kn[i] = p + 4 < end ? keys[p + 4] : ~0u;
                }
#pragma unroll
                for (int i = 0; i < KB; ++i) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int p = p0 + 4 * i * bd + q;
                        const uint32_t k = kc[i][q];
                        const uint32_t before = q == 0 ? kp[i] : kc[i][q - 1];
                        const uint32_t after = q == 3 ? kn[i] : kc[i][q + 1];
                        const uint32_t loc = k - kb;
                        if (p < end && loc < (uint32_t)per_tile) {
                            if (before != k) first[loc] = p;
                            if (after != k) cnt[loc] = p + 1;        // one past the cell's last
                        }
                    }
                }
            }
        }
        __syncthreads();
        // counts, the largest run count and the tile's run count
        int mx = 0;
        uint32_t mruns = 0;
        for (int c = c0; c < c1; ++c) {
            if (cnt[c] > 0) cnt[c] -= first[c];
            mx = max(mx, (cnt[c] + kRunLen - 1) / kRunLen);
            mruns += (uint32_t)((cnt[c] + kRunLen - 1) / kRunLen);
        }
        uint32_t total, truns;
        block_exclusive_scan(mruns, sh, truns);
        atomicMax(&s_max, mx);
        __syncthreads();
        const int nb = s_max;
        const int nb0 = min(nb, kRunsDense);
        int base = 0, lbase = 0;
        for (int b = 0; b < nb0; ++b) {
            // runs (high half) and particles (low half) of this round before my
            // cells: at most 1024 runs and 4096 particles, so the halves never carry
            uint32_t here = 0;
            for (int c = c0; c < c1; ++c) {
                const int left = cnt[c] - b * kRunLen;
                if (left > 0) here += (1u << 16) | (uint32_t)min(kRunLen, left);
            }
            uint32_t pk = block_exclusive_scan(here, sh, total);
            int pos = (int)(pk >> 16), lpos = (int)(pk & 0xffffu);
            for (int c = c0; c < c1; ++c) {
                const int left = cnt[c] - b * kRunLen;
                if (left > 0) {
                    const int len = min(kRunLen, left);
                    const int src = first[c] + b * kRunLen;
                    const int dst = perm_out ? beg + lbase + lpos : src;
                    runs[beg + base + pos] = (dst << 2) | (len - 1);
                    if (perm_out)
                        for (int i = 0; i < len; ++i) perm_out[dst + i] = pbase + (uint32_t)(src + i);
                    ++pos;
                    lpos += len;
                }
            }
            base += (int)(total >> 16);
            lbase += (int)(total & 0xffffu);
        }
        if (nb > nb0) {
            // cells with more than nb0 runs, in cell order: (cell, first
            // sorted position, particle count)
            uint32_t mine_c = 0;
            for (int c = c0; c < c1; ++c) mine_c += cnt[c] > nb0 * kRunLen ? 1u : 0u;
            uint32_t k = block_exclusive_scan(mine_c, sh, total);
            for (int c = c0; c < c1; ++c)
                if (cnt[c] > nb0 * kRunLen) crowd[k++] = make_int4(c, first[c], cnt[c], 0);
            __syncthreads();
            // wave w takes rounds nb0 + w, + NW, ... with its own list of the
            // cells that still have a run in its next round (in cell order).
            // Its first base follows from the rounds before it; after each
            // round it adds the runs and particles of that round and of the
            // NW - 1 rounds the other waves take, all counted on its list.
            constexpr int NW = kRunsBuildThreads / 64;
            const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
            const uint64_t lt = (1ull << lane) - 1ull;
            const int K = (int)total;
            int *mylist = wl + w * kRunsMaxTileCells;
            // runs and particles of one round b on a chunk of cells with counts n
            auto round_counts = [&](bool in, int n, int b, int &r, int &q) {
                const bool a = in && n > b * kRunLen;
                const int d = a ? kRunLen - min(kRunLen, n - b * kRunLen) : 0;
                const uint64_t am = __ballot(a), d0 = __ballot(d & 1), d1 = __ballot(d & 2);
                r += __popcll(am);
                q += kRunLen * __popcll(am) - __popcll(d0) - 2 * __popcll(d1);
            };
            int wb = base, wl0 = lbase, Kw = 0;
            for (int j0 = 0; j0 < K; j0 += 64) {
                const int j = j0 + lane;
                const bool in = j < K;
                const int n = in ? crowd[j].z : 0;
                for (int k = 0; k < w; ++k) round_counts(in, n, nb0 + k, wb, wl0);
                const bool keep = in && n > (nb0 + w) * kRunLen;
                const uint64_t km = __ballot(keep);
                if (keep) mylist[Kw + __popcll(km & lt)] = j;
                Kw += __popcll(km);
            }
            for (int b = nb0 + w; Kw > 0; b += NW) {
                int kept = 0, rpos = 0, ppos = 0, radd = 0, padd = 0;
                for (int j0 = 0; j0 < Kw; j0 += 64) {
                    const int j = j0 + lane;
                    const bool in = j < Kw;
                    const int idx = in ? mylist[j] : 0;
                    const int4 e = in ? crowd[idx] : make_int4(0, 0, 0, 0);
                    const int left = e.z - b * kRunLen;
                    const int len = in ? min(kRunLen, left) : 0;
                    // prefix sums of the run lengths from ballots: kRunLen per
                    // active lane minus the shortfall (0..3) of last runs
                    const int d = in ? kRunLen - len : 0;
                    const uint64_t am = __ballot(in);
                    const uint64_t d0 = __ballot(d & 1), d1 = __ballot(d & 2);
                    const int lpre = kRunLen * __popcll(am & lt) - __popcll(d0 & lt) - 2 * __popcll(d1 & lt);
                    if (in) {
                        const int pos = rpos + __popcll(am & lt);
                        const int src = e.y + b * kRunLen;
                        const int dst = perm_out ? beg + wl0 + ppos + lpre : src;
                        runs[beg + wb + pos] = (dst << 2) | (len - 1);
                        if (perm_out)
                            for (int i = 0; i < len; ++i) perm_out[dst + i] = pbase + (uint32_t)(src + i);
                    }
                    rpos += __popcll(am);
                    ppos += kRunLen * __popcll(am) - __popcll(d0) - 2 * __popcll(d1);
                    for (int k = 1; k < NW; ++k) round_counts(in, e.z, b + k, radd, padd);
                    // the list is read ahead of every write (kept <= j0)
                    const bool keep = in && e.z > (b + NW) * kRunLen;
                    const uint64_t km = __ballot(keep);
                    if (keep) mylist[kept + __popcll(km & lt)] = idx;
                    kept += __popcll(km);
                }
                wb += rpos + radd;
                wl0 += ppos + padd;
                Kw = kept;
            }
            base = (int)truns;
        }
        if (threadIdx.x == 0) runs[np + t] = base;
        __syncthreads();
    }
}

// Work units of the run-based kernel (by one block).  With P = max(ceil(total
// runs / kRunsSplit), kRunsMinPiece), a tile of c runs becomes ceil(c / P)
// pieces (an empty tile none), so at most ntiles + kRunsSplit units exist.
// Tiles cut into pieces or holding more than twice the mean run count go
// first, by decreasing runs per piece (ties by tile index), each followed by
// its pieces in order; then every other non-empty tile in index order.  The
// first kRankMax such tiles (in index order) are ranked; later ones keep index
// order.  Largest-first claiming keeps a crowded tile from finishing last on
// its CU, and splitting keeps one tile from outweighing a CU's share of the
// step.  Every loop that contains a block scan has the same trip count in all
// threads.  A thread takes kUnitTiles consecutive tiles per scan: a scan costs
// about 1.5 us whatever it adds up, and the list of
// 32768 tiles, one per thread and scan, held up the launch that it is part of (256^3
// cells, 4e6 particles: a sort 853 us with a launch of 1024 threads of its own, 995 us
// beside the moves, 783 us with eight tiles per thread).
constexpr int kRankMax = 1024;
constexpr int kUnitTiles = 8;
__device__ __forceinline__ void unit_list(int32_t *runs, int np, int ntiles)
{
    __shared__ uint32_t sh[kPermThreads / 64 + 1];
    __shared__ int rk_tile[kRankMax];
    __shared__ int rk_cnt[kRankMax];
    __shared__ int rk_k[kRankMax];
    __shared__ int by_rank[kRankMax];
    __shared__ unsigned long long s_total;
    const int32_t *cnt = runs + np;
    int32_t *units = runs + runs_units_at(np, ntiles);
    const long long cap = (long long)ntiles + kRunsSplit;
    if (threadIdx.x == 0) s_total = 0ull;
    __syncthreads();
    unsigned long long mine = 0;
    for (int t0 = threadIdx.x; t0 < ntiles; t0 += kUnitTiles * (int)blockDim.x) {
        int c[kUnitTiles];                               // (all of them in flight)
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) {
            const int t = t0 + q * (int)blockDim.x;
            c[q] = t < ntiles ? cnt[t] : 0;
        }
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) mine += (unsigned long long)max(c[q], 0);
    }
    atomicAdd(&s_total, mine);
    __syncthreads();
    const long long total = (long long)s_total;
    const long long pz = max((total + kRunsSplit - 1) / kRunsSplit, (long long)kRunsMinPiece);
    const long long thr = 2 * (total / max(ntiles, 1)) + 1;
    // (runs of an item < 2^29 and pz < 2^20: 32 bits hold the sum)
    auto pieces = [&](int c) -> uint32_t { return ((uint32_t)c + (uint32_t)pz - 1u) / (uint32_t)pz; };
    // this thread's tiles from t on: pieces, and which are split or heavy (bits)
    auto look = [&](int t, uint32_t k[kUnitTiles], int c[kUnitTiles]) -> uint32_t {
        uint32_t heavy = 0;
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) c[q] = t + q < ntiles ? max(cnt[t + q], 0) : 0;
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) {
            k[q] = pieces(c[q]);
            heavy |= (k[q] >= 2 || (long long)c[q] > thr ? 1u : 0u) << q;
        }
        return heavy;
    };
    const int stride = (int)blockDim.x * kUnitTiles;
    typedef int32_t I2 __attribute__((ext_vector_type(2), aligned(4)));
    auto emit = [&](long long at, int t, int k) {
        for (int p = 0; p < k; ++p)
            if (at + p < cap) *reinterpret_cast<I2 *>(units + 2 * (at + p)) = I2{t, p | (k << 16)};
    };
    // ranked tiles: the first kRankMax split or heavy tiles in index order
    uint32_t hbase = 0;
    for (int t0 = 0; t0 < ntiles; t0 += stride) {
        const int t = t0 + (int)threadIdx.x * kUnitTiles;
        uint32_t k[kUnitTiles];
        int c[kUnitTiles];
        const uint32_t heavy = look(t, k, c);
        uint32_t tot;
        uint32_t hp = hbase + block_exclusive_scan((uint32_t)__popc(heavy), sh, tot);
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) {
            if (!((heavy >> q) & 1u)) continue;
            if (hp < (uint32_t)kRankMax) {
                rk_tile[hp] = t + q;
                rk_cnt[hp] = c[q];
                rk_k[hp] = (int)k[q];
            }
            ++hp;
        }
        hbase += tot;
    }
    const int nh = (int)min(hbase, (uint32_t)kRankMax);
    __syncthreads();
    // rank by decreasing runs per piece (cnt / k, compared exactly), ties by tile
    for (int i = threadIdx.x; i < nh; i += blockDim.x) {
        const long long ci = rk_cnt[i], ki = rk_k[i];
        int rank = 0;
        for (int j = 0; j < nh; ++j) {
            const long long a = (long long)rk_cnt[j] * ki, b = ci * (long long)rk_k[j];
            rank += a > b || (a == b && rk_tile[j] < rk_tile[i]);
        }
        by_rank[rank] = i;
    }
    __syncthreads();
    uint32_t nranked = 0;
    for (int r0 = 0; r0 < nh; r0 += blockDim.x) {
        const int r = r0 + (int)threadIdx.x;
        const int i = r < nh ? by_rank[r] : 0;
        const uint32_t k = r < nh ? (uint32_t)rk_k[i] : 0u;
        uint32_t tot;
        const uint32_t at = nranked + block_exclusive_scan(k, sh, tot);
        if (r < nh) emit(at, rk_tile[i], (int)k);
        nranked += tot;
    }
    // every other non-empty tile in index order
    uint32_t hb = 0;
    long long lb = nranked;
    for (int t0 = 0; t0 < ntiles; t0 += stride) {
        const int t = t0 + (int)threadIdx.x * kUnitTiles;
        uint32_t k[kUnitTiles];
        int c[kUnitTiles];
        const uint32_t heavy = look(t, k, c);
        uint32_t toth, totl;
        uint32_t hp = hb + block_exclusive_scan((uint32_t)__popc(heavy), sh, toth);
        uint32_t mine_l = 0;
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) {
            const bool h = (heavy >> q) & 1u;
            if (h && hp < (uint32_t)kRankMax) k[q] = 0;      // ranked
            hp += h ? 1u : 0u;
            mine_l += k[q];
        }
        long long at = lb + block_exclusive_scan(mine_l, sh, totl);
#pragma unroll
        for (int q = 0; q < kUnitTiles; ++q) {
            if (k[q]) emit(at, t + q, (int)k[q]);
            at += k[q];
        }
        hb += toth;
        lb += totl;
    }
    if (threadIdx.x == 0) runs[runs_count_at(np, ntiles)] = (int32_t)min(lb, cap);
}

// (an item without particles)
__global__ __launch_bounds__(kPermThreads) void k_unit_list(int32_t *runs, int np, int ntiles) { unit_list(runs, np, ntiles); }

__global__ void k_fill_i32(int32_t *p, int n, int v)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

int64_t sort_hist_entries(int64_t np) { return kSortHist(np); }

// LSD radix passes over the low `bits` bits of keys[src] with indices idx[src]
// (identity when `identity`); returns the buffer index holding the result.
// Digits of kMaxDigitBits bits, the last pass taking only the bits left.
// (Wider digits, 11 bits in two passes for 21-bit keys, were slower: the
// per-block digit tables cost more than the pass they save.)
// first_hist: the first pass's histogram is in c->hist already.  With few
// blocks the scatter sums the histogram up itself instead of three scan
// launches.
constexpr int kRawBlocks = 128;
static int radix_passes(Ctx *c, int np, int src, bool identity, int bits, bool first_hist)
{
    hipStream_t s = c->stream;
    const int nblocks = sort_blocks(np);
    const bool big = sort_per(np) == kPerThread;
    const bool raw = nblocks <= kRawBlocks;
    bits = std::max(bits, 1);
    const int width = kMaxDigitBits;
    const int npass = (bits + width - 1) / width;
    for (int pass = 0; pass < npass; ++pass) {
        const int shift = width * pass;
        const int dbits = std::min(width, bits - shift);
        if (pass > 0 || !first_hist) {
            hipLaunchKernelGGL(big ? k_hist<kPerThread> : k_hist<kPerThreadSmall>, dim3(nblocks), dim3(kSortThreads), 0, s, c->keys[src], np, shift, dbits, nblocks,
                               c->hist);
            c->stats[0]++;
        }
        if (!raw) {
            const long m = (long)nblocks << dbits;
            const long seg = (m + kScanBlocks - 1) / kScanBlocks;
            const int nparts = (int)((m + seg - 1) / seg);
            uint32_t *part = c->hist_scan + m;
            hipLaunchKernelGGL(k_scan_reduce, dim3(nparts), dim3(256), 0, s, c->hist, m, seg, part);
            hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(kScanBlocks), 0, s, part, nparts);
            hipLaunchKernelGGL(k_scan_apply, dim3(nparts), dim3(256), 0, s, c->hist, m, seg, part, c->hist_scan);
            c->stats[0] += 3;
        }
        hipLaunchKernelGGL(big ? k_scatter<kPerThread> : k_scatter<kPerThreadSmall>, dim3(nblocks), dim3(kSortThreads), (size_t)(kSortWaves << dbits) * 4, s,
                           c->keys[src], (identity && pass == 0) ? (const uint32_t *)nullptr : c->idx[src],
                           c->keys[1 - src], c->idx[1 - src], np, shift, dbits, nblocks, raw ? c->hist : c->hist_scan,
                           raw);
        c->stats[0]++;
        src = 1 - src;
    }
    return src;
}

// Keys of a group's particles by `key_mode`, sorted: the buffer index that holds
// them and their sources.
static int sort_keys(Ctx *c, const SortGroup &g, uint64_t keys)
{
    const int bits = std::max(bits_for(keys), 1), nblocks = sort_blocks(g.total);
    hipLaunchKernelGGL(sort_per(g.total) == kPerThread ? k_keys<kPerThread> : k_keys<kPerThreadSmall>, dim3(nblocks), dim3(kSortThreads), 0, c->stream, g, c->keys[0],
                       std::min(kMaxDigitBits, bits), nblocks, c->hist);
    c->stats[0]++;
    return radix_passes(c, g.total, 0, true, bits, true);
}

// The group of the items args[0 .. count), each with particles; the number of
// distinct keys.
static uint64_t make_group(const SortArgs *args, int count, int key_mode, SortGroup &g)
{
    memset(&g, 0, sizeof(g));
    g.count = count;
    g.prec = args[0].prec;
    g.ndim = args[0].ndim;
    g.key_mode = key_mode;
    uint64_t keys = 0;
    for (int i = 0; i < count; ++i) {
        const SortArgs &a = args[i];
        SortItem &s = g.it[i];
        for (int k = 0; k < 3; ++k) {
            s.n[k] = a.n[k];
            s.tile[k] = a.tile[k];
            s.x[k] = a.x[k];
        }
        s.np = a.np;
        s.ntiles = a.ntiles;
        s.cell = a.cell;
        s.tile_start = a.tile_start;
        s.runs = a.runs;
        g.kbase[i] = (uint32_t)keys;
        g.base[i + 1] = g.base[i] + a.np;
        g.tbase[i + 1] = g.tbase[i] + a.ntiles;
        keys += (uint64_t)a.ntiles * (key_mode == PL_KEY_TILE ? 1 : a.tile[0] * a.tile[1] * a.tile[2]);
    }
    g.total = g.base[count];
    return keys;
}

int bins_buffer(int ntiles)
{
    const int bits = std::max(bits_for((uint64_t)ntiles), 1);
    return ((bits + kMaxDigitBits - 1) / kMaxDigitBits) & 1;
}

hipError_t launch_bins(Ctx *c, const ItemDesc &it)
{
    SortArgs a;
    memset(&a, 0, sizeof(a));
    a.prec = c->d.prec;
    a.ndim = c->d.ndim;
    a.key_mode = PL_KEY_TILE;
    for (int k = 0; k < 3; ++k) {
        a.n[k] = it.n[k];
        a.tile[k] = it.tile[k];
        a.x[k] = a.prec == PL_F64 && k < a.ndim ? (const double *)it.x[k] : nullptr;
    }
    a.np = it.np;
    a.ntiles = it.ntiles;
    a.cell = it.cell;
    a.tile_start = it.tile_start;
    SortGroup g;
    const uint64_t keys = make_group(&a, 1, PL_KEY_TILE, g);
    const int src = sort_keys(c, g, keys);
    hipLaunchKernelGGL(k_tile_start, dim3(std::min((a.np + 255) / 256, 16 * c->num_cu)), dim3(256), 0, c->stream, g,
                       c->keys[src], 0, (int)PL_KEY_TILE);
    c->stats[0]++;
    return hipGetLastError();
}

static hipError_t sort_empty(Ctx *c, const SortArgs &a)
{
    const int grid = std::max(1, (a.ntiles + 256) / 256);
    hipLaunchKernelGGL(k_fill_i32, dim3(grid), dim3(256), 0, c->stream, a.tile_start, a.ntiles + 1, 0);
    c->stats[0]++;
    if (a.runs) {
        hipLaunchKernelGGL(k_fill_i32, dim3(grid), dim3(256), 0, c->stream, a.runs, a.ntiles, 0);
        hipLaunchKernelGGL(k_unit_list, dim3(1), dim3(kPermThreads), 0, c->stream, a.runs, 0, a.ntiles);
        c->stats[0] += 2;
    }
    return hipGetLastError();
}

static hipError_t sort_group(Ctx *c, const SortArgs *args, int count)
{
    hipStream_t s = c->stream;
    const int mode = args[0].key_mode;
    SortGroup g;
    const int grid_of = 16 * c->num_cu;
    int src, shift = 0;
    if (mode == PL_KEY_TILE_RANK) {
        // (one item) phase 1: stable sort by (tile, cell); phase 2: stable sort
        // by (tile, rank in cell, cell) on top of it
        const SortArgs &a = args[0];
        const int per_tile_cells = a.tile[0] * a.tile[1] * a.tile[2], grid_e = std::min((a.np + 255) / 256, grid_of);
        src = sort_keys(c, g, make_group(args, 1, PL_KEY_TILE_CELL, g));
        const int cb = bits_for((uint64_t)per_tile_cells), tb = bits_for((uint64_t)a.ntiles);
        const int rb = std::min(10, 32 - tb - cb);
        hipLaunchKernelGGL(k_cell_start, dim3(grid_e), dim3(256), 0, s, c->keys[src], a.np, c->cell_start);
        hipLaunchKernelGGL(k_rank_keys, dim3(grid_e), dim3(256), 0, s, c->keys[src], a.np, c->cell_start,
                           per_tile_cells, cb, rb);
        c->stats[0] += 2;
        src = radix_passes(c, a.np, src, false, tb + rb + cb, false);
        shift = rb + cb;
    } else {
        const uint64_t keys = make_group(args, count, mode, g);
        src = sort_keys(c, g, keys);
    }
    const bool runs = args[0].runs != nullptr, order = mode == PL_KEY_TILE_RUN;
    if (order && !runs) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_tile_start, dim3(std::min((g.total + 255) / 256, grid_of)), dim3(256), 0, s, g, c->keys[src], shift,
                       mode);
    c->stats[0]++;
    if (runs) {
        // one block per tile: a crowded tile's rounds do not hold up others
        hipLaunchKernelGGL(k_runs_build, dim3(std::max(g.tbase[g.count], 1)), dim3(kRunsBuildThreads), 0, s, g, c->keys[src],
                           order ? c->idx[1 - src] : nullptr);
        c->stats[0]++;
    }
    // run order: every array moved from its place before the sort straight there
    if (order) permute_arrays(c, g, args, c->idx[1 - src], c->idx[src], true);
    else permute_arrays(c, g, args, c->idx[src], nullptr, runs);
    return hipGetLastError();
}

// What the sort of an item reads and writes in the caller's memory.
static int sort_memory(const SortArgs &a, GroupMemory::Range *r)
{
    static_assert(2 * SortArgs::kMaxArrays + 6 <= GroupMemory::kPerItem, "ranges of an item");
    int n = 0;
    auto add = [&](const void *p, size_t bytes, bool write) {
        const uintptr_t b = (uintptr_t)p;
        r[n++] = GroupMemory::Range{b, b + bytes, 0, write};
    };
    for (int k = 0; k < a.narrays; ++k) {
        add(a.src[k], (size_t)a.np * a.esize[k], false);
        add(a.dst[k], (size_t)a.np * a.esize[k], true);
    }
    for (int k = 0; k < 2 && a.nb > 0; ++k) {
        add(a.rsrc[k], (size_t)a.np * a.nb * sizeof(double), false);
        add(a.rdst[k], (size_t)a.np * a.nb * sizeof(double), true);
    }
    add(a.tile_start, ((size_t)a.ntiles + 1) * sizeof(int32_t), true);
    if (a.runs) add(a.runs, (size_t)PL_RUNS_LEN(a.np, a.ntiles) * sizeof(int32_t), true);
    return n;
}

hipError_t launch_sort(Ctx *c, const SortArgs *args, int count, int64_t cap)
{
    for (int i0 = 0, i1 = 0; i0 < count; i0 = i1) {
        i1 = i0 + 1;
        if (args[i0].np == 0) {
            const hipError_t e = sort_empty(c, args[i0]);
            if (e != hipSuccess) return e;
            continue;
        }
        // the items that follow join while the rules of sort_groups.h let them
        auto keys_of = [&](const SortArgs &a) -> uint64_t {
            return (uint64_t)a.ntiles * (a.key_mode == PL_KEY_TILE ? 1 : a.tile[0] * a.tile[1] * a.tile[2]);
        };
        GroupSize size;
        size.np = args[i0].np;
        size.keys = size.most = keys_of(args[i0]);
        GroupMemory mem;
        GroupMemory::Range r[GroupMemory::kPerItem];
        const int first = sort_memory(args[i0], r);
        mem.add(i0, r, first);
        while (args[i0].key_mode != PL_KEY_TILE_RANK && i1 < count && i1 - i0 < kGroup && args[i1].np > 0) {
            const uint64_t k = keys_of(args[i1]);
            if (!group_takes(size, args[i1].np, k, cap)) break;
            const int nr = sort_memory(args[i1], r);
            if (!mem.add(i1, r, nr)) break;
            size.np += args[i1].np;
            size.keys += k;
            size.most = std::max(size.most, k);
            ++i1;
        }
        const hipError_t e = sort_group(c, args + i0, i1 - i0);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Fixed scratch of pl_sort_noalloc: keys and indices (two buffers each) for
// PL_NOALLOC_MAX_NP particles and the digit histograms and their scan.  Every
// GPU the library runs on holds one copy until the process ends; all calls on
// a device share it (calls that overlap on one device race).
// ---------------------------------------------------------------------------

constexpr int64_t kNaNp = PL_NOALLOC_MAX_NP;
constexpr int64_t kNaHist = kSortHist(kNaNp);
constexpr size_t kNaBytes = (size_t)(4 * kNaNp + 2 * kNaHist) * sizeof(uint32_t);

static __device__ __align__(256) unsigned char scratch[kNaBytes];

constexpr int kNaDevices = 64;
static std::mutex na_mu;
static void *na_ptr[kNaDevices];       // device address of `scratch` on each device
static int na_cu[kNaDevices];

hipError_t launch_sort_noalloc(Ctx *c, const SortArgs *a, int count)
{
    for (int i = 0; i < count; ++i)
        if (a[i].np > kNaNp) return hipErrorInvalidValue;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kNaDevices) return hipErrorInvalidDevice;
    void *base = nullptr;
    int cu = 0;
    {
        std::lock_guard<std::mutex> lock(na_mu);
        if (!na_ptr[dev]) {
            // once per device, with that device current: the array's device
            // address (the symbol itself is a host-side stand-in)
            void *p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            int n = 0;
            e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
            if (e != hipSuccess) return e;
            na_cu[dev] = n > 0 ? n : 1;
            na_ptr[dev] = p;
        }
        base = na_ptr[dev];
        cu = na_cu[dev];
    }
    uint32_t *w = static_cast<uint32_t *>(base);
    c->num_cu = cu;
    c->keys[0] = w;
    c->keys[1] = w + kNaNp;
    c->idx[0] = w + 2 * kNaNp;
    c->idx[1] = w + 3 * kNaNp;
    c->hist = w + 4 * kNaNp;
    c->hist_scan = w + 4 * kNaNp + kNaHist;
    c->hist_cap = kNaHist;
    c->cell_start = nullptr;           // PL_KEY_TILE_RANK is refused before this point
    return launch_sort(c, a, count, kNaNp);
}

}  // namespace pl
