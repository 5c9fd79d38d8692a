// Tile kernels that group their particles by cell themselves (template;
// instantiated per precision in k_local_f32.hip and k_local_f64.hip).
//
// A work unit is a chunk of up to `cap` particles of one tile.  The particles
// of a tile are a contiguous range of the item's arrays (the tiled and
// run-based algorithms' tile_start), or of an index list into them (the plain
// algorithm, whose arrays are in no order: the call bins the indices by tile
// first).  Nothing but the tile offsets is taken from the sort, so the
// grouping is that of the particles' present cells.
//
//  * LM_FUSED and LM_DEP count the chunk's particles per cell in the LDS (the
//    tile's cells and one cell around them), order the chunk by cell, and cut
//    every cell's particles into runs of up to one register batch.  The runs
//    are listed by (run inside the cell, cell) for the first rounds, so that
//    the lanes of a wave hold distinct neighbouring cells, and by cell beyond
//    them.  A batch's deposits are summed in float64 registers before one
//    float64 LDS atomic per stencil point and channel.  That is the precision
//    of one float64 atomic per particle with a quarter (float32 form) or half
//    (float64 form) of the LDS atomics, and without lanes of one cell meeting
//    on one LDS address.
//  * LM_PUSH deposits nothing: one particle per lane in the stored order,
//    gathered from 16-byte LDS field records.
//
// What bounds them is the LDS, as in the run-based kernel (its atomics, reads
// and their latency at two waves per SIMD); the plain calls are bound by the
// scattered access to the particles' arrays.  Measured on MI355X against the
// one-particle-per-thread kernel on the same inputs:
//  * plain float64 step, 2^24 particles in random order on 128^3 cells, rho J
//    F: 136.1 ms (3.2e9 global atomics at 2.4e10/s) to 6.1 ms, of which the
//    binning is 0.6 ms;
//  * deposit call on run order (float32, 7.1e6 particles, 8^3 tiles, rho J F):
//    1995 us (four lanes of one cell on one LDS address) to 460 us; push call
//    431 us to 242 us;
//  * tiled fused step by tile key (float32, 1.9e6 particles, 8 channels): 578
//    us to 269 us;
//  * plain push of 1e6 float64 tracers in random order: 677 us to 245 us (165 us
//    and the binning);
//  * push of few particles per tile (72 tracers per 8^3 tile): 62 us per launch;
//    blocks of 256 threads 67 us, with a one-cell field halo 77 us.
#pragma once

#include "k_runs_impl.h"
#include "tile_route.h"

namespace pl {

constexpr int kLocalThreads = 512, kLocalSmall = 256;
static_assert(kLocalThreads <= 8 * 64, "scan words of local_scan");
constexpr int kLocalRounds = 5;        // rounds of runs counted together (11 bits each in 64)
constexpr int kLocalMaxCells = 2047;   // cells of a tile and its ring: fits 11 bits
constexpr int kLocalMaxCap = 8192;     // particles of a chunk: 13 bits of a run entry, 2 bits of length
constexpr int kLocalSums = 8;          // partial particle-side sums per channel (lanes spread over them)

// Particles per register batch, and capacity of the queue of deposits outside
// their batch's cell: about a half of the run-based kernel's (the chunk's
// order takes the rest: with every channel on an 8^3 tile the larger queue
// left chunks of under half a tile).
template <int PREC> struct LocalBatch {
    static constexpr int KR = PREC == PL_F32_OFFSET ? 4 : 2;
    static constexpr int DQ = PREC == PL_F32_OFFSET ? 96 : 64;
};

// Sections of the LDS: field records, deposit tile, work area (cell counts
// while grouping, deposit queue afterwards), queue of particles outside the
// field tile, run list, ordered chunk, sums, control words.
struct LocalLds {
    size_t f, d, work, gq, list, order, sums, ctl, total;
    int cap;
};

template <int PREC, int KIND>
__host__ __device__ inline LocalLds local_lds(int mode, int Lf, int Ld, int E, int nslot, int cap)
{
    using R = typename RealOf<PREC>::T;
    constexpr int DQ = LocalBatch<PREC>::DQ, KR = LocalBatch<PREC>::KR;
    const bool group = mode != LM_PUSH;
    LocalLds s;
    size_t o = 0;
    s.cap = cap;
    s.f = o; o += mode == LM_DEP ? 0 : runs_section((size_t)Lf * FieldRec<PREC, KIND>::FS * sizeof(R));
    s.d = o; o += group ? runs_section((size_t)Ld * nslot * sizeof(double)) : 0;
    size_t work = group ? (size_t)E * 4 + 256 : 0;
    if (mode == LM_FUSED) {
        const size_t q = runs_section((size_t)DQ * 4) + (size_t)DQ * (3 + nslot) * sizeof(R);
        work = work > q ? work : q;
    }
    s.work = o; o += runs_section(work);
    s.gq = o; o += mode == LM_FUSED ? runs_section((size_t)gq_cap(1) * 4) : 0;
    const int nrun = E + cap / KR < cap ? E + cap / KR : cap;
    s.list = o; o += group ? runs_section((size_t)nrun * 2) : 0;
    s.order = o; o += group ? runs_section((size_t)cap * 2) : 0;
    s.sums = o; o += 8 * kLocalSums * sizeof(double);
    s.ctl = o; o += 64;
    s.total = o;
    return s;
}

// Block-wide exclusive sums of a 64-bit and a 32-bit value; the totals go to
// ta and tb.  sh: 16 64-bit words (of up to eight waves).
__device__ __forceinline__ void local_scan(unsigned long long a, unsigned b, unsigned long long *sh,
                                           unsigned long long &ea, unsigned &eb, unsigned long long &ta, unsigned &tb)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    unsigned long long xa = a;
    unsigned xb = b;
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long ya = __shfl_up(xa, off, 64);
        const unsigned yb = __shfl_up(xb, off, 64);
        if (lane >= off) {
            xa += ya;
            xb += yb;
        }
    }
    if (lane == 63) {
        sh[wv] = xa;
        sh[8 + wv] = xb;
    }
    __syncthreads();
    ea = xa - a;
    eb = xb - b;
    ta = 0;
    tb = 0;
    for (int w = 0; w < nw; ++w) {
        if (w == wv) {
            ea += ta;
            eb += tb;
        }
        ta += sh[w];
        tb += (unsigned)sh[8 + w];
    }
    __syncthreads();
}

// Tile and chunk of unit slot l of an item.  Tile t owns the slots from
// t + tile_start[t] / cap to the next tile's first: at least one per chunk of
// its particles, and ntiles + np / cap in all, a number the host knows.  The
// block searches the last tile whose first slot is at most l, blockDim.x
// candidates at a time (one round for up to 512 tiles, two for 262144).
__device__ __forceinline__ int local_tile(const int32_t *ts, int ntiles, int cap, int l, int *sh)
{
    int lo = 0, hi = ntiles;
    while (hi - lo > 1) {                                    // uniform
        const int step = (hi - lo + (int)blockDim.x - 1) / (int)blockDim.x;
        const int t = lo + (int)threadIdx.x * step;
        const bool p = t < hi && t + ts[t < hi ? t : lo] / cap <= l;
        const int n = __popcll(__ballot(p));
        if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = n;
        __syncthreads();
        int c = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) c += sh[w];
        __syncthreads();
        lo += max(c - 1, 0) * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

// Cell of the extended tile (its cells and the ring around them), periodically.
template <int DIM>
__device__ __forceinline__ bool ext_cell(const RunGeo &g, const int n[3], const int c[3], int &e)
{
    bool ok = true;
    int l[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        int v = c[a] - g.lo[a];
        if (v < -1) v += n[a];
        else if (v > g.T[a]) v -= n[a];
        ok = ok && v >= -1 && v <= g.T[a];
        l[a] = v + 1;
    }
    e = l[0] + (g.T[0] + 2) * (l[1] + (DIM >= 3 ? (g.T[1] + 2) * l[2] : 0));
    return ok;
}

// Channel values of a particle that is deposited without a push: charge or
// mass, current, and the force stored by the last push.
template <int PREC, int KIND>
__device__ __forceinline__ void state_values(const UnitC<PREC> &U, int p, const typename RealOf<PREC>::T u[3],
                                             typename RealOf<PREC>::T w, typename RealOf<PREC>::T mu[kMaxCh])
{
    using R = typename RealOf<PREC>::T;
#pragma unroll
    for (int ch = 0; ch < kMaxCh; ++ch) mu[ch] = R(0);
    if constexpr (KIND == PL_LORENTZ) {
        const R g2 = sqrt(fma(fma(u[0], u[0], fma(u[1], u[1], u[2] * u[2])), U.inv_c2, R(1)));
        const R qw = U.q * w;
        mu[0] = qw;
#pragma unroll
        for (int a = 0; a < 3; ++a) mu[1 + a] = qw * u[a] / g2;
    } else {
        mu[0] = U.m * w;
    }
    if (U.fp[0]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) mu[4 + a] = U.fp[a][p];
    }
}

// One particle deposited from its stored state.
template <int PREC, int SHAPE, int DIM, int KIND, int CHS>
__device__ __forceinline__ void state_deposit(const UnitC<PREC> &U, const RunGeo &G, double *lds_d, int p, int &err)
{
    using R = typename RealOf<PREC>::T;
    Pos<PREC, DIM> pos;
    pos.load(U, p, err);
    const R u[3] = {U.u[0][p], U.u[1][p], U.u[2][p]};
    R mu[kMaxCh];
    state_values<PREC, KIND>(U, p, u, U.w ? U.w[p] : U.wdef, mu);
    double mud[kMaxCh];
#pragma unroll
    for (int ch = 0; ch < kMaxCh; ++ch) mud[ch] = (double)mu[ch];
    const R d[3] = {(R)pos.d[0], (R)pos.d[1], (R)pos.d[2]};
    deposit_single<PREC, SHAPE, DIM, CHS>(U, G, lds_d, pos.c, d, mud);
}

// One particle pushed without a deposit.
template <int PREC, int SHAPE, int DIM, int KIND>
__device__ __forceinline__ void particle_push(const UnitC<PREC> &U, const RunGeo &G,
                                              const typename RealOf<PREC>::T *lds_f, int p, bool do_sums,
                                              const RunShared<PREC> &S, int &err)
{
    using R = typename RealOf<PREC>::T;
    constexpr int NC = FieldRec<PREC, KIND>::NC;
    Pos<PREC, DIM> pos;
    pos.load(U, p, err);
    R u[3] = {U.u[0][p], U.u[1][p], U.u[2][p]};
    const R w = U.w ? U.w[p] : U.wdef;
    const R d0[3] = {(R)pos.d[0], (R)pos.d[1], (R)pos.d[2]};
    R wx[3], wy[3], wz[3], F[NC];
    stencil_weights<PREC, SHAPE, DIM>(d0, wx, wy, wz);
    int fb = 0;
    if (field_base<DIM>(G, U.n, pos.c, fb)) gather_rec<PREC, DIM, KIND>(G, lds_f, fb, wx, wy, wz, F);
    else gather<PREC, DIM, NC>(U, nullptr, 0, false, 0, 0, 0, pos.c, wx, wy, wz, F);
    R v[3], mu[kMaxCh];
    push_particle<PREC, KIND>(U, u, F, w, v, mu);
    if (U.fp[0]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) U.fp[a][p] = mu[4 + a];
    }
    if (do_sums) add_sums(S, mu);
    R disp[3] = {R(0), R(0), R(0)};
#pragma unroll
    for (int a = 0; a < DIM; ++a) disp[a] = v[a] * U.dtdx[a];
    pos.advance(disp, U, err);
    pos.store(U, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) U.u[a][p] = u[a];
}

// Stored state of the particles pi[0..len) of a batch.
template <int PREC, int DIM, int KR>
__device__ __forceinline__ void fetch_indexed(const UnitC<PREC> &U, const int pi[KR], int len,
                                              BatchRaw<PREC, DIM, KR> &B)
{
    using R = typename RealOf<PREC>::T;
    B.start = pi[0];
    B.len = len;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        const bool in = j < len;
        if (in) Pos<PREC, DIM>::fetch(U, pi[j], B.pr[j]);
        else B.pr[j] = B.pr[0];
#pragma unroll
        for (int a = 0; a < 3; ++a) B.u[j][a] = in ? U.u[a][pi[j]] : R(0);
        B.w[j] = in ? (U.w ? U.w[pi[j]] : U.wdef) : R(0);
    }
}

// One chunk of a tile.
template <int PREC, int SHAPE, int DIM, int KIND, int MODE, int TS, int CHS, int NT>
__device__ __forceinline__ void local_unit(const ItemDesc &I, int t, int pbeg, int pend, int cap, unsigned flags,
                                           int ctl_at, unsigned char *smem, unsigned *counter, bool &pre, int &err)
{
    using R = typename RealOf<PREC>::T;
    constexpr int KR = LocalBatch<PREC>::KR;
    constexpr bool GROUP = MODE != LM_PUSH;
    const bool do_sums = flags & SF_SUMS;
    RunGeo G;
    G.T[0] = TS ? ts_dim(TS, 0) : I.tile[0];
    G.T[1] = TS ? ts_dim(TS, 1) : I.tile[1];
    G.T[2] = TS ? ts_dim(TS, 2) : I.tile[2];
    G.lo[0] = (t % I.ntile[0]) * G.T[0];
    G.lo[1] = ((t / I.ntile[0]) % I.ntile[1]) * G.T[1];
    G.lo[2] = (t / (I.ntile[0] * I.ntile[1])) * G.T[2];
    G.hf = MODE == LM_PUSH ? ((flags & SF_FHALO2) ? 2 : 1) : 1;
    G.fx = G.T[0] + 2 * G.hf;
    G.fxy = G.fx * (G.T[1] + 2 * G.hf);
    G.Lf = G.fxy * (DIM >= 3 ? G.T[2] + 2 * G.hf : 1);
    G.dx = G.T[0] + 4;
    G.dxy = G.dx * (G.T[1] + 4);
    G.Ld = G.dxy * (DIM >= 3 ? G.T[2] + 4 : 1);
    const int E = (G.T[0] + 2) * (G.T[1] + 2) * (DIM >= 3 ? G.T[2] + 2 : 1);
    UnitC<PREC> U;
    load_unit<PREC>(I, U, G.Ld);
    const int nslot = MODE == LM_PUSH ? 0 : I.nslot;
    const LocalLds L = local_lds<PREC, KIND>(MODE, G.Lf, G.Ld, E, nslot, cap);
    RunShared<PREC> S;
    R *lds_f = reinterpret_cast<R *>(smem + L.f);
    S.lds_f = lds_f;
    S.lds_d = reinterpret_cast<double *>(smem + L.d);
    S.gq = reinterpret_cast<int *>(smem + L.gq);
    S.dq_c = reinterpret_cast<uint32_t *>(smem + L.work);
    S.dq_d = reinterpret_cast<R *>(smem + L.work + runs_section((size_t)LocalBatch<PREC>::DQ * 4));
    S.dq_mu = S.dq_d + 3 * LocalBatch<PREC>::DQ;
    S.dq = LocalBatch<PREC>::DQ;
    S.narrow = false;
    S.ctl = reinterpret_cast<int *>(smem + ctl_at);
    S.sums = reinterpret_cast<double *>(smem + L.sums);
    S.smask = kLocalSums - 1;
    int *ctl = S.ctl;
    const gptr<const uint32_t> idx = (gptr<const uint32_t>)I.idx;
    auto particle = [&](int k) -> int { return idx ? (int)idx[k] : k; };

    if constexpr (MODE != LM_DEP) {
        stage_unit<PREC, DIM, KIND>(U, G, lds_f, S.lds_d, G.Ld * nslot);
    } else {
        for (int k = threadIdx.x; k < G.Ld * nslot; k += blockDim.x) S.lds_d[k] = 0.0;
    }
    if (threadIdx.x == 0) {
        ctl[1] = 0;
        ctl[2] = 0;
    }
    if (threadIdx.x < 8 * kLocalSums) S.sums[threadIdx.x] = 0.0;

    if constexpr (!GROUP) {
        __syncthreads();
        for (int k = pbeg + (int)threadIdx.x; k < pend; k += (int)blockDim.x) {
            const int p = particle(k);
            if constexpr (KIND == PL_TRACER) tracer_particle<PREC, SHAPE, DIM>(U, G, S.lds_f, p, err);
            else particle_push<PREC, SHAPE, DIM, KIND>(U, G, S.lds_f, p, do_sums, S, err);
        }
    } else {
        // group the chunk by cell
        unsigned *cnt = reinterpret_cast<unsigned *>(smem + L.work);
        unsigned long long *scan = reinterpret_cast<unsigned long long *>(smem + L.work + (((size_t)E * 4 + 7) & ~(size_t)7));
        uint16_t *list = reinterpret_cast<uint16_t *>(smem + L.list);
        uint16_t *order = reinterpret_cast<uint16_t *>(smem + L.order);
        for (int e = threadIdx.x; e < E; e += blockDim.x) cnt[e] = 0;
        __syncthreads();
        auto cell_of = [&](int k, int &e) -> bool {
            Pos<PREC, DIM> pos;
            int ignored = 0;
            pos.load(U, particle(k), ignored);
            return ext_cell<DIM>(G, U.n, pos.c, e);
        };
        const int bd = (int)blockDim.x;
#pragma unroll 4
        for (int k = pbeg + (int)threadIdx.x; k < pend; k += bd) {
            int e;
            if (cell_of(k, e)) atomicAdd(&cnt[e], 1u);
        }
        __syncthreads();
        // this thread's cells: particles before them, runs before them in each
        // of the first rounds, and further runs
        constexpr int CPT = (kLocalMaxCells + NT - 1) / NT;
        const int cpt = (E + bd - 1) / bd, c0 = (int)threadIdx.x * cpt;
        unsigned n[CPT];
        unsigned tot = 0, rest = 0;
        unsigned long long rounds = 0;
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            n[q] = (q < cpt && c0 + q < E) ? cnt[c0 + q] : 0u;
            const unsigned nr = (n[q] + KR - 1) / KR;
            tot += n[q];
#pragma unroll
            for (int b = 0; b < kLocalRounds; ++b) rounds += nr > (unsigned)b ? 1ull << (11 * b) : 0ull;
            rest += nr > (unsigned)kLocalRounds ? nr - kLocalRounds : 0u;
        }
        unsigned long long er, tr;
        unsigned ep, et;
        // particles (13 bits and more) and further runs share a 32-bit scan
        local_scan(rounds, tot | rest << 16, scan, er, ep, tr, et);
        unsigned pos = ep & 0xffffu, rpos = ep >> 16;
        unsigned base = 0;
        unsigned rb[kLocalRounds];
#pragma unroll
        for (int b = 0; b < kLocalRounds; ++b) {
            rb[b] = base + (unsigned)((er >> (11 * b)) & 2047u);
            base += (unsigned)((tr >> (11 * b)) & 2047u);
        }
        rpos += base;
        const int nruns = (int)(base + (et >> 16));
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            if (n[q] == 0) continue;
            cnt[c0 + q] = pos;
            const unsigned nr = (n[q] + KR - 1) / KR;
#pragma unroll
            for (int b = 0; b < kLocalRounds; ++b)
                if (nr > (unsigned)b)
                    list[rb[b]++] = (uint16_t)((pos + b * KR) << 2 | (min(n[q] - b * KR, (unsigned)KR) - 1u));
            for (unsigned b = kLocalRounds; b < nr; ++b)
                list[rpos++] = (uint16_t)((pos + b * KR) << 2 | (min(n[q] - b * KR, (unsigned)KR) - 1u));
            pos += n[q];
        }
        __syncthreads();
#pragma unroll 4
        for (int k = pbeg + (int)threadIdx.x; k < pend; k += bd) {
            int e;
            if (cell_of(k, e)) {
                order[atomicAdd(&cnt[e], 1u)] = (uint16_t)(k - pbeg);
            } else {
                // far from its tile: on its own, later (fused) or now
                const int p = particle(k);
                if constexpr (MODE == LM_FUSED) {
                    const int q = atomicAdd(&ctl[1], 1);
                    if (q < gq_cap(1)) S.gq[q] = p;
                    else particle_single<PREC, SHAPE, DIM, KIND, CHS>(U, G, S, p, do_sums, err);
                } else {
                    state_deposit<PREC, SHAPE, DIM, KIND, CHS>(U, G, S.lds_d, p, err);
                }
            }
        }
        __syncthreads();

        // the chunk's runs, one batch each; the next batch is fetched while the
        // current one deposits
        auto run_at = [&](int r, int (&pi)[KR]) -> int {
            const unsigned v = list[r];
            const int s = (int)(v >> 2), len = (int)(v & 3u) + 1;
#pragma unroll
            for (int j = 0; j < KR; ++j) pi[j] = j < len ? particle(pbeg + order[s + j]) : 0;
            return len;
        };
        int r = (int)threadIdx.x;
        bool have = r < nruns;
        int pi[KR];
        BatchRaw<PREC, DIM, KR> cur;
        if (have) {
            const int len = run_at(r, pi);
            fetch_indexed<PREC, DIM, KR>(U, pi, len, cur);
        }
        while (have) {
            r += bd;
            have = r < nruns;
            const BatchRaw<PREC, DIM, KR> now = cur;
            int pn[KR];
#pragma unroll
            for (int j = 0; j < KR; ++j) pn[j] = pi[j];
            auto fetch = [&]() {
                if (have) {
                    const int len = run_at(r, pi);
                    fetch_indexed<PREC, DIM, KR>(U, pi, len, cur);
                }
            };
            if constexpr (MODE == LM_FUSED) {
                run_batch<PREC, SHAPE, DIM, KIND, CHS, KR, false, true>(U, G, S, now, pn, do_sums, err, fetch);
            } else {
                Pos<PREC, DIM> ps[KR];
                R mu[KR][kMaxCh];
                bool in[KR];
#pragma unroll
                for (int j = 0; j < KR; ++j) {
                    in[j] = j < now.len;
                    if (in[j]) {
                        ps[j].set(now.pr[j], U, err);
                        state_values<PREC, KIND>(U, pn[j], now.u[j], now.w[j], mu[j]);
                    } else {
                        ps[j] = ps[0];
#pragma unroll
                        for (int ch = 0; ch < kMaxCh; ++ch) mu[j][ch] = R(0);
                    }
                }
                fetch();
                int db = 0;
                if (dep_base<DIM>(G, U.n, ps[0].c, db))
                    batch_deposit<PREC, SHAPE, DIM, CHS, KR, true>(U, G, S, db, ps, mu, in);
            }
        }
        if constexpr (MODE == LM_FUSED) {
            __syncthreads();
            const int ng = min(ctl[1], gq_cap(1)), nd = min(ctl[2], S.dq);
            for (int i = threadIdx.x; i < ng; i += blockDim.x)
                particle_single<PREC, SHAPE, DIM, KIND, CHS>(U, G, S, S.gq[i], do_sums, err);
            drain_deposits<PREC, SHAPE, DIM, CHS>(U, G, S, nd);
        }
    }
    __syncthreads();
    // the next unit is claimed before the flush, whose atomics hide the round trip
    pre = counter != nullptr;
    if (pre && threadIdx.x == 0) ctl[0] = (int)atomicAdd(counter, 1u);
    if (KIND != PL_TRACER && do_sums && threadIdx.x < 8) {
        double sum = 0.0;
        for (int k = 0; k < kLocalSums; ++k) sum += S.sums[threadIdx.x * kLocalSums + k];
        if (sum != 0.0) global_add(I.psum + threadIdx.x, sum);
    }
    if constexpr (GROUP) flush_unit<PREC, DIM, CHS>(U, G, S.lds_d);
}

template <int PREC, int SHAPE, int DIM, int KIND, int MODE, int TS, int CHS, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(MODE == LM_PUSH ? 4 : 2, MODE == LM_PUSH ? 8 : 2)))
void k_local(const ItemDesc *__restrict__ items, int nitems, int total_units, unsigned *counter, int *errflags,
             unsigned flags, int cap, int ctl_at)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    int *ctl = reinterpret_cast<int *>(smem_raw + ctl_at);
    int err = 0;
    bool pre = false;                      // uniform: ctl[0] already holds the next claim
    // a block for every unit: no claims (see claim_unit)
    const bool direct = (int)gridDim.x >= total_units;
    for (int turn = 0;; ++turn) {
        int g = (int)blockIdx.x;
        if (direct) {
            if (turn > 0) break;                              // uniform
        } else {
            __syncthreads();
            if (!pre && threadIdx.x == 0) ctl[0] = (int)atomicAdd(counter, 1u);
            __syncthreads();
            pre = false;
            g = __builtin_amdgcn_readfirstlane(ctl[0]);
        }
        if (g >= total_units) break;                          // uniform
        const ItemDesc &I = items[find_item(items, nitems, g)];
        const int32_t *ts = I.tile_start;
        // tile offsets must run from 0 to np: otherwise the item was never
        // sorted (or its count changed since): latch it, leave it alone
        if (ts[0] != 0 || ts[I.ntiles] != I.np) {
            if (threadIdx.x == 0) atomicOr(errflags, (int)ERR_UNSORTED);
            continue;                                         // uniform
        }
        const int l = g - I.unit_begin;
        const int t = local_tile(ts, I.ntiles, cap, l, ctl + 4);
        const int beg = min(max(ts[t], 0), I.np), end = min(max(ts[t + 1], beg), I.np);
        const int nch = (end - beg + cap - 1) / cap, j = l - (t + beg / cap);
        if (j < 0 || j >= nch) continue;                      // uniform: an empty slot
        const int pbeg = beg + (int)((long long)(end - beg) * j / nch);
        const int pend = beg + (int)((long long)(end - beg) * (j + 1) / nch);
        local_unit<PREC, SHAPE, DIM, KIND, MODE, TS, CHS, NT>(I, t, pbeg, pend, cap, flags, ctl_at, smem_raw,
                                                                  direct ? nullptr : counter, pre,
                                                                  err);
    }
    runs_latch(err, errflags);
    release_counter(counter, total_units);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

using LocalKernel = void (*)(const ItemDesc *, int, int, unsigned *, int *, unsigned, int, int);

template <int PREC>
static LocalKernel pick_local(int shape, int dim, int kind, int mode, int ts, int chs, int nt)
{
#define PL_LN(S, D, K, M, TS_, CHS_, NT_) \
    if (shape == S && dim == D && kind == K && mode == M && ts == TS_ && chs == CHS_ && nt == NT_) \
        return k_local<PREC, S, D, K, M, TS_, CHS_, NT_>;
#define PL_L(S, D, K, M, TS_, CHS_) PL_LN(S, D, K, M, TS_, CHS_, kLocalThreads)
#define PL_LM(S, D, K) PL_L(S, D, K, LM_FUSED, 0, 0) PL_L(S, D, K, LM_PUSH, 0, 0) PL_L(S, D, K, LM_DEP, 0, 0) \
    PL_LN(S, D, K, LM_FUSED, 0, 0, kLocalSmall) PL_LN(S, D, K, LM_DEP, 0, 0, kLocalSmall)
#define PL_LG(S, D) PL_LM(S, D, PL_LORENTZ) PL_LM(S, D, PL_DUST) PL_L(S, D, PL_TRACER, LM_PUSH, 0, 0)
    PL_LG(PL_TSC, 3) PL_LG(PL_TSC, 2) PL_LG(PL_CIC, 3) PL_LG(PL_CIC, 2)
#define PL_LT(TS_) \
    PL_L(PL_TSC, 3, PL_LORENTZ, LM_FUSED, TS_, 1) PL_L(PL_TSC, 3, PL_LORENTZ, LM_FUSED, TS_, 3) \
    PL_L(PL_TSC, 3, PL_LORENTZ, LM_DEP, TS_, 1) PL_L(PL_TSC, 3, PL_DUST, LM_FUSED, TS_, 2) \
    PL_L(PL_TSC, 3, PL_DUST, LM_DEP, TS_, 2) PL_L(PL_TSC, 3, PL_LORENTZ, LM_PUSH, TS_, 0) \
    PL_L(PL_TSC, 3, PL_DUST, LM_PUSH, TS_, 0) PL_L(PL_TSC, 3, PL_TRACER, LM_PUSH, TS_, 0)
    PL_LT(1) PL_LT(2)
#define PL_LS(K, M, CHS_) PL_LN(PL_TSC, 3, K, M, 4, CHS_, kLocalSmall)
    PL_LS(PL_LORENTZ, LM_FUSED, 1) PL_LS(PL_LORENTZ, LM_FUSED, 3) PL_LS(PL_LORENTZ, LM_DEP, 1)
    PL_LS(PL_DUST, LM_FUSED, 2) PL_LS(PL_DUST, LM_DEP, 2)
#undef PL_LS
#undef PL_LT
#undef PL_LG
#undef PL_LM
#undef PL_L
#undef PL_LN
    return nullptr;
}

template <int PREC>
static LocalLds local_item_lds(const Ctx *c, const ItemDesc &it, int mode, int hf, int cap)
{
    const int d3 = c->d.ndim >= 3;
    const int *T = it.tile;
    const int Lf = (T[0] + 2 * hf) * (T[1] + 2 * hf) * (d3 ? T[2] + 2 * hf : 1);
    const int Ld = (T[0] + 4) * (T[1] + 4) * (d3 ? T[2] + 4 : 1);
    const int E = (T[0] + 2) * (T[1] + 2) * (d3 ? T[2] + 2 : 1);
    if (it.kind == PL_LORENTZ) return local_lds<PREC, PL_LORENTZ>(mode, Lf, Ld, E, it.nslot, cap);
    if (it.kind == PL_DUST) return local_lds<PREC, PL_DUST>(mode, Lf, Ld, E, it.nslot, cap);
    return local_lds<PREC, PL_TRACER>(mode, Lf, Ld, E, 0, cap);
}

// Launch configuration for the items of one species kind: field halo,
// particles per chunk, LDS bytes.  False when it does not pay (tile_route.h;
// binned plain items go by plain_bins), when a tile has too many cells, or when
// its LDS does not fit with chunks of at least kLocalMinCap particles.  Fewer
// particles per tile than threads do not pay either (4096
// particles in 32 tiles: 266 us for ten steps against 251 us of the
// one-particle-per-thread kernel); up to kLocalSmallPerTile a block of 256
// threads holds enough of a tile's runs, and the phases of two blocks on a CU
// overlap (float64 by tile key, 8 x 4 x 4 tiles of 768 particles: eight
// steps and the sort 5.89 ms with 512 threads, 4.16 ms with 256).  The tiles of
// float32 boxes in 3D are larger, and their small blocks have no fixed shapes: dust on
// 8^3 tiles of 1024 particles 72 us with 256 threads, 41 with 512.
constexpr int kLocalMinCap = 1024;
constexpr int kLocalSmallPerTile = 2048;

template <int PREC>
bool local_plan_impl(const Ctx *c, const ItemDesc *host, int nitems, bool push, bool deposit, LocalPlan &pl)
{
    pl = LocalPlan{};
    pl.nt = kLocalThreads;
    if (nitems < 1) return false;
    const int kind = host[0].kind;
    const bool dep = deposit && kind != PL_TRACER;
    if (!push && !dep) return false;
    pl.mode = push ? (dep ? LM_FUSED : LM_PUSH) : LM_DEP;
    const int d3 = c->d.ndim >= 3;
    const bool group = pl.mode != LM_PUSH;
    TileLoad w{0, 0, 0};
    for (int i = 0; i < nitems; ++i) {
        if (host[i].np == 0) continue;
        w.np += host[i].np;
        w.nt += host[i].ntiles;
        w.cells += (int64_t)host[i].n[0] * host[i].n[1] * host[i].n[2];
    }
    if (!host[0].idx && !local_pays(pl.mode, c->d.ndim, PREC, kind, c->d.key_mode, c->num_cu, w)) return false;
    for (int i = 0; i < nitems && group; ++i) {
        const int *T = host[i].tile;
        const int E = (T[0] + 2) * (T[1] + 2) * (d3 ? T[2] + 2 : 1);
        if (E > kLocalMaxCells) return false;
    }
    auto bytes = [&](int hf, int cap) {
        size_t m = 0;
        for (int i = 0; i < nitems; ++i) m = std::max(m, local_item_lds<PREC>(c, host[i], pl.mode, hf, cap).total);
        return m;
    };
    if (!group) {
        // two blocks per CU where a two-cell field halo leaves room for them
        pl.cap = 4096;
        pl.hf = 2 * bytes(2, pl.cap) <= (size_t)c->lds_max ? 2 : 1;
        pl.lds = bytes(pl.hf, pl.cap);
        return pl.lds <= (size_t)c->lds_max;
    }
    const int64_t np = w.np, nt = w.nt;
    pl.hf = 1;
    // tiles of few particles whose LDS lets two blocks share a CU: smaller blocks
    if (np < kLocalSmallPerTile * nt && (PREC == PL_F64 || !d3)) {
        pl.nt = kLocalSmall;
        for (pl.cap = 2048; pl.cap >= kLocalMinCap; pl.cap -= 256) {
            pl.lds = bytes(1, pl.cap);
            if (2 * pl.lds <= (size_t)c->lds_max) break;
        }
        if (pl.cap < kLocalMinCap) pl.nt = kLocalThreads;
    }
    // few particles per thread: no grouping costs less
    if (!host[0].idx && np < pl.nt * nt) return false;
    if (pl.nt == kLocalSmall) return true;
    // chunks: what the LDS holds, and no more than leave each CU one
    const int64_t share = (np / c->num_cu + 255) / 256 * 256;
    pl.cap = (int)std::min<int64_t>(kLocalMaxCap, std::max<int64_t>(kLocalMinCap, share));
    for (; pl.cap >= kLocalMinCap; pl.cap -= 256) {
        pl.lds = bytes(1, pl.cap);
        if (pl.lds <= (size_t)c->lds_max) return true;
    }
    return false;
}

template <int PREC>
hipError_t launch_local_impl(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, const LocalPlan &pl,
                             unsigned sf, unsigned *counter)
{
    int units = 0, ts = 0, chs = 0;
    for (int i = 0; i < nitems; ++i) units = std::max(units, host[i].unit_begin + host[i].nunits);
    if (units <= 0) return hipSuccess;
    const int kind = host[0].kind;
    if (c->d.shape == PL_TSC && c->d.ndim == 3) {
        for (int cand : {1, 2, 4}) {
            if (ts || (cand == 4) != (pl.nt == kLocalSmall)) continue;
            bool all = true;
            for (int i = 0; i < nitems; ++i)
                for (int a = 0; a < 3; ++a) all = all && host[i].tile[a] == ts_dim(cand, a);
            if (all) ts = cand;
        }
        if (ts && pl.mode != LM_PUSH) {
            for (int want : {1, 2, 3}) {
                if ((kind == PL_DUST) != (want == 2) || (want == 3 && pl.mode == LM_DEP)) continue;
                bool all = true;
                for (int i = 0; i < nitems && all; ++i)
                    for (int ch = 0; ch < kMaxCh; ++ch) all = all && host[i].slot[ch] == chs_slot(want, ch);
                if (all) chs = want;
            }
            if (!chs) ts = 0;
        }
    }
    LocalKernel k = pick_local<PREC>(c->d.shape, c->d.ndim, kind, pl.mode, ts, chs, pl.nt);
    if (!k) return hipErrorInvalidValue;
    if (pl.hf == 2) sf |= SF_FHALO2;
    // every item's control words sit at one place: the end of the launch's LDS
    const int grid = std::min(units, resident_blocks(c, (StepKernel)k, pl.nt, pl.lds));
    hipLaunchKernelGGL(k, dim3(grid), dim3(pl.nt), pl.lds, c->stream, table, nitems, units, counter,
                       c->errflags, sf, pl.cap, (int)pl.lds - 64);
    c->stats[0]++;
    c->stats[8]++;
    return hipGetLastError();
}

}  // namespace pl
