// Run-based gather -> push -> deposit kernel for gfx950 (template;
// instantiated per precision in k_runs_f32.hip and k_runs_f64.hip).
//
// Work unit: a piece of one cell tile of one item (the sort cuts a crowded
// tile into pieces of equal run count and lists the units largest first).
// The sort cuts the particles of every cell into runs of up to kRunLen
// consecutive particles and lists the runs of a tile by (index of the run
// inside its cell, cell), so the threads of a wave hold runs of distinct
// neighbouring cells; with the run-order key the runs also lie in memory in
// table order, so a wave's particle loads and stores are contiguous.  A
// thread advances its run in register batches of KR particles that share one
// cell:
//  * each batch particle interpolates its fields from the 27 (9 in 2D)
//    records of its own cell's stencil in the LDS field tile (24 bytes per
//    charged record in float32, 48 in float64);
//  * after the push, the batch's deposits are summed per stencil point and
//    channel before one float64 LDS atomic, cutting LDS atomics by the run
//    length;
//  * the LDS deposit tile carries a two-cell halo, so particles that drifted
//    up to one cell out of the tile since the sort still deposit into LDS;
//    the field tile does too where the LDS allows it (else one cell).
// A particle that moved since the sort is still gathered in its batch, from
// its own cell, while its stencil lies in the field tile; outside the tile it
// is queued in LDS for the single-particle path.  After the push, batch
// particles outside the batch's reference cell queue their deposit.  Queued
// work runs after the runs, or immediately when a queue is full.
// Per particle, gathers and pushes add the same terms in the same order as the
// tiled kernel (explicit fma), so particle states are bit-identical to it.
#pragma once

#include "k_step_impl.h"
#include "runs_lds.h"
#include "runs_sums.h"
#include "unit_chunks.h"

namespace pl {

// Type of a batch's deposit sums.
template <int PREC, bool DACC> struct AccOf { using T = typename RealOf<PREC>::T; };
template <int PREC> struct AccOf<PREC, true> { using T = double; };

// LDS field records.  Lanes of a wave read records of neighbouring cells, so
// the record stride decides the bank pattern: float32 charged particles use a
// plane of 16-byte records and a plane of 8-byte ones (E0 E1 E2 B0 | B1 B2,
// the second after the Lf records of the first), read with one 16- and one
// 8-byte access each: the gather is bound by the LDS bandwidth (a point's
// records take 16 of its cycles per wave at 32 bytes, 12 at 24, against 32
// cycles of fused multiply-adds shared by four SIMDs); float64 charged: one
// 48-byte record E0 E1 E2 B0 B1 B2; three-component kinds: v0 v1 v2 0.
template <int PREC, int KIND> struct FieldRec {
    static constexpr int NC = KIND == PL_LORENTZ ? 6 : 3;
    static constexpr int FS = PREC == PL_F32_OFFSET ? (NC == 6 ? 6 : 4) : (NC == 6 ? 6 : 4);
    static constexpr bool PLANES = PREC == PL_F32_OFFSET && NC == 6;
};

template <int PREC, int KIND>
__device__ __forceinline__ void load_rec(const typename RealOf<PREC>::T *lds_f, int cell, int Lf,
                                         typename RealOf<PREC>::T f[FieldRec<PREC, KIND>::NC])
{
    if constexpr (PREC == PL_F32_OFFSET) {
        const float4 *p = reinterpret_cast<const float4 *>(lds_f);
        const float4 a = p[cell];
        f[0] = a.x; f[1] = a.y; f[2] = a.z;
        if constexpr (KIND == PL_LORENTZ) {
            const float2 b = reinterpret_cast<const float2 *>(p + Lf)[cell];
            f[3] = a.w; f[4] = b.x; f[5] = b.y;
        }
    } else {
        const double2 *p = reinterpret_cast<const double2 *>(lds_f);
        if constexpr (KIND == PL_LORENTZ) {
            double2 a = p[3 * cell], b = p[3 * cell + 1], c = p[3 * cell + 2];
            f[0] = a.x; f[1] = a.y; f[2] = b.x; f[3] = b.y; f[4] = c.x; f[5] = c.y;
        } else {
            double2 a = p[2 * cell], b = p[2 * cell + 1];
            f[0] = a.x; f[1] = a.y; f[2] = b.x;
        }
    }
}

__device__ __forceinline__ int wrap_any(int i, int n)
{
    int r = i % n;
    return r < 0 ? r + n : r;
}

// The same for an index at most one box length outside, as a tile's halo
// cells mostly are (without the division).
__device__ __forceinline__ int wrap_near(int i, int n)
{
    const int r = i < 0 ? i + n : (i >= n ? i - n : i);
    return (unsigned)r < (unsigned)n ? r : wrap_any(i, n);
}

// Geometry of one tile: field tile with an hf-cell halo (1 or 2), deposit
// tile with a two-cell halo.
struct RunGeo {
    int lo[3], T[3];
    int hf;
    int fx, fxy, Lf;
    int dx, dxy, Ld;
};

// LDS index (field tile) of stencil point (-1,-1,-1) of a particle in cell c,
// when the whole stencil lies in the field tile (c at most hf - 1 cells
// outside the tile, periodically).
template <int DIM>
__device__ __forceinline__ bool field_base(const RunGeo &g, const int n[3], const int c[3], int &base)
{
    bool ok = true;
    int l[3] = {0, 0, 0};
    const int h = g.hf - 1;
#pragma unroll
    for (int a = 0; a < DIM; ++a) {
        int v = c[a] - g.lo[a];
        if (v < -h) v += n[a];
        else if (v > g.T[a] - 1 + h) v -= n[a];
        ok = ok && v >= -h && v <= g.T[a] - 1 + h;
        l[a] = v + h;
    }
    base = l[0] + (DIM >= 2 ? l[1] * g.fx : 0) + (DIM >= 3 ? l[2] * g.fxy : 0);
    return ok;
}

template <int DIM>
__device__ __forceinline__ bool inside_tile(const RunGeo &g, const int c[3])
{
    bool ok = true;
#pragma unroll
    for (int a = 0; a < DIM; ++a) ok = ok && (unsigned)(c[a] - g.lo[a]) < (unsigned)g.T[a];
    return ok;
}

// LDS index (deposit tile) of stencil point (-1,-1,-1), when the stencil lies
// in the deposit tile (c at most one cell outside the tile, periodically).
template <int DIM>
__device__ __forceinline__ bool dep_base(const RunGeo &g, const int n[3], const int c[3], int &base)
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
    base = l[0] + (DIM >= 2 ? l[1] * g.dx : 0) + (DIM >= 3 ? l[2] * g.dxy : 0);
    return ok;
}

template <int DIM>
__device__ __forceinline__ bool same_cell(const int a[3], const int b[3])
{
    bool s = a[0] == b[0];
    if (DIM >= 2) s = s && a[1] == b[1];
    if (DIM >= 3) s = s && a[2] == b[2];
    return s;
}

// Push of one particle with interpolated fields F (E, B or the gas velocity):
// updates u, returns the velocity v used for the position update and the
// deposit values mu (charge / mass, current, force, energy) per channel.
template <int PREC, int KIND>
__device__ __forceinline__ void push_particle(const UnitC<PREC> &U, typename RealOf<PREC>::T u[3],
                                              const typename RealOf<PREC>::T *F, typename RealOf<PREC>::T w,
                                              typename RealOf<PREC>::T v[3], typename RealOf<PREC>::T mu[kMaxCh])
{
    using R = typename RealOf<PREC>::T;
    if constexpr (KIND == PL_LORENTZ) {
        R du[3];
        R uo[3] = {u[0], u[1], u[2]};
        R u_old2 = fma(u[0], u[0], fma(u[1], u[1], u[2] * u[2]));
        boris<R>(u, F, F + 3, U.h, U.inv_c2, du);
        R u_new2 = fma(u[0], u[0], fma(u[1], u[1], u[2] * u[2]));
        const R gn2 = fma(u_new2, U.inv_c2, R(1));
        R gn = sqrt(gn2);
        R go = sqrt(fma(u_old2, U.inv_c2, R(1)));
        R ig = div_sqrt_ge1(R(1), gn2);
#pragma unroll
        for (int a = 0; a < 3; ++a) v[a] = u[a] * ig;
        R qw = U.q * w, mw = U.m * w;
        mu[0] = qw;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            mu[1 + a] = qw * v[a];
            mu[4 + a] = mw * du[a] * U.inv_dt;
        }
        if constexpr (PREC == PL_F64) {
            mu[7] = mw * U.c2 * (gn - go) * U.inv_dt;
        } else {
            R dd = fma(du[0], u[0] + uo[0], fma(du[1], u[1] + uo[1], du[2] * (u[2] + uo[2])));
            mu[7] = mw * dd / (gn + go) * U.inv_dt;
        }
    } else {
        R du[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            du[a] = (F[a] - u[a]) * U.one_m_decay;
            u[a] = F[a] + (u[a] - F[a]) * U.decay;
            v[a] = u[a];
        }
        R mw = U.m * w;
        mu[0] = mw;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            mu[1 + a] = R(0);
            mu[4 + a] = mw * du[a] * U.inv_dt;
        }
        mu[7] = R(0);
    }
}

// Offset of channel ch's plane in the LDS deposit tile (compile-time for
// CHS != 0), -1 when the channel is inactive.
template <int CHS, class U_>
__device__ __forceinline__ int ch_off(const U_ &U, int ch, int Ld)
{
    if constexpr (CHS != 0) return chs_slot(CHS, ch) >= 0 ? chs_slot(CHS, ch) * Ld : -1;
    else return U.soff[ch];
}

template <int PREC> struct RunShared {
    using R = typename RealOf<PREC>::T;
    const R *lds_f;
    double *lds_d;
    int *gq;
    uint32_t *dq_c;
    R *dq_d;      // 3 x dq
    R *dq_mu;     // nslot x dq
    int *ctl;     // [1] queued particles, [2] queued deposits
    int dq;       // capacity of the deposit queue
    bool narrow;  // only particles inside the tile join their batch's deposit sums
    double *sums; // 8 particle-side sums of the unit, smask + 1 partial sums each
    int smask;
};

// Particle-side conservation sums (only with SF_SUMS): LDS accumulation per
// unit, one global add per unit.
template <int PREC>
__device__ __forceinline__ void add_sums(const RunShared<PREC> &S, const typename RealOf<PREC>::T mu[kMaxCh])
{
#pragma unroll
    for (int k = 0; k < 8; ++k)
        __hip_atomic_fetch_add(S.sums + k * (S.smask + 1) + ((int)threadIdx.x & S.smask), (double)mu[k],
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Interpolate the fields of the LDS field tile to a particle whose stencil
// starts at record `fb`: the 27 (9 in 2D) records are read kPrefetch points
// ahead of their use, so several LDS reads are in flight while the previous
// points are summed.  Terms are added in the order (k, j, i) with explicit
// fused multiply-adds, the order of the tiled kernel.
constexpr int kPrefetch = 4;

template <int PREC, int DIM, int KIND>
__device__ __forceinline__ void gather_rec(const RunGeo &G, const typename RealOf<PREC>::T *lds_f, int fb,
                                           const typename RealOf<PREC>::T wx[3], const typename RealOf<PREC>::T wy[3],
                                           const typename RealOf<PREC>::T wz[3],
                                           typename RealOf<PREC>::T F[FieldRec<PREC, KIND>::NC])
{
    using R = typename RealOf<PREC>::T;
    constexpr int NC = FieldRec<PREC, KIND>::NC;
    constexpr int SY = Stencil<DIM>::SY, SZ = Stencil<DIM>::SZ;
    constexpr int NPT = SZ * SY * 3;
    constexpr int NB = kPrefetch + 1;
    R buf[NB][NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) F[q] = R(0);
#pragma unroll
    for (int pt = 0; pt < kPrefetch && pt < NPT; ++pt)
        load_rec<PREC, KIND>(lds_f, fb + (pt / 9) * G.fxy + ((pt / 3) % 3) * G.fx + pt % 3, G.Lf, buf[pt % NB]);
    R wyz = R(0);
#pragma unroll
    for (int pt = 0; pt < NPT; ++pt) {
        const int nx = pt + kPrefetch;
        if (nx < NPT)
            load_rec<PREC, KIND>(lds_f, fb + (nx / 9) * G.fxy + ((nx / 3) % 3) * G.fx + nx % 3, G.Lf, buf[nx % NB]);
        const int k = pt / 9, j = (pt / 3) % 3, i = pt % 3;
        if (i == 0) wyz = wz[k] * wy[j];
        const R wt = wyz * wx[i];
#pragma unroll
        for (int q = 0; q < NC; ++q) F[q] = fma(wt, buf[pt % NB][q], F[q]);
    }
}

// Deposit one particle (cell c, offset d, values mu per channel) into the LDS
// deposit tile when its stencil fits, else into the grids.
template <int PREC, int SHAPE, int DIM, int CHS>
__device__ __forceinline__ void deposit_single(const UnitC<PREC> &U, const RunGeo &G, double *lds_d, const int c[3],
                                               const typename RealOf<PREC>::T d[3], const double mu[kMaxCh])
{
    using R = typename RealOf<PREC>::T;
    R wx[3], wy[3], wz[3];
    stencil_weights<PREC, SHAPE, DIM>(d, wx, wy, wz);
    int base = 0;
    bool inl = dep_base<DIM>(G, U.n, c, base);
    deposit<PREC, DIM, CHS>(U, lds_d, inl, base, G.dx, G.dxy, G.Ld, c, wx, wy, wz, mu);
}

// The whole step of one particle on its own: gather from the LDS field tile
// when its stencil fits, else from the grids; push; store; deposit.
template <int PREC, int SHAPE, int DIM, int KIND, int CHS>
__device__ __forceinline__ void particle_single(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S, int p,
                                             bool do_sums, int &err)
{
    using R = typename RealOf<PREC>::T;
    constexpr int NC = FieldRec<PREC, KIND>::NC;
    Pos<PREC, DIM> pos;
    pos.load(U, p, err);
    R u[3] = {U.u[0][p], U.u[1][p], U.u[2][p]};
    R w = U.w ? U.w[p] : U.wdef;
    R d0[3] = {(R)pos.d[0], (R)pos.d[1], (R)pos.d[2]};
    R wx[3], wy[3], wz[3];
    stencil_weights<PREC, SHAPE, DIM>(d0, wx, wy, wz);
    R F[NC];
    int fb = 0;
    if (field_base<DIM>(G, U.n, pos.c, fb)) {
        gather_rec<PREC, DIM, KIND>(G, S.lds_f, fb, wx, wy, wz, F);
    } else {
        gather<PREC, DIM, NC>(U, nullptr, 0, false, 0, 0, 0, pos.c, wx, wy, wz, F);
    }
    R v[3], mu[kMaxCh];
    push_particle<PREC, KIND>(U, u, F, w, v, mu);
    if (U.fp[0]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) U.fp[a][p] = mu[4 + a];
    }
    R disp[3] = {R(0), R(0), R(0)};
#pragma unroll
    for (int a = 0; a < DIM; ++a) disp[a] = v[a] * U.dtdx[a];
    pos.advance(disp, U, err);
    pos.store(U, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) U.u[a][p] = u[a];
    double mud[kMaxCh];
#pragma unroll
    for (int ch = 0; ch < kMaxCh; ++ch) mud[ch] = (double)mu[ch];
    if (do_sums) add_sums(S, mu);
    R dn[3] = {(R)pos.d[0], (R)pos.d[1], (R)pos.d[2]};
    deposit_single<PREC, SHAPE, DIM, CHS>(U, G, S.lds_d, pos.c, dn, mud);
}

// Deposit of the queued records: one stencil row of one record per lane, so
// that a few dozen records keep every wave of the block busy for a few atomics
// instead of one wave for all of theirs (the block waits for the queue's end).
template <int PREC, int SHAPE, int DIM, int CHS>
__device__ __forceinline__ void drain_deposits(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S, int nd)
{
    using R = typename RealOf<PREC>::T;
    constexpr int SY = Stencil<DIM>::SY, SZ = Stencil<DIM>::SZ, NROW = SY * SZ;
    const int DQ = S.dq;
    for (int task = threadIdx.x; task < nd * NROW; task += blockDim.x) {
        const int i = task / NROW, row = task % NROW, kk = row / 3, jj = row % 3;
        int c[3];
        unpack_cell(S.dq_c[i], c[0], c[1], c[2]);
        const R d[3] = {S.dq_d[i], S.dq_d[DQ + i], S.dq_d[2 * DQ + i]};
        R wx[3], wy[3], wz[3];
        stencil_weights<PREC, SHAPE, DIM>(d, wx, wy, wz);
        auto pick = [](const R w[3], int k) -> R { return k == 0 ? w[0] : k == 1 ? w[1] : w[2]; };
        const R wyz = pick(wz, kk) * pick(wy, jj);
        double mu[kMaxCh];
#pragma unroll
        for (int ch = 0; ch < kMaxCh; ++ch) {
            const int so = ch_off<CHS>(U, ch, G.Ld);
            mu[ch] = so >= 0 ? (double)S.dq_mu[(so / G.Ld) * DQ + i] : 0.0;
        }
        int base = 0;
        if (dep_base<DIM>(G, U.n, c, base)) {
            double *at = S.lds_d + base + kk * G.dxy + jj * G.dx;
#pragma unroll
            for (int ii = 0; ii < 3; ++ii) {
                const double w = (double)(wyz * wx[ii]);
#pragma unroll
                for (int ch = 0; ch < kMaxCh; ++ch) {
                    const int so = ch_off<CHS>(U, ch, G.Ld);
                    if (so >= 0)
                        __hip_atomic_fetch_add(at + so + ii, w * mu[ch], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        } else {
            const int gy = DIM >= 2 ? wrap_cell(c[1] + jj - 1, U.n[1]) : 0;
            const int gz = DIM >= 3 ? wrap_cell(c[2] + kk - 1, U.n[2]) : 0;
            const long grow = (long)U.n[0] * (gy + (long)U.n[1] * gz);
#pragma unroll
            for (int ii = 0; ii < 3; ++ii) {
                const double w = (double)(wyz * wx[ii]) * U.inv_dv;
                const long gc = grow + wrap_cell(c[0] + ii - 1, U.n[0]);
#pragma unroll
                for (int ch = 0; ch < kMaxCh; ++ch)
                    if (ch_off<CHS>(U, ch, G.Ld) >= 0) global_add(U.M[ch] + gc, w * mu[ch]);
            }
        }
    }
}

// Deposit of the batch particles in the reference cell (dco[j]): their values
// are summed per stencil point and channel before each LDS atomic, in the
// particles' type, or in float64 (DACC: the precision of one float64 atomic
// per particle, for the kernels that stand in for that).
template <int PREC, int SHAPE, int DIM, int CHS, int KR, bool DACC>
__device__ __forceinline__ void batch_deposit(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S, int db,
                                              const Pos<PREC, DIM> pos[KR], typename RealOf<PREC>::T mu[KR][kMaxCh],
                                              const bool dco[KR])
{
    using R = typename RealOf<PREC>::T;
    using A = typename AccOf<PREC, DACC>::T;
    constexpr int SY = Stencil<DIM>::SY, SZ = Stencil<DIM>::SZ;
    R wx[KR][3], wy[KR][3], wz[KR][3];
    A mua[KR][kMaxCh];
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        R dn[3] = {(R)pos[j].d[0], (R)pos[j].d[1], (R)pos[j].d[2]};
        stencil_weights<PREC, SHAPE, DIM>(dn, wx[j], wy[j], wz[j]);
#pragma unroll
        for (int ch = 0; ch < kMaxCh; ++ch) mua[j][ch] = dco[j] ? (A)mu[j][ch] : A(0);
    }
#pragma unroll
    for (int k = 0; k < SZ; ++k)
#pragma unroll
        for (int jj = 0; jj < SY; ++jj) {
            R wyz[KR];
#pragma unroll
            for (int j = 0; j < KR; ++j) wyz[j] = wz[j][k] * wy[j][jj];
            const int row = db + k * G.dxy + jj * G.dx;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                A wt[KR];
#pragma unroll
                for (int j = 0; j < KR; ++j) wt[j] = (A)(wyz[j] * wx[j][i]);
#pragma unroll
                for (int ch = 0; ch < kMaxCh; ++ch) {
                    const int so = ch_off<CHS>(U, ch, G.Ld);
                    if (so < 0) continue;
                    A s = wt[0] * mua[0][ch];
#pragma unroll
                    for (int j = 1; j < KR; ++j) s = fma(wt[j], mua[j][ch], s);
                    __hip_atomic_fetch_add(S.lds_d + so + row + i, (double)s, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
}

// K consecutive elements of one particle array in one access.  The sort keeps
// a run's particles consecutive, and with the run order the runs of a wave
// follow one another, so these loads and stores cover contiguous stretches.
// Only element alignment is known (a batch starts at any particle), so the
// vector type declares exactly that; gfx950's multi-dword global accesses
// need dword alignment only.
template <class T, int K> struct Vec {
    typedef T V __attribute__((ext_vector_type(K), aligned(sizeof(T))));
    typedef __attribute__((address_space(1))) V *P;
    typedef const __attribute__((address_space(1))) V *CP;
};

// (n < 2^29 with the run-based algorithm, so a 32-bit byte offset from an
// array's base holds every element: one scalar base and one offset register per
// batch instead of a 64-bit address per array)
template <class T>
__device__ __forceinline__ gptr<T> at32(gptr<T> base, int i)
{
    return (gptr<T>)((gptr<char>)base + (uint32_t)((uint32_t)i * (uint32_t)sizeof(T)));
}

template <class T>
__device__ __forceinline__ gptr<const T> at32c(gptr<const T> base, int i)
{
    return (gptr<const T>)((gptr<const char>)base + (uint32_t)((uint32_t)i * (uint32_t)sizeof(T)));
}

template <class T, int K>
__device__ __forceinline__ void load_vec(gptr<const T> base, int i, T (&out)[K])
{
    const typename Vec<T, K>::V v = *reinterpret_cast<typename Vec<T, K>::CP>(at32c<T>(base, i));
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = v[k];
}

template <class T, int K>
__device__ __forceinline__ void store_vec(gptr<T> base, int i, const T (&in)[K])
{
    typename Vec<T, K>::V v;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = in[k];
    *reinterpret_cast<typename Vec<T, K>::P>(at32<T>(base, i)) = v;
}

// State of a whole batch (every slot handled in place) written back with one
// access per array.
template <int PREC, int DIM, int KR>
__device__ __forceinline__ void store_batch(const UnitC<PREC> &U, int start, const Pos<PREC, DIM> pos[KR],
                                            const typename RealOf<PREC>::T u[KR][3],
                                            const typename RealOf<PREC>::T mu[KR][kMaxCh])
{
    using R = typename RealOf<PREC>::T;
    R t[KR];
    if constexpr (PREC == PL_F32_OFFSET) {
        uint32_t cv[KR];
#pragma unroll
        for (int j = 0; j < KR; ++j)
            cv[j] = pack_cell(pos[j].c[0], DIM > 1 ? pos[j].c[1] : 0, DIM > 2 ? pos[j].c[2] : 0);
        store_vec<uint32_t, KR>(U.cell, start, cv);
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
#pragma unroll
            for (int j = 0; j < KR; ++j) t[j] = pos[j].d[a];
            store_vec<R, KR>(U.x[a], start, t);
        }
    } else {
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
#pragma unroll
            for (int j = 0; j < KR; ++j) t[j] = pos[j].x[a];
            store_vec<R, KR>(U.x[a], start, t);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int j = 0; j < KR; ++j) t[j] = u[j][a];
        store_vec<R, KR>(U.u[a], start, t);
    }
    if (U.fp[0]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int j = 0; j < KR; ++j) t[j] = mu[j][4 + a];
            store_vec<R, KR>(U.fp[a], start, t);
        }
    }
}

// Gather and push of the batch particles whose stencil lies in the
// LDS field tile (co[j]); fb[j] is the field record of stencil point
// (-1,-1,-1) of particle j, pi[j] its index (SEQ: pi[0] + j).
template <int PREC, int SHAPE, int DIM, int KIND, int KR, bool SEQ>
__device__ __forceinline__ void batch_push(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S,
                                           const int pi[KR], const int fb[KR], Pos<PREC, DIM> pos[KR], typename RealOf<PREC>::T u[KR][3],
                                           const typename RealOf<PREC>::T w[KR], const bool co[KR],
                                           typename RealOf<PREC>::T mu[KR][kMaxCh], bool do_sums, int &err)
{
    using R = typename RealOf<PREC>::T;
    constexpr int NC = FieldRec<PREC, KIND>::NC;

    // a batch of consecutive particles whose slots are all handled here is
    // written back at the end with one access per array; otherwise every slot
    // is stored on its own
    bool whole = SEQ;
#pragma unroll
    for (int j = 0; j < KR; ++j) whole = whole && co[j];

    // gather and push one particle at a time (each stencil point is one
    // interleaved LDS record read); keep what the batched deposit needs
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        const int p = SEQ ? pi[0] + j : pi[j];
        R wx[3], wy[3], wz[3];
        R d0[3] = {(R)pos[j].d[0], (R)pos[j].d[1], (R)pos[j].d[2]};
        stencil_weights<PREC, SHAPE, DIM>(d0, wx, wy, wz);
        R F[NC];
        gather_rec<PREC, DIM, KIND>(G, S.lds_f, fb[j], wx, wy, wz, F);
        R v[3];
        push_particle<PREC, KIND>(U, u[j], F, w[j], v, mu[j]);
        R disp[3] = {R(0), R(0), R(0)};
#pragma unroll
        for (int a = 0; a < DIM; ++a) disp[a] = v[a] * U.dtdx[a];
        int e2 = 0;
        pos[j].advance(disp, U, e2);
        if (co[j]) {
            err |= e2;
            if (!whole) {
                if constexpr (SEQ) {
                    const Pos<PREC, DIM> one[1] = {pos[j]};
                    const R uo[1][3] = {{u[j][0], u[j][1], u[j][2]}};
                    const R mo[1][kMaxCh] = {{R(0), R(0), R(0), R(0), mu[j][4], mu[j][5], mu[j][6], R(0)}};
                    store_batch<PREC, DIM, 1>(U, p, one, uo, mo);
                } else {
                    pos[j].store(U, p);
#pragma unroll
                    for (int a = 0; a < 3; ++a) U.u[a][p] = u[j][a];
                    if (U.fp[0]) {
#pragma unroll
                        for (int a = 0; a < 3; ++a) U.fp[a][p] = mu[j][4 + a];
                    }
                }
            }
            if (do_sums) add_sums(S, mu[j]);
        }
    }
    if (whole) store_batch<PREC, DIM, KR>(U, pi[0], pos, u, mu);
}

// Deposit of a pushed batch.  The batch particles in the reference cell are
// summed before each LDS atomic; the others are queued.  The reference is the
// new cell of the first batch particle, or of the second when the first shares
// its cell with no other batch particle.  co: the batch particles handled here,
// own: those of them that may join the sums.
template <int PREC, int SHAPE, int DIM, int CHS, int KR, bool DACC>
__device__ __forceinline__ void batch_dep(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S,
                                          const Pos<PREC, DIM> pos[KR], typename RealOf<PREC>::T mu[KR][kMaxCh],
                                          const bool co[KR], const bool own[KR])
{
    using R = typename RealOf<PREC>::T;
    const int DQ = S.dq;
    int f0 = -1, f1 = -1;
#pragma unroll
    for (int j = KR - 1; j >= 0; --j) {
        if (own[j]) {
            f1 = f0;
            f0 = j;
        }
    }
    int rc[3] = {0, 0, 0};
#pragma unroll
    for (int j = 0; j < KR; ++j)
        if (j == f0)
#pragma unroll
            for (int a = 0; a < 3; ++a) rc[a] = pos[j].c[a];
    bool alone = true;
#pragma unroll
    for (int j = 0; j < KR; ++j) alone = alone && (j == f0 || !(own[j] && same_cell<DIM>(pos[j].c, rc)));
    if (alone && f1 >= 0) {
#pragma unroll
        for (int j = 0; j < KR; ++j)
            if (j == f1)
#pragma unroll
                for (int a = 0; a < 3; ++a) rc[a] = pos[j].c[a];
    }
    int db = 0;
    const bool dep_in = f0 >= 0 && dep_base<DIM>(G, U.n, rc, db);
    bool dco[KR];
    bool any_dco = false;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        dco[j] = own[j] && dep_in && same_cell<DIM>(pos[j].c, rc);
        any_dco = any_dco || dco[j];
    }
    unsigned ovf_d = 0;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        if (co[j] && !dco[j]) {
            int q = atomicAdd(&S.ctl[2], 1);
            if (q < DQ) {
                S.dq_c[q] = pack_cell(pos[j].c[0], DIM > 1 ? pos[j].c[1] : 0, DIM > 2 ? pos[j].c[2] : 0);
#pragma unroll
                for (int a = 0; a < 3; ++a) S.dq_d[a * DQ + q] = (R)pos[j].d[a];
#pragma unroll
                for (int ch = 0; ch < kMaxCh; ++ch) {
                    int so = ch_off<CHS>(U, ch, G.Ld);
                    if (so >= 0) S.dq_mu[(so / G.Ld) * DQ + q] = mu[j][ch];
                }
            } else {
                ovf_d |= 1u << j;
            }
        }
    }
    // deposits that found the queue full
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        if (ovf_d & (1u << j)) {
            double mud[kMaxCh];
#pragma unroll
            for (int ch = 0; ch < kMaxCh; ++ch) mud[ch] = (double)mu[j][ch];
            R dn[3] = {(R)pos[j].d[0], (R)pos[j].d[1], (R)pos[j].d[2]};
            deposit_single<PREC, SHAPE, DIM, CHS>(U, G, S.lds_d, pos[j].c, dn, mud);
        }
    }
    if (any_dco) batch_deposit<PREC, SHAPE, DIM, CHS, KR, DACC>(U, G, S, db, pos, mu, dco);
}

// Stored state of one batch (up to KR particles): fetched when the batch starts
// (run kernel) or while the batch before it deposits (self-grouping kernels).
template <int PREC, int DIM, int KR> struct BatchRaw {
    using R = typename RealOf<PREC>::T;
    typename Pos<PREC, DIM>::Raw pr[KR];
    R u[KR][3], w[KR];
    int start, len;
};

template <int PREC, int DIM, int KR>
__device__ __forceinline__ void fetch_batch(const UnitC<PREC> &U, int start, int len, BatchRaw<PREC, DIM, KR> &B)
{
    using R = typename RealOf<PREC>::T;
    B.start = start;
    B.len = len;
    if (len == KR) {
        // a whole batch: one access per array
        R t[KR];
        if constexpr (PREC == PL_F32_OFFSET) {
            uint32_t cv[KR];
            load_vec<uint32_t, KR>((gptr<const uint32_t>)U.cell, start, cv);
#pragma unroll
            for (int j = 0; j < KR; ++j) B.pr[j].cell = cv[j];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (a < DIM) load_vec<R, KR>((gptr<const R>)U.x[a], start, t);
#pragma unroll
                for (int j = 0; j < KR; ++j) B.pr[j].o[a] = a < DIM ? t[j] : 0.0f;
            }
        } else {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (a < DIM) load_vec<R, KR>((gptr<const R>)U.x[a], start, t);
#pragma unroll
                for (int j = 0; j < KR; ++j) B.pr[j].x[a] = a < DIM ? t[j] : 0.0;
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            load_vec<R, KR>((gptr<const R>)U.u[a], start, t);
#pragma unroll
            for (int j = 0; j < KR; ++j) B.u[j][a] = t[j];
        }
        if (U.w) {
            load_vec<R, KR>(U.w, start, t);
#pragma unroll
            for (int j = 0; j < KR; ++j) B.w[j] = t[j];
        } else {
#pragma unroll
            for (int j = 0; j < KR; ++j) B.w[j] = U.wdef;
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        const int p = start + j;
        if (j < len) {
            if constexpr (PREC == PL_F32_OFFSET) {
                B.pr[j].cell = *at32<uint32_t>(U.cell, p);
#pragma unroll
                for (int a = 0; a < 3; ++a) B.pr[j].o[a] = a < DIM ? *at32<R>(U.x[a], p) : 0.0f;
            } else {
#pragma unroll
                for (int a = 0; a < 3; ++a) B.pr[j].x[a] = a < DIM ? *at32<R>(U.x[a], p) : 0.0;
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) B.u[j][a] = *at32<R>(U.u[a], p);
            B.w[j] = U.w ? *at32c<R>(U.w, p) : U.wdef;
        } else {
            B.pr[j] = B.pr[0];
#pragma unroll
            for (int a = 0; a < 3; ++a) B.u[j][a] = R(0);
            B.w[j] = R(0);
        }
    }
}

// One batch of up to KR particles of one run, of indices pi[j] (SEQ: pi[0] + j).
// mid() is called between the push and the deposit: the caller issues the next
// batch's loads there, where the gather's registers are free and the deposit
// covers them.
template <int PREC, int SHAPE, int DIM, int KIND, int CHS, int KR, bool SEQ, bool DACC, class Mid>
__device__ __forceinline__ void run_batch(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S,
                                          const BatchRaw<PREC, DIM, KR> &Bt, const int pi[KR], bool do_sums, int &err,
                                          Mid mid)
{
    using R = typename RealOf<PREC>::T;
    const int len = Bt.len;
    Pos<PREC, DIM> pos[KR];
    R u[KR][3], w[KR];
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        if (j < len) pos[j].set(Bt.pr[j], U, err);
        else pos[j] = pos[0];
#pragma unroll
        for (int a = 0; a < 3; ++a) u[j][a] = Bt.u[j][a];
        w[j] = Bt.w[j];
    }
    // every particle whose stencil lies in the LDS field tile is gathered in
    // the batch from its own cell (lanes read distinct records anyway)
    int fb[KR];
    bool co[KR], own[KR];
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        co[j] = field_base<DIM>(G, U.n, pos[j].c, fb[j]) && j < len;
        own[j] = co[j] && !(S.narrow && !inside_tile<DIM>(G, pos[j].c));
        if (!co[j]) fb[j] = 0;       // computed but unused: keep its reads inside the field tile
    }
    // particles outside the tile: queue for the single-particle path (when
    // the queue is full they run on their own after the batch)
    unsigned ovf_g = 0;
#pragma unroll
    for (int j = 0; j < KR; ++j) {
        if (j < len && !co[j]) {
            int q = atomicAdd(&S.ctl[1], 1);
            if (q < gq_cap(G.hf)) S.gq[q] = SEQ ? pi[0] + j : pi[j];
            else ovf_g |= 1u << j;
        }
    }
    bool any = false;
#pragma unroll
    for (int j = 0; j < KR; ++j) any = any || co[j];
    R mu[KR][kMaxCh];
    if (any) batch_push<PREC, SHAPE, DIM, KIND, KR, SEQ>(U, G, S, pi, fb, pos, u, w, co, mu, do_sums, err);
    mid();
    if (any) batch_dep<PREC, SHAPE, DIM, CHS, KR, DACC>(U, G, S, pos, mu, co, own);
    while (ovf_g) {
        const int j = __builtin_ctz(ovf_g);
        ovf_g &= ovf_g - 1u;
        int p = pi[0] + j;
        if constexpr (!SEQ) {
#pragma unroll
            for (int k = 1; k < KR; ++k)
                if (k == j) p = pi[k];
        }
        particle_single<PREC, SHAPE, DIM, KIND, CHS>(U, G, S, p, do_sums, err);
    }
}

// Control words: queued particles, queued deposits, chunks passed, and
// the two next units (item or -1, tile, particles, runs); then the launch's unit
// table.
enum RunsCtl { RC_QP = 1, RC_QD = 2, RC_QI = 3, RC_UNIT = 4 };
enum RunsUnit { RU_ITEM = 0, RU_TILE, RU_PBEG, RU_PEND, RU_RLO, RU_RHI, RU_WORDS };
constexpr int RU_NONE = -1, RU_LATER = -2, RU_HEAVY = 1 << 30;     // RU_ITEM: no unit left, not claimed yet, a heavy unit
enum { RC_ENDS = 16 };                 // unit table: first word
static_assert(RC_UNIT + 2 * RU_WORDS <= RC_ENDS && 4 * (RC_ENDS + kRunsGroups) == kRunsCtlBytes, "control words");

template <int PREC, int KIND>
__host__ __device__ inline size_t runs_lds_bytes(int Lf, int Ld, int nslot, int hf, int threads, size_t offs[6])
{
    using R = typename RealOf<PREC>::T;
    return runs_lds_layout(sizeof(R), FieldRec<PREC, KIND>::FS, Lf, Ld, nslot, hf, threads, offs);
}

// Threads per block of the run kernel.  One block per CU (the LDS tiles take
// most of the 160 KB), so two waves per SIMD: the compiler may spend registers
// on reads in flight.
constexpr int kRunsThreads = 512;

// Gas velocity at a position of the Runge-Kutta scheme: from the LDS field
// records when the stencil lies in the tile's field tile, else from the grid.
template <int PREC, int SHAPE, int DIM>
__device__ __forceinline__ void tracer_velocity(const UnitC<PREC> &U, const RunGeo &G,
                                                const typename RealOf<PREC>::T *lds_f, const Pos<PREC, DIM> &q,
                                                typename RealOf<PREC>::T k[3])
{
    using R = typename RealOf<PREC>::T;
    R dm[3] = {(R)q.d[0], (R)q.d[1], (R)q.d[2]};
    R sx[3], sy[3], sz[3];
    stencil_weights<PREC, SHAPE, DIM>(dm, sx, sy, sz);
    int fb = 0;
    if (field_base<DIM>(G, U.n, q.c, fb)) gather_rec<PREC, DIM, PL_TRACER>(G, lds_f, fb, sx, sy, sz, k);
    else gather<PREC, DIM, 3>(U, nullptr, 0, false, 0, 0, 0, q.c, sx, sy, sz, k);
}

// One passive tracer on the gas velocity frozen over the step (Eq. 1):
// Heun's two-stage scheme, or the three-stage SSP scheme of Shu and Osher,
// x + dt (k1 + k2 + 4 k3) / 6 with k1 = v(x), k2 = v(x + dt k1),
// k3 = v(x + dt (k1 + k2) / 4); the stored velocity is the step's mean.
// The same terms in the same order as the tiled kernel's tracer path.
template <int PREC, int SHAPE, int DIM>
__device__ __forceinline__ void tracer_particle(const UnitC<PREC> &U, const RunGeo &G,
                                                const typename RealOf<PREC>::T *lds_f, int p, int &err)
{
    using R = typename RealOf<PREC>::T;
    Pos<PREC, DIM> pos;
    pos.load(U, p, err);
    R k1[3], k2[3], v[3];
    tracer_velocity<PREC, SHAPE, DIM>(U, G, lds_f, pos, k1);
    // velocity of the stage at x + dt * s (s in cells per unit time)
    auto stage = [&](const R sv[3], R k[3]) {
        Pos<PREC, DIM> mid = pos;
        R dd[3] = {R(0), R(0), R(0)};
#pragma unroll
        for (int a = 0; a < DIM; ++a) dd[a] = sv[a] * U.dtdx[a];
        mid.advance(dd, U, err);
        tracer_velocity<PREC, SHAPE, DIM>(U, G, lds_f, mid, k);
    };
    stage(k1, k2);
    if (U.rk == 3) {
        R hq[3], k3[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) hq[a] = R(0.25) * (k1[a] + k2[a]);
        stage(hq, k3);
#pragma unroll
        for (int a = 0; a < 3; ++a) v[a] = (k1[a] + k2[a] + R(4) * k3[a]) / R(6);
    } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) v[a] = R(0.5) * (k1[a] + k2[a]);
    }
    R disp[3] = {R(0), R(0), R(0)};
#pragma unroll
    for (int a = 0; a < DIM; ++a) disp[a] = v[a] * U.dtdx[a];
    pos.advance(disp, U, err);
    pos.store(U, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) U.u[a][p] = v[a];
}

// Grid cell of field record e of a tile (hf-cell halo).
template <int PREC, int DIM>
__device__ __forceinline__ long rec_cell(const UnitC<PREC> &U, const RunGeo &G, int e)
{
    const int Ly = G.T[1] + 2 * G.hf;
    const int lx = e % G.fx, ly = (e / G.fx) % Ly, lz = e / G.fxy;
    const int gx = wrap_near(G.lo[0] + lx - G.hf, U.n[0]);
    const int gy = DIM >= 2 ? wrap_near(G.lo[1] + ly - G.hf, U.n[1]) : 0;
    const int gz = DIM >= 3 ? wrap_near(G.lo[2] + lz - G.hf, U.n[2]) : 0;
    return gx + (long)U.n[0] * (gy + (long)U.n[1] * gz);
}

template <int PREC, int DIM, int KIND>
__device__ __forceinline__ void rec_load(const UnitC<PREC> &U, const RunGeo &G, int e,
                                         double (&v)[FieldRec<PREC, KIND>::NC])
{
    const long gc = rec_cell<PREC, DIM>(U, G, e);
#pragma unroll
    for (int q = 0; q < FieldRec<PREC, KIND>::NC; ++q) v[q] = U.gf[q][gc];
}

// (conflict-free: consecutive threads write consecutive records)
template <int PREC, int KIND>
__device__ __forceinline__ void rec_store(const RunGeo &G, typename RealOf<PREC>::T *lds_f, int e,
                                          const double (&v)[FieldRec<PREC, KIND>::NC])
{
    using R = typename RealOf<PREC>::T;
    using FR = FieldRec<PREC, KIND>;
    constexpr int NC = FR::NC, FS = FR::FS;
    if constexpr (FR::PLANES) {
        float4 *p = reinterpret_cast<float4 *>(lds_f);
        p[e] = make_float4((R)v[0], (R)v[1], (R)v[2], (R)v[3]);
        reinterpret_cast<float2 *>(p + G.Lf)[e] = make_float2((R)v[4], (R)v[5]);
    } else {
        R w[FS];
#pragma unroll
        for (int q = 0; q < FS; ++q) w[q] = q < NC ? (R)v[q] : R(0);
        if constexpr (PREC == PL_F32_OFFSET) {
            *reinterpret_cast<float4 *>(lds_f + FS * e) = make_float4(w[0], w[1], w[2], w[3]);
        } else {
#pragma unroll
            for (int k = 0; k < FS / 2; ++k)
                *reinterpret_cast<double2 *>(lds_f + FS * e + 2 * k) = make_double2(w[2 * k], w[2 * k + 1]);
        }
    }
}

// Stage the field records of a tile and clear its deposit tile (ndep values).
// Float32 form: two-deep pipeline, a record's loads are issued before the
// previous record is stored, and the first loads overlap the clearing.  The
// caller synchronises.
template <int PREC, int DIM, int KIND>
__device__ __forceinline__ void stage_unit(const UnitC<PREC> &U, const RunGeo &G, typename RealOf<PREC>::T *lds_f,
                                           double *lds_d, int ndep)
{
    constexpr int NC = FieldRec<PREC, KIND>::NC;
    if constexpr (PREC == PL_F32_OFFSET) {
        double cur[NC];
        int e = threadIdx.x;
        if (e < G.Lf) rec_load<PREC, DIM, KIND>(U, G, e, cur);
        for (int k = threadIdx.x; k < ndep; k += blockDim.x) lds_d[k] = 0.0;
        for (; e < G.Lf; e += blockDim.x) {
            double nxt[NC];
            const int en = e + (int)blockDim.x;
            if (en < G.Lf) rec_load<PREC, DIM, KIND>(U, G, en, nxt);
            rec_store<PREC, KIND>(G, lds_f, e, cur);
#pragma unroll
            for (int q = 0; q < NC; ++q) cur[q] = nxt[q];
        }
    } else {
        // float64 records: one at a time (the pipeline's registers spill there)
        for (int e = threadIdx.x; e < G.Lf; e += blockDim.x) {
            double v[NC];
            rec_load<PREC, DIM, KIND>(U, G, e, v);
            rec_store<PREC, KIND>(G, lds_f, e, v);
        }
        for (int k = threadIdx.x; k < ndep; k += blockDim.x) lds_d[k] = 0.0;
    }
}

// Flush of a deposit tile, which it leaves cleared: one float64 global atomic
// per touched cell and channel.  A cell's values are read before the previous
// cell's atomics are issued.
template <int PREC, int DIM, int CHS>
__device__ __forceinline__ void flush_unit(const UnitC<PREC> &U, const RunGeo &G, double *lds_d)
{
    const int Ly = G.T[1] + 4;
    auto take = [&](int e, double (&v)[kMaxCh]) {
#pragma unroll
        for (int ch = 0; ch < kMaxCh; ++ch) {
            const int so = ch_off<CHS>(U, ch, G.Ld);
            v[ch] = so >= 0 ? lds_d[so + e] : 0.0;
        }
    };
    double v[kMaxCh];
    int e = threadIdx.x;
    if (e < G.Ld) take(e, v);
    for (; e < G.Ld; e += blockDim.x) {
        double nv[kMaxCh];
        const int en = e + (int)blockDim.x;
        if (en < G.Ld) take(en, nv);
        bool any = false;
#pragma unroll
        for (int ch = 0; ch < kMaxCh; ++ch) {
            const int so = ch_off<CHS>(U, ch, G.Ld);
            if (so >= 0) lds_d[so + e] = 0.0;
            any = any || v[ch] != 0.0;
        }
        if (any) {
            const int lx = e % G.dx, ly = (e / G.dx) % Ly, lz = e / G.dxy;
            const int gx = wrap_near(G.lo[0] + lx - 2, U.n[0]);
            const int gy = DIM >= 2 ? wrap_near(G.lo[1] + ly - 2, U.n[1]) : 0;
            const int gz = DIM >= 3 ? wrap_near(G.lo[2] + lz - 2, U.n[2]) : 0;
            const long gc = gx + (long)U.n[0] * (gy + (long)U.n[1] * gz);
#pragma unroll
            for (int ch = 0; ch < kMaxCh; ++ch) {
                const int so = ch_off<CHS>(U, ch, G.Ld);
                if (so >= 0) global_add(U.M[ch] + gc, v[ch] * U.inv_dv);
            }
        }
#pragma unroll
        for (int ch = 0; ch < kMaxCh; ++ch) v[ch] = nv[ch];
    }
}

// Geometry of tile t of an item, and a unit's LDS sections.
template <int DIM, int HF, int TS>
__device__ __forceinline__ void unit_geo(const ItemDesc &I, int t, unsigned flags, RunGeo &G)
{
    G.T[0] = TS ? ts_dim(TS, 0) : I.tile[0];
    G.T[1] = TS ? ts_dim(TS, 1) : I.tile[1];
    G.T[2] = TS ? ts_dim(TS, 2) : I.tile[2];
    G.lo[0] = (t % I.ntile[0]) * G.T[0];
    G.lo[1] = ((t / I.ntile[0]) % I.ntile[1]) * G.T[1];
    G.lo[2] = (t / (I.ntile[0] * I.ntile[1])) * G.T[2];
    G.hf = HF ? HF : ((flags & SF_FHALO2) ? 2 : 1);
    G.fx = G.T[0] + 2 * G.hf;
    G.fxy = G.fx * (G.T[1] + 2 * G.hf);
    G.Lf = G.fxy * (DIM >= 3 ? G.T[2] + 2 * G.hf : 1);
    G.dx = G.T[0] + 4;
    G.dxy = G.dx * (G.T[1] + 4);
    G.Ld = G.dxy * (DIM >= 3 ? G.T[2] + 4 : 1);
}

template <int PREC, int KIND>
__device__ __forceinline__ void unit_shared(const RunGeo &G, int nslot, unsigned char *smem_raw, int lds_bytes,
                                            unsigned flags, RunShared<PREC> &S)
{
    using R = typename RealOf<PREC>::T;
    size_t offs[6];
    const int dq = runs_queue(sizeof(R), (int)blockDim.x);
    runs_lds_bytes<PREC, KIND>(G.Lf, G.Ld, nslot, G.hf, (int)blockDim.x, offs);
    S.narrow = PREC == PL_F32_OFFSET && (flags & SF_NARROW);
    S.lds_f = reinterpret_cast<R *>(smem_raw + offs[0]);
    S.lds_d = reinterpret_cast<double *>(smem_raw + offs[1]);
    S.gq = reinterpret_cast<int *>(smem_raw + offs[2]);
    S.dq_c = reinterpret_cast<uint32_t *>(smem_raw + offs[3]);
    S.dq_d = reinterpret_cast<R *>(smem_raw + offs[4]);
    S.dq_mu = S.dq_d + 3 * dq;
    S.dq = dq;
    S.ctl = reinterpret_cast<int *>(smem_raw + lds_bytes - kRunsCtlBytes);
    S.sums = reinterpret_cast<double *>(smem_raw + offs[5]);
    S.smask = 0;
}

__device__ __forceinline__ void run_entry(int e, int pbeg, int pend, int &rs, int &rl)
{
    rs = min(max(e >> 2, pbeg), pend - 1);
    rl = min((e & 3) + 1, pend - rs);
}

// The runs [r_lo, r_hi) of a unit, one per thread at a time (r = r_lo + tid,
// + blockDim, ...; entry: the first one's), each cut into batches of KR.  A
// batch is loaded when it starts: with the next batch in flight the float32
// kernel needed all its registers (1.38 ms on the 128^3 box with 2^24
// particles against 1.32 before the units were pipelined).  A long piece is taken in segments of 4 * blockDim
// runs with the LDS queues drained between segments when half full; every piece
// ends with a drain.  Segment count, drain decisions and barriers are uniform
// across the block.  The last wave (it has the fewest runs) calls last() when it
// is through, before the block meets.  Pieces of one tile on
// several CUs meet only in the global atomics of the flush.
template <int PREC, int SHAPE, int DIM, int KIND, int CHS, int KR, class Ahead, class Last>
__device__ __forceinline__ void unit_runs(const UnitC<PREC> &U, const RunGeo &G, const RunShared<PREC> &S,
                                          gptr<const int32_t> runs, int pbeg, int pend, int r_lo, int r_hi, int entry,
                                          bool do_sums, int &err, Ahead ahead, Last last)
{
    const int bd = (int)blockDim.x, seg = 4 * bd;
    for (int s0 = r_lo; s0 < r_hi; s0 += seg) {
        const int s1 = min(r_hi, s0 + seg);
        int r = s0 + (int)threadIdx.x, b = 0, rs = 0, rl = 0;
        if (r < s1) run_entry(s0 > r_lo ? runs[r] : entry, pbeg, pend, rs, rl);
        while (r < s1) {
            BatchRaw<PREC, DIM, KR> now;
            fetch_batch<PREC, DIM, KR>(U, rs + b, min(KR, rl - b), now);
            const int pi[KR] = {now.start};
            run_batch<PREC, SHAPE, DIM, KIND, CHS, KR, true, false>(U, G, S, now, pi, do_sums, err, []() {});
            b += KR;
            if (b >= rl) {
                r += bd;
                b = 0;
                if (r < s1) run_entry(runs[r], pbeg, pend, rs, rl);
            }
        }
        const bool end = s1 >= r_hi;
        if (end) ahead();
        if (end && (int)threadIdx.x >= bd - 64) last();
        __syncthreads();
        const int qg = S.ctl[RC_QP], qd = S.ctl[RC_QD];
        if (end || 2 * qg > gq_cap(G.hf) || 2 * qd > S.dq) {
            drain_deposits<PREC, SHAPE, DIM, CHS>(U, G, S, min(qd, S.dq));
            const int ng = min(qg, gq_cap(G.hf));
            if (ng > 0) {
                for (int i = threadIdx.x; i < ng; i += blockDim.x)
                    particle_single<PREC, SHAPE, DIM, KIND, CHS>(U, G, S, S.gq[i], do_sums, err);
                // (rare: the loads again rather than their registers held through the gathers)
                if (end) ahead();
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                S.ctl[RC_QP] = 0;
                S.ctl[RC_QD] = 0;
            }
        }
        if (!end) __syncthreads();      // all threads hold the same counts before anyone queues again
    }
}

// One work unit of the kernel that takes every species kind (a piece of tile t
// of item I): stage the tile's field records (and clear its deposit tile),
// advance the piece's runs, and flush the deposits; passive tracers are
// advanced one particle at a time from the same field records.  last(): see
// unit_runs.
template <int PREC, int SHAPE, int DIM, int KIND, int HF, int TS, int CHS, class Last>
__device__ __forceinline__ void runs_unit(const ItemDesc &I, int t, int pbeg, int pend, int r_lo, int r_hi,
                                          unsigned flags, int lds_bytes, unsigned char *smem_raw, int &err, Last last)
{
    constexpr int KR = PREC == PL_F32_OFFSET ? 4 : 2;
    const bool do_sums = flags & SF_SUMS;
    RunGeo G;
    unit_geo<DIM, HF, TS>(I, t, flags, G);
    UnitC<PREC> U;
    load_unit<PREC>(I, U, G.Ld);
    RunShared<PREC> S;
    unit_shared<PREC, KIND>(G, I.nslot, smem_raw, lds_bytes, flags, S);
    stage_unit<PREC, DIM, KIND>(U, G, const_cast<typename RealOf<PREC>::T *>(S.lds_f), S.lds_d, G.Ld * I.nslot);
    if (threadIdx.x == 0) {
        S.ctl[RC_QP] = 0;
        S.ctl[RC_QD] = 0;
    }
    if (threadIdx.x < 8) S.sums[threadIdx.x] = 0.0;
    __syncthreads();
    const gptr<const int32_t> runs = (gptr<const int32_t>)(I.runs + pbeg);
    if constexpr (KIND == PL_TRACER) {
        // passive tracers deposit nothing: thread k advances the particles of
        // runs r_lo + k, + blockDim, ... on their own
        for (int r = r_lo + (int)threadIdx.x; r < r_hi; r += (int)blockDim.x) {
            int rs = 0, rl = 0;
            run_entry(runs[r], pbeg, pend, rs, rl);
            for (int q = 0; q < rl; ++q) tracer_particle<PREC, SHAPE, DIM>(U, G, S.lds_f, rs + q, err);
        }
        if ((int)threadIdx.x >= (int)blockDim.x - 64) last();
    } else {
        const int entry = r_lo + (int)threadIdx.x < r_hi ? runs[r_lo + (int)threadIdx.x] : 0;
        unit_runs<PREC, SHAPE, DIM, KIND, CHS, KR>(U, G, S, runs, pbeg, pend, r_lo, r_hi, entry, do_sums, err, []() {}, last);
        if (do_sums && threadIdx.x < 8 && S.sums[threadIdx.x] != 0.0) global_add(I.psum + threadIdx.x, S.sums[threadIdx.x]);
        flush_unit<PREC, DIM, CHS>(U, G, S.lds_d);
    }
}

// Work units of a launch.  Item k has as many units as its sort listed, largest
// first as (tile, piece | npieces << 16); the launch numbers the units of all
// its items in order.  Every block adds the counts up for itself: entry k of
// its unit table is the end of the units of the k-th group of ceil(nitems /
// kRunsGroups) items.  An item whose tables do not cover its particles (tile
// offsets from 0 to np, at least one unit when np > 0: never sorted, or its
// count changed since) is latched and left alone.
__device__ __forceinline__ int item_units(const ItemDesc &I, bool &stale)
{
    const int nu = min(max(I.runs[runs_count_at(I.np, I.ntiles)], 0), I.nunits > 0 ? I.nunits + kRunsSplit : 0);
    stale = I.tile_start[0] != 0 || I.tile_start[I.ntiles] != I.np || (I.np > 0 && nu == 0);
    return stale ? 0 : nu;
}

__device__ __forceinline__ void runs_units(const ItemDesc *__restrict__ items, int nitems, int *errflags, int *ctl)
{
    if (threadIdx.x < kRunsGroups) {
        const int per = (nitems + kRunsGroups - 1) / kRunsGroups, k0 = (int)threadIdx.x * per;
        int n = 0;
        bool any = false;
        for (int k = k0; k < min(nitems, k0 + per); ++k) {
            bool stale;
            n += item_units(items[k], stale);
            any = any || stale;
        }
        if (any) atomicOr(errflags, (int)ERR_UNSORTED);
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(n, off, 64);
            if ((int)threadIdx.x >= off) n += y;
        }
        ctl[RC_ENDS + threadIdx.x] = n;
    }
}
static_assert(kRunsGroups == 64, "the unit table is one wave's scan");

// Claims.  The parts of the launch's units are dealt to kQueues chunks, kDeal
// consecutive ones at a time (neighbouring tiles share a chunk), each chunk with
// its own counter; block b starts on chunk b % kQueues and moves to the next
// chunk with parts left when its own is exhausted (qi chunks passed, mirrored in
// ctl[RC_QI]).  Blocks are dispatched to the XCDs in turn, so the blocks of one
// XCD mostly share a chunk and find its field records in their L2; results do
// not depend on that placement.  The dealing spreads an item's crowded tiles,
// which its list has first, over the chunks: in eight contiguous ones the blocks
// of the first had all of them, one after another.  Measured per pass of 8
// steps and a sort, contiguous and dealt in 64, 16 and 4: clumped 64^3 float64
// 2414, 2034, 1840 and 1862 us, clumped 128^3 float32 11.04, 8.95, 9.11 and 9.13 ms; even
// 128^3 float32 10.75, 10.62, 10.62 and 10.71 ms, eleven items at once 15.0,
// 15.2, 14.9 and 14.8 ms.  With fewer units than blocks every unit is claimed in
// `sub` parts of its runs (of at least kRunsMinSub), so a small box fills the chip too.
// Every part flushes a whole tile, and a launch's atomics are bound at about
// 5e10/s: 32^3 cells with 2.6e5 particles (64 tiles for 256 CUs) took 67 us per
// launch whole, 56 us in four parts of 300 runs, 54.5 us in two.
constexpr int kRunsMinSub = 512;

__device__ __forceinline__ int runs_sub(int total)
{
    return total > 0 && total < (int)gridDim.x ? (int)gridDim.x / total : 1;
}

// The next claim of the block (by one whole wave, uniformly): a part of a unit
// in [0, parts), or -1 when every chunk is exhausted.  A chunk found exhausted
// costs one round trip; the counters of the others are then read together.
__device__ __forceinline__ int runs_take(int parts, unsigned *counter, int &qi)
{
    const int lane = (int)threadIdx.x & 63, home = (int)(blockIdx.x % kQueues);
    while (qi < kQueues) {
        const int q = (home + qi) % kQueues, size = chunk_size(q, parts);
        if (size > 0) {
            int n = 0;
            if (lane == 0) n = (int)atomicAdd(counter + q, 1u);
            n = __builtin_amdgcn_readfirstlane(n);
            if (n < size) return chunk_part(q, n);
        }
        // lane k: whether the chunk after k passed ones has units left
        const int p = (home + lane) % kQueues;
        unsigned seen = ~0u;
        if (lane < kQueues) seen = __hip_atomic_load(counter + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const bool left = lane < kQueues && lane > qi && seen < (unsigned)chunk_size(p, parts);
        const uint64_t m = __ballot(left);
        qi = m ? (int)__builtin_ctzll(m) : kQueues;
    }
    return -1;
}

// The runs of claim g (one whole wave, uniformly): item (with RU_HEAVY where
// the part has more than kHeavy times the particles of the item's mean unit),
// tile, particles and runs of one unit's part; false when it has none (or the
// unit list is damaged).
constexpr float kHeavy = 1.5f;
__device__ __forceinline__ bool runs_lookup(const ItemDesc *__restrict__ items, int nitems, const int *ctl, int g, int sub,
                                            int *u)
{
    int s = 0;
    if (sub > 1) {
        s = g % sub;
        g /= sub;
    }
    const int lane = (int)threadIdx.x & 63, per = (nitems + kRunsGroups - 1) / kRunsGroups;
    const int end = ctl[RC_ENDS + lane];
    const int grp = min((int)__popcll(__ballot(end <= g)), kRunsGroups - 1);
    int local = g - (grp > 0 ? __builtin_amdgcn_readlane(end, grp - 1) : 0), k = grp * per;
    const int kend = min(nitems, k + per);
    for (; k < kend - 1; ++k) {
        bool stale;
        const int n = item_units(items[k], stale);
        if (local < n) break;
        local -= n;
    }
    if (k >= kend) return false;
    const ItemDesc &I = items[k];
    const int32_t *unit = I.runs + runs_units_at(I.np, I.ntiles) + 2 * local;
    const int nu = __builtin_amdgcn_readfirstlane(I.runs[runs_count_at(I.np, I.ntiles)]);
    const int t = __builtin_amdgcn_readfirstlane(unit[0]), w = __builtin_amdgcn_readfirstlane(unit[1]);
    const int piece = w & 0xffff, npieces = w >> 16;
    if ((unsigned)t >= (unsigned)I.ntiles || npieces < 1 || piece >= npieces) return false;
    const int beg = I.tile_start[t], last = I.tile_start[t + 1], cnt = I.runs[I.np + t];
    const int pbeg = min(max(__builtin_amdgcn_readfirstlane(beg), 0), I.np);
    const int pend = min(max(__builtin_amdgcn_readfirstlane(last), pbeg), I.np);
    const int nruns = min(max(__builtin_amdgcn_readfirstlane(cnt), 0), pend - pbeg);
    int lo = 0, hi = nruns;
    if (npieces > 1) {
        lo = (int)((long long)nruns * piece / npieces);
        hi = (int)((long long)nruns * (piece + 1) / npieces);
    }
    const bool heavy = (float)(pend - pbeg) * (float)nu > kHeavy * (float)I.np * (float)npieces;
    if (sub > 1) {
        // parts of at least kRunsMinSub runs, the last ones empty
        const int n = hi - lo, parts = max(1, min(sub, n / kRunsMinSub));
        if (s >= parts) return false;
        hi = lo + (int)((long long)n * (s + 1) / parts);
        lo = lo + (int)((long long)n * s / parts);
    }
    u[RU_ITEM] = k | (heavy ? RU_HEAVY : 0);
    u[RU_TILE] = t;
    u[RU_PBEG] = pbeg;
    u[RU_PEND] = pend;
    u[RU_RLO] = lo;
    u[RU_RHI] = hi;
    return hi > lo;
}

// The next unit with runs, claimed and looked up by one whole wave into a
// unit's control words (item -1: none left); whether it is a heavy one.
__device__ __forceinline__ bool runs_next(const ItemDesc *__restrict__ items, int nitems, unsigned *counter, int *ctl,
                                          int *unit)
{
    const int total = __builtin_amdgcn_readfirstlane(ctl[RC_ENDS + kRunsGroups - 1]), sub = runs_sub(total);
    int qi = __builtin_amdgcn_readfirstlane(ctl[RC_QI]);
    bool heavy = false;
    for (;;) {
        int g = -1;
        if (total * sub <= (int)gridDim.x) {
            // a block for every part: block b takes part b (see claim_unit)
            if (qi == 0 && (int)blockIdx.x < total * sub) g = (int)blockIdx.x;
            qi = kQueues;
        } else {
            g = runs_take(total * sub, counter, qi);
        }
        if (g < 0) {
            unit[RU_ITEM] = RU_NONE;
            break;
        }
        if (runs_lookup(items, nitems, ctl, g, sub, unit)) {
            heavy = __builtin_amdgcn_readfirstlane(unit[RU_ITEM]) & RU_HEAVY;
            break;
        }
    }
    ctl[RC_QI] = qi;
    return heavy;
}

// The last block to finish resets the chunk counters for the next launch (a
// launch with a block for every part claimed nothing).
__device__ __forceinline__ void release_queues(unsigned *counter, const int *ctl)
{
    const int total = ctl[RC_ENDS + kRunsGroups - 1];
    if (total * runs_sub(total) <= (int)gridDim.x) return;            // uniform
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        unsigned done = atomicAdd(counter + kQueues, 1u);
        if (done == gridDim.x - 1) {
            for (int q = 0; q < kQueues; ++q) atomicExch(counter + q, 0u);
            atomicExch(counter + kQueues, 0u);
        }
    }
}

__device__ __forceinline__ void runs_latch(int err, int *errflags)
{
    unsigned long long any = __ballot(err != 0);
    if (any) {
        int e = err;
        for (int off = 32; off > 0; off >>= 1) e |= __shfl_xor(e, off, 64);
        if ((threadIdx.x & 63) == 0) atomicOr(errflags, e);
    }
}

// HF: field halo width (1 or 2) fixed at compile time, or 0 to take it from
// the launch flags; TS and HF fixed make every LDS stencil offset an
// immediate.  NT: threads per block; with kRunsSmall two blocks share a CU.
template <int PREC, int SHAPE, int DIM, int KIND, int HF, int TS, int CHS, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_runs(const ItemDesc *__restrict__ items, int nitems,
                                             unsigned *counter, int *errflags, unsigned flags, int lds_bytes)
{
    using R = typename RealOf<PREC>::T;
    constexpr int KR = PREC == PL_F32_OFFSET ? 4 : 2;
    constexpr int NC = FieldRec<PREC, KIND>::NC;
    // records of the next unit that a thread loads ahead of the flush
    constexpr int NPRE = 2;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    int *ctl = reinterpret_cast<int *>(smem_raw + lds_bytes - kRunsCtlBytes);
    const bool do_sums = flags & SF_SUMS;
    int err = 0;
    if (threadIdx.x == 0) {
        ctl[RC_QP] = 0;
        ctl[RC_QD] = 0;
        ctl[RC_QI] = 0;
    }
    runs_units(items, nitems, errflags, ctl);
    __syncthreads();
    if (threadIdx.x < 64) runs_next(items, nitems, counter, ctl, ctl + RC_UNIT);
    __syncthreads();
    // Unit by unit, two known ahead (the last wave looks the second up while the
    // others work), but none beyond a heavy one: a block that holds two crowded
    // pieces does them in turn while others have run out (clumped 48^3 in float64,
    // 8 steps and a sort: 1302 us with the pieces held, 1125 us without).  Past a
    // heavy unit the next is claimed at its end (RU_LATER) and staged without
    // loads ahead.  The loads of the next unit's fields go out before this
    // unit's flush and come back before its atomics, and the LDS has them right
    // after it.  What it measured, share of the waves' time on the 128^3 box
    // with 2^24 particles (float32, rho J F): staging 9.4 to 3 %, claims 4.4 to 0
    // %, the queue's drain and its wait 7.0 to 5 %, flush 10.6 % as before (bound
    // by the round trips of its device-scope atomics); with the smaller records
    // and no batch prefetch 1.38 to 1.15 ms per launch.
    struct Ref {
        int iti, t, pbeg, pend, r_lo, r_hi;
    };
    auto known = [&](int slot) -> Ref {
        const int *w = ctl + RC_UNIT + RU_WORDS * slot;
        auto word = [&](int k) -> int { return __builtin_amdgcn_readfirstlane(w[k]); };
        const int it = word(RU_ITEM);
        return Ref{it < 0 ? it : it & ~RU_HEAVY, word(RU_TILE), word(RU_PBEG), word(RU_PEND), word(RU_RLO), word(RU_RHI)};
    };
    Ref cur = known(0);
    if (cur.iti >= 0) {
        RunGeo G;
        UnitC<PREC> U;
        RunShared<PREC> S;
        const int tid = (int)threadIdx.x, bd = (int)blockDim.x;
        unit_geo<DIM, HF, TS>(items[cur.iti], cur.t, flags, G);
        load_unit<PREC>(items[cur.iti], U, G.Ld);
        unit_shared<PREC, KIND>(G, items[cur.iti].nslot, smem_raw, lds_bytes, flags, S);
        stage_unit<PREC, DIM, KIND>(U, G, const_cast<R *>(S.lds_f), S.lds_d, G.Ld * items[cur.iti].nslot);
        if (tid < 8) S.sums[tid] = 0.0;
        if (tid >= bd - 64) {
            int *next = ctl + RC_UNIT + RU_WORDS;
            if (__builtin_amdgcn_readfirstlane(ctl[RC_UNIT]) & RU_HEAVY) next[RU_ITEM] = RU_LATER;
            else runs_next(items, nitems, counter, ctl, next);
        }
        auto first_entry = [&](const Ref &u) -> int {
            return u.iti >= 0 && u.r_lo + tid < u.r_hi
                       ? ((gptr<const int32_t>)(items[u.iti].runs + u.pbeg))[u.r_lo + tid] : 0;
        };
        int entry = first_entry(cur);
        __syncthreads();
        Ref nxt = known(1);
        for (int slot = 0;; slot ^= 1) {
            const gptr<const int32_t> runs = (gptr<const int32_t>)(items[cur.iti].runs + cur.pbeg);
            const int entry_n = first_entry(nxt);
            RunGeo Gn = G;
            double pre[NPRE][NC];
            auto ahead = [&]() {
                if (nxt.iti < 0) return;                         // uniform
                const ItemDesc &In = items[nxt.iti];
                UnitC<PREC> V;           // (what the field loads need of it)
                for (int a = 0; a < 3; ++a) {
                    V.n[a] = In.n[a];
                    V.gf[a] = (gptr<const double>)(KIND == PL_LORENTZ ? In.E[a] : In.vg[a]);
                    V.gf[3 + a] = (gptr<const double>)(KIND == PL_LORENTZ ? In.B[a] : nullptr);
                }
                unit_geo<DIM, HF, TS>(In, nxt.t, flags, Gn);
#pragma unroll
                for (int k = 0; k < NPRE; ++k)
                    if (tid + k * bd < Gn.Lf) rec_load<PREC, DIM, KIND>(V, Gn, tid + k * bd, pre[k]);
            };
            unit_runs<PREC, SHAPE, DIM, KIND, CHS, KR>(
                U, G, S, runs, cur.pbeg, cur.pend, cur.r_lo, cur.r_hi, entry, do_sums, err, ahead, [&]() {
                    // this unit's words take the claim after the next one; the
                    // words of a next one not claimed yet, the claim after that
                    int *mine = ctl + RC_UNIT + RU_WORDS * slot, *other = ctl + RC_UNIT + RU_WORDS * (slot ^ 1);
                    const bool both = nxt.iti == RU_LATER;
                    bool hold = nxt.iti >= 0 && (__builtin_amdgcn_readfirstlane(other[RU_ITEM]) & RU_HEAVY);
#pragma unroll 1
                    for (int k = 0; k < (both ? 2 : 1); ++k) {
                        int *w = k ? other : mine;
                        if (hold) w[RU_ITEM] = RU_LATER;
                        else hold = runs_next(items, nitems, counter, ctl, w);
                    }
                });
            if (do_sums && tid < 8) {
                const double v = S.sums[tid];
                S.sums[tid] = 0.0;
                if (v != 0.0) global_add(items[cur.iti].psum + tid, v);
            }
            flush_unit<PREC, DIM, CHS>(U, G, S.lds_d);
            const bool later = nxt.iti == RU_LATER;              // uniform, as are all of its values
            if (later) nxt = known(slot);
            if (nxt.iti < 0) break;                              // uniform
            if (later) unit_geo<DIM, HF, TS>(items[nxt.iti], nxt.t, flags, Gn);
            if (nxt.iti != cur.iti) {
                load_unit<PREC>(items[nxt.iti], U, Gn.Ld);
                if (TS == 0) {
                    // another item's tile may lay the sections out otherwise
                    __syncthreads();
                    unit_shared<PREC, KIND>(Gn, items[nxt.iti].nslot, smem_raw, lds_bytes, flags, S);
                    for (int k = tid; k < Gn.Ld * items[nxt.iti].nslot; k += bd) S.lds_d[k] = 0.0;
                    if (tid < 8) S.sums[tid] = 0.0;
                }
                    }
            G = Gn;
            R *lds_f = const_cast<R *>(S.lds_f);
            if (!later) {
#pragma unroll
                for (int k = 0; k < NPRE; ++k)
                    if (tid + k * bd < G.Lf) rec_store<PREC, KIND>(G, lds_f, tid + k * bd, pre[k]);
            }
            for (int e = tid + (later ? 0 : NPRE * bd); e < G.Lf; e += bd) {
                double v[NC];
                rec_load<PREC, DIM, KIND>(U, G, e, v);
                rec_store<PREC, KIND>(G, lds_f, e, v);
            }
            cur = nxt;
            entry = later ? first_entry(cur) : entry_n;
            nxt = known(later ? slot ^ 1 : slot);
            if (later) slot ^= 1;                                // (cur stays where it is)
            __syncthreads();
        }
    }
    runs_latch(err, errflags);
    release_queues(counter, ctl);
}

// One persistent launch over the items of every species kind of a call: each
// claimed unit runs the unit body of its item's kind (uniform per block).
// CHL and CHD fix the channel sets of the charged (rho J F) and dust (rho F)
// items, or are 0 to take them at run time.  The last wave claims and looks up
// the next unit when it is through its own runs, while the others finish theirs.
template <int PREC, int SHAPE, int DIM, int HF, int TS, int CHL, int CHD>
__global__ __launch_bounds__(kRunsThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_runs_mix(const ItemDesc *__restrict__ items, int nitems,
                                             unsigned *counter, int *errflags, unsigned flags, int lds_bytes)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    int *ctl = reinterpret_cast<int *>(smem_raw + lds_bytes - kRunsCtlBytes);
    int err = 0;
    if (threadIdx.x == 0) ctl[RC_QI] = 0;
    runs_units(items, nitems, errflags, ctl);
    __syncthreads();
    if (threadIdx.x < 64) runs_next(items, nitems, counter, ctl, ctl + RC_UNIT);
    for (int slot = 0;; slot ^= 1) {
        __syncthreads();
        const int *mine = ctl + RC_UNIT + RU_WORDS * slot;
        auto word = [&](int k) -> int { return __builtin_amdgcn_readfirstlane(mine[k]); };
        if (word(RU_ITEM) < 0) break;                         // uniform
        const ItemDesc &I = items[word(RU_ITEM) & ~RU_HEAVY];
        const int t = word(RU_TILE), pbeg = word(RU_PBEG), pend = word(RU_PEND), lo = word(RU_RLO), hi = word(RU_RHI);
        const int kind = __builtin_amdgcn_readfirstlane(I.kind);
        auto last = [&]() { runs_next(items, nitems, counter, ctl, ctl + RC_UNIT + RU_WORDS * (slot ^ 1)); };
        if (kind == PL_LORENTZ)
            runs_unit<PREC, SHAPE, DIM, PL_LORENTZ, HF, TS, CHL>(I, t, pbeg, pend, lo, hi, flags, lds_bytes, smem_raw, err, last);
        else if (kind == PL_DUST)
            runs_unit<PREC, SHAPE, DIM, PL_DUST, HF, TS, CHD>(I, t, pbeg, pend, lo, hi, flags, lds_bytes, smem_raw, err, last);
        else
            runs_unit<PREC, SHAPE, DIM, PL_TRACER, HF, TS, 0>(I, t, pbeg, pend, lo, hi, flags, lds_bytes, smem_raw, err, last);
    }
    runs_latch(err, errflags);
    release_queues(counter, ctl);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

using RunsKernel = void (*)(const ItemDesc *, int, unsigned *, int *, unsigned, int);

// The variants with fixed shapes are those whose LDS (160 KB) allows them and
// that no wider halo replaces: with a two-cell field halo, and in float64 on 8^3
// tiles with one cell and seven channels; float64 with every channel has no room
// on 8^3.  A launch that none of them fits takes the run-time shapes.
template <int PREC>
static RunsKernel pick_runs(int shape, int dim, int kind, int hf, int ts, int chs, int nt)
{
#define PL_RN(S, D, K, HF_, TS_, CHS_, NT_) \
    if (shape == S && dim == D && kind == K && hf == HF_ && ts == TS_ && chs == CHS_ && nt == NT_) \
        return k_runs<PREC, S, D, K, HF_, TS_, CHS_, NT_>;
#define PL_R(S, D, K, HF_, TS_, CHS_) PL_RN(S, D, K, HF_, TS_, CHS_, kRunsThreads)
#define PL_RG(S, D) PL_R(S, D, PL_LORENTZ, 0, 0, 0) PL_R(S, D, PL_DUST, 0, 0, 0)
    PL_RG(PL_TSC, 3) PL_RG(PL_TSC, 2) PL_RG(PL_CIC, 3) PL_RG(PL_CIC, 2)
    PL_RN(PL_TSC, 2, PL_LORENTZ, 0, 0, 0, kRunsSmall) PL_RN(PL_TSC, 2, PL_DUST, 0, 0, 0, kRunsSmall)
    PL_RN(PL_CIC, 2, PL_LORENTZ, 0, 0, 0, kRunsSmall) PL_RN(PL_CIC, 2, PL_DUST, 0, 0, 0, kRunsSmall)
    PL_RN(PL_TSC, 2, PL_LORENTZ, 2, 3, 1, kRunsSmall) PL_RN(PL_TSC, 2, PL_LORENTZ, 2, 3, 3, kRunsSmall)
    PL_RN(PL_TSC, 2, PL_DUST, 2, 3, 2, kRunsSmall)
    PL_R(PL_TSC, 3, PL_DUST, 2, 1, 2) PL_R(PL_TSC, 3, PL_DUST, 2, 2, 2)
    PL_R(PL_TSC, 3, PL_LORENTZ, 2, 2, 1) PL_R(PL_TSC, 3, PL_LORENTZ, 2, 2, 3)
    if constexpr (PREC == PL_F32_OFFSET) {
        PL_R(PL_TSC, 3, PL_LORENTZ, 2, 1, 1) PL_R(PL_TSC, 3, PL_LORENTZ, 2, 1, 3)
    } else {
        PL_R(PL_TSC, 3, PL_LORENTZ, 1, 1, 1)
    }
#undef PL_RG
#undef PL_R
#undef PL_RN
    return nullptr;
}

// (float64 on 8^3: with charged items one cell, dust and tracers alone two)
template <int PREC>
static RunsKernel pick_runs_mix(int shape, int dim, int hf, int ts, int chl, int chd)
{
#define PL_M(S, D, HF_, TS_, CL, CD) \
    if (shape == S && dim == D && hf == HF_ && ts == TS_ && chl == CL && chd == CD) \
        return k_runs_mix<PREC, S, D, HF_, TS_, CL, CD>;
    PL_M(PL_TSC, 3, 0, 0, 0, 0) PL_M(PL_TSC, 2, 0, 0, 0, 0) PL_M(PL_CIC, 3, 0, 0, 0, 0) PL_M(PL_CIC, 2, 0, 0, 0, 0)
    PL_M(PL_TSC, 3, 2, 1, 1, 2) PL_M(PL_TSC, 3, 2, 2, 1, 2) PL_M(PL_TSC, 3, 2, 2, 3, 2)
    if constexpr (PREC == PL_F32_OFFSET) {
        PL_M(PL_TSC, 3, 2, 1, 3, 2)
    } else {
        PL_M(PL_TSC, 3, 1, 1, 1, 2)
    }
#undef PL_M
    return nullptr;
}

template <int PREC>
static size_t runs_item_lds(const Ctx *c, const ItemDesc &it, int hf, int nt)
{
    const int d3 = c->d.ndim >= 3;
    const int Lf = (it.tile[0] + 2 * hf) * (it.tile[1] + 2 * hf) * (d3 ? it.tile[2] + 2 * hf : 1);
    const int Ld = (it.tile[0] + 4) * (it.tile[1] + 4) * (d3 ? it.tile[2] + 4 : 1);
    size_t offs[6];
    if (it.kind == PL_LORENTZ) return runs_lds_bytes<PREC, PL_LORENTZ>(Lf, Ld, it.nslot, hf, nt, offs);
    if (it.kind == PL_DUST) return runs_lds_bytes<PREC, PL_DUST>(Lf, Ld, it.nslot, hf, nt, offs);
    return runs_lds_bytes<PREC, PL_TRACER>(Lf, Ld, 0, hf, nt, offs);
}

// Whether the footprint that the float32 sums go by (runs_sums.h) fits for every
// item of a launch with an hf-cell field halo.
template <int PREC>
static bool runs_sums_fit(const Ctx *c, const ItemDesc *host, int nitems, int hf)
{
    for (int i = 0; i < nitems; ++i)
        if (runs_sums_bytes(host[i].kind == PL_LORENTZ, host[i].tile, c->d.ndim,
                            host[i].kind == PL_TRACER ? 0 : host[i].nslot, hf) > (size_t)c->lds_max)
            return false;
    return true;
}

// Launch configuration of the run kernel for the items of one launch.
template <int PREC>
bool runs_plan_impl(const Ctx *c, const ItemDesc *host, int nitems, RunsPlan &pl)
{
    pl = RunsPlan{};
    pl.nt = kRunsThreads;
    if (nitems < 1) return false;
    bool kinds[3] = {false, false, false};
    for (int i = 0; i < nitems; ++i) kinds[host[i].kind] = true;
    pl.mixed = kinds[PL_TRACER] || (kinds[PL_LORENTZ] && kinds[PL_DUST]);
    // compile-time tile shape (8^3 or 8x8x4) and channel sets when every item
    // allows them: charged rho J F or all eight, dust rho F.  (With run-time
    // shapes the LDS offsets are registers and the kernel spills: 5.3e6
    // charged particles on 96^3 and eight 32^3 boxes, eight channels, 980 us
    // against 613 us fixed; float64 on 96^3, 7.1e6 particles: 1105 us
    // against 799 us, both with the changes of k_runs.)
    const bool d2 = c->d.ndim == 2;
    if (c->d.shape == PL_TSC && !(d2 && pl.mixed)) {
        auto set_of = [&](const ItemDesc &it, int want) {
            for (int ch = 0; ch < kMaxCh; ++ch)
                if (it.slot[ch] != chs_slot(want, ch)) return false;
            return true;
        };
        int chl = 0;
        bool chall = true;
        for (int i = 0; i < nitems && chall; ++i) {
            if (host[i].kind == PL_DUST) chall = set_of(host[i], 2);
            if (host[i].kind != PL_LORENTZ) continue;
            const int got = set_of(host[i], 1) ? 1 : set_of(host[i], 3) ? 3 : 0;
            chall = got && (chl == 0 || chl == got);
            chl = got;
        }
        for (int cand = d2 ? 3 : 1; cand <= (d2 ? 3 : 2) && pl.ts == 0 && chall; ++cand) {
            bool all = true;
            for (int i = 0; i < nitems; ++i)
                for (int a = 0; a < 3; ++a) all = all && host[i].tile[a] == ts_dim(cand, a);
            if (all) pl.ts = cand;
        }
        if (pl.ts) {
            pl.chl = chl ? chl : 1;
            pl.chd = 2;
        }
    }
    auto bytes = [&](int hf, int nt) {
        size_t lds = 0;
        for (int i = 0; i < nitems; ++i) lds = std::max(lds, runs_item_lds<PREC>(c, host[i], hf, nt));
        return lds;
    };
    // 2D tiles small enough for two blocks on a CU: a unit of an 8 x 8 tile has
    // fewer runs than a large block has threads, and a large block's staging,
    // runs and flush wait on each other (512^2 cells, 16 particles per cell: 285
    // us per launch with one large block of run-time shape, 190 us with two of
    // 256 threads; with four of 128 or eight of 64 threads a launch of the same
    // kernel took 1.1 and 1.4 times as long)
    if (d2 && !pl.mixed && 2 * bytes(2, kRunsSmall) <= (size_t)c->lds_max) pl.nt = kRunsSmall;
    else if (d2) pl.ts = pl.chl = pl.chd = 0;
    // (else the self-grouping kernel and its float64 sums)
    if (PREC == PL_F32_OFFSET && !runs_sums_fit<PREC>(c, host, nitems, 1)) return false;
    // LDS of the launch: a two-cell field halo when it fits, else one cell
    for (int hf = 2; hf >= 1; --hf) {
        pl.hf = hf;
        pl.lds = bytes(hf, pl.nt);
        pl.narrow = PREC == PL_F32_OFFSET && hf == 2 && !runs_sums_fit<PREC>(c, host, nitems, 2);
        if (pl.lds <= (size_t)c->lds_max) return true;
    }
    return false;
}

template <int PREC>
hipError_t launch_runs_impl(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, int total_units,
                            unsigned sf, unsigned *counter)
{
    if (total_units <= 0) return hipSuccess;
    RunsPlan pl;
    if (!runs_plan_impl<PREC>(c, host, nitems, pl)) return hipErrorInvalidConfiguration;
    if (pl.hf == 2) sf |= SF_FHALO2;
    if (pl.narrow) sf |= SF_NARROW;
    RunsKernel k = nullptr;
    int chs = 0;
    auto pick = [&]() {
        // compile-time halo in the fixed-shape kernels, from the flags otherwise
        const int kind = host[0].kind, hf = pl.ts ? pl.hf : 0;
        chs = pl.mixed || kind == PL_LORENTZ ? pl.chl : pl.chd;
        k = pl.mixed ? pick_runs_mix<PREC>(c->d.shape, c->d.ndim, hf, pl.ts, pl.chl, pl.chd)
                     : pick_runs<PREC>(c->d.shape, c->d.ndim, kind, hf, pl.ts, chs, pl.nt);
    };
    pick();
    if (!k) {
        pl.ts = pl.chl = pl.chd = 0;
        pick();
    }
    if (!k) return hipErrorInvalidConfiguration;
    const int rb = pl.nt;
    // every item has kRunsSplit units beyond its tiles for the pieces of crowded tiles
    const int units = total_units + nitems * kRunsSplit;
    const int grid = std::min(units, resident_blocks(c, (StepKernel)k, rb, pl.lds));
    hipLaunchKernelGGL(k, dim3(grid), dim3(rb), pl.lds, c->stream, table, nitems, counter, c->errflags, sf,
                       (int)pl.lds);
    c->stats[0]++;
    c->stats[4]++;
    if (pl.ts) c->stats[6]++;
    c->stats[7] = pl.ts | chs << 4 | pl.hf << 8 | (pl.mixed ? 1 << 12 : 0);
    return hipGetLastError();
}

}  // namespace pl
