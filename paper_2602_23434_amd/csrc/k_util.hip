// Step dispatch (one persistent launch per species kind), zeroing, sums and
// pack / unpack kernels.
#include <hip/hip_runtime.h>

#include <string.h>

#include <algorithm>
#include <vector>

#include "pl_device.h"
#include "plain_cost.h"

namespace pl {

hipError_t launch_group_f32(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, int total_units,
                            unsigned sf, bool push, bool deposit, unsigned *counter);
hipError_t launch_group_f64(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, int total_units,
                            unsigned sf, bool push, bool deposit, unsigned *counter);
hipError_t launch_runs_f32(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, int total_units,
                           unsigned sf, unsigned *counter);
hipError_t launch_runs_f64(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, int total_units,
                           unsigned sf, unsigned *counter);
hipError_t launch_local_f32(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, const LocalPlan &pl,
                            unsigned sf, unsigned *counter);
hipError_t launch_local_f64(Ctx *c, const ItemDesc *table, const ItemDesc *host, int nitems, const LocalPlan &pl,
                            unsigned sf, unsigned *counter);

// Items of one launch: those of one species kind; an item whose indices the
// call bins (plain algorithm) has one of its own.
int group_end(const std::vector<ItemDesc> &host, int i0)
{
    int i1 = i0 + 1;
    if (host[i0].idx) return i1;
    while (i1 < (int)host.size() && host[i1].kind == host[i0].kind && !host[i1].idx) ++i1;
    return i1;
}

// Fused run-based steps of charged and dust species take the run-based kernel
// (its tables come from the sort).  What else has tiles takes a self-grouping
// kernel, which needs only the tile offsets, where that pays (tile_route.h) and
// the tile and its LDS allow it; else the one-particle-per-thread kernel.
Route group_route(const Ctx *c, const ItemDesc *host, int nitems, bool push, bool deposit, LocalPlan &pl)
{
    RunsPlan rp;
    if (c->d.algo == PL_ALGO_RUNS && push && deposit && host[0].kind != PL_TRACER && runs_plan(c, host, nitems, rp))
        return ROUTE_RUNS;
    if ((c->d.algo != PL_ALGO_PLAIN || host[0].idx) && local_plan(c, host, nitems, push, deposit, pl))
        return ROUTE_LOCAL;
    return ROUTE_STEP;
}

// Tiles of a binned item: 8^3 cells (float32) or 8 x 8 x 4 (float64), 32 x 32
// or 32 x 16 in 2D, the largest whose LDS leaves chunks of a tile's particles;
// they need not divide the box (a tile past its edge wraps).  Their number.
static int64_t bin_tiles(const Ctx *c, const ItemDesc &it, int tile[3], int ntile[3])
{
    const bool d3 = c->d.ndim == 3, f64 = c->d.prec == PL_F64;
    tile[0] = d3 ? 8 : 32;
    tile[1] = d3 ? 8 : (f64 ? 16 : 32);
    tile[2] = d3 ? (f64 || it.nslot > 7 ? 4 : 8) : 1;
    int64_t nt = 1;
    for (int a = 0; a < 3; ++a) {
        ntile[a] = (it.n[a] + tile[a] - 1) / tile[a];
        nt *= ntile[a];
    }
    return nt;
}

void plain_bins(const Ctx *c, std::vector<ItemDesc> &host, bool push, bool deposit)
{
    if (c->d.algo != PL_ALGO_PLAIN) return;
    const int n = (int)host.size();
    std::vector<PlainItem> rule(n, PlainItem{0, 0, 0, false, false});
    std::vector<ItemDesc> bins;
    for (int i0 = 0, i1 = 0; i0 < n; i0 = i1) {
        const int kind = host[i0].kind;
        bool any = false;
        for (i1 = i0; i1 < n && host[i1].kind == kind; ++i1) {
            const ItemDesc &it = host[i1];
            const bool dep = deposit && kind != PL_TRACER && it.nslot > 0;
            if (it.np == 0 || !(push || dep)) continue;
            int tile[3], ntile[3];
            const int64_t nt = bin_tiles(c, it, tile, ntile), cells = (int64_t)it.n[0] * it.n[1] * it.n[2];
            const bool want = dep ? it.np >= kBinMinDeposit : push_bins(it.np, cells, nt, c->d.ndim, c->d.prec, kind);
            bool fits = false;
            if (want && nt <= c->bin_cap) {
                if (bins.empty()) bins = host;
                ItemDesc &d = bins[i1];
                for (int a = 0; a < 3; ++a) {
                    d.tile[a] = tile[a];
                    d.ntile[a] = ntile[a];
                }
                d.ntiles = (int)nt;
                d.tile_start = c->bin_start;
                d.idx = c->idx[bins_buffer(d.ntiles)];
                LocalPlan pl;
                fits = local_plan(c, &d, 1, push, deposit, pl);
            }
            if (dep) rule[i1] = PlainItem{it.np, nt, it.nslot, fits, false};
            else if (fits) rule[i1].binned = any = true;     // (a rule of its own: no deposit)
            any = any || fits;
        }
        if (!any) continue;
        std::vector<PlainItem> dep(rule.begin() + i0, rule.begin() + i1);
        choose_bins(dep.data(), i1 - i0, c->d.ndim, c->d.prec, kind, c->num_cu);
        for (int i = i0; i < i1; ++i)
            if (rule[i].binned || dep[i - i0].binned) host[i] = bins[i];
        std::stable_partition(host.begin() + i0, host.begin() + i1, [](const ItemDesc &d) { return d.idx != nullptr; });
    }
}

// The host table is ordered by species kind, then by particle count.  A fused
// run-based step is one launch over every item; otherwise every group of items
// (group_end) is one launch with a work counter of its kind.
hipError_t launch_step(Ctx *c, const ItemDesc *table, const std::vector<ItemDesc> &host, int nitems,
                       int total_units, unsigned flags, bool deposit, bool push)
{
    (void)total_units;
    const bool f64 = c->d.prec == PL_F64;
    unsigned sf = (push ? SF_PUSH : 0u) | (deposit ? SF_DEPOSIT : 0u) | ((flags & PL_SUMS) ? SF_SUMS : 0u) |
                  (c->runs ? SF_RUNS : 0u);
    // a fused run-based step with every kind in one launch (the item table
    // numbers units across all items then: see build_table)
    RunsPlan pl;
    if (c->one_launch && c->d.algo == PL_ALGO_RUNS && push && deposit && runs_plan(c, host.data(), nitems, pl)) {
        int units = 0;
        for (int i = 0; i < nitems; ++i) units += host[i].nunits;
        return f64 ? launch_runs_f64(c, table, host.data(), nitems, units, sf, c->counters)
                   : launch_runs_f32(c, table, host.data(), nitems, units, sf, c->counters);
    }
    for (int i0 = 0, i1 = 0; i0 < nitems; i0 = i1) {
        i1 = group_end(host, i0);
        const ItemDesc *h = host.data() + i0, *t = table + i0;
        const int n = i1 - i0;
        unsigned *counter = c->counters + kCounterStride * h->kind;
        int units = 0;
        for (int i = 0; i < n; ++i) units += h[i].nunits;
        LocalPlan lp;
        const Route r = group_route(c, h, n, push, deposit, lp);
        hipError_t e = hipSuccess;
        if (h->idx) e = launch_bins(c, *h);
        if (e != hipSuccess) return e;
        if (r == ROUTE_RUNS) {
            e = f64 ? launch_runs_f64(c, t, h, n, units, sf, counter) : launch_runs_f32(c, t, h, n, units, sf, counter);
        } else {
            if (c->d.algo == PL_ALGO_RUNS && push && deposit && h->kind != PL_TRACER) c->stats[5]++;
            if (r == ROUTE_LOCAL)
                e = f64 ? launch_local_f64(c, t, h, n, lp, sf, counter) : launch_local_f32(c, t, h, n, lp, sf, counter);
            else
                e = f64 ? launch_group_f64(c, t, h, n, units, sf, push, deposit, counter)
                        : launch_group_f32(c, t, h, n, units, sf, push, deposit, counter);
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// Zeroing, sums, pack / unpack
// ---------------------------------------------------------------------------

__global__ void k_zero(double *p, long n)
{
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = 0.0;
}

// Every active moment channel of every item of a call in one launch: block
// row y zeroes channel y % kMaxCh of item y / kMaxCh (items from the device
// table of the call).
__global__ void k_zero_items(const ItemDesc *items)
{
    const ItemDesc &it = items[blockIdx.y / kMaxCh];
    const int ch = blockIdx.y % kMaxCh;
    if (it.kind == PL_TRACER || it.slot[ch] < 0) return;
    double *p = it.M[ch];
    const long n = (long)it.n[0] * it.n[1] * it.n[2];
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = 0.0;
}

// The same for a call of a few items, whose descriptors come as arguments and
// are written to the call's table: one launch instead of a copy from pinned
// memory, an event and a launch.  zero = false: the table only.  A step of a
// 32 x 32 box with 4096 particles took 23.9 us from call to call with the copy
// and 18.8 us with this kernel (10 eager steps and a sort: 239 and 188 us).  More
// items than fit 4 KB of arguments take the ring.
template <int N>
__global__ void k_zero_table(TableArgs<N> t, int n, bool zero, ItemDesc *table)
{
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        const int words = n * (int)(sizeof(ItemDesc) / 4);
        const uint32_t *src = reinterpret_cast<const uint32_t *>(&t);
        for (int i = threadIdx.x; i < words; i += blockDim.x) reinterpret_cast<uint32_t *>(table)[i] = src[i];
    }
    if (!zero) return;
    const ItemDesc &it = t.d[blockIdx.y / kMaxCh];
    const int ch = blockIdx.y % kMaxCh;
    if (it.kind == PL_TRACER || it.slot[ch] < 0) return;
    double *p = it.M[ch];
    const long cells = (long)it.n[0] * it.n[1] * it.n[2];
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < cells; i += (long)gridDim.x * blockDim.x) p[i] = 0.0;
}

template <int N>
hipError_t launch_table_n(Ctx *c, const std::vector<ItemDesc> &host, bool zero, ItemDesc *table)
{
    TableArgs<N> t;
    memset(&t, 0, sizeof(t));
    long cells = 0;
    for (size_t i = 0; i < host.size(); ++i) {
        t.d[i] = host[i];
        if (host[i].kind != PL_TRACER && host[i].nslot > 0)
            cells = std::max(cells, (long)host[i].n[0] * host[i].n[1] * host[i].n[2]);
    }
    zero = zero && cells > 0;
    const int channels = zero ? (int)host.size() * kMaxCh : 1;
    const long per = std::min<long>((cells + 255) / 256, (8L * c->num_cu + channels - 1) / channels * 4);
    const int gx = zero ? (int)std::max<long>(1, per) : 1;
    hipLaunchKernelGGL(k_zero_table<N>, dim3(gx, channels), dim3(256), 0, c->stream, t, (int)host.size(), zero, table);
    if (zero) c->stats[0]++;
    return hipGetLastError();
}

hipError_t launch_table(Ctx *c, const std::vector<ItemDesc> &host, bool zero, ItemDesc *table)
{
    if (host.empty() || host.size() > (size_t)kTableArgs) return hipErrorInvalidValue;
    return host.size() == 1 ? launch_table_n<1>(c, host, zero, table) : launch_table_n<kTableArgs>(c, host, zero, table);
}

hipError_t launch_zero(Ctx *c, const ItemDesc *table, const std::vector<ItemDesc> &host)
{
    long cells = 0;
    for (const ItemDesc &it : host)
        if (it.kind != PL_TRACER) cells = std::max(cells, (long)it.n[0] * it.n[1] * it.n[2]);
    if (cells == 0 || host.empty()) return hipSuccess;
    const int channels = (int)host.size() * kMaxCh;
    const int gx = (int)std::max<long>(1, std::min<long>((cells + 255) / 256, (8L * c->num_cu + channels - 1) / channels * 4));
    hipLaunchKernelGGL(k_zero_items, dim3(gx, channels), dim3(256), 0, c->stream, table);
    c->stats[0]++;
    return hipGetLastError();
}

hipError_t launch_zero_sums(Ctx *c, double *sums, int n)
{
    hipLaunchKernelGGL(k_zero, dim3(1), dim3(256), 0, c->stream, sums, (long)n);
    c->stats[0]++;
    return hipGetLastError();
}

__global__ void k_grid_sum(const double *p, long n, double scale, double *out)
{
    double s = 0.0;
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) s += p[i];
    s = wave_sum(s);
    __shared__ double part[16];
    int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) part[wv] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += part[k];
        global_add(out, t * scale);
    }
}

hipError_t launch_grid_sums(Ctx *c, const ItemDesc &it, double *out8)
{
    long cells = (long)it.n[0] * it.n[1] * it.n[2];
    double dv = 1.0 / it.inv_dv;
    int grid = (int)std::min<long>((cells + 255) / 256, 4L * c->num_cu);
    for (int ch = 0; ch < kMaxCh; ++ch) {
        if (!it.M[ch]) continue;
        hipLaunchKernelGGL(k_grid_sum, dim3(grid), dim3(256), 0, c->stream, it.M[ch], cells, dv, out8 + ch);
        c->stats[0]++;
    }
    return hipGetLastError();
}

template <int PREC>
__global__ void k_pack(ItemDesc it, int ndim, const double *x0, const double *x1, const double *x2,
                       const double *u0, const double *u1, const double *u2, int *errflags)
{
    const double *xs[3] = {x0, x1, x2};
    const double *us[3] = {u0, u1, u2};
    int err = 0;
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < it.np; p += gridDim.x * blockDim.x) {
        int c[3] = {0, 0, 0};
        double xw[3] = {0.0, 0.0, 0.0};
        for (int a = 0; a < 3; ++a)
            if (!isfinite(us[a][p])) err |= ERR_NONFINITE;
        for (int a = 0; a < ndim; ++a) {
            double v = xs[a][p];
            double nn = (double)it.n[a];
            if (!(v >= 0.0 && v < nn)) {
                if (!isfinite(v)) { v = 0.0; err |= ERR_NONFINITE; }
                v = v - nn * floor(v / nn);
                if (v >= nn || v < 0.0) v = 0.0;
            }
            xw[a] = v;
        }
        if (PREC == PL_F64) {
            for (int a = 0; a < ndim; ++a) ((double *)it.x[a])[p] = xw[a];
            for (int a = 0; a < 3; ++a) ((double *)it.u[a])[p] = us[a][p];
        } else {
            for (int a = 0; a < ndim; ++a) {
                double f = floor(xw[a]);
                int ci = (int)f;
                float o = (float)(xw[a] - f - 0.5);
                if (o >= 0.5f) {
                    o = -0.5f;
                    ci = ci + 1 == it.n[a] ? 0 : ci + 1;
                }
                c[a] = ci;
                ((float *)it.x[a])[p] = o;
            }
            it.cell[p] = pack_cell(c[0], c[1], c[2]);
            for (int a = 0; a < 3; ++a) ((float *)it.u[a])[p] = (float)us[a][p];
        }
    }
    if (err) atomicOr(errflags, err);
}

template <int PREC>
__global__ void k_unpack(ItemDesc it, int ndim, double *x0, double *x1, double *x2, double *u0, double *u1,
                         double *u2)
{
    double *xs[3] = {x0, x1, x2};
    double *us[3] = {u0, u1, u2};
    for (int p = blockIdx.x * blockDim.x + threadIdx.x; p < it.np; p += gridDim.x * blockDim.x) {
        if (PREC == PL_F64) {
            for (int a = 0; a < ndim; ++a) xs[a][p] = ((const double *)it.x[a])[p];
            for (int a = 0; a < 3; ++a) us[a][p] = ((const double *)it.u[a])[p];
        } else {
            int c[3];
            unpack_cell(it.cell[p], c[0], c[1], c[2]);
            for (int a = 0; a < ndim; ++a) xs[a][p] = (double)c[a] + 0.5 + (double)((const float *)it.x[a])[p];
            for (int a = 0; a < 3; ++a) us[a][p] = (double)((const float *)it.u[a])[p];
        }
    }
}

hipError_t launch_pack(Ctx *c, const ItemDesc &it, int prec, int ndim, const double *x[3], const double *u[3])
{
    if (it.np == 0) return hipSuccess;
    int grid = std::min((it.np + 255) / 256, 16 * c->num_cu);
    if (prec == PL_F64)
        hipLaunchKernelGGL(k_pack<PL_F64>, dim3(grid), dim3(256), 0, c->stream, it, ndim, x[0], x[1], x[2], u[0],
                           u[1], u[2], c->errflags);
    else
        hipLaunchKernelGGL(k_pack<PL_F32_OFFSET>, dim3(grid), dim3(256), 0, c->stream, it, ndim, x[0], x[1], x[2],
                           u[0], u[1], u[2], c->errflags);
    c->stats[0]++;
    return hipGetLastError();
}

hipError_t launch_unpack(Ctx *c, const ItemDesc &it, int prec, int ndim, double *x[3], double *u[3])
{
    if (it.np == 0) return hipSuccess;
    int grid = std::min((it.np + 255) / 256, 16 * c->num_cu);
    if (prec == PL_F64)
        hipLaunchKernelGGL(k_unpack<PL_F64>, dim3(grid), dim3(256), 0, c->stream, it, ndim, x[0], x[1], x[2], u[0],
                           u[1], u[2]);
    else
        hipLaunchKernelGGL(k_unpack<PL_F32_OFFSET>, dim3(grid), dim3(256), 0, c->stream, it, ndim, x[0], x[1], x[2],
                           u[0], u[1], u[2]);
    c->stats[0]++;
    return hipGetLastError();
}

}  // namespace pl
