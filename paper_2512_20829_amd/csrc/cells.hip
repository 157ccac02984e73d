// FLA projection on general meshes: the cells are points (their centroids)
// with volumes, as on an unstructured finite-volume mesh.  The estimator
// (eqs. kernel-estimator, kernel, smoothing-length, coupling-terms-kernel)
// needs nothing of a cell but the point where it is evaluated, and the mesh
// enters the result only through the per-cell factor n_hat of App. A
// (eq. mv-scal: proportional to the cell volume).
//
// Spatial index (built once per mesh): a rectilinear grid of buckets whose
// per-axis edges sit at quantiles of the centroid coordinates, so that the
// buckets of a stretched or clustered mesh hold similar numbers of cells;
// cells sorted by bucket.  Trajectories are keyed by home bucket and
// neighbourhood class (distance in buckets to the farthest bucket their
// cutoff sphere reaches) and sorted, as on the Cartesian mesh.
//
// Gather: one wave per work item of up to kCellsPerItem cells of one bucket,
// each lane owning kCellsPerLane cells.  The wave scans the records of the
// buckets within reach, 64 at a time, one per lane, and keeps those whose
// cutoff sphere meets the bounding box of its cells; batches of 64 of these
// are evaluated two at a time, each lane with the binary64 offsets and the inclusion test of
// the Cartesian gather (so both paths, and the oracle, take the same
// decisions).
#include <type_traits>

#include "internal.hpp"
#include "kernels.hpp"
#include "prepass.hpp"

namespace flp {

typedef float F4 __attribute__((ext_vector_type(4)));

// Number of interior edges e[1..nb-1] that are <= p: the bucket of p along
// one axis, clamped to [0, nb - 1].
__device__ inline int bucket_of(const double* e, int nb, double p)
{
    int l = 0, r = nb - 1;
    while (l < r) {
        const int mid = (l + r + 1) >> 1;
        if (e[mid] <= p)
            l = mid;
        else
            r = mid - 1;
    }
    return l;
}

// Histogram of the centroid coordinates per axis (kCellsHistBins equal bins
// over [lo, hi]) and validation: a centroid outside the box or not finite, or
// a volume that is negative or not finite, counts in *bad.
__global__ void k_cells_hist(int dim, int64_t M, const double* x0, const double* x1, const double* x2, double lo0,
                             double lo1, double lo2, double hi0, double hi1, double hi2, uint32_t* hist, uint32_t* bad,
                             const double* vol)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= M) return;
    const double* xs[3] = {x0, x1, x2};
    const double los[3] = {lo0, lo1, lo2}, his[3] = {hi0, hi1, hi2};
    bool ok = !vol || (isfinite(vol[c]) && vol[c] >= 0.0);
    for (int a = 0; a < dim; ++a) {
        const double x = xs[a][c];
        if (!(x >= los[a] && x <= his[a])) {       // also rejects NaN
            ok = false;
            continue;
        }
        double f = (x - los[a]) / (his[a] - los[a]) * (double)kCellsHistBins;
        int bin = (int)fmin(fmax(floor(f), 0.0), (double)(kCellsHistBins - 1));
        atomicAdd(&hist[(int64_t)a * kCellsHistBins + bin], 1u);
    }
    if (!ok) atomicAdd(bad, 1u);
}

hipError_t launch_cells_hist(int dim, int64_t M, const double* const* xc, const double* lo, const double* hi,
                             uint32_t* hist, uint32_t* bad, const double* vol, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const int64_t blocks = (M + 255) / 256;
    FLA_LAUNCH(k_cells_hist, dim3((unsigned)blocks), dim3(256), 0, s, dim, M, xc[0], xc[1],
                       dim == 3 ? xc[2] : xc[0], lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], hist, bad, vol);
    return hipGetLastError();
}

// Sort key of each cell: its bucket (linear index, axis 0 fastest) and, below,
// its eighth of the bucket along the bucket's longest edge, so that the first
// and the second 64 cells of a work item fill boxes of their own; and the
// identity value.
__global__ void k_cells_key(CellGridDev g, int64_t M, const double* x0, const double* x1, const double* x2,
                            uint32_t* keys, uint32_t* vals)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= M) return;
    const double* xs[3] = {x0, x1, x2};
    int64_t lin = 0, stride = 1;
    double longest = -1.0, at = 0.0;
    for (int a = 0; a < g.dim; ++a) {
        const int b = bucket_of(g.edges[a], g.nb[a], xs[a][c]);
        const double lo = g.edges[a][b], len = g.edges[a][b + 1] - lo;
        if (len > longest) {
            longest = len;
            at = (xs[a][c] - lo) / len;
        }
        lin += stride * b;
        stride *= g.nb[a];
    }
    constexpr int parts = 1 << kCellsSubBits;
    const int sub = (int)fmin(fmax(at * parts, 0.0), (double)(parts - 1));
    keys[c] = ((uint32_t)lin << kCellsSubBits) | (uint32_t)sub;
    vals[c] = (uint32_t)c;
}

hipError_t launch_cells_key(const CellGridDev& g, int64_t M, const double* const* xc, uint32_t* keys, uint32_t* vals,
                            hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const int64_t blocks = (M + 255) / 256;
    FLA_LAUNCH(k_cells_key, dim3((unsigned)blocks), dim3(256), 0, s, g, M, xc[0], xc[1],
                       g.dim == 3 ? xc[2] : xc[0], keys, vals);
    return hipGetLastError();
}

// Centroids and volumes in bucket order, and the permutation back.
__global__ void k_cells_sorted(int dim, int64_t M, const uint32_t* order, const double* x0, const double* x1,
                               const double* x2, const double* vol, double* s0, double* s1, double* s2, double* vs,
                               uint32_t* perm)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= M) return;
    const uint32_t c = order[p];
    s0[p] = x0[c];
    s1[p] = x1[c];
    if (dim == 3) s2[p] = x2[c];
    if (vol) vs[p] = vol[c];
    perm[p] = c;
}

hipError_t launch_cells_sorted(int dim, int64_t M, const uint32_t* order, const double* const* xc, const double* vol,
                               double* const* xs, double* vs, uint32_t* perm, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const int64_t blocks = (M + 255) / 256;
    FLA_LAUNCH(k_cells_sorted, dim3((unsigned)blocks), dim3(256), 0, s, dim, M, order, xc[0], xc[1],
                       dim == 3 ? xc[2] : xc[0], vol, xs[0], xs[1], dim == 3 ? xs[2] : xs[0], vs, perm);
    return hipGetLastError();
}

// Sort key of a trajectory on the bucket grid: home bucket and the largest
// per-axis distance in buckets (circular on periodic axes; a support that
// spans a whole periodic axis counts as the axis's bucket count) from the
// home bucket to a bucket that can hold a centroid within rc.  The support
// interval is widened by 1e-12 of |x| + rc + L, far more than the rounding of
// x -+ rc and of the periodic wrap.  Returns false when the interval misses
// a closed box (every centroid lies in the box).
template <int D>
struct BucketKey {
    const CellGridDev& g;
    __device__ uint32_t stride() const { return (uint32_t)g.nbuckets; }
    __device__ bool operator()(const double* x, double rc, int64_t& bl, int& reach) const
    {
        int hb[3] = {0, 0, 0};
        reach = 0;
        bool support = true;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            const int nb = g.nb[a];
            const double* e = g.edges[a];
            const double sl = 1e-12 * (fabs(x[a]) + rc + g.L[a]);
            const double plo = x[a] - rc - sl, phi = x[a] + rc + sl;
            int ra;
            if (g.periodic[a]) {
                const double xw = x[a] - floor((x[a] - g.lo[a]) / g.L[a]) * g.L[a];
                hb[a] = bucket_of(e, nb, xw);
                if (!(phi - plo < g.L[a])) {
                    ra = nb;
                } else {
                    const double lw = plo - floor((plo - g.lo[a]) / g.L[a]) * g.L[a];
                    const double hw = phi - floor((phi - g.lo[a]) / g.L[a]) * g.L[a];
                    const int blo = bucket_of(e, nb, lw), bhi = bucket_of(e, nb, hw);
                    // where the support wraps, its end can lie in the home
                    // bucket again, one turn away
                    int dl = hb[a] - blo, dr = bhi - hb[a];
                    dl = dl < 0 || (dl == 0 && lw > xw) ? dl + nb : dl;
                    dr = dr < 0 || (dr == 0 && hw < xw) ? dr + nb : dr;
                    ra = dl > dr ? dl : dr;
                }
            } else {
                if (phi < g.lo[a] || plo > g.hi[a]) support = false;
                const double xc = fmin(fmax(x[a], g.lo[a]), g.hi[a]);
                hb[a] = bucket_of(e, nb, xc);
                const int blo = bucket_of(e, nb, fmax(plo, g.lo[a])), bhi = bucket_of(e, nb, fmin(phi, g.hi[a]));
                ra = hb[a] - blo;
                if (bhi - hb[a] > ra) ra = bhi - hb[a];
            }
            if (ra < 0) ra = 0;
            if (ra > kClasses) ra = kClasses;
            if (ra > reach) reach = ra;
        }
        bl = hb[0] + (int64_t)g.nb[0] * (hb[1] + (int64_t)g.nb[1] * hb[2]);
        return support;
    }
};

constexpr int kCellsPrepassPerThread = 4;

template <typename R, int D>
__global__ __launch_bounds__(256) void k_cells_prepass(TrajDev t, CellGridDev g, PhysDev ph, const float* hfac,
                                                       uint32_t* keys, uint32_t* vals, double4* rpos, R* rw,
                                                       unsigned long long* stats)
{
    const int64_t i0 = (int64_t)blockIdx.x * blockDim.x * kCellsPrepassPerThread + threadIdx.x;
    const uint32_t sentinel = (uint32_t)kClasses * (uint32_t)g.nbuckets;
    unsigned long long skipped = 0, nosup = 0;
    const BucketKey<D> key{g};
#pragma unroll
    for (int u = 0; u < kCellsPrepassPerThread; ++u) {
        const int64_t i = i0 + (int64_t)u * blockDim.x;
        if (i < t.count)
            prepass_traj<R, D>(t, key, ph, hfac, 0, i, i, 0u, sentinel, keys, vals, rpos, rw, nullptr, skipped,
                               nosup);
    }
    wave_count_sum(stats, ST_SKIPPED, (unsigned)skipped);
    wave_count_sum(stats, ST_NOSUPPORT, (unsigned)nosup);
}

template <typename R, int D>
hipError_t launch_cells_prepass(const TrajDev& t, const CellGridDev& g, const PhysDev& ph, const float* hfac,
                                uint32_t* keys, uint32_t* vals, double4* rpos, R* rw, unsigned long long* stats,
                                hipStream_t s)
{
    if (t.count == 0) return hipSuccess;
    const int64_t per = 256 * kCellsPrepassPerThread;
    const int64_t blocks = (t.count + per - 1) / per;
    FLA_LAUNCH((k_cells_prepass<R, D>), dim3((unsigned)blocks), dim3(256), 0, s, t, g, ph, hfac, keys, vals,
                       rpos, rw, stats);
    return hipGetLastError();
}

// Buckets within reach r of bucket b along one axis, as at most two runs
// [s, e] (a periodic axis wraps; a reach that covers the axis lists every
// bucket once).
__device__ inline int axis_runs(int b, int r, int nb, int periodic, int* s, int* e)
{
    s[1] = 0;
    e[1] = -1;
    if (periodic) {
        if (2 * r + 1 >= nb) {
            s[0] = 0;
            e[0] = nb - 1;
            return 1;
        }
        const int lo = b - r, hi = b + r;
        if (lo < 0) {
            s[0] = lo + nb;
            e[0] = nb - 1;
            s[1] = 0;
            e[1] = hi;
            return 2;
        }
        if (hi >= nb) {
            s[0] = lo;
            e[0] = nb - 1;
            s[1] = 0;
            e[1] = hi - nb;
            return 2;
        }
        s[0] = lo;
        e[0] = hi;
        return 1;
    }
    s[0] = b - r < 0 ? 0 : b - r;
    e[0] = b + r > nb - 1 ? nb - 1 : b + r;
    return 1;
}

__device__ inline double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ inline double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    return v;
}
__device__ inline double uniform(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Rows of buckets within reach of a bucket for one class: runs along x, then
// y, then z, each axis in at most two pieces.
struct CellRows {
    int nx, xs[2], xe[2];
    int y0[2], ny, nyt;      // first bucket of the pieces, length of the first, of both
    int z0[2], nz, nzt;
};

// records evaluated per batch
constexpr int kCellsBatch = kWave;
constexpr int kCellsFold = 8;    // records of a binary32 partial sum
constexpr int kCellsNone = kCellsBatch + kWave;   // slot of the record that reaches nothing

template <typename R> struct CellsLds {
    double4 pos[kCellsNone + 1];              // kept records: position and 1/h
    R w[kCellsNone + 1][kRecW];               // and weights
    double shift[kCellsNone + 1][3];            // periodic image of the offsets
    CellRows rows[kClasses];
    int base[kClasses + 1];                   // first run of each class
};

// What bounds it: instruction issue, 90% of the time busy.  A tested pair of a
// record and 64 cells takes about 23 vector instructions (binary64 offsets,
// squares and conversions, the exponential, the denominator) and one matrix
// instruction, and 39% of its lanes hold an included pair; the scan adds a
// tenth.  A record is read once per wave into LDS and from there, the same
// words for every lane, so nothing waits on memory in the pair loop; the image
// of a record's offsets is found once per record where the wave's box lies in
// one image (three additions), and per pair only where it straddles two.  The
// 6.2e9 pairs of 2M trajectories on 128^3 scattered cells take 15.8 ms; one
// record at a time through scalar loads, with a branch per pair and axis for
// the image, took 40.7 ms.  Two waves to a SIMD: at three the registers spill
// and it takes 16.1 ms where two take 15.0 (sums of 16); partial sums of 8
// records cost 1.1 ms against 16 and halve the error.
template <typename R, int D, bool COUNT>
__global__ __launch_bounds__(kWave, 2) void k_cells_gather(CellsGatherArgs a)
{
    constexpr int C = D + 1;
    constexpr int CPL = kCellsPerLane, NB = kCellsBatch;
    static_assert(CPL == 2 && NB == kWave, "one lane per record");
    constexpr bool kMfma = sizeof(R) == 4;
    using L = CellsLds<R>;
    __shared__ L my;
    const int lane = threadIdx.x;
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    if (item >= a.nwork) return;
    const int4 wk = a.work[item];
    const int b = wk.x, first = wk.y, ncell = wk.z;
    int bc[3];
    bc[0] = b % a.g.nb[0];
    bc[1] = (b / a.g.nb[0]) % a.g.nb[1];
    bc[2] = D == 3 ? b / (a.g.nb[0] * a.g.nb[1]) : 0;

    double xc[CPL][D];
    bool act[CPL];
#pragma unroll
    for (int u = 0; u < CPL; ++u) {
        const int k = u * kWave + lane;
        act[u] = k < ncell;
        const int p = first + (act[u] ? k : 0);
#pragma unroll
        for (int ax = 0; ax < D; ++ax) xc[u][ax] = a.xc[ax][p];
    }
    // bounding boxes, centre and half extent per axis: of the wave's cells, and
    // of the first and of the second 64 of them
    double cb[D], eh[D], cu[CPL][D], eu[CPL][D];
#pragma unroll
    for (int ax = 0; ax < D; ++ax) {
        double lo = 0.0, hi = 0.0;
#pragma unroll
        for (int u = 0; u < CPL; ++u) {
            const double l = wave_min(xc[u][ax]), h = wave_max(xc[u][ax]);
            cu[u][ax] = uniform(0.5 * (l + h));
            eu[u][ax] = uniform(0.5 * (h - l) * (1.0 + 1e-12) + 1e-300);
            lo = u ? fmin(lo, l) : l;
            hi = u ? fmax(hi, h) : h;
        }
        cb[ax] = uniform(0.5 * (lo + hi));
        eh[ax] = uniform(0.5 * (hi - lo) * (1.0 + 1e-12) + 1e-300);
    }
    R c2;
    {
#pragma clang fp contract(off)
        const R c = (R)a.cutoff;
        c2 = c * c;
    }

    // binary32: the denominator on the vector unit, the channels on the matrix
    // unit; partial sums run over at most kCellsFold records, then go to binary64
    R sum[CPL][C + 1];
    F4 acc[CPL];
    double tot[CPL][C + 1];
    uint32_t np[CPL];
#pragma unroll
    for (int u = 0; u < CPL; ++u) {
        np[u] = 0;
        acc[u] = F4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q <= C; ++q) {
            sum[u][q] = 0;
            tot[u][q] = 0.0;
        }
    }

    // scaled squared distance from a record to a box (nearest image) within reach
    auto meets = [&](const double4 P, const double* c, const double* h) {
        const double x[3] = {P.x, P.y, P.z};
        double acc = 0.0;
#pragma unroll
        for (int ax = 0; ax < D; ++ax) {
            double d = fabs(c[ax] - x[ax]);
            if (a.g.periodic[ax]) {
                if (d > 1.25 * a.g.L[ax]) d = fabs(min_image(d, a.g.L[ax]));
                d = fmin(d, fabs(d - a.g.L[ax]));
            }
            const double u = fmax(d - h[ax], 0.0) * P.w;
            acc = fma(u, u, acc);
        }
        return acc <= a.filt2;
    };

    // ---- one batch of n <= NB kept records
    auto process = [&](int n) {
        wave_sync();
        bool reach[CPL] = {false, false}, moved = false, mixed = false;
        if (lane < n) {
            const double4 P = my.pos[lane];
#pragma unroll
            for (int u = 0; u < CPL; ++u) reach[u] = meets(P, cu[u], eu[u]);
            // the image of the wave's box: none, one for the whole box, or mixed
            const double x[3] = {P.x, P.y, P.z};
#pragma unroll
            for (int ax = 0; ax < D; ++ax) {
                double sh = 0.0;
                if (a.g.periodic[ax]) {
                    const double La = a.g.L[ax], hi = 0.5 * La * (1.0 + 1e-9), lo = 0.5 * La * (1.0 - 1e-9);
                    const double d = cb[ax] - x[ax], dl = d - eh[ax], dh = d + eh[ax];
                    if (!(fmax(fabs(dl), fabs(dh)) < lo)) {
                        const double far = La * (1.0 - 1e-9);
                        if (dl > hi && dh < far)
                            sh = -La;
                        else if (dh < -hi && dl > -far)
                            sh = La;
                        else
                            mixed = true;
                    }
                }
                moved = moved || sh != 0.0;
                my.shift[lane][ax] = sh;
            }
        }
        const uint64_t r0 = __ballot(reach[0]), r1 = __ballot(reach[1]);
        const uint64_t mx = __ballot(mixed), mv = __ballot(moved) & ~mx;
        wave_sync();
        // the records of `bits`, two at a time so that the chains of their
        // pairs interleave, over the cells u0 to u1 of every lane; IMG: 0
        // offsets as they are, 1 the record's shift, 2 the minimum image of
        // every pair
        auto pass = [&](uint64_t bits, auto u0c, auto u1c, auto img) {
            constexpr int U0 = decltype(u0c)::value, U1 = decltype(u1c)::value, IMG = decltype(img)::value;
            while (bits) {
#pragma unroll 1
                for (int k = 0; k < kCellsFold / 2 && bits; ++k) {
                    // the last one of an odd number goes with the record that
                    // reaches nothing
                    const int e0 = __builtin_ctzll(bits);
                    bits &= ~(1ull << e0);
                    const int e1 = bits ? __builtin_ctzll(bits) : kCellsNone;
                    bits &= ~(1ull << (e1 & 63));
                    double x[2][D], inv_h[2], sh[2][D];
                    R w[2][C + 1];
                    float aw[2];   // q_m/h on lane m of every four (0 past the channels)
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const int e = r ? e1 : e0;
                        const double4 P = my.pos[e];
                        const double px[3] = {P.x, P.y, P.z};
                        inv_h[r] = P.w;
#pragma unroll
                        for (int ax = 0; ax < D; ++ax) {
                            x[r][ax] = px[ax];
                            sh[r][ax] = IMG == 1 ? my.shift[e][ax] : 0.0;
                        }
#pragma unroll
                        for (int q = 0; q <= (kMfma ? 0 : C); ++q) w[r][q] = my.w[e][q];
                        if (kMfma) aw[r] = (float)my.w[e][1 + (lane & 3)];
                    }
                    R ss[2][CPL], ev[2][CPL];
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int u = U0; u < U1; ++u) {
                            R s[3];
#pragma unroll
                            for (int ax = 0; ax < D; ++ax) {
                                double d;
                                {
#pragma clang fp contract(off)
                                    d = xc[u][ax] - x[r][ax];
                                    if (IMG == 1) d = d + sh[r][ax];
                                }
                                if (IMG == 2 && a.g.periodic[ax]) d = min_image(d, a.g.L[ax]);
                                s[ax] = (R)scaled_sq(d, inv_h[r]);
                            }
                            {
#pragma clang fp contract(off)
                                ss[r][u] = s[0] + s[1];
                                if (D == 3) ss[r][u] = ss[r][u] + s[2];
                            }
                        }
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int u = U0; u < U1; ++u) {
                            const bool inc = ss[r][u] <= c2;
                            if (COUNT) np[u] += inc && act[u] ? 1u : 0u;
                            ev[r][u] = (R)0;
                            if (sizeof(R) == 4 || __any(inc)) {   // the binary64 exponential is long
                                const R g = gauss_factor(ss[r][u]);
                                ev[r][u] = inc ? g : (R)0;
                            }
                        }
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int u = U0; u < U1; ++u)
#pragma unroll
                            for (int q = 0; q <= (kMfma ? 0 : C); ++q) sum[u][q] = fma(ev[r][u], w[r][q], sum[u][q]);
                    if constexpr (kMfma) {
                        // one 4x4x1 matrix instruction per 64 pairs: register k of a
                        // lane takes channel k of its cell.  They stay together:
                        // between vector instructions each costs about three times
                        // its 8 cycles.
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int u = U0; u < U1; ++u)
                                acc[u] = __builtin_amdgcn_mfma_f32_4x4x1f32(aw[r], (float)ev[r][u], acc[u], 4, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                if constexpr (kMfma) {
#pragma unroll
                    for (int u = U0; u < U1; ++u) {
                        tot[u][0] += (double)sum[u][0];
                        sum[u][0] = 0;
#pragma unroll
                        for (int q = 0; q < C; ++q) tot[u][1 + q] += (double)acc[u][q];
                        acc[u] = F4{0.f, 0.f, 0.f, 0.f};
                    }
                }
            }
        };
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        const uint64_t plain = ~(mx | mv);
        pass(r0 & r1 & plain, I0{}, I2{}, I0{});
        pass(r0 & ~r1 & plain, I0{}, I1{}, I0{});
        pass(r1 & ~r0 & plain, I1{}, I2{}, I0{});
        pass((r0 | r1) & mv, I0{}, I2{}, I1{});
        pass((r0 | r1) & mx, I0{}, I2{}, I2{});
        wave_sync();
    };

    // infinitely far in units of its h; no weight
    if (lane < kRecW) {
        my.w[kCellsNone][lane] = 0;
        if (lane < 3) my.shift[kCellsNone][lane] = 0.0;
        if (lane == 0) my.pos[kCellsNone] = make_double4(0.0, 0.0, 0.0, INFINITY);
    }

    // ---- scan.  Lane l holds run l of the current 64 runs of the sequence
    // class by class, z, y, piece of x: records s0 to s1 and its first chunk of
    // 64; the next chunk's records and the next runs are loaded ahead.
    if (lane < kClasses) {
        const uint32_t* bs = a.bstart + (int64_t)lane * a.g.nbuckets;
        int n = 0;
        if (bs[0] != bs[a.g.nbuckets]) {
            const int r = (lane == kClasses - 1) ? (1 << 28) : lane;
            CellRows cr;
            int s[2], t[2];
            cr.nx = axis_runs(bc[0], r, a.g.nb[0], a.g.periodic[0], cr.xs, cr.xe);
            axis_runs(bc[1], r, a.g.nb[1], a.g.periodic[1], s, t);
            cr.y0[0] = s[0];
            cr.y0[1] = s[1];
            cr.ny = t[0] - s[0] + 1;
            cr.nyt = cr.ny + (t[1] - s[1] + 1);
            cr.z0[0] = cr.z0[1] = 0;
            cr.nz = cr.nzt = 1;
            if (D == 3) {
                axis_runs(bc[2], r, a.g.nb[2], a.g.periodic[2], s, t);
                cr.z0[0] = s[0];
                cr.z0[1] = s[1];
                cr.nz = t[0] - s[0] + 1;
                cr.nzt = cr.nz + (t[1] - s[1] + 1);
            }
            n = cr.nx * cr.nyt * cr.nzt;
            my.rows[lane] = cr;
        }
        int incl = n;
#pragma unroll
        for (int o = 1; o < kClasses; o <<= 1) {
            const int t = __shfl_up(incl, o, kClasses);
            if (lane >= o) incl += t;
        }
        my.base[lane + 1] = incl;
        if (lane == 0) my.base[0] = 0;
    }
    wave_sync();
    const int nrun = my.base[kClasses];
    auto run_of = [&](int f, uint32_t& j0, uint32_t& j1) {
        j0 = j1 = 0;
        if (f >= nrun) return;
        int k = 0;
        while (my.base[k + 1] <= f) ++k;
        const CellRows& cr = my.rows[k];
        const int j = f - my.base[k], q = cr.nx == 2 ? j & 1 : 0, row = cr.nx == 2 ? j >> 1 : j;
        const int iz = row / cr.nyt, iy = row - iz * cr.nyt;
        const int y = iy < cr.ny ? cr.y0[0] + iy : cr.y0[1] + (iy - cr.ny);
        const int z = iz < cr.nz ? cr.z0[0] + iz : cr.z0[1] + (iz - cr.nz);
        const uint32_t* bs = a.bstart + (int64_t)k * a.g.nbuckets + (int64_t)a.g.nb[0] * (y + (int64_t)a.g.nb[1] * z);
        j0 = bs[cr.xs[q]];
        j1 = bs[cr.xe[q] + 1];
    };
    constexpr int NQ = (int)(kRecW * sizeof(R) / sizeof(uint4));
    uint32_t s0 = 0, s1 = 0, first_chunk = 0, s0n, s1n, c = 0, nchunk = 0;
    int f0 = 0, ncand = 0;
    run_of(lane, s0n, s1n);
    double4 Pn = make_double4(0, 0, 0, 0);
    uint4 wqn[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) wqn[q] = make_uint4(0, 0, 0, 0);
    bool okn = false;
    const uint64_t ltmask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (bool more = true; more;) {
        const double4 P = Pn;
        uint4 wq[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) wq[q] = wqn[q];
        const bool inr = okn;
        okn = false;
        while (c >= nchunk) {
            c = nchunk = 0;
            if (f0 >= nrun) {
                more = false;
                break;
            }
            s0 = s0n;
            s1 = s1n;
            f0 += kWave;
            run_of(f0 + lane, s0n, s1n);
            const uint32_t nc = (s1 - s0 + kWave - 1) / kWave;
            uint32_t incl = nc;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const uint32_t t = __shfl_up(incl, o, kWave);
                if (lane >= o) incl += t;
            }
            first_chunk = incl - nc;
            nchunk = __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        if (more) {
            const int j = __popcll(__ballot(first_chunk <= c)) - 1;
            const uint32_t p = __builtin_amdgcn_readlane(s0, j) +
                               (c - __builtin_amdgcn_readlane(first_chunk, j)) * kWave + lane;
            okn = p < __builtin_amdgcn_readlane(s1, j);
            ++c;
            if (okn) {
                Pn = a.rpos[p];
                const uint4* w = reinterpret_cast<const uint4*>((const R*)a.rw + (int64_t)p * kRecW);
#pragma unroll
                for (int q = 0; q < NQ; ++q) wqn[q] = w[q];
            }
        }
        const bool ok = inr && meets(P, cb, eh);
        const uint64_t bal = __ballot(ok);
        if (ok) {
            const int at = ncand + __popcll(bal & ltmask);
            my.pos[at] = P;
            uint4* w = reinterpret_cast<uint4*>(my.w[at]);
#pragma unroll
            for (int q = 0; q < NQ; ++q) w[q] = wq[q];
        }
        ncand += __popcll(bal);
        while (ncand >= (more ? NB : 1)) {
            const int n = ncand < NB ? ncand : NB;
            process(n);
            const int rem = ncand - n;
            if (rem > 0) {
                const int at = n + (lane < rem ? lane : 0);
                const double4 mp = my.pos[at];
                uint4 mw[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) mw[q] = reinterpret_cast<const uint4*>(my.w[at])[q];
                wave_sync();
                if (lane < rem) {
                    my.pos[lane] = mp;
#pragma unroll
                    for (int q = 0; q < NQ; ++q) reinterpret_cast<uint4*>(my.w[lane])[q] = mw[q];
                }
            }
            ncand = rem;
        }
    }

    unsigned long long wave_pairs = 0;
#pragma unroll
    for (int u = 0; u < CPL; ++u) {
        if (!act[u]) continue;
        const int p = first + u * kWave + lane;
        const uint32_t cell = a.perm[p];
        const double den = sizeof(R) == 4 ? tot[u][0] : (double)sum[u][0];
        double f;
        {
#pragma clang fp contract(off)
            f = -a.scale * (a.use_vol ? a.vol[p] : 1.0);
        }
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const double num = sizeof(R) == 4 ? tot[u][1 + q] : (double)sum[u][1 + q];
            const double S = den > 0.0 ? f * (num / den) : 0.0;
            ((R*)a.out[q])[cell] = (R)S;
        }
        if (a.den) ((R*)a.den)[cell] = (R)den;
        if (COUNT) {
            if (a.pairs) a.pairs[cell] = np[u];
            wave_pairs += np[u];
        }
    }
    // the weights beyond the range of R (split_over), to the cells that include
    // their records: infinities, which leave nothing of the finite sums
    if (a.stats[ST_OVER]) {
        R over[CPL][C + 1];
        bool hit[CPL] = {false, false};
#pragma unroll
        for (int u = 0; u < CPL; ++u)
#pragma unroll
            for (int q = 0; q <= C; ++q) over[u][q] = 0;
        for (int f = 0; f < nrun; ++f) {
            uint32_t j0, j1;
            run_of(f, j0, j1);
            for (uint32_t p0 = j0; p0 < j1; p0 += kWave) {
                const uint32_t p = p0 + lane;
                const int code = p < j1 ? (int)((const R*)a.rw)[(int64_t)p * kRecW + kRecOver] : 0;
                for (uint64_t bits = __ballot(code != 0); bits; bits &= bits - 1) {
                    const int e = __builtin_ctzll(bits);
                    const int oc = __builtin_amdgcn_readlane(code, e);
                    const double4 P = a.rpos[p0 + e];
                    const double px[3] = {P.x, P.y, P.z};
#pragma unroll
                    for (int u = 0; u < CPL; ++u) {
                        R ss = 0;
#pragma unroll
                        for (int ax = 0; ax < D; ++ax) {
                            double d = xc[u][ax] - px[ax];
                            if (a.g.periodic[ax]) d = min_image(d, a.g.L[ax]);
                            const R s = (R)scaled_sq(d, P.w);
                            ss = ax ? ss + s : s;
                        }
                        if (ss <= c2) {
                            hit[u] = true;
#pragma unroll
                            for (int q = 0; q <= C; ++q)
                                if ((oc >> (2 * q)) & 3) over[u][q] += gauss_factor(ss) * over_weight<R>(oc, q);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < CPL; ++u) {
            if (!act[u] || !hit[u]) continue;
            const int p = first + u * kWave + lane;
            const uint32_t cell = a.perm[p];
            const double f = -a.scale * (a.use_vol ? a.vol[p] : 1.0);
            const bool over_den = over[u][0] != (R)0;
            const double den = over_den ? (double)over[u][0] : 1.0;
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const double num = (double)over[u][1 + q];
                if (num == 0.0 && !over_den) continue;
                ((R*)a.out[q])[cell] = (R)(den > 0.0 ? f * (num / den) : 0.0);
            }
            if (over_den && a.den) ((R*)a.den)[cell] = over[u][0];
        }
    }
    if (COUNT) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) wave_pairs += __shfl_xor(wave_pairs, o, kWave);
        if (lane == 0 && wave_pairs) atomicAdd(&a.stats[ST_PAIRS], wave_pairs);
    }
}

template <typename R, int D>
hipError_t launch_cells_gather(const CellsGatherArgs& a, bool count, hipStream_t s)
{
    if (a.nwork == 0) return hipSuccess;
    // one wave a workgroup: their times differ, and four together held the
    // registers and LDS of the finished ones
    const int blocks = a.nwork;
    if (count)
        FLA_LAUNCH((k_cells_gather<R, D, true>), dim3(blocks), dim3(kWave), 0, s, a);
    else
        FLA_LAUNCH((k_cells_gather<R, D, false>), dim3(blocks), dim3(kWave), 0, s, a);
    return hipGetLastError();
}

template hipError_t launch_cells_prepass<float, 2>(const TrajDev&, const CellGridDev&, const PhysDev&, const float*,
                                                   uint32_t*, uint32_t*, double4*, float*, unsigned long long*,
                                                   hipStream_t);
template hipError_t launch_cells_prepass<float, 3>(const TrajDev&, const CellGridDev&, const PhysDev&, const float*,
                                                   uint32_t*, uint32_t*, double4*, float*, unsigned long long*,
                                                   hipStream_t);
template hipError_t launch_cells_prepass<double, 2>(const TrajDev&, const CellGridDev&, const PhysDev&, const float*,
                                                    uint32_t*, uint32_t*, double4*, double*, unsigned long long*,
                                                    hipStream_t);
template hipError_t launch_cells_prepass<double, 3>(const TrajDev&, const CellGridDev&, const PhysDev&, const float*,
                                                    uint32_t*, uint32_t*, double4*, double*, unsigned long long*,
                                                    hipStream_t);
template hipError_t launch_cells_gather<float, 2>(const CellsGatherArgs&, bool, hipStream_t);
template hipError_t launch_cells_gather<float, 3>(const CellsGatherArgs&, bool, hipStream_t);
template hipError_t launch_cells_gather<double, 2>(const CellsGatherArgs&, bool, hipStream_t);
template hipError_t launch_cells_gather<double, 3>(const CellsGatherArgs&, bool, hipStream_t);

}  // namespace flp
