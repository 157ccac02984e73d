// Cell-centric gather of the Nadaraya-Watson numerator and denominator
// (eqs. kernel-estimator, kernel and coupling-terms-kernel; App. B steps
// 1c, 1d, 2a, 2c) with the epilogue fused in.  No atomics touch the fields:
// every cell is owned by exactly one lane of one wave, and each lane visits
// the trajectories of its tile in a fixed order, so results are bitwise
// reproducible.
//
// Work decomposition: a tile is TE^D cells, a workgroup owns a tile or (3-D,
// binary64) one half of it across x; the waves of the workgroup (four in
// 3-D, two in 2-D) take the candidate chunks in turn and their sums are added
// in wave order at the end; the workgroups are persistent and take their
// XCD's parts in heaviest-first order (k_gather).
//  * candidate trajectories come from the buckets (class k, home tile) of
//    the neighbourhood of the tile: a class-k trajectory reaches at most k
//    tiles from its home tile (the last class spans whole axes);
//  * a conservative binary64 sphere/box test compacts candidates into an
//    LDS list (order preserved with wave ballots);
//  * per batch of candidates the lanes build, in LDS, the per-axis factors
//    s = (d/h)^2 and e = exp(-s/2) for the cell centres of the workgroup on
//    every axis (the Gaussian is separable on a Cartesian mesh), in
//    straight-line code (the minimum image and the delta records take one
//    branch per axis);
//  * every lane then walks the batch over its cells, skipping what a record
//    reaches nowhere (an exact, wave-uniform skip).
// Weights beyond the range of the precision are left out of these sums and added
// afterwards (add_overs).  Two tile bodies share this frame:
//  * gather_planes (binary32, 3-D): a lane owns a column of cells, and what
//    depends on z alone is the same on every lane (few tiles of many records:
//    four workgroups to each, k_gather_split);
//  * gather_tile (binary64, and 2-D): the tile is split into 2^D sub-blocks
//    of SB^D cells and lane l owns the cell with in-block coordinates lc(l)
//    in every sub-block.
// Binary32 partial sums run over at most 64 records before they are folded
// (into binary64 or compensated totals); binary64 sums need no compensation.
//
// Plan codes plan + kGatherPlans * shape (fla_autotune times them all): the
// plan is the granularity of the skips, the shape the part of a tile that a
// workgroup owns (in binary32 the whole tile in either shape).
//
// This header holds the kernels and their launchers; the units
// gather_{f32,f64}_{2d,3d}.hip instantiate them per precision and dimension,
// so that they compile in parallel.
#pragma once
#include <type_traits>

#include "internal.hpp"
#include "kernels.hpp"

namespace flp {

// Gather mode of the Nadaraya-Watson estimator on any mesh (uniform or
// rectilinear axes); FLA_NW itself assumes uniform axes.
constexpr int kNwGeneral = 2;

constexpr int kCap = 2 * kWave;

typedef float F4 __attribute__((ext_vector_type(4)));

// A value that is the same on every lane, moved to scalar registers (the
// vector unit computes binary64 and binary32 values into vector registers).
__device__ inline double uniform_value(double v)
{
    const unsigned long long b = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ inline float uniform_value(float v)
{
    return __int_as_float((int)__builtin_amdgcn_readfirstlane((unsigned)__float_as_int(v)));
}

template <typename R> __device__ inline R r_inf();
template <> __device__ inline float r_inf<float>() { return __builtin_inff(); }
template <> __device__ inline double r_inf<double>() { return __builtin_inf(); }

template <typename R>
__device__ inline void two_sum_acc(R& hi, R& lo, R p)
{
    R s = hi + p;
    R bp = s - hi;
    R err = (hi - (s - bp)) + (p - bp);
    hi = s;
    lo += err;
}

// waves per workgroup (all work on one tile or part): four; two in binary32
// 2-D, whose tiles have twice the cells per axis and whose staging tables are
// larger
template <typename R, int D> struct GatherWaves { static constexpr int value = D == 3 || sizeof(R) == 8 ? 4 : 2; };

// Workgroups per tile (the shape).  With TP = 2 (binary64) each workgroup owns
// one half of the tile along x, which halves the registers of its sums and its
// staging space, so that more workgroups share a compute unit, at the cost of
// scanning and staging every candidate once per half.  They stage 32 records
// at a time, two lanes to a record: half the space again, so that two
// workgroups fit a compute unit instead of one and the binary64 chains of one
// cover the other's (61 x 47 x 53 cells, 120k trajectories: 382 -> 284 us).  In
// 2-D, two halves of four waves in place of one tile of two also spread a small
// mesh over four times the waves (64^2 cells: 87 -> 32 us); whole tiles are
// staged in the same way and are taken where records are few (whole_tiles).
template <typename R> __host__ __device__ constexpr int tile_parts(int D, int shape)
{
    return sizeof(R) == 8 && shape == 0 ? 2 : 1;
}

// Waves per SIMD the register allocation is held to (binary32 in 3-D: the
// sums of eight planes take 120 registers; at three waves the rest spills
// into the loops, 6.9 instead of 5.0 ms on the 128^3 case; binary64: two where
// the staging space lets two workgroups in).
template <typename R, int D, int TP> struct GatherOcc {
    static constexpr int value = sizeof(R) == 4 || TP == 2 || D == 2 ? 2 : 1;
};

template <typename R, int D, int TP>
struct GatherLds {
    using R4 = typename V4<R>::T;
    using R2 = typename V2<R>::T;
    static constexpr int SB = Geo<D>::SB, NA = D + 2;
    static constexpr int NT = TP == 2 ? D - 1 : D;   // axes staged for both halves (split: y, z)
    // records staged at a time, lanes that stage one
    static constexpr int NB = TP == 2 || (D == 2 && sizeof(R) == 8) ? kWave / 2 : kWave, LPR = kWave / NB;
    uint32_t cand[kCap];               // compacted candidate record indices
    R4 tab[NB][NT][SB];                // {s, e} at in-block position l and l + SB
    R2 tabs[NB][TP == 2 ? SB : 1];     // split axis x: {s, e} of the owned half
    R wts[NB][NA];                     // {1/h, q/h ...} of each staged record
    int mask[NB];                      // sub-blocks holding at least one included pair
};

// Per-axis factors of one record for the tile at tile coordinates tc, whose
// cell centres are xcs: tab[a][l] = {s, e} at in-block positions l and
// l + SB of axis a, with s = (d/h)^2 (binary64 rounded to R) and
// e = exp(-s/2); with the split, axis x is staged for the owned half
// only, tabs[l] = {s, e} at position soff + l.  A delta record (1/h < 0) has
// factor 1 at its home cell and 0 elsewhere.  Returns the visit mask of the
// workgroup's sub-blocks: bit b is set iff the sum of the per-axis minima of
// s over sub-block b passes the cutoff (sums are monotone in each term, so
// no sub-block holding an included pair is skipped).
template <typename R, int D, int TP>
__device__ __forceinline__ int stage_record(const MeshDev& m, const double (*xcs)[Geo<D>::TE], const int* tc,
                                            const int soff, const double4 P, const R c2, const int part,
                                            typename V4<R>::T (*tab)[Geo<D>::SB], typename V2<R>::T* tabs)
{
    using G = Geo<D>;
    constexpr int TE = G::TE, SB = G::SB, NSB = G::NSB / TP;
    // positions l of a half tile that this lane takes: all of them, or (two
    // lanes to a record, 32 apart) its half of them
    constexpr int LPR = GatherLds<R, D, TP>::LPR, NL = SB / LPR, NP = 2 * NL;
    const int l0 = part * NL;
    auto whole = [](R v) { return LPR == 2 ? fmin(v, __shfl_xor(v, kWave / 2, kWave)) : v; };
    using R4 = typename V4<R>::T;
    using R2 = typename V2<R>::T;
    double x[3] = {P.x, P.y, P.z};
    const bool delta = P.w < 0.0;
    const double inv_h = delta ? -P.w : P.w;
    R mn[3][2];
    // Straight-line code per axis (the positions are independent chains);
    // the minimum image and the delta records take one branch per axis.
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const bool one = TP == 2 && a == 0;   // one half of this axis, at soff
        const int np = one ? NL : NP;
        double d[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            // positions l and l + SB of the sub-blocks, or soff + l
            const int pp = l0 + (one ? soff + p : p < NL ? p : p - NL + SB);
            d[p] = (p < np) ? xcs[a][pp] - x[a] : 0.0;
        }
        if (m.periodic[a]) {
            // centres of cells beyond the mesh are NaN, ignored by fmax
            double dm = 0.0;
#pragma unroll
            for (int p = 0; p < NP; ++p) dm = fmax(dm, fabs(d[p]));
            if (LPR == 2) dm = fmax(dm, __shfl_xor(dm, kWave / 2, kWave));
            const double L = m.L[a];
            if (dm > 0.5 * L) {
                if (dm < L) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
#pragma clang fp contract(off)
                        const double w = d[p] > 0.0 ? d[p] - L : d[p] + L;
                        d[p] = fabs(d[p]) <= 0.5 * L ? d[p] : w;
                    }
                } else {
#pragma unroll
                    for (int p = 0; p < NP; ++p) d[p] = min_image(d[p], L);
                }
            }
        }
        // s = (d/h)^2 rounded to R, e = exp(-s/2); a NaN centre gives a NaN s,
        // which never passes the test and is ignored by the minima
        R sv[NP], ev[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            sv[p] = (R)scaled_sq(d[p], inv_h);
            ev[p] = gauss_factor(sv[p]);
        }
        if (delta) {
            // whole amount into the home cell: factor 1 there, 0 elsewhere
            const int64_t hcell = home_index(m, a, x[a]);
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int pp = l0 + (one ? soff + p : p < NL ? p : p - NL + SB);
                const bool home = (int64_t)tc[a] * TE + pp == hcell;
                sv[p] = home ? (R)0 : r_inf<R>();
                ev[p] = home ? (R)1 : (R)0;
            }
        }
        R mlo = r_inf<R>(), mhi = r_inf<R>();
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            if (one) {
                R2 t2;
                t2.x = sv[l];
                t2.y = ev[l];
                tabs[l0 + l] = t2;
            } else {
                R4 t4;
                t4.x = sv[l];
                t4.y = ev[l];
                t4.z = sv[l + NL];
                t4.w = ev[l + NL];
                tab[TP == 2 ? a - 1 : a][l0 + l] = t4;
                mhi = fmin(mhi, sv[l + NL]);
            }
            mlo = fmin(mlo, sv[l]);
        }
        mn[a][0] = whole(mlo);
        mn[a][1] = whole(mhi);
    }
    // visit mask: the sub-block can hold an included pair (the sum of
    // the per-axis minima passes; binary32/64 sums are monotone in each
    // term, so the skip never drops an included pair)
    int mk = 0;
#pragma unroll
    for (int b = 0; b < NSB; ++b) {
        // sub-block bits: (x, y, z), or (y, z) with x split
        const int bx = TP == 2 ? 0 : b & 1;
        const int by = TP == 2 ? b & 1 : (b >> 1) & 1;
        const int bz = TP == 2 ? (b >> 1) & 1 : (b >> 2) & 1;
        R smin = mn[0][bx] + mn[1][by];
        if (D == 3) smin = smin + mn[2][bz];
        mk |= (smin <= c2) ? (1 << b) : 0;
    }
    return mk;
}

// Rows of home tiles that the tile at tile coordinates tc must consider for
// neighbourhood class k: the home tiles within k tiles of tc on every axis
// (the last class: whole axes), in rows along x, ordered z, then y; along x
// the home tiles of a row are contiguous in the sorted order (one run, or two
// across a periodic wrap, with tile ranges runs[q]).
struct ClassRows {
    uint32_t kb;        // first bucket of the class
    int lo_t[3], cnt_t[3];
    int runs[2][2];
    int nruns, nrows;
};

template <int D>
__device__ __forceinline__ void class_rows(const MeshDev& m, const int* tc, int k, ClassRows& cr)
{
    cr.kb = (uint32_t)k * (uint32_t)m.ntiles;
    const int r = (k == kClasses - 1) ? (1 << 28) : k;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (a >= D) {
            cr.lo_t[a] = 0;
            cr.cnt_t[a] = 1;
            continue;
        }
        int nt = m.nt[a];
        if (2 * (int64_t)r + 1 >= nt) {
            cr.lo_t[a] = 0;
            cr.cnt_t[a] = nt;
        } else if (m.periodic[a]) {
            cr.lo_t[a] = tc[a] - r;
            cr.cnt_t[a] = 2 * r + 1;
        } else {
            int l0 = tc[a] - r < 0 ? 0 : tc[a] - r;
            int l1 = tc[a] + r >= nt ? nt - 1 : tc[a] + r;
            cr.lo_t[a] = l0;
            cr.cnt_t[a] = l1 - l0 + 1;
        }
    }
    const int x0 = cr.lo_t[0], x1 = cr.lo_t[0] + cr.cnt_t[0] - 1;
    cr.nruns = 1;
    if (x0 < 0) {
        cr.runs[0][0] = x0 + m.nt[0];
        cr.runs[0][1] = m.nt[0] - 1;
        cr.runs[1][0] = 0;
        cr.runs[1][1] = x1;
        cr.nruns = 2;
    } else if (x1 >= m.nt[0]) {
        cr.runs[0][0] = x0;
        cr.runs[0][1] = m.nt[0] - 1;
        cr.runs[1][0] = 0;
        cr.runs[1][1] = x1 - m.nt[0];
        cr.nruns = 2;
    } else {
        cr.runs[0][0] = x0;
        cr.runs[0][1] = x1;
        cr.runs[1][0] = 0;
        cr.runs[1][1] = -1;
    }
    cr.nrows = cr.cnt_t[1] * cr.cnt_t[2];
}

// First bucket of row `row` of a class.
template <int D>
__device__ __forceinline__ uint32_t row_bucket(const MeshDev& m, const ClassRows& cr, int row)
{
    const int jz = row / cr.cnt_t[1], jy = row - jz * cr.cnt_t[1];
    int hz = cr.lo_t[2] + jz;
    if (D == 3) hz = (int)posmod(hz, m.nt[2]);
    const int hy = (int)posmod(cr.lo_t[1] + jy, m.nt[1]);
    return cr.kb + (uint32_t)m.nt[0] * ((uint32_t)hy + (uint32_t)m.nt[1] * (uint32_t)hz);
}

// Calls fn(s0, s1) for every non-empty run [s0, s1) of sorted records that
// the tile at tile coordinates tc must consider, class by class, row by row
// (class_rows).  The bucket bounds of up to 64 rows are fetched at once, one
// row per lane, and read back with readlane, so the rows do not wait on one
// scalar load each.
template <int D, typename F>
__device__ __forceinline__ void for_each_run(const MeshDev& m, const uint32_t* bstart, const int* tc,
                                             const int lane, F&& fn)
{
    for (int k = 0; k < kClasses; ++k) {
        const uint32_t kb = (uint32_t)k * (uint32_t)m.ntiles;
        if (bstart[kb] == bstart[kb + m.ntiles]) continue;
        ClassRows cr;
        class_rows<D>(m, tc, k, cr);
        for (int g0 = 0; g0 < cr.nrows; g0 += kWave) {
            // lane j fetches the bounds of row g0 + j
            uint32_t b00 = 0, b01 = 0, b10 = 0, b11 = 0;
            const int row = g0 + lane;
            if (row < cr.nrows) {
                const uint32_t rowb = row_bucket<D>(m, cr, row);
                b00 = bstart[rowb + cr.runs[0][0]];
                b01 = bstart[rowb + cr.runs[0][1] + 1];
                if (cr.nruns == 2) {
                    b10 = bstart[rowb + cr.runs[1][0]];
                    b11 = bstart[rowb + cr.runs[1][1] + 1];
                }
            }
            // runs in order: row by row, the runs of a row in x order
            const int nr = cr.nrows - g0 < kWave ? cr.nrows - g0 : kWave;
            for (int j = 0; j < nr * cr.nruns; ++j) {
                const int jr = cr.nruns == 2 ? j >> 1 : j;
                const bool second = cr.nruns == 2 && (j & 1);
                const uint32_t a0 = __builtin_amdgcn_readlane(b00, jr), a1 = __builtin_amdgcn_readlane(b01, jr);
                const uint32_t c0 = __builtin_amdgcn_readlane(b10, jr), c1 = __builtin_amdgcn_readlane(b11, jr);
                const uint32_t s0 = second ? c0 : a0, s1 = second ? c1 : a1;
                if (s0 < s1) fn(s0, s1);
            }
        }
    }
}

// Conservative test of one record against the tile: a delta record (1/h < 0)
// belongs to the tile of its home cell; any other record passes if the
// scaled binary64 distance from its position to the tile's box of cell
// centres (mid bmid, half-widths bhalf; axes where the box spans half a
// periodic box or more are not tested) is within filt2.
template <int D>
__device__ __forceinline__ bool candidate_ok(const MeshDev& m, const double4 P, const int* tc, const double* bmid,
                                             const double* bhalf, const bool* faxis, double filt2)
{
    constexpr int TE = Geo<D>::TE;
    double x[3] = {P.x, P.y, P.z};
    if (P.w < 0.0) {
        bool ok = true;
#pragma unroll
        for (int a = 0; a < D; ++a) ok = ok && (home_index(m, a, x[a]) / TE == tc[a]);
        return ok;
    }
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        if (!faxis[a]) continue;
        double d = fabs(axis_offset(m, a, bmid[a], x[a])) - bhalf[a];
        if (d > 0.0) {
            double u = d * P.w;
            acc += u * u;
        }
    }
    return acc <= filt2;
}

// Adds the weights beyond the range of R (split_over) to the fields of the lane's
// cell `lin` with indices cidx, where it includes their records: infinities,
// which leave nothing of the finite sums.  Called by whole waves, after the cells
// have been written, only where a record of the call has an over code.
template <typename R, int D, int MODE>
__device__ __forceinline__ void add_overs(const GatherArgs& g, const int* tc, const int lane, const int64_t* cidx,
                                          const int64_t lin, const bool inside)
{
    constexpr int NA = D + 2;
    const MeshDev& m = g.m;
    const R c2 = (R)g.cutoff * (R)g.cutoff;
    double xc[D];
#pragma unroll
    for (int a = 0; a < D; ++a)
        xc[a] = cidx[a] < m.n[a] ? cell_centre(m, a, cidx[a]) : __builtin_nan("");
    R sum[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) sum[k] = 0;
    bool hit = false;
    for_each_run<D>(m, g.bstart, tc, lane, [&](const uint32_t s0, const uint32_t s1) {
        for (uint32_t p0 = s0; p0 < s1; p0 += kWave) {
            const uint32_t p = p0 + lane;
            const int code = p < s1 ? (int)((const R*)g.rw)[(size_t)p * kRecW + kRecOver] : 0;
            for (uint64_t bits = __ballot(code != 0); bits; bits &= bits - 1) {
                const int e = __builtin_ctzll(bits);
                const int c = __builtin_amdgcn_readlane(code, e);
                const double4 P = g.rpos[p0 + e];
                const double x[3] = {P.x, P.y, P.z};
                const bool delta = MODE == FLA_DEPOSIT && P.w < 0.0;
                R s = 0, ev = 1;
#pragma unroll
                for (int a = 0; a < D; ++a) {
                    R sa = (R)scaled_sq(axis_offset(m, a, xc[a], x[a]), P.w), ea = gauss_factor(sa);
                    if (delta) {
                        const bool home = cidx[a] == home_index(m, a, x[a]);
                        sa = home ? (R)0 : r_inf<R>();
                        ea = (R)1;
                    }
                    s = a ? s + sa : sa;
                    ev *= ea;
                }
                if (s <= c2) {
                    hit = true;
#pragma unroll
                    for (int k = 0; k < NA; ++k)
                        if ((c >> (2 * k)) & 3) sum[k] += ev * over_weight<R>(c, k);
                }
            }
        }
    });
    if (!hit || !inside) return;
    const double f = -g.scale * (g.cell_scale ? (double)((const R*)g.cell_scale)[lin] : 1.0);
    const bool over_den = sum[0] != (R)0;          // also where it is NaN
    const double den = over_den ? (double)sum[0] : 1.0;
#pragma unroll
    for (int k = 0; k <= D; ++k) {
        const double q = (double)sum[1 + k];
        if (q == 0.0 && !over_den) continue;
        ((R*)g.out[k])[lin] = (R)(MODE != FLA_DEPOSIT ? (den > 0.0 ? f * (q / den) : 0.0) : f * q / m.vol);
    }
    if (over_den && g.den) ((R*)g.den)[lin] = sum[0];
}

// ---------------------------------------------------------------------------
// Binary32, 3-D: whole planes of a tile per wave.
// ---------------------------------------------------------------------------
// Lane l owns the column of cells (x, y) = (l % 8, l / 8) of the tile; the
// eight planes are taken in turn, so that everything that depends on z alone
// is the same on all 64 lanes:
//  * the test s_x + s_y + s_z <= c^2 is the comparison of s_x + s_y with a
//    threshold T(s_z), the largest binary32 t with fl(t + s_z) <= c^2, so the
//    decision is that of the sum, bit for bit;
//  * e_z goes into the record's weights (e_z/h, e_z q_k/h), so that a pair's
//    kernel weight is e_x e_y alone, formed once per record and column.
// A pair then costs one subtraction (scaled threshold minus scaled s_x + s_y),
// one median (the weight where the difference is positive, else 0), one
// multiply-add for the denominator and a quarter of a 4x4x1 matrix
// instruction for the four channels.  The plane's threshold and denominator
// weight come out of one register per 16 (record, plane) pairs by a row
// broadcast inside the vector instruction, the channel weights out of one
// register by the matrix instruction's own block broadcast: a pair of records
// costs seven LDS reads for all of its planes.
constexpr int kPlaneRecs = 2;              // records per register of row broadcasts
struct PlaneGroup {
    float2 x[kPlaneRecs][8], y[kPlaneRecs][8];   // {s B, e} at the tile's positions
    float2 td[kPlaneRecs][8];                    // per plane: scaled threshold, e_z/h
    float ez[kPlaneRecs][8];
    float q[kPlaneRecs][4];                      // q_k/h
};
struct PlaneLds {
    static constexpr int NB = 32;          // records per batch (two lanes stage one record)
    PlaneGroup grp[NB / kPlaneRecs + 1];   // the last one is read ahead, never written or used
    double4 pos[NB + kWave];               // compacted candidates: position and 1/h,
    float4 wa[NB + kWave];                 // {1/h, q_0/h, q_1/h, q_2/h}
    float wb[NB + kWave];                  // and q_3/h
};

struct PlaneWavesLds {
    PlaneLds w[GatherWaves<float, 3>::value];
};
// of a workgroup whose waves work on the same batches (SPLIT)
struct PlaneSplitLds {
    static constexpr int W = GatherWaves<float, 3>::value, N = 2 * W * kWave;
    PlaneGroup grp[W][PlaneLds::NB / kPlaneRecs + 1];
    double4 pos[N];                        // candidates of all waves
    float4 wa[N];
    float wb[N];
    int cnt[W], more[W];
};

// Home-tile rows of the classes of a tile, in the order they are visited
// (class by class, row by row, the runs of a row in x order), as one sequence
// of runs of sorted records.
struct RunTable {
    ClassRows cls[kClasses];
    int base[kClasses + 1];                // first run of each class
};

// lane j of the row of 16 lanes, on every lane of the row
template <int J> __device__ __forceinline__ float row_bcast(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + J, 0xF, 0xF, true));
}

// Weights of one record in two planes and their part of the denominators:
// a, b hold scaled threshold minus scaled s_x + s_y and become the kernel
// weight where that is positive, else 0; the planes' denominator weights are
// lanes J0 and J1 of each row of dz.  As one block because the compiler does
// not fold a row broadcast into a multiply-add (a move and a multiply-add
// instead: one vector instruction in four more); the two medians in front
// keep the two wait states that a row broadcast needs after any write of dz.
template <int J0, int J1>
__device__ __forceinline__ void weigh2(float& a, float& b, const float e, const float dz, float& da, float& db)
{
    asm("v_med3_f32 %0, %0, %4, 0\n\t"
        "v_med3_f32 %1, %1, %4, 0\n\t"
        "v_fmac_f32_dpp %2, %5, %0 row_newbcast:%c6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %3, %5, %1 row_newbcast:%c7 row_mask:0xf bank_mask:0xf"
        : "+v"(a), "+v"(b), "+v"(da), "+v"(db)
        : "v"(e), "v"(dz), "n"(J0), "n"(J1));
}

template <int I, int N, typename F> __device__ __forceinline__ void static_for(F&& f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// Conservative test of one record against the tile, as candidate_ok but
// without a branch per axis: the distance to the nearest image of a box centre
// takes one fold below 5 L / 4 (the margin of filt2 covers its rounding).
template <bool DELTA>
__device__ __forceinline__ bool near_tile(const MeshDev& m, const double4 P, const int* tc, const double* bmid,
                                          const double* bhalf, const bool* faxis, double filt2)
{
    const double x[3] = {P.x, P.y, P.z};
    if (DELTA && P.w < 0.0) {
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) ok = ok && (home_index(m, a, x[a]) / Geo<3>::TE == tc[a]);
        return ok;
    }
    double acc = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!faxis[a]) continue;
        double d = fabs(bmid[a] - x[a]);
        if (m.periodic[a]) {
            if (d > 1.25 * m.L[a]) d = fabs(min_image(d, m.L[a]));
            d = fmin(d, fabs(d - m.L[a]));
        }
        const double u = fmax(d - bhalf[a], 0.0) * P.w;
        acc = fma(u, u, acc);
    }
    return acc <= filt2;
}

// The fields of cell lin from its sums: divided (NW) or scaled by 1/V_c
// (deposition), sign, scale.
template <int MODE>
__device__ __forceinline__ void write_cell(const GatherArgs& g, const int64_t lin, const double* sum)
{
    const double f = -g.scale * (g.cell_scale ? (double)((const float*)g.cell_scale)[lin] : 1.0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double val = MODE != FLA_DEPOSIT ? (sum[0] > 0.0 ? f * (sum[1 + k] / sum[0]) : 0.0)
                                               : f * sum[1 + k] / g.m.vol;
        ((float*)g.out[k])[lin] = (float)val;
    }
    if (g.den) ((float*)g.den)[lin] = (float)sum[0];
}

// The work of one workgroup in binary32 and 3-D: the planes of `own` (a bit
// per two) of one tile.  The four waves
// take the chunks of 64 candidates in turn and keep their own sums.
//
// What bounds it: instruction issue.  A plane of one record takes 22 cycles (a
// probe of the loop alone: three vector instructions 12.6, the matrix
// instruction 9.4; they do not overlap, from one wave or from several), which
// is three fifths of the kernel; the rest are the group's words, the staging
// and the scan.  Two waves per SIMD hold the sums of eight planes (120
// registers) without spills, so no wave waits on memory that it has not asked
// for a step ahead: the bounds of the next 64 runs, the next chunk's positions
// and weights and the next group's LDS words are in flight while the current
// ones are used.  Against sub-blocks of 4^3 cells with a sum, a compare, a
// select and two products per pair (half tiles, three waves per SIMD): 2M
// trajectories on 128^3 cells 4.79 -> 3.8 ms (24.5 TFLOP/s of the 15 flops
// per included pair), 32.8M on 256^3 272 -> 198 ms (40 TFLOP/s).
//
// SPLIT: the workgroup takes the chunks of one of those four waves, number
// `share`, and writes its sums of the tile to `part` (k_split_sum adds them).  Its
// waves scan that one's chunks together and sum 64 candidates each, and the sums of
// every 64 are added in the candidates' order: bit for bit those of the one wave.
template <int MODE, bool COUNT, int PLAN, bool OVERS, bool SPLIT>
__device__ __forceinline__ void gather_planes(const GatherArgs& g, const int tile, const int share, const int shares,
                                              double* part)
{
    using L = PlaneLds;
    constexpr int W = GatherWaves<float, 3>::value, TE = Geo<3>::TE, ZP = TE, C = 4, NA = 5;
    constexpr int NB = L::NB, HZ = ZP / 2, GR = kPlaneRecs;
    constexpr bool kGeneral = MODE == kNwGeneral;
    static_assert(GR * ZP == 16, "one row of lanes per group");
    static_assert(sizeof(L) * W >= sizeof(double) * W * 4 * NA * kWave, "four planes of sums must fit");
    __shared__ std::conditional_t<SPLIT, PlaneSplitLds, PlaneWavesLds> lds;
    __shared__ RunTable runs;
    __shared__ double xcs[3][TE];

    const MeshDev& m = g.m;
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const uint32_t own = SPLIT ? (1u << (ZP / 2)) - 1u : ((1u << (ZP / 2 / shares)) - 1u) << (share * (ZP / 2 / shares));
    int tc[3];
    tc[0] = tile % m.nt[0];
    tc[1] = (tile / m.nt[0]) % m.nt[1];
    tc[2] = tile / (m.nt[0] * m.nt[1]);

    if (threadIdx.x < 3 * TE) {
        const int a = threadIdx.x / TE, p = threadIdx.x % TE;
        const int64_t idx = (int64_t)tc[a] * TE + p;
        xcs[a][p] = idx < m.n[a] ? (kGeneral ? cell_centre(m, a, idx) : uniform_centre(m, a, idx))
                                 : __builtin_nan("");
    }
    if (threadIdx.x >= kWave && threadIdx.x < kWave + kClasses) {
        const int k = threadIdx.x - kWave;
        const uint32_t kb = (uint32_t)k * (uint32_t)m.ntiles;
        int n = 0;
        if (g.bstart[kb] != g.bstart[kb + m.ntiles]) {
            ClassRows cr;
            class_rows<3>(m, tc, k, cr);
            n = cr.nrows * cr.nruns;
            runs.cls[k] = cr;
        }
        int incl = n;
#pragma unroll
        for (int o = 1; o < kClasses; o <<= 1) {
            const int t = __shfl_up(incl, o, kClasses);
            if (k >= o) incl += t;
        }
        runs.base[k + 1] = incl;
        if (k == 0) runs.base[0] = 0;
    }
    const int lx = lane & 7, ly = lane >> 3;
    // Scaled squares: B = 2^bexp takes c^2 to about 2^64, so that differences
    // of scaled sums are 0, negative or far above 1 (bexp is even: 2^(bexp/2)
    // scales 1/h).  cmid: the real number below which (tie: up to which) a sum
    // of two binary32 numbers rounds to at most c^2.
    const float c2 = uniform_value((float)g.cutoff * (float)g.cutoff);
    const int bexp = (64 - (c2 > 0.0f ? ilogbf(c2) : -150)) & ~1;
    const float c2b = uniform_value(ldexpf(c2, bexp));
    const bool tiny = bexp > 100;          // the factor below would be subnormal
    const float ek = uniform_value(ldexpf(-0.72134752044448170368f, tiny ? 0 : -bexp));
    // just below cmid where the tie rounds up, so that a sum equal to it fails
    double cmid = ldexp(0.5 * ((double)c2 + (double)__int_as_float(__float_as_int(c2) + 1)), bexp);
    if (__float_as_int(c2) & 1) cmid = __longlong_as_double(__double_as_longlong(cmid) - 1);
    cmid = uniform_value(cmid);

    __syncthreads();
    double bmid[3], bhalf[3];
    bool faxis[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double f, l;
        if (kGeneral && m.edges[a]) {
            int p1 = TE - 1;
            const int last = (int)(m.n[a] - 1 - (int64_t)tc[a] * TE);
            if (p1 > last) p1 = last;
            f = xcs[a][0];
            l = xcs[a][p1];
        } else {
            const int64_t c0 = (int64_t)tc[a] * TE;
            f = uniform_centre(m, a, c0);
            l = uniform_centre(m, a, c0 + TE - 1);
        }
        bmid[a] = uniform_value(0.5 * (f + l));
        bhalf[a] = uniform_value(0.5 * (l - f));
        faxis[a] = !(m.periodic[a] && 4.0 * bhalf[a] >= m.L[a]);
    }

    F4 acc[ZP];
    float den[ZP];
    double tot[ZP][NA];
    double ptot[2][NA] = {};               // SPLIT: of planes wave and wave + W
    static_assert(ZP == 2 * W, "two planes a wave");
    uint32_t cnt[ZP];
#pragma unroll
    for (int z = 0; z < ZP; ++z) {
        acc[z] = F4{0.f, 0.f, 0.f, 0.f};
        den[z] = 0.f;
        cnt[z] = 0;
#pragma unroll
        for (int k = 0; k < NA; ++k) tot[z][k] = 0.0;
    }
    auto fold = [&]() {
#pragma unroll
        for (int z = 0; z < ZP; ++z) {
            tot[z][0] += (double)den[z];
            den[z] = 0.f;
#pragma unroll
            for (int k = 0; k < C; ++k) tot[z][1 + k] += (double)acc[z][k];
            acc[z] = F4{0.f, 0.f, 0.f, 0.f};
        }
    };
    const uint64_t ltmask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    // ---- one batch of n <= NB candidates of this wave.  Lanes e and e + 32
    // stage record e: the lower half takes x and the first half of the planes,
    // the upper half y and the others (12 positions each).
    auto stage = [&](PlaneGroup* grp, const double4* pos, const float4* was, const float* wbs, int n, uint32_t* reach) {
        const int e = lane & (NB - 1), half = lane / NB;
        PlaneGroup& gp = grp[e / GR];
        const int er = e % GR;
        // least s B of the lane's 8 positions along x or y, largest threshold
        // of its planes by twos
        float smin = r_inf<float>(), thi[2] = {-3.0e38f, -3.0e38f};
        if (e < n) {
            const double4 P = pos[e];
            const bool delta = MODE == FLA_DEPOSIT && P.w < 0.0;
            const double hb = ldexp(delta ? -P.w : P.w, bexp / 2);
            // np positions of axis a from position p0 on: s B and e
            auto axis = [&](int a, double xa, int p0, double mid, double halfw, auto npc, float* sv, float* ev) {
                constexpr int np = decltype(npc)::value;
                double d[np];
#pragma unroll
                for (int q = 0; q < np; ++q) d[q] = xcs[a][p0 + q] - xa;
                if (m.periodic[a]) {
                    // the tile's box bounds the offsets
                    const double dm = fabs(mid - xa) + halfw, La = m.L[a];
                    if (dm > 0.5 * La) {
                        if (dm < La) {
#pragma unroll
                            for (int q = 0; q < np; ++q) {
#pragma clang fp contract(off)
                                const double w = d[q] > 0.0 ? d[q] - La : d[q] + La;
                                d[q] = fabs(d[q]) <= 0.5 * La ? d[q] : w;
                            }
                        } else {
#pragma unroll
                            for (int q = 0; q < np; ++q) d[q] = min_image(d[q], La);
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < np; ++q) {
                    sv[q] = (float)scaled_sq(d[q], hb);
                    ev[q] = __builtin_amdgcn_exp2f((tiny ? ldexpf(sv[q], -bexp) : sv[q]) * ek);
                }
                if (MODE == FLA_DEPOSIT && delta) {
                    // whole amount into the home cell: factor 1 there, 0 elsewhere
                    const int64_t hcell = home_index(m, a, xa);
#pragma unroll
                    for (int q = 0; q < np; ++q) {
                        const bool home = (int64_t)tc[a] * TE + p0 + q == hcell;
                        sv[q] = home ? 0.f : r_inf<float>();
                        ev[q] = home ? 1.f : 0.f;
                    }
                }
            };
            float sv[TE], ev[TE];
            axis(half, half ? P.y : P.x, 0, half ? bmid[1] : bmid[0], 1.001 * (half ? bhalf[1] : bhalf[0]),
                 std::integral_constant<int, TE>{}, sv, ev);
            float4* row = (float4*)(half ? gp.y[er] : gp.x[er]);
#pragma unroll
            for (int q = 0; q < TE; ++q) smin = fminf(smin, sv[q]);   // ignores NaN (a centre beyond the mesh)
#pragma unroll
            for (int q = 0; q < TE; q += 2) row[q / 2] = make_float4(sv[q], ev[q], sv[q + 1], ev[q + 1]);
            axis(2, P.z, half * HZ, bmid[2], 1.001 * bhalf[2], std::integral_constant<int, HZ>{}, sv, ev);
            const float4 wa = was[e];
            float tv[HZ];
#pragma unroll
            for (int q = 0; q < HZ; ++q) {
                // the binary32 number after c^2 (middle) - s_z truncated: the
                // least that s_x + s_y must stay below
                const uint64_t r = __double_as_longlong(cmid - (double)sv[q]);
                const uint32_t tr = __builtin_amdgcn_alignbit((uint32_t)(r >> 32) - (896u << 20), (uint32_t)r, 29);
                tv[q] = sv[q] <= c2b ? __int_as_float((int)(tr + 1)) : -3.0e38f;
            }
#pragma unroll
            for (int q = 0; q < 2; ++q) thi[q] = fmaxf(tv[2 * q], tv[2 * q + 1]);
            float4* td = (float4*)&gp.td[er][half * HZ];
            td[0] = make_float4(tv[0], wa.x * ev[0], tv[1], wa.x * ev[1]);
            td[1] = make_float4(tv[2], wa.x * ev[2], tv[3], wa.x * ev[3]);
            *(float4*)&gp.ez[er][half * HZ] = make_float4(ev[0], ev[1], ev[2], ev[3]);
            if (half) *(float4*)gp.q[er] = make_float4(wa.y, wa.z, wa.w, wbs[e]);
        } else if (e < (n + GR - 1) / GR * GR) {
            // slots that fill up the last group reach nothing
            const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f), none = make_float4(-3.0e38f, 0.f, -3.0e38f, 0.f);
            float4* row = (float4*)(half ? gp.y[er] : gp.x[er]);
#pragma unroll
            for (int q = 0; q < TE / 2; ++q) row[q] = zero;
            float4* td = (float4*)&gp.td[er][half * HZ];
            td[0] = none;
            td[1] = none;
            *(float4*)&gp.ez[er][half * HZ] = zero;
            if (half) *(float4*)gp.q[er] = zero;
        }
        // records that reach planes 2 h and 2 h + 1 (sums of the least terms: no
        // pair is missed), one bit each; lower lanes hold h = 0, 1, upper ones
        // h = 2, 3
        {
            const auto mn = __builtin_amdgcn_permlane32_swap(__float_as_uint(smin), __float_as_uint(smin), false, false);
            const float mxy = __uint_as_float(mn[0]) + __uint_as_float(mn[1]);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint64_t any = __ballot(mxy < thi[q]);
                reach[q] = (uint32_t)any;
                reach[q + 2] = (uint32_t)(any >> 32);
            }
        }
    };
    // ---- sums the n records of staged groups over the planes of `own`
    auto evaluate = [&](const PlaneGroup* grp, int n, uint32_t* reach) {
#pragma unroll
        for (int h = 0; h < ZP / 2; ++h) reach[h] = own >> h & 1 ? reach[h] : 0u;
        // the next group's words are read while the current group is summed
        struct Words {
            float2 td, fx[GR], fy[GR];
            float ez, q;
        };
        auto load = [&](const PlaneGroup& p, Words& w) {
            w.td = (&p.td[0][0])[lane & 15];
            w.ez = (&p.ez[0][0])[lane >> 2];
            w.q = p.q[lane >> 5][lane & 3];
#pragma unroll
            for (int r = 0; r < GR; ++r) {
                w.fx[r] = p.x[r][lx];
                w.fy[r] = p.y[r][ly];
            }
        };
        constexpr int UG = 4;              // groups per step of the loop
        Words w, nx;
        load(grp[0], nx);
#pragma unroll 1
        for (int g0 = 0; g0 * GR < n; g0 += UG) {
            static_for<0, UG>([&](auto gc) {
                constexpr int u = decltype(gc)::value;
                w = nx;
                load(grp[g0 + u + 1], nx);   // past the last group: words that are not used
                const float tz = w.td.x, dz = w.td.y, aw = w.ez * w.q;
                float sxy[GR], exy[GR];
#pragma unroll
                for (int r = 0; r < GR; ++r) {
                    sxy[r] = w.fx[r].x + w.fy[r].x;
                    exy[r] = w.fx[r].y * w.fy[r].y;
                }
                // both records in planes z and z + 1
                auto planes2 = [&](auto zc) {
                    constexpr int z = decltype(zc)::value, j = ZP + z;
                    float a0 = row_bcast<z>(tz) - sxy[0], b0 = row_bcast<z + 1>(tz) - sxy[0];
                    float a1 = row_bcast<j>(tz) - sxy[1], b1 = row_bcast<j + 1>(tz) - sxy[1];
                    if (COUNT) {
                        cnt[z] += (a0 > 0.f ? 1u : 0u) + (a1 > 0.f ? 1u : 0u);
                        cnt[z + 1] += (b0 > 0.f ? 1u : 0u) + (b1 > 0.f ? 1u : 0u);
                    }
                    weigh2<z, z + 1>(a0, b0, exy[0], dz, den[z], den[z + 1]);
                    weigh2<j, j + 1>(a1, b1, exy[1], dz, den[z], den[z + 1]);
                    // the matrix instructions stay together: each costs about
                    // three times its 8 cycles between vector instructions
                    __builtin_amdgcn_sched_barrier(0);
                    acc[z] = __builtin_amdgcn_mfma_f32_4x4x1f32(aw, a0, acc[z], 4, z, 0);
                    acc[z + 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(aw, b0, acc[z + 1], 4, z + 1, 0);
                    acc[z] = __builtin_amdgcn_mfma_f32_4x4x1f32(aw, a1, acc[z], 4, j, 0);
                    acc[z + 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(aw, b1, acc[z + 1], 4, j + 1, 0);
                    __builtin_amdgcn_sched_barrier(0);
                };
                // PLAN: granularity of the skips (a skipped pair only saves
                // additions of zero): 1 two planes, 2 four, 3 all
                constexpr int S = PLAN == 1 ? 2 : PLAN == 2 ? 4 : ZP;
                static_for<0, ZP / S>([&](auto hc) {
                    constexpr int h = decltype(hc)::value;
                    uint32_t any = 0;
#pragma unroll
                    for (int v = 0; v < S / 2; ++v) any |= reach[h * (S / 2) + v];
                    if (any & (((1u << GR) - 1) << (GR * u)))
                        static_for<0, S / 2>([&](auto zc) {
                            planes2(std::integral_constant<int, S * h + 2 * decltype(zc)::value>{});
                        });
                });
            });
#pragma unroll
            for (int h = 0; h < ZP / 2; ++h) reach[h] >>= GR * UG;
        }
    };

    // ---- scan.  Lane l holds run l of the current 64 runs: records s0 to s1
    // and its first chunk; chunk c, c + CS, ... are this wave's.
    constexpr int CS = SPLIT ? W * W : W;
    const int nrun = runs.base[kClasses];
    auto run_of = [&](int f, uint32_t& a0, uint32_t& a1) {
        a0 = a1 = 0;
        if (f >= nrun) return;
        int k = 0;
        while (runs.base[k + 1] <= f) ++k;
        const ClassRows& cr = runs.cls[k];
        const int j = f - runs.base[k];
        const int q = cr.nruns == 2 ? j & 1 : 0;
        const uint32_t rb = row_bucket<3>(m, cr, cr.nruns == 2 ? j >> 1 : j);
        a0 = g.bstart[rb + cr.runs[q][0]];
        a1 = g.bstart[rb + cr.runs[q][1] + 1];
    };
    uint32_t s0 = 0, s1 = 0, first = 0, s0n, s1n;
    int f0 = 0;
    uint32_t c = SPLIT ? (uint32_t)(share + W * wave) : (uint32_t)wave, nchunk = 0;
    run_of(lane, s0n, s1n);
    double4 Pn = make_double4(0, 0, 0, 0);
    float4 wan = make_float4(0, 0, 0, 0);
    float wbn = 0.f;
    bool okn = false;
    int ncand = 0, nfold = 0;
    for (bool more = true; more;) {
        const double4 P = Pn;
        const float4 wa = wan;
        const float wb = wbn;
        const bool inr = okn;
        // the next chunk, if there is one
        okn = false;
        while (c >= nchunk) {
            c -= nchunk;
            nchunk = 0;
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
            first = incl - nc;
            nchunk = __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        if (more) {
            const int j = __popcll(__ballot(first <= c)) - 1;
            const uint32_t p = __builtin_amdgcn_readlane(s0, j) + (c - __builtin_amdgcn_readlane(first, j)) * kWave + lane;
            okn = p < __builtin_amdgcn_readlane(s1, j);
            c += CS;
            if (okn) {
                Pn = g.rpos[p];
                const float* w = (const float*)g.rw + (size_t)p * kRecW;
                wan = *(const float4*)w;
                wbn = w[4];
            }
        }
        const bool ok = inr && near_tile<MODE == FLA_DEPOSIT>(m, P, tc, bmid, bhalf, faxis, g.filt2);
        const uint64_t bal = __ballot(ok);
        if constexpr (SPLIT) {
            // the waves' candidates in the order of their chunks
            if (lane == 0) {
                lds.cnt[wave] = __popcll(bal);
                lds.more[wave] = more;
            }
            __syncthreads();
            int at = ncand + __popcll(bal & ltmask);
            more = false;
#pragma unroll
            for (int t = 0; t < W; ++t) {
                const int ct = __builtin_amdgcn_readfirstlane(lds.cnt[t]);
                at += t < wave ? ct : 0;
                ncand += ct;
                more = more || __builtin_amdgcn_readfirstlane(lds.more[t]) != 0;
            }
            if (ok) {
                lds.pos[at] = P;
                lds.wa[at] = wa;
                lds.wb[at] = wb;
            }
            __syncthreads();
            while (ncand >= (more ? W * kWave : 1)) {
                // each wave sums 64 records over all planes, as one wave sums them
                // between two folds
                const int n = ncand < W * kWave ? ncand : W * kWave;
#pragma unroll 1
                for (int o = wave * kWave; o < (wave + 1) * kWave && o < n; o += NB) {
                    const int nu = n - o < NB ? n - o : NB;
                    uint32_t reach[ZP / 2];
                    wave_sync();
                    stage(lds.grp[wave], lds.pos + o, lds.wa + o, lds.wb + o, nu, reach);
                    wave_sync();
                    evaluate(lds.grp[wave], nu, reach);
                }
                // their sums, in the order of the records, to those of planes wave
                // and wave + 4
                float* ex = reinterpret_cast<float*>(lds.grp);   // [wave][plane][k][lane]
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    __syncthreads();
#pragma unroll
                    for (int u = 0; u < W; ++u) {
                        float* e = ex + (wave * W + u) * NA * kWave + lane;
                        e[0] = den[W * h + u];
#pragma unroll
                        for (int k = 0; k < C; ++k) e[(1 + k) * kWave] = acc[W * h + u][k];
                        den[W * h + u] = 0.f;
                        acc[W * h + u] = F4{0.f, 0.f, 0.f, 0.f};
                    }
                    __syncthreads();
#pragma unroll
                    for (int v = 0; v < W; ++v)
#pragma unroll
                        for (int k = 0; k < NA; ++k)
                            ptot[h][k] += (double)ex[((v * W + wave) * NA + k) * kWave + lane];
                }
                const int rem = ncand - n, tid = threadIdx.x, from = n + (tid < rem ? tid : 0);
                const double4 mp = lds.pos[from];
                const float4 ma = lds.wa[from];
                const float mb = lds.wb[from];
                __syncthreads();
                if (tid < rem) {
                    lds.pos[tid] = mp;
                    lds.wa[tid] = ma;
                    lds.wb[tid] = mb;
                }
                __syncthreads();
                ncand = rem;
            }
        } else {
            L& my = lds.w[wave];
            if (ok) {
                const int at = ncand + __popcll(bal & ltmask);
                my.pos[at] = P;
                my.wa[at] = wa;
                my.wb[at] = wb;
            }
            ncand += __popcll(bal);
            while (ncand >= (more ? NB : 1)) {
                const int n = ncand < NB ? ncand : NB;
                uint32_t reach[ZP / 2];
                wave_sync();
                stage(my.grp, my.pos, my.wa, my.wb, n, reach);
                wave_sync();
                evaluate(my.grp, n, reach);
                wave_sync();
                // binary32 partial sums run over at most 64 records
                if (++nfold == kWave / NB) {
                    fold();
                    nfold = 0;
                }
                const int rem = ncand - n;
                if (rem > 0) {
                    const int at = n + (lane < rem ? lane : 0);
                    const double4 mp = my.pos[at];
                    const float4 ma = my.wa[at];
                    const float mb = my.wb[at];
                    wave_sync();
                    if (lane < rem) {
                        my.pos[lane] = mp;
                        my.wa[lane] = ma;
                        my.wb[lane] = mb;
                    }
                }
                ncand = rem;
            }
        }
    }
    if (!SPLIT) fold();

    const int64_t cx = (int64_t)tc[0] * TE + lx, cy = (int64_t)tc[1] * TE + ly;
    const bool in_xy = cx < m.n[0] && cy < m.n[1];
    if constexpr (SPLIT) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < NA; ++k) part[((W * h + wave) * NA + k) * kWave + lane] = ptot[h][k];
    } else {
        // ---- the waves' sums, four planes at a time through LDS, added in wave
        // order
        double* red = reinterpret_cast<double*>(&lds);   // [wave][plane][k][lane]
#pragma unroll
        for (int z0 = 0; z0 < ZP; z0 += 4) {
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < NA; ++k) red[((wave * 4 + u) * NA + k) * kWave + lane] = tot[z0 + u][k];
            __syncthreads();
            const int64_t cz = (int64_t)tc[2] * TE + z0 + wave;
            if (in_xy && cz < m.n[2] && (own >> ((z0 + wave) / 2) & 1)) {
                double sum[NA];
#pragma unroll
                for (int k = 0; k < NA; ++k) {
                    double a = 0.0;
#pragma unroll
                    for (int v = 0; v < W; ++v) a += red[((v * 4 + wave) * NA + k) * kWave + lane];
                    sum[k] = a;
                }
                write_cell<MODE>(g, cx + (int64_t)m.n[0] * (cy + (int64_t)m.n[1] * cz), sum);
            }
        }
    }
    if (OVERS && g.stats[ST_OVER])
        for (int z = wave; z < ZP; z += W) {
            const int64_t ci[3] = {cx, cy, (int64_t)tc[2] * TE + z};
            if (!(own >> (z / 2) & 1)) continue;
            add_overs<float, 3, MODE>(g, tc, lane, ci, cx + (int64_t)m.n[0] * (cy + (int64_t)m.n[1] * ci[2]),
                                      in_xy && ci[2] < m.n[2]);
        }
    if (COUNT) {
        // every wave holds counts for all of the workgroup's cells; integer
        // sums do not depend on the order of the atomic additions
        unsigned long long npairs = 0;
#pragma unroll
        for (int z = 0; z < ZP; ++z) {
            if (!(own >> (z / 2) & 1)) continue;
            npairs += cnt[z];
            const int64_t cz = (int64_t)tc[2] * TE + z;
            if (g.pairs && cnt[z] && in_xy && cz < m.n[2])
                atomicAdd(&g.pairs[cx + (int64_t)m.n[0] * (cy + (int64_t)m.n[1] * cz)], cnt[z]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) npairs += __shfl_xor(npairs, o, kWave);
        if (lane == 0 && npairs) atomicAdd(&g.stats[ST_PAIRS], npairs);
    }
}

// The work of one workgroup: the sub-blocks of its share (every one
// where `shares` is 1) of part `work % TP` of tile `work / TP` of the mesh of g.
template <typename R, int D, int MODE, bool COUNT, int PLAN, int TP, bool OVERS>
__device__ __forceinline__ void gather_tile(const GatherArgs& g, const int work, const int share, const int shares)
{
    constexpr int kGatherWaves = GatherWaves<R, D>::value;
    using G = Geo<D>;
    constexpr int TE = G::TE, SB = G::SB, NSB = G::NSB / TP, C = D + 1, NA = C + 1;
    constexpr int NB = GatherLds<R, D, TP>::NB, LPR = GatherLds<R, D, TP>::LPR;
    constexpr int NT = GatherLds<R, D, TP>::NT;
    constexpr bool kComp = sizeof(R) == 4;
    using R4 = typename V4<R>::T;
    using R2 = typename V2<R>::T;
    using L = GatherLds<R, D, TP>;
    static_assert(sizeof(L) * kGatherWaves >= sizeof(R) * kGatherWaves * NSB * NA * kWave,
                  "reduction buffer must fit in the staging space");
    __shared__ L lds[kGatherWaves];
    __shared__ double xcs[D][TE];

    const int own = ((1 << (NSB / shares)) - 1) << (share * (NSB / shares));

    const MeshDev& m = g.m;
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
    L& my = lds[wave];
    const int tile = work / TP;
    const int soff = (TP == 2) ? (work % TP) * SB : 0;   // first owned cell of the tile along x
    int tc[3];
    tc[0] = tile % m.nt[0];
    tc[1] = (tile / m.nt[0]) % m.nt[1];
    tc[2] = (D == 3) ? tile / (m.nt[0] * m.nt[1]) : 0;
    // a part lying wholly beyond the mesh has no cells (uniform over the workgroup)
    if (TP == 2 && (int64_t)tc[0] * TE + soff >= m.n[0]) return;

    // kNwGeneral takes any mesh (rectilinear axes read their edges); the
    // other modes assume uniform axes and compute the centres
    constexpr bool kGeneral = MODE == kNwGeneral;
    if (threadIdx.x < D * TE) {
        int a = threadIdx.x / TE, p = threadIdx.x % TE;
        int64_t idx = (int64_t)tc[a] * TE + p;
        xcs[a][p] = idx < m.n[a] ? (kGeneral ? cell_centre(m, a, idx) : uniform_centre(m, a, idx))
                                 : __builtin_nan("");
    }
    int lc[3];
    if (D == 3) {
        lc[0] = lane & 3;
        lc[1] = (lane >> 2) & 3;
        lc[2] = lane >> 4;
    } else {
        lc[0] = lane & 7;
        lc[1] = lane >> 3;
        lc[2] = 0;
    }
    R c2;
    {
        R c = (R)g.cutoff;
        c2 = uniform_value(c * c);
    }
    // conservative tile box of cell centres for the candidate filter: on
    // uniform axes from the formula (extrapolated past the last cell), on
    // rectilinear axes from the existing centres in the table.  (The box
    // decides which records are staged, hence where the binary32 partial
    // sums are folded: a uniform axis gets the same box in either mode, so
    // a uniform snapshot of a batch that also holds rectilinear ones keeps
    // the bits of its own call.)
    if (kGeneral) __syncthreads();
    double bmid[3] = {0, 0, 0}, bhalf[3] = {0, 0, 0};
    bool faxis[3] = {false, false, false};
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const bool one = TP == 2 && a == 0;
        double f, l;
        if (kGeneral && m.edges[a]) {
            const int p0 = one ? soff : 0;
            int p1 = p0 + (one ? SB : TE) - 1;
            const int last = (int)(m.n[a] - 1 - (int64_t)tc[a] * TE);
            if (p1 > last) p1 = last;
            f = xcs[a][p0];
            l = xcs[a][p1];
        } else {
            const int64_t c0 = (int64_t)tc[a] * TE + (one ? soff : 0);
            f = uniform_centre(m, a, c0);
            l = uniform_centre(m, a, c0 + (one ? SB : TE) - 1);
        }
        bmid[a] = uniform_value(0.5 * (f + l));
        bhalf[a] = uniform_value(0.5 * (l - f));
        faxis[a] = !(m.periodic[a] && 4.0 * bhalf[a] >= m.L[a]);
    }

    // Binary32: the C source channels of a sub-block are accumulated on the
    // matrix unit (see `sub` below), the denominator on the vector unit.
    constexpr bool kMfma = sizeof(R) == 4;
    R part[NSB][NA];
    R hi[NSB][NA];
    R lo[NSB][NA];
    F4 acc[NSB];
#pragma unroll
    for (int b = 0; b < NSB; ++b) {
        acc[b] = F4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            part[b][k] = 0;
            hi[b][k] = 0;
            lo[b][k] = 0;
        }
    }
    // included pairs per sub-block of this lane (counted calls only)
    uint32_t cntb[NSB];
#pragma unroll
    for (int b = 0; b < NSB; ++b) cntb[b] = 0;
    const uint64_t ltmask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    __syncthreads();

    // ---- one batch of n <= NB staged candidates of this wave
    auto process = [&](int n) {
        wave_sync();
        const int rec = lane % NB;
        if (rec < n) {
            uint32_t p = my.cand[rec];
            double4 P = g.rpos[p];
            const R* w = (const R*)g.rw + (size_t)p * kRecW;
#pragma unroll
            for (int k = 0; k < NA; ++k) my.wts[rec][k] = w[k];
            my.mask[rec] =
                stage_record<R, D, TP>(m, xcs, tc, soff, P, c2, LPR == 2 ? lane / NB : 0, my.tab[rec], my.tabs[rec]);
        }
        wave_sync();
        // every lane keeps the mask of one staged record (read with readlane,
        // no LDS round trip)
        const int maskv = (lane < n) ? my.mask[lane < NB ? lane : 0] : 0;
        // one sub-block of one record: the per-pair inclusion test, then the
        // denominator multiply-add and the C channel multiply-adds.  In
        // binary32 the channels go to one v_mfma_f32_4x4x1_16b_f32: with A
        // broadcast from lanes 0..3 (cbsz 4, abid 0) it forms, in every
        // 4-lane block, the outer product of the record's channel weights
        // (lane m of A holds q_m/h) and the four lanes' kernel weights (B),
        // so that register k of lane l accumulates channel k of the lane's
        // cell: the layout of the vector path, with 4 multiply-adds per lane
        // moved off the vector unit.
        auto sub = [&](int b, const R4* t, const R2& ts, const R* wv, float wq) {
            R s, ew;
            if constexpr (TP == 2) {
                // x split: ts holds the owned half of x, t the y and z tables
                const int by = b & 1, bz = (b >> 1) & 1;
                s = ts.x + (by ? t[0].z : t[0].x);
                ew = ts.y * (by ? t[0].w : t[0].y);
                if constexpr (D == 3) {
                    s = s + (bz ? t[1].z : t[1].x);
                    ew = ew * (bz ? t[1].w : t[1].y);
                }
            } else {
                const int bx = b & 1, by = (b >> 1) & 1, bz = (b >> 2) & 1;
                s = (bx ? t[0].z : t[0].x) + (by ? t[1].z : t[1].x);
                ew = (bx ? t[0].w : t[0].y) * (by ? t[1].w : t[1].y);
                if constexpr (D == 3) {
                    s = s + (bz ? t[2].z : t[2].x);
                    ew = ew * (bz ? t[2].w : t[2].y);
                }
            }
            bool in = s <= c2;
            ew = in ? ew : (R)0;
            if constexpr (kMfma) {
                part[b][0] = fma(ew, wv[0], part[b][0]);
                acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(wq, (float)ew, acc[b], 4, 0, 0);
            } else {
#pragma unroll
                for (int k = 0; k < NA; ++k) part[b][k] = fma(ew, wv[k], part[b][k]);
            }
            if (COUNT) cntb[b] += in ? 1u : 0u;
        };
        // PLAN sets the granularity of the wave-uniform skips of a record that
        // reaches the workgroup's part: 0 one branch per sub-block, 1 per
        // pair of sub-blocks along z (3-D), 2 per half tile (whole tiles
        // have 8 sub-blocks; with the x split the part has 4, so 2 and 3
        // coincide), 3 none (every sub-block evaluated, masked by the pair
        // test); in 2-D, 1 and 2 evaluate the whole tile.  All plans add the
        // same products; a skipped sub-block only saves additions of zero.
        auto accumulate = [&](int e, const R4* t, const R2& ts, const R* wv, float wq) {
            const int mk = __builtin_amdgcn_readlane(maskv, e) & own;
            if (mk == 0) return;
            if (PLAN == 3 || (D == 2 && PLAN != 0) || (PLAN == 2 && NSB == 4)) {
#pragma unroll
                for (int b = 0; b < NSB; ++b) sub(b, t, ts, wv, wq);
            } else if (PLAN == 2) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    if (mk & (0x0F << (4 * h))) {
#pragma unroll
                        for (int b = 4 * h; b < 4 * h + 4; ++b) sub(b, t, ts, wv, wq);
                    }
            } else if (PLAN == 1) {
#pragma unroll
                for (int q = 0; q < NSB / 2; ++q)
                    if (mk & (((1 << (NSB / 2)) | 1) << q)) {
                        sub(q, t, ts, wv, wq);
                        sub(q + NSB / 2, t, ts, wv, wq);
                    }
            } else {
#pragma unroll
                for (int b = 0; b < NSB; ++b)
                    if (mk & (1 << b)) sub(b, t, ts, wv, wq);
            }
        };
        // weights of staged record e: {1/h, q/h ...} on every lane, and, for
        // the matrix unit, q_m/h on lane m < C of each 4-lane group (0 on the
        // others)
        const int wm = lane & 3;
        auto load_w = [&](int e, R* w, float& wq) {
            if constexpr (kMfma) {
                w[0] = my.wts[e][0];
                wq = wm < C ? (float)my.wts[e][1 + (wm < C ? wm : 0)] : 0.0f;
            } else {
#pragma unroll
                for (int k = 0; k < NA; ++k) w[k] = my.wts[e][k];
                wq = 0.0f;
            }
        };
        // factors of staged record e at the lane's cells
        auto load_t = [&](int e, R4* t, R2& ts) {
#pragma unroll
            for (int a = 0; a < NT; ++a) t[a] = my.tab[e][a][lc[TP == 2 ? a + 1 : a]];
            if (TP == 2) ts = my.tabs[e][lc[0]];
        };
        R4 tA[NT], tB[NT];
        R2 hA, hB;
        R wA[NA], wB[NA];
        float qA, qB;
        {
            // one record at a time; the factors of the next record are read
            // while the current one is accumulated
            load_t(0, tA, hA);
            load_w(0, wA, qA);
            for (int e = 0; e < n; e += 2) {
                if (e + 1 < n) {
                    load_t(e + 1, tB, hB);
                    load_w(e + 1, wB, qB);
                }
                accumulate(e, tA, hA, wA, qA);
                if (e + 1 >= n) break;
                if (e + 2 < n) {
                    load_t(e + 2, tA, hA);
                    load_w(e + 2, wA, qA);
                }
                accumulate(e + 1, tB, hB, wB, qB);
            }
        }
        if (kComp) {
#pragma unroll
            for (int b = 0; b < NSB; ++b) {
                two_sum_acc(hi[b][0], lo[b][0], part[b][0]);
                part[b][0] = 0;
#pragma unroll
                for (int k = 1; k < NA; ++k) {
                    two_sum_acc(hi[b][k], lo[b][k], kMfma ? (R)acc[b][k - 1] : part[b][k]);
                    part[b][k] = 0;
                }
                acc[b] = F4{0.f, 0.f, 0.f, 0.f};
            }
        }
        wave_sync();
    };

    int ncand = 0;
    uint32_t chunk = 0;          // chunks of 64 candidates are dealt round-robin to the waves
    for_each_run<D>(m, g.bstart, tc, lane, [&](const uint32_t s0, const uint32_t s1) {
        // this wave's chunks of the run: base0, base0 + 4*64, ...
        const uint32_t nch = (s1 - s0 + kWave - 1) / kWave;
        const uint32_t first = (uint32_t)((wave - (int)(chunk % kGatherWaves) + kGatherWaves) % kGatherWaves);
        chunk += nch;
        double4 Pn = make_double4(0, 0, 0, 0);
        if (first < nch && s0 + first * kWave + lane < s1) Pn = g.rpos[s0 + first * kWave + lane];
        for (uint32_t c = first; c < nch; c += kGatherWaves) {
            const uint32_t base = s0 + c * kWave;
            uint32_t p = base + lane;
            double4 P = Pn;
            const uint32_t pn = base + kGatherWaves * kWave + lane;
            if (pn < s1) Pn = g.rpos[pn];
            const bool ok = p < s1 && candidate_ok<D>(m, P, tc, bmid, bhalf, faxis, g.filt2);
            uint64_t bal = __ballot(ok);
            if (ok) my.cand[ncand + __popcll(bal & ltmask)] = p;
            ncand += __popcll(bal);
            while (ncand >= NB) {
                process(NB);
                int rem = ncand - NB;
                uint32_t mv = (lane < rem) ? my.cand[NB + lane] : 0u;
                wave_sync();
                if (lane < rem) my.cand[lane] = mv;
                ncand = rem;
            }
        }
    });
    if (ncand > 0) process(ncand);

    // ---- fixed-order reduction of the waves' partial sums through LDS
    __syncthreads();
    R* red = reinterpret_cast<R*>(lds);   // [wave][b][k][lane]
#pragma unroll
    for (int b = 0; b < NSB; ++b)
#pragma unroll
        for (int k = 0; k < NA; ++k)
            red[((wave * NSB + b) * NA + k) * kWave + lane] = kComp ? hi[b][k] + lo[b][k] : part[b][k];
    __syncthreads();

    // linear index of the lane's cell in sub-block b; false beyond the mesh
    auto cell_of = [&](int b, int64_t* cidx, int64_t& lin) {
        bool inside = true;
        cidx[2] = 0;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            int half;
            if (TP == 2)
                half = a == 0 ? soff : ((b >> (a > 0 ? a - 1 : 0)) & 1) * SB;
            else
                half = ((b >> a) & 1) * SB;
            cidx[a] = (int64_t)tc[a] * TE + half + lc[a];
            inside = inside && cidx[a] < m.n[a];
        }
        lin = cidx[0] + (int64_t)m.n[0] * (cidx[1] + (int64_t)m.n[1] * cidx[2]);
        return inside;
    };

    // ---- epilogue: divide (NW) or scale by 1/V_c (deposition), sign, scale
    for (int b = wave; b < NSB; b += kGatherWaves) {
        int64_t lin, ci[3];
        if (!(own >> b & 1) || !cell_of(b, ci, lin)) continue;
        double tot[NA];
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            double acc = 0.0;
            for (int v = 0; v < kGatherWaves; ++v) acc += (double)red[((v * NSB + b) * NA + k) * kWave + lane];
            tot[k] = acc;
        }
        double den = tot[0];
        double cs = g.cell_scale ? (double)((const R*)g.cell_scale)[lin] : 1.0;
        double f = -g.scale * cs;
#pragma unroll
        for (int k = 0; k < C; ++k) {
            double val;
            if (MODE != FLA_DEPOSIT)
                val = (den > 0.0) ? f * (tot[1 + k] / den) : 0.0;
            else
                val = f * tot[1 + k] / m.vol;
            ((R*)g.out[k])[lin] = (R)val;
        }
        if (g.den) ((R*)g.den)[lin] = (R)den;
    }
    if (OVERS && g.stats[ST_OVER])
        for (int b = wave; b < NSB; b += kGatherWaves) {
            if (!(own >> b & 1)) continue;
            int64_t lin, ci[3];
            const bool inside = cell_of(b, ci, lin);
            add_overs<R, D, MODE>(g, tc, lane, ci, lin, inside);
        }
    if (COUNT) {
        // every wave holds counts for all of the workgroup's cells (the
        // waves split the candidates, not the cells); integer sums do not
        // depend on the order of the atomic additions
        unsigned long long npairs = 0;
#pragma unroll
        for (int b = 0; b < NSB; ++b) {
            if (!(own >> b & 1)) continue;
            npairs += cntb[b];
            int64_t lin, ci[3];
            if (g.pairs && cntb[b] && cell_of(b, ci, lin)) atomicAdd(&g.pairs[lin], cntb[b]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) npairs += __shfl_xor(npairs, o, kWave);
        if (lane == 0 && npairs) atomicAdd(&g.stats[ST_PAIRS], npairs);
    }
}

// Share `share` of `shares` of work item `work`, by the body of its precision
// and dimension.  OVERS: with the weights beyond the range of R (add_overs),
// which the persistent gathers and gather_planes leave to a launch of their own
// (k_gather_overs): in them they cost 5 to 13%, by the registers alone.
template <typename R, int D> constexpr bool kPlanes = sizeof(R) == 4 && D == 3;   // gather_planes
template <typename R, int D, int MODE, bool COUNT, int PLAN, int TP, bool OVERS>
__device__ __forceinline__ void gather_work(const GatherArgs& g, const int work, const int share = 0,
                                            const int shares = 1)
{
    if constexpr (kPlanes<R, D>)
        gather_planes<MODE, COUNT, PLAN, OVERS, false>(g, work, share, shares, nullptr);
    else
        gather_tile<R, D, MODE, COUNT, PLAN, TP, OVERS>(g, work, share, shares);
}

// Slot b of the launch belongs to XCD b % kXcds and computes the work item
// order[xcd_remap(b)] (the heaviest items of each XCD first).  The workgroups
// (as many as the compute units hold) take their XCD's slots x, x + kXcds,
// ... in order from that XCD's counter until they pass the end, so a
// workgroup that finishes early starts the next item at once (128^3: 4.93 ->
// 4.80 ms).  Which workgroup computes an item does not change its results.
template <typename R, int D, int MODE, bool COUNT, int PLAN, int TP>
static __global__ __launch_bounds__((kWave * GatherWaves<R, D>::value), (GatherOcc<R, D, TP>::value)) void k_gather(GatherArgs g)
{
    const int total = g.m.ntiles * TP;
    __shared__ int s_slot;
    const int x = blockIdx.x % kXcds;
    for (;;) {
        __syncthreads();   // every lane has read the previous slot
        if (threadIdx.x == 0) s_slot = x + kXcds * (int)atomicAdd(&g.queue[x], 1u);
        __syncthreads();
        const int slot = s_slot;
        if (slot >= total) break;
        int w = xcd_remap(slot, total);
        w = g.order[w];
        gather_work<R, D, MODE, COUNT, PLAN, TP, false>(g, w);
    }
}

// add_overs for every tile, one workgroup each.
template <typename R, int D, int MODE>
__device__ __forceinline__ void overs_tile(const GatherArgs& g, const int tile)
{
    constexpr int TE = Geo<D>::TE, cells = D == 3 ? TE * TE * TE : TE * TE;
    const MeshDev& m = g.m;
    const int tc[3] = {tile % m.nt[0], (tile / m.nt[0]) % m.nt[1], D == 3 ? tile / (m.nt[0] * m.nt[1]) : 0};
    for (int i = threadIdx.x; i < cells; i += 256) {      // whole waves
        const int q[3] = {i % TE, (i / TE) % TE, i / (TE * TE)};
        int64_t ci[3] = {0, 0, 0};
        bool inside = true;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            ci[a] = (int64_t)tc[a] * TE + q[a];
            inside = inside && ci[a] < m.n[a];
        }
        add_overs<R, D, MODE>(g, tc, threadIdx.x % kWave, ci, ci[0] + (int64_t)m.n[0] * (ci[1] + (int64_t)m.n[1] * ci[2]),
                              inside);
    }
}
template <typename R, int D, int MODE>
static __global__ __launch_bounds__(256) void k_gather_overs(GatherArgs g)
{
    if (!g.stats[ST_OVER]) return;
    overs_tile<R, D, MODE>(g, blockIdx.x);
}

// Every share of every part of every tile with a workgroup of its own (small
// meshes).  A kernel beside the one above, which pays 2% for the shares on the
// 128^3 case; the plan that skips most finely, since a share skips the cells of
// the others.
template <typename R, int D, int MODE, bool COUNT, int TP>
static __global__ __launch_bounds__((kWave * GatherWaves<R, D>::value), (GatherOcc<R, D, TP>::value)) void k_gather_small(
    GatherArgs g, int shares)
{
    const int w = xcd_remap(blockIdx.x, g.m.ntiles * TP * shares);
    gather_work<R, D, MODE, COUNT, (sizeof(R) == 4 && D == 3 ? 1 : 0), TP, !kPlanes<R, D>>(g, w / shares, w % shares, shares);
}

// Binary32 3-D meshes of few tiles with many records each: four workgroups to a
// tile, each with the chunks of one of the four waves that the tile would have (so
// the sums keep their bits), and its sums in part, 20 KiB a workgroup: those of
// waves 0 and 1 of all tiles in part01, of 2 and 3 in part23.
constexpr int kSplitWords = 8 * 5 * kWave;
template <int MODE, bool COUNT>
static __global__ __launch_bounds__(256, 2) void k_gather_split(GatherArgs g, double* part01, double* part23)
{
    const int w = xcd_remap(blockIdx.x, g.m.ntiles * 4), tile = w / 4, v = w % 4;
    double* part = (v < 2 ? part01 : part23) + (size_t)(tile * 2 + v % 2) * kSplitWords;
    gather_planes<MODE, COUNT, 1, false, true>(g, tile, v, 1, part);
}
// The fields from those sums, added in the order of the waves: four planes of a
// tile to a workgroup.
template <int MODE>
__device__ __forceinline__ void split_sum(const GatherArgs& g, const int tile, const int at, const double* part01,
                                          const double* part23)
{
    constexpr int TE = Geo<3>::TE, NA = 5;
    const MeshDev& m = g.m;
    const int lane = threadIdx.x % kWave, z = blockIdx.x % 2 * 4 + threadIdx.x / kWave;
    const int64_t cx = (int64_t)(tile % m.nt[0]) * TE + lane % TE;
    const int64_t cy = (int64_t)((tile / m.nt[0]) % m.nt[1]) * TE + lane / TE;
    const int64_t cz = (int64_t)(tile / (m.nt[0] * m.nt[1])) * TE + z;
    if (cx >= m.n[0] || cy >= m.n[1] || cz >= m.n[2]) return;
    double sum[NA];
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        double a = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            a += ((v < 2 ? part01 : part23) + (size_t)(at * 2 + v % 2) * kSplitWords)[(z * NA + k) * kWave + lane];
        sum[k] = a;
    }
    write_cell<MODE>(g, cx + (int64_t)m.n[0] * (cy + (int64_t)m.n[1] * cz), sum);
}
template <int MODE>
static __global__ __launch_bounds__(256) void k_split_sum(GatherArgs g, const double* part01, const double* part23)
{
    split_sum<MODE>(g, blockIdx.x / 2, blockIdx.x / 2, part01, part23);
}

// Estimated work of every tile: the number of candidate records its scan
// visits (the bucket sizes over its class neighbourhoods).  One wave per
// tile, a row per lane.
template <int D>
static __global__ __launch_bounds__(256) void k_tile_cost(GatherArgs g)
{
    const MeshDev& m = g.m;
    const int tile = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kWave);
    const int lane = threadIdx.x % kWave;
    if (tile >= m.ntiles) return;   // whole waves
    int tc[3];
    tc[0] = tile % m.nt[0];
    tc[1] = (tile / m.nt[0]) % m.nt[1];
    tc[2] = (D == 3) ? tile / (m.nt[0] * m.nt[1]) : 0;
    uint32_t c = 0;
    for (int k = 0; k < kClasses; ++k) {
        const uint32_t kb = (uint32_t)k * (uint32_t)m.ntiles;
        if (g.bstart[kb] == g.bstart[kb + m.ntiles]) continue;
        ClassRows cr;
        class_rows<D>(m, tc, k, cr);
        for (int row = lane; row < cr.nrows; row += kWave) {
            const uint32_t rowb = row_bucket<D>(m, cr, row);
            for (int q = 0; q < cr.nruns; ++q)
                c += g.bstart[rowb + cr.runs[q][1] + 1] - g.bstart[rowb + cr.runs[q][0]];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if (lane == 0) g.tile_cost[tile] = c;
}

// Work order of the single-snapshot gather.  Workgroups are dealt
// round-robin over the XCDs and xcd_remap gives each XCD a contiguous range
// of slots; inside its range (one workgroup of this kernel per XCD) the work
// units are placed in descending classes of their tile's cost (four classes
// per power of two), so that the heaviest tiles start first and the light
// ones fill the end.  The order inside a class is immaterial: a work unit's
// results do not depend on the slot that computes it.
constexpr int kOrderBins = 33 * 4;
static __global__ __launch_bounds__(1024) void k_tile_order(const uint32_t* __restrict__ cost, int nunits, int zs,
                                                     int* __restrict__ order, uint32_t* __restrict__ queue)
{
    __shared__ uint32_t cnt[kOrderBins];
    const int x = blockIdx.x;
    if (threadIdx.x == 0) queue[x] = 0;    // the gather's counter of this XCD
    const int q = nunits / kXcds, rem = nunits % kXcds;
    const int s0 = x * q + (x < rem ? x : rem), n = q + (x < rem ? 1 : 0);
    auto bin = [](uint32_t c) {
        const int b = 32 - __clz(c);   // 0 for c = 0, else 1 + floor(log2 c)
        const int sub = b >= 3 ? (int)((c >> (b - 3)) & 3u) : 0;
        return b * 4 + sub;
    };
    for (int i = threadIdx.x; i < kOrderBins; i += blockDim.x) cnt[i] = 0;
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) atomicAdd(&cnt[bin(cost[(s0 + i) / zs])], 1u);
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int b = kOrderBins - 1; b >= 0; --b) {
            const uint32_t t = cnt[b];
            cnt[b] = acc;
            acc += t;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t pos = atomicAdd(&cnt[bin(cost[(s0 + i) / zs])], 1u);
        order[s0 + pos] = s0 + i;
    }
}

// Work item of workgroup `bid` of a batch of `nwork` items.  Workgroups are
// dealt round-robin over the XCDs in launch order; in every full chunk of
// kXcds * chunk items, XCD x receives the `chunk` consecutive items
// x * chunk ... x * chunk + chunk - 1, so neighbouring tiles of one snapshot
// share an L2 while the chunks still start in work-list order.
static __device__ inline int batch_work_item(int bid, int nwork, int chunk)
{
    const int span = kXcds * chunk;
    const int c = bid / span, off = bid % span;
    if ((c + 1) * span > nwork) return bid;
    return c * span + (off % kXcds) * chunk + off / kXcds;
}

// Last snapshot whose first work item is <= j.
static __device__ inline int batch_snapshot(const BatchItem* __restrict__ items, int nsnap, int j)
{
    int lo = 0, hi = nsnap - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].tile_base <= j)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

template <typename R, int D, int MODE>
static __global__ __launch_bounds__(256) void k_gather_batch_overs(const BatchItem* __restrict__ items, int nsnap)
{
    if (!items[0].g.stats[ST_OVER]) return;    // of the whole call
    const int j = blockIdx.x, i = batch_snapshot(items, nsnap, j);
    overs_tile<R, D, MODE>(items[i].g, j - items[i].tile_base);
}

// k_gather_split and k_split_sum over the tiles of a batch.
template <int MODE, bool COUNT>
static __global__ __launch_bounds__(256, 2) void k_gather_split_batch(const BatchItem* __restrict__ items, int nsnap,
                                                                      double* part01, double* part23)
{
    const int j = blockIdx.x / 4, v = blockIdx.x % 4, i = batch_snapshot(items, nsnap, j);   // heaviest first
    double* part = (v < 2 ? part01 : part23) + (size_t)(j * 2 + v % 2) * kSplitWords;
    gather_planes<MODE, COUNT, 1, false, true>(items[i].g, j - items[i].tile_base, v, 1, part);
}
template <int MODE>
static __global__ __launch_bounds__(256) void k_split_sum_batch(const BatchItem* __restrict__ items, int nsnap,
                                                                const double* part01, const double* part23)
{
    const int j = blockIdx.x / 2, i = batch_snapshot(items, nsnap, j);
    split_sum<MODE>(items[i].g, j - items[i].tile_base, j, part01, part23);
}

// Persistent workgroups over nwork work items of a batch from `first` on, one
// (snapshot, tile part) at a time.  The snapshots are stored in work-list order:
// items[s].tile_base is the first work item of snapshot s.  Slot b of the
// ordered launch (batch_work_item) belongs to XCD b % kXcds; each XCD has
// its own counter (queue[x], zeroed before the launch), from which its
// workgroups take that XCD's slots x, x + kXcds, ... in order until they
// pass the end.  Every item is taken exactly once, by a workgroup of the XCD
// the ordered launch gives it, and a workgroup that finishes early takes the
// next one instead of waiting for the dispatcher (on the 64-snapshot batch
// 37.5 against 38.4 ms).  Which workgroup computes an item does not change
// its results.
template <typename R, int D, int MODE, bool COUNT, int PLAN, int TP>
static __global__ __launch_bounds__((kWave * GatherWaves<R, D>::value), (GatherOcc<R, D, TP>::value)) void k_gather_batch(
    const BatchItem* __restrict__ items, int nsnap, int first, int nwork, int chunk, uint32_t* __restrict__ queue)
{
    __shared__ int s_slot;
    const int total = nwork * TP;
    const int x = blockIdx.x % kXcds;
    for (;;) {
        __syncthreads();   // every lane has read the previous slot
        if (threadIdx.x == 0) s_slot = x + kXcds * (int)atomicAdd(&queue[x], 1u);
        __syncthreads();
        const int slot = s_slot;
        if (slot >= total) break;
        const int u = batch_work_item(slot, total, chunk);
        const int j = first + u / TP;         // tile-level work item
        const int lo = batch_snapshot(items, nsnap, j);
        gather_work<R, D, MODE, COUNT, PLAN, TP, false>(items[lo].g, (j - items[lo].tile_base) * TP + u % TP);
    }
}

// Plan 0 of binary32 in 3-D is plan 1: two planes of two records are the
// finest unit of its skips.
template <typename R, int D> constexpr int finest_plan() { return sizeof(R) == 4 && D == 3 ? 1 : 0; }

template <typename R, int D, int MODE, bool COUNT, int TP>
static void launch_plan(const GatherArgs& g, int plan, dim3 grid, dim3 block, hipStream_t s)
{
    constexpr int kFinest = finest_plan<R, D>();
    switch (plan) {
    case 1: FLA_LAUNCH((k_gather<R, D, MODE, COUNT, 1, TP>), grid, block, 0, s, g); break;
    case 2: FLA_LAUNCH((k_gather<R, D, MODE, COUNT, 2, TP>), grid, block, 0, s, g); break;
    case 3: FLA_LAUNCH((k_gather<R, D, MODE, COUNT, 3, TP>), grid, block, 0, s, g); break;
    default: FLA_LAUNCH((k_gather<R, D, MODE, COUNT, kFinest, TP>), grid, block, 0, s, g); break;
    }
}

// Workgroups that the compute units hold at once (waves per SIMD from the
// register budget, 4 SIMDs per unit).
template <typename R, int D, int TP>
static int64_t resident_workgroups(int ncu)
{
    return (int64_t)(ncu > 0 ? ncu : 1) * GatherOcc<R, D, TP>::value * 4 / GatherWaves<R, D>::value;
}

template <typename R, int D, int MODE, bool COUNT, int TP>
static void launch_batch_plan(const BatchItem* items, int nsnap, int first, int nwork, int chunk, int plan, uint32_t* queue,
                              int ncu, hipStream_t s)
{
    // as many workgroups as the compute units hold, at most one per item
    int64_t nb = resident_workgroups<R, D, TP>(ncu);
    const int64_t total = (int64_t)nwork * TP;
    if (nb > total) nb = total;
    if (nb < 1) nb = 1;
    dim3 grid((unsigned)nb), block(kWave * GatherWaves<R, D>::value);
    constexpr int kFinest = finest_plan<R, D>();
    switch (plan) {
    case 1: FLA_LAUNCH((k_gather_batch<R, D, MODE, COUNT, 1, TP>), grid, block, 0, s, items, nsnap, first, nwork, chunk, queue); break;
    case 2: FLA_LAUNCH((k_gather_batch<R, D, MODE, COUNT, 2, TP>), grid, block, 0, s, items, nsnap, first, nwork, chunk, queue); break;
    case 3: FLA_LAUNCH((k_gather_batch<R, D, MODE, COUNT, 3, TP>), grid, block, 0, s, items, nsnap, first, nwork, chunk, queue); break;
    default: FLA_LAUNCH((k_gather_batch<R, D, MODE, COUNT, kFinest, TP>), grid, block, 0, s, items, nsnap, first, nwork, chunk, queue); break;
    }
}

template <typename R, int D, int TP>
static void launch_batch_shape(const BatchItem* items, int nsnap, int first, int nwork, int chunk, bool count, int plan,
                               bool general, uint32_t* queue, int ncu, hipStream_t s)
{
    if (general) {
        if (count)
            launch_batch_plan<R, D, kNwGeneral, true, TP>(items, nsnap, first, nwork, chunk, plan, queue, ncu, s);
        else
            launch_batch_plan<R, D, kNwGeneral, false, TP>(items, nsnap, first, nwork, chunk, plan, queue, ncu, s);
    } else {
        if (count)
            launch_batch_plan<R, D, FLA_NW, true, TP>(items, nsnap, first, nwork, chunk, plan, queue, ncu, s);
        else
            launch_batch_plan<R, D, FLA_NW, false, TP>(items, nsnap, first, nwork, chunk, plan, queue, ncu, s);
    }
}

// Whether four workgroups to a tile (k_gather_split) take less time than one.  They
// do where compute units would be left idle: up to one tile to a unit always
// (whole calls in binary32, one workgroup or up to four that share a tile's planes,
// against split: 20^3 cells and 1M trajectories 2477 -> 988 us, 40^3 and 1M 1010 ->
// 525, 30^3 and 100k 342 -> 181); above, where the last units' second or third
// tile costs more than the tenth that the exchange of the sums does (343 tiles and
// 1M 733 -> 666, 320 tiles 744 -> 637, but 512 tiles 631 -> 694).  And only where
// the sums, 80 KiB a tile, fit into the spare records: at fewer records a tile
// the scan is short and there is little to share.
static_assert(kSplitRecords * sizeof(double4) >= 2 * kSplitWords * sizeof(double), "the sums fit into the spare records");
template <int MODE> static bool split_pays(int64_t tiles, int64_t records, int ncu)
{
    if (records < kSplitRecords * tiles || tiles > 3 * (int64_t)ncu) return false;
    const int64_t whole = (tiles + ncu - 1) / ncu, quarters = (4 * tiles + ncu - 1) / ncu;
    return whole <= 1 || (MODE == FLA_DEPOSIT ? 10 * quarters <= 40 * whole : 11 * quarters < 40 * whole);
}

// 2-D binary64: whole tiles in place of halves where a tile has few records, since
// each half stages a record's y factors anew and waves of few records idle: 1000^2
// cells with 2001 records 577 -> 354 us, with 200k 399 -> 339; with 250 and more to a
// tile the halves' skips and number win, 300^2 and 200k 213 -> 180.
static bool whole_tiles(int64_t tiles, int64_t records) { return records < 128 * tiles; }

template <int MODE, bool COUNT>
static void launch_split_batch(const BatchItem* items, int nsnap, int nwork, const GatherSpare& spare, hipStream_t s)
{
    FLA_LAUNCH((k_gather_split_batch<MODE, COUNT>), dim3((unsigned)nwork * 4), dim3(256), 0, s, items, nsnap, spare.a,
               spare.b);
    FLA_LAUNCH((k_split_sum_batch<MODE>), dim3((unsigned)nwork * 2), dim3(256), 0, s, items, nsnap,
               (const double*)spare.a, (const double*)spare.b);
}

// plan_code = plan + kGatherPlans * shape (shape 1: whole tiles, 3-D only).  The first nsplit work items, of binary32 3-D snapshots that the caller has found
// heavy, go to four workgroups each.
template <typename R, int D>
hipError_t launch_gather_batch(const BatchItem* items, int nsnap, int nwork, int nsplit, int chunk, bool count,
                               int plan_code, bool general, uint32_t* queue, int ncu, const GatherSpare& spare,
                               hipStream_t s)
{
    if (nwork <= 0) return hipSuccess;
    const int plan = plan_code % kGatherPlans, shape = plan_code / kGatherPlans;
    int first = 0;
    if constexpr (kPlanes<R, D>) {
        if (nsplit > 0) {
            if (general)
                count ? launch_split_batch<kNwGeneral, true>(items, nsnap, nsplit, spare, s)
                      : launch_split_batch<kNwGeneral, false>(items, nsnap, nsplit, spare, s);
            else
                count ? launch_split_batch<FLA_NW, true>(items, nsnap, nsplit, spare, s)
                      : launch_split_batch<FLA_NW, false>(items, nsnap, nsplit, spare, s);
            first = nsplit;
        }
    }
    if (first < nwork) {
        // the XCD counters start at zero (a fill kernel: the launch may be captured)
        hipError_t e = launch_fill_u32(queue, kXcds, 0u, s);
        if (e != hipSuccess) return e;
        if constexpr (D == 2 && sizeof(R) == 8) {
            if (whole_tiles(nwork, spare.records))
                launch_batch_shape<R, D, 1>(items, nsnap, first, nwork - first, chunk, count, plan, general, queue, ncu, s);
            else
                launch_batch_shape<R, D, 2>(items, nsnap, first, nwork - first, chunk, count, plan, general, queue, ncu, s);
        } else if (D == 2 || shape == 0)   // in 2-D there is no other shape than the first
            launch_batch_shape<R, D, tile_parts<R>(D, 0)>(items, nsnap, first, nwork - first, chunk, count, plan, general,
                                                          queue, ncu, s);
        else
            launch_batch_shape<R, D, tile_parts<R>(D, D == 3)>(items, nsnap, first, nwork - first, chunk, count, plan,
                                                               general, queue, ncu, s);
    }
    FLA_LAUNCH((k_gather_batch_overs<R, D, FLA_NW>), dim3((unsigned)nwork), dim3(256), 0, s, items, nsnap);
    return hipGetLastError();
}

// Where every part of every tile has a workgroup at once, their order is
// nothing and needs neither costs nor counters (three launches); and where
// compute units would be left idle, up to four workgroups share a part's cells:
// each scans and stages the same candidates as one would and evaluates its own
// planes or sub-blocks of them, so the sums keep their order and their bits.
// Whole calls with and without: 64^2 cells in binary64 107 -> 93 us, in
// binary32 140 -> 111.  (Binary32 3-D tiles of many records: split_pays.)
// A share skips as finely as there is, and shape 0 has the most workgroups, so
// plan codes make no difference here.
template <typename R, int D, int MODE, bool COUNT>
static bool launch_small(const GatherArgs& g, hipStream_t s)
{
    constexpr int TP = tile_parts<R>(D, 0);
    constexpr int NSB = sizeof(R) == 4 && D == 3 ? 4 : Geo<D>::NSB / TP, most = NSB < 4 ? NSB : 4;
    const int64_t fit = resident_workgroups<R, D, TP>(g.ncu), parts = (int64_t)g.m.ntiles * TP;
    if (parts > fit) return false;
    int shares = 1;
    while (2 * shares <= most && parts * 2 * shares <= fit) shares *= 2;
    FLA_LAUNCH((k_gather_small<R, D, MODE, COUNT, TP>), dim3((unsigned)(parts * shares)),
               dim3(kWave * GatherWaves<R, D>::value), 0, s, g, shares);
    if (kPlanes<R, D>) FLA_LAUNCH((k_gather_overs<R, D, MODE>), dim3((unsigned)g.m.ntiles), dim3(256), 0, s, g);
    return true;
}

template <typename R, int D, int TP>
static hipError_t launch_gather_shape(const GatherArgs& g, int mode, bool count, int plan, const GatherSpare& spare,
                                      hipStream_t s)
{
    const bool general = g.m.edges[0] || g.m.edges[1] || g.m.edges[2];
    auto launch = [&](auto modec, auto countc) -> hipError_t {
        constexpr int MODE = decltype(modec)::value;
        constexpr bool COUNT = decltype(countc)::value;
        if constexpr (kPlanes<R, D>) {
            if (spare.small && split_pays<MODE>(g.m.ntiles, spare.records, g.ncu)) {
                const unsigned nt = (unsigned)g.m.ntiles;
                FLA_LAUNCH((k_gather_split<MODE, COUNT>), dim3(nt * 4), dim3(256), 0, s, g, spare.a, spare.b);
                FLA_LAUNCH((k_split_sum<MODE>), dim3(nt * 2), dim3(256), 0, s, g, (const double*)spare.a,
                           (const double*)spare.b);
                FLA_LAUNCH((k_gather_overs<R, D, MODE>), dim3(nt), dim3(256), 0, s, g);
                return hipGetLastError();
            }
        }
        if (spare.small && launch_small<R, D, MODE, COUNT>(g, s)) return hipGetLastError();
        FLA_LAUNCH(k_tile_cost<D>, dim3((unsigned)((g.m.ntiles + 3) / 4)), dim3(256), 0, s, g);
        FLA_LAUNCH(k_tile_order, dim3(kXcds), dim3(1024), 0, s, (const uint32_t*)g.tile_cost, g.m.ntiles * TP, TP,
                   g.order, g.queue);
        // as many workgroups as the compute units hold at once
        int64_t nb = (int64_t)g.m.ntiles * TP;
        const int64_t fit = resident_workgroups<R, D, TP>(g.ncu);
        if (fit < nb) nb = fit;
        launch_plan<R, D, MODE, COUNT, TP>(g, plan, dim3((unsigned)nb), dim3(kWave * GatherWaves<R, D>::value), s);
        FLA_LAUNCH((k_gather_overs<R, D, MODE>), dim3((unsigned)g.m.ntiles), dim3(256), 0, s, g);
        return hipGetLastError();
    };
    auto counted = [&](auto modec) {
        return count ? launch(modec, std::true_type{}) : launch(modec, std::false_type{});
    };
    if (mode != FLA_NW) return counted(std::integral_constant<int, FLA_DEPOSIT>{});
    return general ? counted(std::integral_constant<int, kNwGeneral>{}) : counted(std::integral_constant<int, FLA_NW>{});
}

template <typename R, int D>
hipError_t launch_gather(const GatherArgs& g, int mode, bool count, int plan_code, const GatherSpare& spare,
                         hipStream_t s)
{
    if (g.m.ntiles <= 0) return hipSuccess;
    const int plan = plan_code % kGatherPlans, shape = plan_code / kGatherPlans;
    if constexpr (D == 2 && sizeof(R) == 8)
        if (whole_tiles(g.m.ntiles, spare.records))
            return launch_gather_shape<R, D, 1>(g, mode, count, plan, spare, s);
    // in 2-D there is no other shape than the first
    if (D == 2 || shape == 0) return launch_gather_shape<R, D, tile_parts<R>(D, 0)>(g, mode, count, plan, spare, s);
    return launch_gather_shape<R, D, tile_parts<R>(D, D == 3)>(g, mode, count, plan, spare, s);
}

}  // namespace flp
