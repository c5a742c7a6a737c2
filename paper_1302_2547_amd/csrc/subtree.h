// subtree.h -- the coarse correction of a whole subtree of small levels in one
// workgroup, with every level's matrix and vectors in LDS and registers (gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include "amg_internal.h"
#include "wave_ops.h"

namespace amg {
namespace {

constexpr int kSubWaves = kSubtreeThreads / kWave;
constexpr int kSubUnroll = 4;  // entries per lane in flight

struct SubShared {
    // a reduction's wavefront sums, value d of wavefront w at 4 w + d (the second set:
    // the threshold test's)
    double part[2][4 * kSubWaves];
};

// The coefficients of a finished coarse correction: e = a1 c1 (+ a2 c2 when two).
struct SubCoef {
    double a1, a2;
    bool two;
};

// Sums of four values over the block, in two parts around a barrier.
__device__ __forceinline__ void sub_partials(const double (&v)[4], double *part)
{
    const int lane = threadIdx.x & (kWave - 1);
    const double t = spread4_sum(v);
    if (lane < 4) part[threadIdx.x / kWave * 4 + lane] = t;
}
// After the barrier: the totals, the same in every thread.
__device__ __forceinline__ void sub_totals(const double *part, double (&v)[4])
{
    const int lane = threadIdx.x & (kWave - 1);
    const double t = mod4_sum(lane < 4 * kSubWaves ? part[lane] : 0.0);
#pragma unroll
    for (int d = 0; d < 4; d++) v[d] = lane_value(t, d);
}

// LDS, in bytes at compile-time places (the offsets are part of the instructions, and
// no address is held in registers): the exact solve's residual and solution, then the
// vectors g, c1 and c2 of levels 1, 2, ...  A level of K slots per thread has room for
// K kSubtreeThreads rows, and a zero after them.
constexpr int kSubExactRc = 0, kSubExactC1 = 8 * kInlineCoarse;
constexpr int kSubExactRows = kInlineCoarse + kSubtreeThreads;
constexpr int kSubLevel1 = kSubExactC1 + 8 * kSubExactRows;
constexpr int sub_vector(int K) { return 8 * (K * kSubtreeThreads + 1); }
template <int D, int K>
struct SubLds {
    static constexpr int g = kSubLevel1 + (D - 1) * 3 * sub_vector(1);
    static constexpr int c1 = g + sub_vector(K), c2 = c1 + sub_vector(K);
    static constexpr int above = c2 + sub_vector(K);  // the residual that the level above the top one hands down
    static constexpr int end = above + sub_vector(K);
};
template <int K>
struct SubLds<0, K> {
    static constexpr int c1 = kSubExactC1, c2 = kSubExactC1;
};
template <class P>
__device__ __forceinline__ P *sub_at(char *lds, int off)
{
    return reinterpret_cast<P *>(lds + off);
}

// Keeps a value that is cheap to recompute from being computed ahead of a loop and
// held in registers through it.
__device__ __forceinline__ int sub_here(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// What a kernel of the subtree works with.
struct SubCtx {
    const Subtree &S;
    char *lds;
    SubShared &sh;
    double theta2;  // squared K-cycle threshold, 0: none
    int *flag;
    int wave;       // this wavefront (uniform)
};

// One lane's part of a row.  A row of a level is served by G lanes of one wavefront, G
// the power of two that gives each at most kSubUnroll entries (and the members of its
// aggregate in two steps); the rows are ordered by G, so the aligned groups fill the
// wavefronts whatever the lengths.  The entries, the diagonal and the row's part of
// the level's vectors stay in registers from one visit to the next (every lane of the
// group holds the latter); index pairs are packed and unpacked where they are used.
// Padding entries have the value 0 and column n, where every vector holds a zero.
template <class T>
struct SubRow {
    T a[kSubUnroll];
    int c[kSubUnroll / 2];
    int ig;   // row (n: none); log2 G; 1 on the group's first lane
    int sbe;  // this lane's members of the row's aggregate on the level above: sb, sb + G, ... < se
    int agg;  // the row's coarse position; log2 G of the wavefront's widest group
    double minv, rc;
    double keep;  // t of the first step, then c1

    static __device__ __forceinline__ int low(int v) { return v & 0xffff; }
    static __device__ __forceinline__ int high(int v) { return (int)((unsigned)v >> 16); }

    __device__ __forceinline__ void load(const SubSlots &src, int s)
    {
        const T *va = static_cast<const T *>(src.va), *m = static_cast<const T *>(src.minv);
#pragma unroll
        for (int u = 0; u < kSubUnroll; u++) a[u] = va[u * src.count + s];
        const int2 k = src.ci[s];
        c[0] = k.x;
        c[1] = k.y;
        ig = src.ig[s];
        sbe = src.sbe[s];
        agg = src.agg[s];
        minv = (double)m[s];
        rc = keep = 0.0;
    }
    static_assert(kSubUnroll == 4, "two packed pairs of columns");
    __device__ __forceinline__ int at() const { return low(sub_here(ig)); }
    __device__ __forceinline__ bool writer() const { return sub_here(ig) < 0; }
    __device__ __forceinline__ int coarse() const { return low(sub_here(agg)); }
    // sum over the row's group of lanes
    __device__ __forceinline__ double sum(double s) const
    {
        const int widest = __builtin_amdgcn_readfirstlane(high(sub_here(agg)));
        if (widest > 0) {
            const int g = high(sub_here(ig)) & 7;
            s += g >= 1 ? dpp_f64<kDppQuadXor1>(s) : 0.0;
            if (widest > 1) {
                s += g >= 2 ? dpp_f64<kDppQuadXor2>(s) : 0.0;
                if (widest > 2) {
                    s += g >= 3 ? dpp_f64<kDppRowHalfMirror>(s) : 0.0;
                    s += g >= 4 ? dpp_f64<kDppRowMirror>(s) : 0.0;
                    if (widest > 4) {
                        const double h = rows_pair_sum(s);
                        s = g >= 5 ? h : s;
                        const double w = halves_sum(s);
                        s = g >= 6 ? w : s;
                    }
                }
            }
        }
        return s;
    }
    // sum of a_ij v_j over the row; over: the wavefront's slot, which is a row with
    // more entries than its lanes hold when it is below the level's count of those
    __device__ __forceinline__ double times(const SubCtx &x, const SubLevel &F, const double *v, int slot) const
    {
        double t[kSubUnroll];
#pragma unroll
        for (int u = 0; u < kSubUnroll; u += 2) {
            const int k = sub_here(c[u / 2]);
            t[u] = v[low(k)];
            t[u + 1] = v[high(k)];
        }
        double s = (double)a[0] * t[0];
#pragma unroll
        for (int u = 1; u < kSubUnroll; u++) s += (double)a[u] * t[u];
        if (slot < F.nover) {
            const int *ptr = sub_at<const int>(x.lds, F.optr);
            const T *va = sub_at<const T>(x.lds, F.ova);
            const uint16_t *ci = sub_at<const uint16_t>(x.lds, F.oci);
#pragma unroll 1
            for (int p = ptr[slot] + (threadIdx.x & (kWave - 1)); p < ptr[slot + 1]; p += kWave)
                s += (double)va[p] * v[ci[p]];
        }
        return sum(s);
    }
    // sum of the fine values t over the row's aggregate (t[n] = 0)
    __device__ __forceinline__ double members(const double *t, int n) const
    {
        const int q = sub_here(sbe), b = low(q), e = high(q), step = 1 << (high(sub_here(ig)) & 7);
        double v[kSubUnroll], s = 0.0;
#pragma unroll
        for (int u = 0; u < kSubUnroll; u++) v[u] = t[b + u * step < e ? b + u * step : n];
#pragma unroll
        for (int u = 0; u < kSubUnroll; u++) s += v[u];
#pragma unroll 1
        for (int p = b + kSubUnroll * step; p < e; p += step) s += t[p];
        return sum(s);
    }
};

// The rows of levels 1 .. D: K slots per lane on level D, one on the levels below.
template <class T, int D, int K>
struct SubRegs {
    SubRow<T> row[K];
    SubRegs<T, D - 1, 1> below;
};
constexpr int kSubExact = kInlineCoarse / 8;  // columns of the inverse per lane
template <class T, int K>
struct SubRegs<T, 0, K> {
    double ainv[kSubExact];  // row t / 8, columns t % 8 + 8 u
    double dinv;             // decoupled unknown t >> dlanes
    int sbe, dsbe;           // this lane's members of coupled unknown t / 8 and of that decoupled unknown
    int at;                  // their places, 16 bits each
};

template <class T, int D, int K>
__device__ __forceinline__ void sub_load_rows(const SubCtx &x, SubRegs<T, D, K> &R)
{
    const Subtree &S = x.S;
    if constexpr (D > 0) {
#pragma unroll
        for (int k = 0; k < K; k++)
            if (k * kSubWaves + x.wave < S.lev[D].waves) R.row[k].load(S.lev[D].slots, k * kSubtreeThreads + threadIdx.x);
        sub_load_rows<T, D - 1, 1>(x, R.below);
    } else {
#pragma unroll
        for (int u = 0; u < kSubExact; u++)
            R.ainv[u] = x.wave * 8 < S.m ? S.exact_ainv[u * kSubtreeThreads + threadIdx.x] : 0.0;
        R.dinv = S.exact_dinv[threadIdx.x];
        R.sbe = S.exact_index[threadIdx.x];
        R.dsbe = S.exact_index[kSubtreeThreads + threadIdx.x];
        R.at = S.exact_index[2 * kSubtreeThreads + threadIdx.x];
    }
}

// The exact solve of the coarsest level from the residual t of the level above: eight
// lanes per coupled unknown and row of the inverse, 2^dlanes per decoupled unknown (as
// many as the block has: their aggregates hold up to some twenty members, and with one
// lane each the longest took 1,000 cycles of every visit).
template <class T>
__device__ __forceinline__ void sub_exact(const SubCtx &x, const SubRegs<T, 0, 1> &R, const double *t)
{
    const Subtree &S = x.S;
    double *rc = sub_at<double>(x.lds, kSubExactRc), *c1 = sub_at<double>(x.lds, kSubExactC1);
    const int sub = threadIdx.x & 7, k = threadIdx.x / 8;
    auto members = [&](int q, int step) {
        const int e = (int)((unsigned)q >> 16);
        double s = 0.0;
#pragma unroll 2
        for (int p = q & 0xffff; p < e; p += step) s += t[p];
        return s;
    };
    if (x.wave * 8 < S.m) {
        const double s = group_sum<8>(members(sub_here(R.sbe), 8));
        if (sub == 0) rc[k] = s;  // kInlineCoarse of them, zeros past m
    }
    const int lg = S.dlanes;
    if (x.wave * kWave < S.nd << lg) {
        double s = members(sub_here(R.dsbe), 1 << lg);
        if (lg >= 1) s += dpp_f64<kDppQuadXor1>(s);
        if (lg >= 2) s += dpp_f64<kDppQuadXor2>(s);
        if (lg >= 3) s += dpp_f64<kDppRowHalfMirror>(s);
        const int d = threadIdx.x >> lg;
        if (d < S.nd && d << lg == (int)threadIdx.x) c1[(unsigned)sub_here(R.at) >> 16] = s * R.dinv;
    }
    __syncthreads();
    if (S.m > 0) {
        if (x.wave * 8 < S.m) {
            double v[kSubExact], s = 0.0;
#pragma unroll
            for (int u = 0; u < kSubExact; u++) v[u] = rc[sub + 8 * u];
#pragma unroll
            for (int u = 0; u < kSubExact; u++) s += 8 * u + sub < S.m ? R.ainv[u] * v[u] : 0.0;
            s = group_sum<8>(s);
            if (sub == 0 && k < S.m) c1[sub_here(R.at) & 0xffff] = s;
        }
        __syncthreads();
    }
}

// alpha1 / rho1 of a first step from its products d = (c1, A c1), (c1, rc): 0 and the
// breakdown flag when A turns out not to be SPD; a zero coarse residual gives c1 = 0
// and no correction.  *rho: rho1, or 0 where there is no correction.
__device__ __forceinline__ double sub_first(const SubCtx &x, const double (&d)[4], double *rho)
{
    const double rho1 = d[0], alpha1 = d[1];
    const bool ok = rho1 > 0.0;
    if (threadIdx.x == 0 && !ok && !(rho1 == 0.0 && alpha1 == 0.0)) atomicOr(x.flag, 1);
    *rho = lane_value(ok ? rho1 : 0.0, 0);
    return lane_value(ok ? alpha1 / rho1 : 0.0, 0);
}
// The correction's coefficients after the second step: d = (c2, A c2), (c2, rt), (c2, A c1).
// gamma / rho1 is a quotient, not a product with 1 / rho1, which is infinite for a
// subnormal rho1 (residuals of about 1e-154).
__device__ __forceinline__ SubCoef sub_second(const SubCtx &x, const double (&d)[4], double q1, double rho1)
{
    const double beta = d[0], alpha2 = d[1], gamma = d[2];
    SubCoef c{q1, 0.0, true};
    if (rho1 != 0.0) {
        const double g1 = gamma / rho1, rho2 = beta - gamma * g1;
        if (rho2 > 0.0) {
            c.a2 = lane_value(alpha2 / rho2, 0);
            c.a1 = q1 - g1 * c.a2;
        } else if (threadIdx.x == 0 && !(beta == 0.0 && alpha2 == 0.0)) {
            atomicOr(x.flag, 1);
        }
    }
    return c;
}
// Threshold test (Sec. 4.3) from this thread's shares of (rc, rc) and (rt, rt): true
// when the second step is skipped.
__device__ __forceinline__ bool sub_skip(const SubCtx &x, double rcrc, double rtrt)
{
    double v[4] = {rcrc, rtrt, 0.0, 0.0};
    sub_partials(v, x.sh.part[1]);
    __syncthreads();
    sub_totals(x.sh.part[1], v);
    __syncthreads();
    return v[1] < x.theta2 * v[0];
}

// The coarse correction of level D of the subtree (0: the coarsest level) from the
// residual tup of the level above (tn: its size, where tup holds a zero): nu
// flexible-CG steps, each preconditioned by a visit of the level, whose coarse
// correction is that of level D - 1.  Returns the coefficients of the level's c1 and
// c2 (the same in every thread).
//
// A visit turns the residual r into c = K(r).  Every line is one pass over the
// level's rows between two barriers; r, M^-1 and c1 of a row stay in its lanes:
//   r = sum of tup over the row's aggregate, g = M^-1 r     (first step)
//   t = r - A g                                  -> coarse correction, e
//   g = M^-1 r + P e
//   c = g + M^-1 (r - A g)                           (c1, then c2)
//   A c and the step's inner products; after the first step y = A c1, g = M^-1 y
// and the second step's t needs no pass of its own for rt = r - q y, q = alpha1/rho1:
// t = rt - A M^-1 rt = t1 - q (y - A g), so the product A g runs while q is reduced.
// (c2, A c1) is formed as (A c2, c1): A is symmetric.  c2's storage holds t while the
// levels below work.

template <class T, int D, int K>
__device__ __forceinline__ SubCoef sub_correct(const SubCtx &x, SubRegs<T, D, K> &R, const double *tup, int tn)
{
    if constexpr (D == 0) {
        sub_exact<T>(x, R, tup);
        return SubCoef{1.0, 0.0, false};
    } else {
        using L = SubLds<D, K>;
        double *g = sub_at<double>(x.lds, L::g), *c1 = sub_at<double>(x.lds, L::c1), *c2 = sub_at<double>(x.lds, L::c2);
        const SubLevel &F = x.S.lev[D];
        // f(row, k, slot of the wavefront) for this wavefront's slots of the level
        auto each = [&](auto f) {
#pragma unroll
            for (int k = 0; k < K; k++) {
                const int slot = k * kSubWaves + x.wave;
                if (slot < F.waves) f(R.row[k], k, slot);
            }
        };
        each([&](SubRow<T> &w, int, int) {
            w.rc = w.members(tup, tn);
            if (w.writer()) g[w.at()] = w.minv * w.rc;
        });
        __syncthreads();
        each([&](SubRow<T> &w, int, int slot) {
            w.keep = w.rc - w.times(x, F, g, slot);
            if (w.writer()) c2[w.at()] = w.keep;
        });
        __syncthreads();
        SubCoef c{0.0, 0.0, false};
        double q = 0.0, rho1 = 0.0;
#pragma unroll 1
        for (int step = 0; step < 2; step++) {
            const SubCoef e = sub_correct<T, D - 1, 1>(x, R.below, c2, K * kSubtreeThreads);
            const double *d1 = sub_at<const double>(x.lds, SubLds<D - 1, 1>::c1);
            const double *d2 = sub_at<const double>(x.lds, SubLds<D - 1, 1>::c2);
            double o[K] = {}, y[K] = {}, s[K] = {};
            each([&](SubRow<T> &w, int k, int) {
                const int J = w.coarse();
                double v = e.a1 * d1[J];
                if (e.two) v += e.a2 * d2[J];
                o[k] = w.minv * w.rc + v;
                if (w.writer()) g[w.at()] = o[k];
            });
            __syncthreads();
            double *out = step ? c2 : c1;
            each([&](SubRow<T> &w, int k, int slot) {
                o[k] += w.minv * (w.rc - w.times(x, F, g, slot));
                if (w.writer()) out[w.at()] = o[k];
            });
            __syncthreads();
            double d[4] = {0.0, 0.0, 0.0, 0.0};
            each([&](SubRow<T> &w, int k, int slot) {
                y[k] = w.times(x, F, out, slot);
                if (w.writer()) {
                    d[0] += o[k] * y[k];
                    d[1] += o[k] * w.rc;
                    if (step) d[2] += w.keep * y[k];
                    else g[w.at()] = w.minv * y[k];
                }
            });
            sub_partials(d, x.sh.part[0]);
            __syncthreads();
            if (step) {
                sub_totals(x.sh.part[0], d);
                return sub_second(x, d, q, rho1);
            }
            // q is reduced while A M^-1 y is formed
            if (x.S.nu == 2) each([&](SubRow<T> &w, int k, int slot) { s[k] = w.times(x, F, g, slot); });
            sub_totals(x.sh.part[0], d);
            q = sub_first(x, d, &rho1);
            c = SubCoef{q, 0.0, false};
            if (x.S.nu == 1) break;
            double rcrc = 0.0, rtrt = 0.0;
            each([&](SubRow<T> &w, int k, int) {
                const double rt = w.rc - q * y[k];
                if (w.writer()) {
                    rcrc += w.rc * w.rc;
                    rtrt += rt * rt;
                    c2[w.at()] = w.keep - q * (y[k] - s[k]);
                }
                w.rc = rt;
                w.keep = o[k];
            });
            if (x.theta2 > 0.0 && sub_skip(x, rcrc, rtrt)) break;
            __syncthreads();
        }
        return c;
    }
}

}  // namespace
}  // namespace amg
