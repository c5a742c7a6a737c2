// subtree.hip -- the small levels at the bottom of a hierarchy in one launch
// (gfx950).
//
// The K-cycle visits level k 2^k times, so its bottom levels -- a thousand unknowns
// and fewer -- take most of its launches, each a few microseconds of latency for a
// few kilobytes of work.  Where one workgroup can hold the last levels (matrices in
// registers: 512 threads, about 230 of them each; vectors in LDS), the whole coarse
// correction of the top one runs in one workgroup per right-hand side (k_subtree):
// every pass of the recursion below -- about 9 for each visit of a level -- is a
// sweep between two block barriers instead of a launch.  What bounds it is the chain of
// those passes: the instructions of one wavefront, LDS latency and cross-lane sums, 450
// to 900 clocks a pass.  On a top level of four slots per thread, whose code is larger
// than the instruction cache holds beside the other levels', a pass takes 4,000 to 8,000.
// Hence 512 threads and no more rows per thread than needed, rows packed by length (2^c
// lanes, four entries a lane), LDS places known at compile time, and one body of code for
// both inner steps.
//
// Measured: 38.3 us for the levels of 971, 286, 108 and 37 rows under the 1003x997 grid,
// 21.4 us for 990, 191 and 50; the 20 launches that the first replaces took about 110 us.
// A solve of that grid went from 58.8 to 22.2 ms, a K-cycle of a 33x31 grid
// from 102 to 38 us (with the cycle on the caller's vectors).
#include <algorithm>

#include "subtree.h"

namespace amg {
namespace {

// e = the coarse correction for the restricted residual rc of the subtree's top level
// (both column-major, the level's size apart).  D: levels above the coarsest one, K:
// slots per thread on the top one.
template <class T, int D, int K>
__global__ void __launch_bounds__(kSubtreeThreads) k_subtree(Subtree S, const T *__restrict__ rc,
                                                             T *__restrict__ eout, int *__restrict__ flag,
                                                             const int *__restrict__ gate, double theta2)
{
    if (gate && gate[blockIdx.y] == 0) return;
    extern __shared__ __align__(16) char lds[];
    __shared__ SubShared sh;
    const int t0 = threadIdx.x;
    const SubLevel &F = S.lev[D];
    rc += (size_t)blockIdx.y * F.n;
    eout += (size_t)blockIdx.y * F.n;
    const SubCtx x{S, lds, sh, theta2, flag, __builtin_amdgcn_readfirstlane(t0 / kWave)};
    SubRegs<T, D, K> regs;
    sub_load_rows<T, D, K>(x, regs);
    using L = SubLds<D, K>;
    double *r = sub_at<double>(lds, L::above);
    for (int i = t0; i < F.n; i += kSubtreeThreads) r[i] = (double)rc[i];
    if (t0 < D) {  // the zeros that padding reads
        double *z = sub_at<double>(lds, SubLds<1, 1>::g) + t0 * 3 * (kSubtreeThreads + 1);
        const int rows = (t0 == D - 1 ? K : 1) * kSubtreeThreads;
        for (int v = 1; v <= (t0 == D - 1 ? 4 : 3); v++) z[v * rows + v - 1] = 0.0;
    }
    for (int i = t0; i < S.over_bytes / 8; i += kSubtreeThreads)
        sub_at<double>(lds, S.over_at)[i] = static_cast<const double *>(S.over)[i];
    __syncthreads();
    const SubCoef c = sub_correct<T, D, K>(x, regs, r, K * kSubtreeThreads);
    const double *c1 = sub_at<const double>(lds, L::c1), *c2 = sub_at<const double>(lds, L::c2);
    for (int i = t0; i < F.n; i += kSubtreeThreads) {
        const double e = c.a1 * c1[i];
        eout[i] = (T)(c.two ? e + c.a2 * c2[i] : e);
    }
}

// Classes of rows: class c < 7 takes 2^c lanes, class 7 the whole wavefront with
// entries left over.
constexpr int kSubClasses = 8;
__device__ inline int row_class(int len, int members)
{
    const int lanes = max((len + kSubUnroll - 1) / kSubUnroll, (members + 2 * kSubUnroll - 1) / (2 * kSubUnroll));
    if (len > kWave * kSubUnroll) return 7;
    int c = 0;
    while (c < 6 && (1 << c) < lanes) c++;
    return c;
}
__device__ inline int class_lanes(int c) { return 1 << (c < 6 ? c : 6); }

struct SubOrder {
    int count[kSubClasses];  // rows of the class
    int base[kSubClasses];   // first lane slot: the widest class first
    int lanes;
};

// Counts the classes of level d's rows; place(i, class, rank in the class) is called
// for every row.  The whole block takes part.
template <class Place>
__device__ void order_rows(const SubtreeSource &P, int d, int count, SubOrder &o, Place place)
{
    constexpr int kW = kSubtreeThreads / kWave;
    __shared__ int wave_count[kSubClasses][kW];
    const SubtreeSource::Lev &X = P.lev[d];
    const int *seg = d + 1 < count ? P.lev[d + 1].seg : nullptr;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (threadIdx.x < kSubClasses) o.count[threadIdx.x] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < X.n; i0 += kSubtreeThreads) {
        const int i = i0 + threadIdx.x;
        const int mine = i < X.n ? row_class(X.rp[i + 1] - X.rp[i], seg ? seg[i + 1] - seg[i] : 1) : -1;
        int before = 0;  // rows of my class in earlier lanes
        for (int c = 0; c < kSubClasses; c++) {
            const unsigned long long b = __ballot(mine == c);
            if (lane == 0) wave_count[c][w] = __popcll(b);
            if (mine == c) before = __popcll(b & ((1ull << lane) - 1ull));
        }
        __syncthreads();
        if (mine >= 0) {
            int rank = o.count[mine] + before;
            for (int k = 0; k < w; k++) rank += wave_count[mine][k];
            place(i, mine, rank);
        }
        __syncthreads();
        if (threadIdx.x < kSubClasses)
            for (int k = 0; k < kW; k++) o.count[threadIdx.x] += wave_count[threadIdx.x][k];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        int at = 0;
        for (int c = kSubClasses - 1; c >= 0; c--) {
            o.base[c] = at;
            at += o.count[c] * class_lanes(c);
        }
        o.lanes = at;
    }
    __syncthreads();
}

__global__ void __launch_bounds__(kSubtreeThreads) k_subtree_needs(SubtreeSource P, int count, SubtreeNeed *need)
{
    __shared__ SubOrder o;
    __shared__ int over;
    const int d = blockIdx.x + 1;
    const SubtreeSource::Lev &X = P.lev[d];
    if (threadIdx.x == 0) over = 0;
    order_rows(P, d, count, o, [&](int i, int c, int) {
        if (c == 7) atomicAdd(&over, X.rp[i + 1] - X.rp[i] - kWave * kSubUnroll);
    });
    if (threadIdx.x == 0) need[d] = SubtreeNeed{(o.lanes + kWave - 1) / kWave, o.count[7], over};
}

// Fills the slot arrays of level d = blockIdx.x + 1 (block 0 of the grid's last column:
// the exact solve's).
template <class T>
__global__ void __launch_bounds__(kSubtreeThreads) k_subtree_pack(Subtree S, SubtreeSource P, char *over_image)
{
    extern __shared__ __align__(16) char dyn[];
    const int t = threadIdx.x, D = S.levels - 1;
    if ((int)blockIdx.x == D) {
        double *ainv = const_cast<double *>(S.exact_ainv), *dinv = const_cast<double *>(S.exact_dinv);
        int *index = const_cast<int *>(S.exact_index);
        const int *seg = P.lev[1].seg;
        const int i = t / 8, sub = t & 7;
        for (int u = 0; u < kSubExact; u++) {
            const int j = sub + 8 * u;
            ainv[u * kSubtreeThreads + t] = i < S.m && j < S.m ? P.cs.ainv[i * S.m + j] : 0.0;
        }
        const int J = i < S.m ? (P.cs.idx ? P.cs.idx[i] : i) : 0;
        index[t] = i < S.m ? (seg[J] + sub) | seg[J + 1] << 16 : 0;
        const int q = t >> S.dlanes, qs = t & ((1 << S.dlanes) - 1);
        const int K = q < S.nd ? P.cs.didx[q] : 0;
        dinv[t] = q < S.nd ? P.cs.dinv[q] : 0.0;
        index[kSubtreeThreads + t] = q < S.nd ? (seg[K] + qs) | seg[K + 1] << 16 : 0;
        index[2 * kSubtreeThreads + t] = J | K << 16;
        return;
    }
    const int d = blockIdx.x + 1;
    const SubLevel &F = S.lev[d];
    const SubtreeSource::Lev &X = P.lev[d];
    const int slots = F.slots.count;
    __shared__ SubOrder o;
    int *owner = reinterpret_cast<int *>(dyn);                       // row and class of each slot's group, -1: none
    uint16_t *rank = reinterpret_cast<uint16_t *>(owner + slots);    // per row
    uint16_t *cls = rank + (X.n + 1) / 2 * 2;
    for (int s = t; s < slots; s += kSubtreeThreads) owner[s] = -1;
    order_rows(P, d, S.levels, o, [&](int i, int c, int r) {
        rank[i] = (uint16_t)r;
        cls[i] = (uint16_t)c;
    });
    for (int i = t; i < X.n; i += kSubtreeThreads) {
        const int c = cls[i], at = o.base[c] + rank[i] * class_lanes(c);
        for (int k = 0; k < class_lanes(c); k++) owner[at + k] = i;
    }
    __syncthreads();
    const int *seg = d + 1 < S.levels ? P.lev[d + 1].seg : nullptr;
    T *va = static_cast<T *>(const_cast<void *>(F.slots.va)), *minv = static_cast<T *>(const_cast<void *>(F.slots.minv));
    int2 *ci = const_cast<int2 *>(F.slots.ci);
    int *ig = const_cast<int *>(F.slots.ig), *sbe = const_cast<int *>(F.slots.sbe), *agg = const_cast<int *>(F.slots.agg);
    const T *xva = static_cast<const T *>(X.va), *xm = static_cast<const T *>(X.minv);
    for (int s = t; s < slots; s += kSubtreeThreads) {
        const int i = owner[s], first = owner[s & ~(kWave - 1)];
        const int lg = i >= 0 ? min((int)cls[i], 6) : 0, G = 1 << lg, sub = s & (G - 1);
        const int widest = first >= 0 ? min((int)cls[first], 6) : 0;
        const int b = i >= 0 ? X.rp[i] + sub : 0, e = i >= 0 ? X.rp[i + 1] : 0;
        int k[kSubUnroll];
        for (int u = 0; u < kSubUnroll; u++) {
            const int q = b + u * G;
            k[u] = q < e ? X.ci[q] : slots;  // the zero after the rows
            va[u * slots + s] = q < e ? xva[q] : T(0);
        }
        ci[s] = int2{k[0] | k[1] << 16, k[2] | k[3] << 16};
        minv[s] = i >= 0 ? xm[i] : T(0);
        ig[s] = (i >= 0 ? i : slots) | lg << 16 | (i >= 0 && sub == 0 ? 1 << 31 : 0);
        const int sb = i >= 0 ? (seg ? seg[i] : i) : 0, se = i >= 0 ? (seg ? seg[i + 1] : i + 1) : 0;
        sbe[s] = (sb + sub) | se << 16;
        agg[s] = (i >= 0 ? X.agg[i] : 0) | widest << 16;
    }
    // the long rows' other entries (LDS offsets, here into the image)
    char *img = over_image - S.over_at;
    int *optr = sub_at<int>(img, F.optr);
    T *ova = sub_at<T>(img, F.ova);
    uint16_t *oci = sub_at<uint16_t>(img, F.oci);
    int at = 0;
    for (int r = 0; r < F.nover; r++) {
        const int i = owner[r * kWave], b = X.rp[i] + kWave * kSubUnroll, len = X.rp[i + 1] - b;
        if (t == 0) optr[r] = at;
        for (int p = t; p < len; p += kSubtreeThreads) {
            ova[at + p] = xva[b + p];
            oci[at + p] = (uint16_t)X.ci[b + p];
        }
        at += len;
    }
    if (t == 0) optr[F.nover] = at;
}

// Takes sizes out of one block, 16 bytes aligned.
struct Carve {
    char *base;
    size_t at = 0;
    template <class P>
    P *take(size_t count)
    {
        P *p = reinterpret_cast<P *>(base + at);
        at += (count * sizeof(P) + 15) / 16 * 16;
        return p;
    }
};
// value_bytes: of type T
size_t carve(Subtree &S, int value_bytes, char *base)
{
    Carve c{base};
    for (int d = 1; d < S.levels; d++) {
        SubSlots &L = S.lev[d].slots;
        L.count = (d == S.levels - 1 ? S.width : 1) * kSubtreeThreads;
        L.va = c.take<char>((size_t)L.count * kSubUnroll * value_bytes);
        L.minv = c.take<char>((size_t)L.count * value_bytes);
        L.ci = c.take<int2>(L.count);
        L.ig = c.take<int>(L.count);
        L.sbe = c.take<int>(L.count);
        L.agg = c.take<int>(L.count);
    }
    S.exact_ainv = c.take<double>(kSubExact * kSubtreeThreads);
    S.exact_dinv = c.take<double>(kSubtreeThreads);
    S.exact_index = c.take<int>(3 * kSubtreeThreads);
    S.over = c.take<char>(S.over_bytes);
    return c.at;
}

template <class T, int D>
void launch_depth(const Subtree &S, const T *rc, T *e, int *flag, hipStream_t s, int ncol, const int *gate,
                  double theta2)
{
    if constexpr (D <= kSubtreeDepth) {
        if (S.levels - 1 != D) return launch_depth<T, D + 1>(S, rc, e, flag, s, ncol, gate, theta2);
        const dim3 grid(1, ncol);
        const size_t lds = (size_t)S.lds_bytes;
        switch (S.width) {
        case 1: k_subtree<T, D, 1><<<grid, kSubtreeThreads, lds, s>>>(S, rc, e, flag, gate, theta2); break;
        case 2: k_subtree<T, D, 2><<<grid, kSubtreeThreads, lds, s>>>(S, rc, e, flag, gate, theta2); break;
        default: k_subtree<T, D, 4><<<grid, kSubtreeThreads, lds, s>>>(S, rc, e, flag, gate, theta2); break;
        }
        AMG_HIP(hipGetLastError());
    }
}

}  // namespace

void launch_subtree_needs(const SubtreeSource &P, int count, SubtreeNeed *need, hipStream_t s)
{
    k_subtree_needs<<<count - 1, kSubtreeThreads, 0, s>>>(P, count, need);
    AMG_HIP(hipGetLastError());
}

bool layout_subtree(int count, const int *n, const SubtreeNeed *need, const CoarseSolve &cs, int value_bytes,
                    int lds_limit, Subtree &S)
{
    if (cs.m > kInlineCoarse || cs.nd > kSubtreeThreads) return false;  // n[0] = m + nd
    // The top level may have several slots per thread, the ones below it one: a level is
    // swept twice as often as the one above it, and more than four slots (or two on two
    // levels) do not fit the registers.  Every level more that fits is taken: each halves
    // the launches of a K-cycle.  That pays also where its four slots make a pass as long
    // as a launch (4,000 to 8,000 clocks; 4 to 5 us): the levels above stop at a lower
    // count of visits.  K-cycle with a top level of up to 4 / 2 / 1 slots per thread, in
    // us: 45x45 46 / 77 / 76, 131x67 110 / 130 / 134, 1003x997 1,278 / 1,565 / 1,561, graph
    // of 5,000 points 59 / 91 / 92, of 150,000 1,257 / 1,401 / 1,402; top level of two
    // slots: 33x31 41 / 41 / 70, 41x37x29 395 / 397 / 565, 300,000 points 1,985 / 1,973 /
    // 2,728.  No problem of these is slower with the wider level.
    int top = 0;
    for (int d = 1; d < count && d <= kSubtreeDepth; d++) {
        if (need[d].waves <= 4 * kSubWaves) top = d;
        if (need[d].waves > kSubWaves) break;
    }
    for (; top >= 1; top--) {
        const int waves = need[top].waves;
        S.levels = top + 1;
        S.width = waves <= kSubWaves ? 1 : (waves <= 2 * kSubWaves ? 2 : 4);
        S.m = cs.m;
        S.nd = cs.nd;
        S.dlanes = 0;
        while (S.dlanes < 3 && cs.nd << (S.dlanes + 1) <= kSubtreeThreads) S.dlanes++;
        // the vectors' places are fixed (SubLds); the long rows' other entries come after them
        S.over_at = kSubLevel1 + (top - 1) * 3 * sub_vector(1) + 4 * sub_vector(S.width);
        int64_t at = S.over_at;
        auto take = [&](int64_t bytes) {
            const int64_t o = at;
            at += (bytes + 7) / 8 * 8;
            return (int)o;
        };
        for (int d = 0; d <= top; d++) {
            SubLevel &F = S.lev[d];
            F = SubLevel{};
            F.n = n[d];
            if (d == 0) continue;
            F.waves = need[d].waves;
            F.nover = need[d].nover;
            F.optr = take(4 * ((int64_t)F.nover + 1));
            F.ova = take((int64_t)need[d].over * value_bytes);
            F.oci = take(2 * (int64_t)need[d].over);
        }
        S.over_bytes = (int)(at - S.over_at);
        S.lds_bytes = (int)at;
        if (at <= lds_limit) return true;
    }
    S = Subtree{};
    return false;
}

size_t subtree_bytes(const Subtree &S, int value_bytes)
{
    Subtree c = S;
    return carve(c, value_bytes, nullptr);
}

int subtree_lds_limit()
{
    int dev = 0, lds = 0;
    AMG_HIP(hipGetDevice(&dev));
    AMG_HIP(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    return lds - (int)((sizeof(SubShared) + 127) / 128 * 128);
}

template <class T>
void launch_subtree_pack(Subtree &S, const SubtreeSource &P, void *base, hipStream_t s)
{
    carve(S, sizeof(T), static_cast<char *>(base));
    size_t lds = 0;
    for (int d = 1; d < S.levels; d++)
        lds = std::max(lds, sizeof(int) * (size_t)S.lev[d].slots.count + 4 * (size_t)(S.lev[d].n + 2));
    k_subtree_pack<T><<<S.levels, kSubtreeThreads, lds, s>>>(S, P, static_cast<char *>(const_cast<void *>(S.over)));
    AMG_HIP(hipGetLastError());
}

template <class T>
void launch_subtree(const Subtree &S, const T *rc, T *e, int *flag, hipStream_t s, int ncol, const int *gate,
                    double theta2)
{
    launch_depth<T, 1>(S, rc, e, flag, s, ncol, gate, theta2);
}

template void launch_subtree_pack<double>(Subtree &, const SubtreeSource &, void *, hipStream_t);
template void launch_subtree_pack<float>(Subtree &, const SubtreeSource &, void *, hipStream_t);
template void launch_subtree<double>(const Subtree &, const double *, double *, int *, hipStream_t, int, const int *,
                                     double);
template void launch_subtree<float>(const Subtree &, const float *, float *, int *, hipStream_t, int, const int *,
                                    double);

}  // namespace amg
