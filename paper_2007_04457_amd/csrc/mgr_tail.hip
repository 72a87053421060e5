// Small coarse levels in one workgroup, entirely in LDS.
//
// Once the level grid is small (a few thousand nodes) every stage of a level
// step is latency bound and a separate launch per stage costs more than the
// work.  This kernel runs all remaining level steps (decomposition: the
// finest of them first; recomposition: the coarsest first) in one workgroup
// of kTailThreads lanes.  Global memory is touched only at the boundary: the
// input level grid, the coefficients of each level (written to / read from the
// caller's array at stride 2^k), the coarsest values and the tables, all of
// whose loads are issued before the first of them is waited for.
//
// What bounds it is latency: the chain of phases between barriers.  So
//  - the load vector and the correction solve of a dimension are one linear
//    map, z = B c with B = M_{l-1}^{-1} R M_l (rows of the product, built on
//    the host in FP64; M^{-1} decays by about 0.27 a row, so long rows are
//    cut where what is left is below the working precision): one phase of
//    independent dot products per dimension instead of a stencil pass and a
//    serial elimination;
//  - a level's coarse nodes live in an array of their own (G) and its fine
//    nodes in U, which is zero at coarse nodes, so the coefficients are
//    formed in place, no pass needs a mask, and the last dimension's phase
//    adds the correction and hands the values to the next level;
//  - a recomposition's corrections depend on the stored coefficients alone:
//    those of all levels share the three phases, and the coarse-to-fine chain
//    keeps one phase per level.
// A dot-product task is four neighbouring outputs of one fibre: lanes take
// fibres (their reads are contiguous or at an odd stride: no bank conflicts),
// the four table entries of a tap are one broadcast read.  (Two fibres a lane
// halve those reads' share of the LDS bandwidth but lengthen each phase's
// chain: 16.0 -> 17.7 us in the kernel at 17^3.)  Coefficients and
// interpolation go by cells: a coarse node and the up to seven fine nodes
// after it share its eight corners.
//
// Per call, the launch included (FP32): 17^3 decomposed in 28.6 -> 18 us with
// these phases in place of stencil passes and a serial elimination per
// dimension, recomposed in 34 -> 19; 513 nodes 79 -> 24, 93 -> 25; 65^2 41 -> 30,
// 50 -> 30.  What is left is the chain itself: 2000 to 4000 cycles a phase, of
// LDS round trips and of the address arithmetic that the first loads wait for.
//
// Four dimensions never come here; level grids of any length do (View3: the
// LDS arrays hold the phantom nodes, which are zero; user's and packed arrays
// have none).
#include "mgr_internal.h"

namespace mgr {
namespace {

constexpr int kT = kTailThreads;
constexpr int kWaves = kT / 64;
constexpr int kTB = (5 * 1024) / kT;  // loads of the finest grid in flight per lane
constexpr int kTailOffs = 516;        // nodes of the finest grid per dimension (at most kTailMaxSide)
static_assert(kTailOffs >= kTailMaxSide && kTailOffs <= kT, "one pass");

// idx / n for idx < 2^20 and r = 1 / n: the quotient of idx + 1/2 lies at least
// 1 / (2 n) from a whole number, further than its rounding.  (Integer products
// here are of small numbers: 24-bit multiplies, four times the rate of 32-bit
// ones.)
__device__ __forceinline__ int fdiv(int idx, float r) { return (int)fmaf((float)idx, r, 0.5f * r); }

__device__ __forceinline__ bool phantom(const TailLevel& L, int j0, int j1, int j2)
{
    return j0 == L.d[0].ph || j1 == L.d[1].ph || j2 == L.d[2].ph;
}
// Place of node (j0, j1, j2) in the packed grid (without phantoms).
__device__ __forceinline__ int packed_at(const TailLevel& L, int j0, int j1, int j2)
{
    return __mul24(__mul24(min(j0, L.d[0].act - 1), L.d[1].act) + min(j1, L.d[1].act - 1), L.d[2].act) +
           min(j2, L.d[2].act - 1);
}
// Index j0, j1, j2 of node idx of a box of sizes (., n1, n2).
__device__ __forceinline__ void split(int idx, int n1, float r1, int n2, float r2, int& j0, int& j1, int& j2)
{
    const int q = fdiv(idx, r2);
    j2 = idx - __mul24(q, n2);
    j0 = fdiv(q, r1);
    j1 = q - __mul24(j0, n1);
}
__device__ __forceinline__ void node_of(const TailLevel& L, int idx, int& j0, int& j1, int& j2)
{
    split(idx, L.d[1].m, L.d[1].rm, L.d[2].m, L.d[2].rm, j0, j1, j2);
}
__device__ __forceinline__ void coarse_of(const TailLevel& L, int c, int& i0, int& i1, int& i2)
{
    split(c, L.d[1].mc, L.d[1].rmc, L.d[2].mc, L.d[2].rmc, i0, i1, i2);
}

// The four table entries of a tap, one read.
template <typename T>
struct Tap {
    typedef T V __attribute__((ext_vector_type(4), aligned(16)));
};

// Dot products of one dimension: the array `in` is (outer, m, inner); n results
// at a time go to out(o, inner, n, v): v[k] is element o + k inner of (outer,
// mc, inner).  m and mc are the level grid and its coarse nodes with the rows
// of B (kStep 8: input nodes per group of four outputs), the other way round
// with its columns (the adjoints: kStep 2).
template <int kStep, typename T, class Out>
__device__ __forceinline__ void tail_dots(const TailDim& D, const T* B, const T* in, int outer, int inner, float rinner,
                                          Out out)
{
    constexpr bool kRows = kStep == 8;
    const int m = kRows ? D.m : D.mc, mc = kRows ? D.mc : D.m;
    const float rmc = kRows ? D.rmc : D.rm;
    const int nt = uni(D.nt), off = D.off, smax = m - nt, nfib = uni(outer * inner);
    auto start_of = [&](int g) { return min(max(kStep * g - off, 0), smax); };
    if (nfib >= 32) {
        const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
        const int nch = (nfib + 63) >> 6, units = nch * ((uni(mc) + 3) >> 2);
        const float rch = __builtin_amdgcn_rcpf((float)nch);
        for (int u = wave; u < units; u += kWaves) {
            const int g = uni(fdiv(u, rch)), f = (u - g * nch) * 64 + lane;
            const int fc = min(f, nfib - 1), q = fdiv(fc, rinner), r = fc - __mul24(q, inner);
            const T* x = in + __mul24(__mul24(q, m) + start_of(g), inner) + r;
            const T* b = B + 4 * nt * g;
            T a0 = T(0), a1 = T(0), a2 = T(0), a3 = T(0);
#pragma unroll 4
            for (int t = 0; t < nt; t++) {
                const T v = *x;
                x += inner;
                const typename Tap<T>::V w = *reinterpret_cast<const typename Tap<T>::V*>(b);
                b += 4;
                a0 = fma(w.x, v, a0);
                a1 = fma(w.y, v, a1);
                a2 = fma(w.z, v, a2);
                a3 = fma(w.w, v, a3);
            }
            if (f < nfib) {
                const T v[4] = {a0, a1, a2, a3};
                out(__mul24(__mul24(q, mc) + 4 * g, inner) + r, inner, uni(min(4, mc - 4 * g)), v);
            }
        }
    } else {
        // few fibres: a lane per output
        for (int e = threadIdx.x; e < nfib * mc; e += kT) {
            const int f = fdiv(e, rmc), i = e - __mul24(f, mc), g = i >> 2;
            const int q = fdiv(f, rinner), r = f - __mul24(q, inner);
            const T* x = in + __mul24(__mul24(q, m) + start_of(g), inner) + r;
            const T* b = B + 4 * __mul24(nt, g) + (i & 3);
            T a = T(0);
#pragma unroll 4
            for (int t = 0; t < nt; t++) {
                a = fma(*b, *x, a);
                b += 4;
                x += inner;
            }
            const T v[1] = {a};
            out(__mul24(__mul24(q, mc) + i, inner) + r, inner, 1, v);
        }
    }
}

// Phase ps (0 .. na - 1) of a level's correction, the active dimensions last
// first; the last phase gives the z of coarse nodes to fin(c, step, n, z): z[k] is
// that of node c + k step.  A: the level's arrays.
template <typename T, class Fin>
__device__ __forceinline__ void tail_phase(const TailLevel& L, const T* tab, T* A, int ps, Fin fin)
{
    const int na = uni(L.na), d = uni((L.dims >> (2 * ps)) & 3);
    const bool last = ps == na - 1;
    const T* const in = A + (ps == 0 ? 0 : ps == 1 ? L.p1 : L.p2);
    T* const o = A + (ps == 0 ? L.p1 : L.p2);
    const int outer = (d == 2) ? L.d[0].m * L.d[1].m : (d == 1) ? L.d[0].m : 1;
    const int inner = (d == 2) ? 1 : (d == 1) ? L.d[2].mc : L.d[1].mc * L.d[2].mc;
    const float rinner = (d == 2) ? 1.0f : (d == 1) ? L.d[2].rmc : L.d[1].rmc * L.d[2].rmc;
    tail_dots<8>(L.d[d], tab + L.d[d].B, in, outer, inner, rinner, [&](int c, int step, int n, const auto& v) {
        if (last) {
            fin(c, step, n, v);
        } else {
#pragma unroll
            for (int k = 0; k < (int)(sizeof(v) / sizeof(T)); k++)
                if (k < n) o[c + k * step] = v[k];
        }
    });
}

// Cells of a level: for every coarse node i, fn(i, ok, u, p, g): u[e] is the
// value of U at node 2 i + e of the level grid (e: bit d set, odd along
// dimension d), p[e] its interpolant from the coarse values G, ok[e] whether
// e > 0 is a fine node there; g the coarse value.  The interpolant is a sum
// over the corners, the neighbours along dim 0 first and along dim 2 last,
// each weighted by the product of its one-dimensional weights.  Every LDS read
// of a cell is issued before the first is used.
template <typename T, class Fn>
__device__ __forceinline__ void tail_cells(const TailLevel& L, const T* tab, const T* U, const T* G, Fn fn)
{
    const int Vc = uni(L.Vc), mc1 = L.d[1].mc, mc2 = L.d[2].mc, m2 = L.d[2].m, m12 = __mul24(L.d[1].m, m2);
    for (int c = threadIdx.x; c < Vc; c += kT) {
        int i[3];
        coarse_of(L, c, i[0], i[1], i[2]);
        bool has[3];
        T wl[3], wh[3];
        int up[3], fu[3];
        const int cs[3] = {__mul24(mc1, mc2), mc2, 1}, fs[3] = {m12, m2, 1};
#pragma unroll
        for (int d = 0; d < 3; d++) {
            const bool in = i[d] < L.d[d].mc - 1;
            has[d] = in && 2 * i[d] + 1 != L.d[d].ph;
            up[d] = in ? cs[d] : 0;
            fu[d] = in ? fs[d] : 0;
            // (of an inactive dimension no node is fine: any readable entry)
            const T* w = tab + (in ? L.d[d].w + 4 * i[d] + 2 : 0);
            wl[d] = w[0];
            wh[d] = w[1];
        }
        const int u0 = 2 * (__mul24(i[0], m12) + __mul24(i[1], m2) + i[2]);
        T g[8], u[8], p[8];
        bool ok[8];
#pragma unroll
        for (int e = 0; e < 8; e++) {
            g[e] = G[c + ((e & 1) ? up[0] : 0) + ((e & 2) ? up[1] : 0) + ((e & 4) ? up[2] : 0)];
            u[e] = U[u0 + ((e & 1) ? fu[0] : 0) + ((e & 2) ? fu[1] : 0) + ((e & 4) ? fu[2] : 0)];
        }
        p[0] = T(0);
        ok[0] = false;
#pragma unroll
        for (int e = 1; e < 8; e++) {
            ok[e] = (!(e & 1) || has[0]) && (!(e & 2) || has[1]) && (!(e & 4) || has[2]);
            T acc = T(0);
#pragma unroll
            for (int k = 0; k < 8; k++) {
                if (k & ~e) continue;
                T w = T(1);
#pragma unroll
                for (int d = 0; d < 3; d++)
                    if (e >> d & 1) w *= (k >> d & 1) ? wh[d] : wl[d];
                acc = fma(w, g[k], acc);
            }
            p[e] = acc;
        }
        fn(i, u0, fs, ok, u, p, g[0]);
    }
}

struct TailStatic {
    // offsets in the user's arrays of the finest tail level's nodes, per
    // dimension (node j of l levels on is node min(j 2^l, m - 1) there)
    int64_t off0[kTailOffs], off1[kTailOffs], off2[kTailOffs];
    // the levels' descriptions (each phase needs a dozen of their fields: from
    // LDS, since a scalar load that misses its cache waits some 600 cycles)
    TailLevel lv[kMaxTail];
};
static_assert(sizeof(TailStatic) + kTailLdsBytes <= 163840, "fits a CU's LDS");

// Offsets in the user's arrays of node (j0, j1, j2) of the level l steps after
// the tail's first.
struct TailUser {
    const int64_t *off0, *off1, *off2;
    int x0, x1, x2;
    __device__ __forceinline__ int64_t at0(int l, int j) const { return off0[min(j << l, x0)]; }
    __device__ __forceinline__ int64_t at1(int l, int j) const { return off1[min(j << l, x1)]; }
    __device__ __forceinline__ int64_t at2(int l, int j) const { return off2[min(j << l, x2)]; }
    __device__ __forceinline__ int64_t operator()(int l, int j0, int j1, int j2) const
    {
        return at0(l, j0) + at1(l, j1) + at2(l, j2);
    }
};

// What the input is: the finest level grid (the next ones are formed by the
// kernel), in the user's array or the workspace, there plus its correction or
// alone; or the classes, in the user's array.
enum TailIn { kTailGridZ, kTailGrid, kTailClasses };

// Descriptions, offsets, tables and input to LDS.
template <typename T, TailIn kIn, bool kLdsTab>
__device__ __forceinline__ TailUser tail_load(const TailArgs<T>& a, const T* src, T* lds, TailStatic& sm)
{
    constexpr bool kDec = kIn != kTailClasses;
    int64_t *const off0 = sm.off0, *const off1 = sm.off1, *const off2 = sm.off2;
    TailLevel* const lv = sm.lv;
    const int tid = threadIdx.x, nlev = a.nlev, k0 = a.k0;
    {
        const int* q = reinterpret_cast<const int*>(a.lv);
        int* o = reinterpret_cast<int*>(lv);
        for (int e = tid; e < nlev * (int)(sizeof(TailLevel) / 4); e += kT) o[e] = q[e];
    }
    // the tables are one contiguous range: their loads go out first
    constexpr int kTT = 4;
    const int ntab = kLdsTab ? a.tab_elems : 0;
    T tt[kTT];
    if (kLdsTab) {
#pragma unroll
        for (int q = 0; q < kTT; q++) tt[q] = a.tab[min(q * kT + tid, ntab - 1)];
    }
    if (tid < kTailOffs) {
        off0[tid] = min((int64_t)tid * (a.st[0] << k0), a.last[0]);
        off1[tid] = min((int64_t)tid * (a.st[1] << k0), a.last[1]);
        off2[tid] = min((int64_t)tid * (a.st[2] << k0), a.last[2]);
    }
    __syncthreads();  // descriptions, offsets
    const TailLevel L0 = lv[0];
    const int base = uni(L0.cum);
    T* const ltab = lds + a.data_elems;
    const TailUser user = {off0, off1, off2, L0.d[0].m - 1, L0.d[1].m - 1, L0.d[2].m - 1};
    // node idx of a level (its value v) to its LDS arrays A
    auto put = [&](const TailLevel& L, T* A, int idx, int j0, int j1, int j2, T v) {
        const bool coarse = ((j0 | j1 | j2) & 1) == 0;
        if (kDec && coarse)
            A[L.g + __mul24(__mul24(j0 >> 1, L.d[1].mc) + (j1 >> 1), L.d[2].mc) + (j2 >> 1)] = v;
        A[idx] = (coarse || phantom(L, j0, j1, j2)) ? T(0) : v;
    };
    // ---- loads: the finest level grid, then (recomposition) the coarser
    // levels' coefficients and the coarsest values, all issued before the
    // first is waited for
    T tmp[kTB];
    auto load0 = [&](int b0) {
#pragma unroll
        for (int q = 0; q < kTB; q++) {
            const int idx = min(b0 + q * kT + tid, L0.V - 1);
            int j0, j1, j2;
            node_of(L0, idx, j0, j1, j2);
            if (kDec && k0 > 0) {
                const int pk = packed_at(L0, j0, j1, j2);
                tmp[q] = (kIn == kTailGridZ) ? a.Wk[pk] + a.Z0[pk] : a.Wk[pk];
            } else {
                tmp[q] = src[user(0, j0, j1, j2)];
            }
        }
    };
    auto put0 = [&](int b0) {
#pragma unroll
        for (int q = 0; q < kTB; q++) {
            const int idx = b0 + q * kT + tid;
            int j0, j1, j2;
            node_of(L0, min(idx, L0.V - 1), j0, j1, j2);
            if (idx < L0.V) put(L0, lds, idx, j0, j1, j2, tmp[q]);
        }
    };
    load0(0);
    if (kDec) {
        // the coarser levels' arrays: their coarse nodes and phantoms stay zero
        for (int e = (nlev > 1 ? lv[1].cum - base : a.data_elems) + tid; e < a.data_elems; e += kT) lds[e] = T(0);
    } else {
        // nodes of the levels after the first, level by level, then the
        // coarsest values: element e of the sequence
        int rest = 0;
        for (int l = 1; l < nlev; l++) rest += lv[l].V;
        const TailLevel& Lt = lv[nlev - 1];
        const int all = rest + Lt.Vc;
        constexpr int kTC = 2;
        for (int b0 = 0; b0 < all; b0 += kTC * kT) {
            T v[kTC];
            int at[kTC];
            bool zero[kTC];
#pragma unroll
            for (int q = 0; q < kTC; q++) {
                int e = min(b0 + q * kT + tid, all - 1);
                int64_t o = 0;
                at[q] = 0;
                zero[q] = false;
                if (e >= rest) {
                    int i0, i1, i2;
                    coarse_of(Lt, e - rest, i0, i1, i2);
                    o = user(nlev, i0, i1, i2);
                    at[q] = Lt.cum - base + Lt.g + (e - rest);
                } else {
                    for (int l = 1; l < nlev; l++) {
                        const TailLevel& L = lv[l];
                        if (e >= 0 && e < L.V) {
                            int j0, j1, j2;
                            node_of(L, e, j0, j1, j2);
                            o = user(l, j0, j1, j2);
                            at[q] = L.cum - base + e;
                            zero[q] = ((j0 | j1 | j2) & 1) == 0 || phantom(L, j0, j1, j2);
                        }
                        e -= L.V;
                    }
                }
                v[q] = src[o];
            }
#pragma unroll
            for (int q = 0; q < kTC; q++)
                if (b0 + q * kT + tid < all) lds[at[q]] = zero[q] ? T(0) : v[q];
        }
    }
    put0(0);
    for (int b0 = kTB * kT; b0 < L0.V; b0 += kTB * kT) {
        load0(b0);
        put0(b0);
    }
    if (kLdsTab) {
#pragma unroll
        for (int q = 0; q < kTT; q++)
            if (q * kT + tid < ntab) ltab[q * kT + tid] = tt[q];
        for (int e = kTT * kT + tid; e < ntab; e += kT) ltab[e] = a.tab[e];
    }
    __syncthreads();
    return user;
}

template <typename T, bool kDec, bool kLdsTab>
__device__ __forceinline__ void tail_body(const TailArgs<T>& a, const T* src, T* dst, T* lds, TailStatic& sm)
{
    const TailUser user = tail_load<T, kDec ? kTailGridZ : kTailClasses, kLdsTab>(a, src, lds, sm);
    TailLevel* const lv = sm.lv;
    const int nlev = a.nlev, k0 = a.k0;
    const TailLevel& L0 = lv[0];
    const int base = uni(L0.cum), tbase = uni(L0.tab);
    T* const ltab = lds + a.data_elems;
    // tables of a level
    auto tables = [&](const TailLevel& L) -> const T* {
        return (kLdsTab ? (const T*)ltab : a.tab) + (L.tab - tbase);
    };

    if (kDec) {
        for (int l = 0; l < nlev; l++) {
            const TailLevel& L = lv[l];
            const T* const tab = tables(L);
            T* const A = lds + (L.cum - base);
            const T* const G = A + L.g;
            tail_cells(L, tab, A, G,
                       [&](const int (&i)[3], int u0, const int (&fs)[3], const bool (&ok)[8], const T (&u)[8],
                           const T (&p)[8], T) {
                           int64_t o[3][2];
#pragma unroll
                           for (int b = 0; b < 2; b++) {
                               o[0][b] = user.at0(l, 2 * i[0] + b);
                               o[1][b] = user.at1(l, 2 * i[1] + b);
                               o[2][b] = user.at2(l, 2 * i[2] + b);
                           }
#pragma unroll
                           for (int e = 1; e < 8; e++) {
                               const T v = u[e] - p[e];
                               if (ok[e]) {
                                   A[u0 + ((e & 1) ? fs[0] : 0) + ((e & 2) ? fs[1] : 0) + ((e & 4) ? fs[2] : 0)] = v;
                                   dst[o[0][e & 1] + o[1][e >> 1 & 1] + o[2][e >> 2]] = v;
                               }
                           }
                       });
            __syncthreads();
            // z added to the coarse values, which are the next level's grid
            const bool lastl = l + 1 == nlev;
            const TailLevel& N = lv[lastl ? l : l + 1];
            T* const An = lds + (N.cum - base);
            const int e0 = L.d[0].mc - 1, e1 = L.d[1].mc - 1, e2 = L.d[2].mc - 1;
            const int f0 = N.d[0].m - 1, f1 = N.d[1].m - 1, f2 = N.d[2].m - 1;
            const int g1 = N.d[1].mc, g2 = N.d[2].mc, gn = N.g;
            auto fin = [&](int c, int step, int n, const auto& z) {
                constexpr int NZ = (int)(sizeof(z) / sizeof(T));
                T v[NZ];
#pragma unroll
                for (int k = 0; k < NZ; k++) v[k] = G[c + (k < n ? k * step : 0)] + z[k];
#pragma unroll
                for (int k = 0; k < NZ; k++) {
                    if (k >= n) break;
                    int i0, i1, i2;
                    coarse_of(L, c + k * step, i0, i1, i2);
                    if (lastl) {
                        dst[user(l + 1, i0, i1, i2)] = v[k];
                        continue;
                    }
                    // index in the next level grid with its phantom
                    const int j0 = (i0 == e0) ? f0 : i0, j1 = (i1 == e1) ? f1 : i1, j2 = (i2 == e2) ? f2 : i2;
                    const int s = ((j0 | j1 | j2) & 1) ? 0 : 1;
                    An[(s ? gn : 0) + __mul24(__mul24(j0 >> s, s ? g1 : f1 + 1) + (j1 >> s), s ? g2 : f2 + 1) + (j2 >> s)] = v[k];
                }
            };
            const int na = uni(L.na);
            for (int ps = 0; ps < na; ps++) {
                tail_phase(L, tab, A, ps, fin);
                __syncthreads();
            }
        }
    } else {
        // every level's correction, then the chain; z_l goes to the level's
        // own G, except the coarsest level's, which is subtracted at once
        // from the coarsest values there
        const int na = uni(L0.na);
        for (int ps = 0; ps < na; ps++) {
            for (int l = 0; l < nlev; l++) {
                const TailLevel& L = lv[l];
                T* const A = lds + (L.cum - base);
                T* const G = A + L.g;
                const bool top = l + 1 == nlev;
                tail_phase(L, tables(L), A, ps, [&](int c, int step, int n, const auto& z) {
                    constexpr int NZ = (int)(sizeof(z) / sizeof(T));
                    T v[NZ];
#pragma unroll
                    for (int k = 0; k < NZ; k++) v[k] = top ? G[c + (k < n ? k * step : 0)] - z[k] : z[k];
#pragma unroll
                    for (int k = 0; k < NZ; k++)
                        if (k < n) G[c + k * step] = v[k];
                });
            }
            __syncthreads();
        }
        for (int l = nlev - 1; l >= 0; l--) {
            const TailLevel& L = lv[l];
            const T* const A = lds + (L.cum - base);
            // node (j0, j1, j2) of this level's grid: subtract the next finer
            // level's z (it is that level's coarse node), or write it out
            const bool last = l == 0;
            const TailLevel& N = lv[last ? 0 : l - 1];
            T* const Gn = lds + (N.cum - base) + N.g;
            tail_cells(L, tables(L), A, A + L.g,
                       [&](const int (&i)[3], int, const int (&)[3], const bool (&ok)[8], const T (&u)[8], const T (&p)[8],
                           T g) {
                           // places in the packed grid, or in the user's array
                           int k[3][2];
                           int64_t o[3][2];
#pragma unroll
                           for (int b = 0; b < 2; b++) {
                               k[0][b] = __mul24(__mul24(min(2 * i[0] + b, L.d[0].act - 1), L.d[1].act), L.d[2].act);
                               k[1][b] = __mul24(min(2 * i[1] + b, L.d[1].act - 1), L.d[2].act);
                               k[2][b] = min(2 * i[2] + b, L.d[2].act - 1);
                               if (last && k0 == 0) {
                                   o[0][b] = user.at0(0, 2 * i[0] + b);
                                   o[1][b] = user.at1(0, 2 * i[1] + b);
                                   o[2][b] = user.at2(0, 2 * i[2] + b);
                               }
                           }
                           T z[8];
#pragma unroll
                           for (int e = 0; e < 8; e++)
                               z[e] = last ? T(0) : Gn[k[0][e & 1] + k[1][e >> 1 & 1] + k[2][e >> 2]];
#pragma unroll
                           for (int e = 0; e < 8; e++) {
                               const T v = (e == 0) ? g : u[e] + p[e];
                               if (e > 0 && !ok[e]) continue;
                               const int pk = k[0][e & 1] + k[1][e >> 1 & 1] + k[2][e >> 2];
                               if (!last)
                                   Gn[pk] = v - z[e];
                               else if (k0 == 0)
                                   dst[o[0][e & 1] + o[1][e >> 1 & 1] + o[2][e >> 2]] = v;
                               else
                                   a.Wk[pk] = v;
                           }
                       });
            __syncthreads();
        }
    }
}

// ---- adjoints ---------------------------------------------------------------
// The transposes of the same steps, with the columns of B (t = B^T y, expanded
// dimension by dimension, 0 first, through the arrays that the reductions use
// in reverse).  Adjoint of the decomposition, coarse to fine:
//   O = g + B^T G at the fine nodes, O = G - P^T O at the coarse ones,
// which is the next finer level's G; of the recomposition, fine to coarse:
//   G' = G + P^T g (the next level grid), out = g - B^T G' at the fine nodes,
// where the expansions of all levels follow the chain of the G and share three
// phases.  The last steps of a 257^3 FP32 adjoint, from 17^3 nodes on, took seven
// launches (58 us in the kernels) and a copy per step; 23 us here.

// P^T U at coarse node (i0, i1, i2): its up to 26 fine neighbours (U is zero at
// coarse nodes).
template <typename T>
__device__ __forceinline__ T tail_restrict(const TailLevel& L, const T* tab, const T* U, const int (&i)[3])
{
    const int m2 = L.d[2].m, m12 = __mul24(L.d[1].m, m2);
    const int fs[3] = {m12, m2, 1};
    T w[3][2];
    int o[3][2];
#pragma unroll
    for (int d = 0; d < 3; d++) {
        const bool lo = i[d] > 0, hi = i[d] < L.d[d].mc - 1;
        const T* q = tab + L.d[d].w + 4 * i[d];
        w[d][0] = lo ? q[-1] : T(0);
        w[d][1] = hi ? q[2] : T(0);
        o[d][0] = lo ? -fs[d] : 0;
        o[d][1] = hi ? fs[d] : 0;
    }
    const T* const u = U + 2 * (__mul24(i[0], m12) + __mul24(i[1], m2) + i[2]);
    T r[3];
#pragma unroll
    for (int b0 = 0; b0 < 3; b0++) {
        T q[3];
#pragma unroll
        for (int b1 = 0; b1 < 3; b1++) {
            const T* x = u + (b0 == 0 ? o[0][0] : b0 == 2 ? o[0][1] : 0) + (b1 == 0 ? o[1][0] : b1 == 2 ? o[1][1] : 0);
            q[b1] = fma(w[2][1], x[o[2][1]], fma(w[2][0], x[o[2][0]], x[0]));
        }
        r[b0] = fma(w[1][1], q[2], fma(w[1][0], q[0], q[1]));
    }
    return fma(w[0][1], r[2], fma(w[0][0], r[0], r[1]));
}

// Phase ps (0 .. na - 1) of B^T G; the last one gives the t of the level's nodes
// to fin(idx, step, n, t).
template <typename T, class Fin>
__device__ __forceinline__ void tail_adj_phase(const TailLevel& L, const T* tab, T* A, int ps, Fin fin)
{
    const int na = uni(L.na), q = na - 1 - ps, d = uni((L.dims >> (2 * q)) & 3);
    const T* const in = A + (ps == 0 ? L.g : q == 0 ? L.p1 : L.p2);
    T* const o = A + (q == 1 ? L.p1 : L.p2);
    const int outer = (d == 2) ? L.d[0].m * L.d[1].m : (d == 1) ? L.d[0].m : 1;
    const int inner = (d == 2) ? 1 : (d == 1) ? L.d[2].mc : L.d[1].mc * L.d[2].mc;
    const float rinner = (d == 2) ? 1.0f : (d == 1) ? L.d[2].rmc : L.d[1].rmc * L.d[2].rmc;
    tail_dots<2>(L.d[d], tab + L.d[d].B, in, outer, inner, rinner, [&](int c, int step, int n, const auto& v) {
        if (q == 0) {
            fin(c, step, n, v);
        } else {
#pragma unroll
            for (int k = 0; k < (int)(sizeof(v) / sizeof(T)); k++)
                if (k < n) o[c + k * step] = v[k];
        }
    });
}

template <typename T, bool kRec, bool kLdsTab>
__device__ __forceinline__ void tail_adj_body(const TailArgs<T>& a, T* lds, TailStatic& sm)
{
    const TailUser user = tail_load<T, kRec ? kTailGrid : kTailClasses, kLdsTab>(a, a.src, lds, sm);
    TailLevel* const lv = sm.lv;
    const int nlev = a.nlev, k0 = a.k0;
    const TailLevel& L0 = lv[0];
    const int base = uni(L0.cum), tbase = uni(L0.tab), na = uni(L0.na);
    T* const ltab = lds + a.data_elems;
    auto tables = [&](const TailLevel& L) -> const T* {
        return (kLdsTab ? (const T*)ltab : a.tab) + (L.tab - tbase);
    };
    T* const dst = a.dst;
    if (!kRec) {
        for (int l = nlev - 1; l >= 0; l--) {
            const TailLevel& L = lv[l];
            const T* const tab = tables(L);
            T* const A = lds + (L.cum - base);
            T* const G = A + L.g;
            // O at node idx: the next finer level's G, or out
            const TailLevel& N = lv[max(l - 1, 0)];
            T* const Gn = lds + (N.cum - base) + N.g;
            auto put = [&](int idx, int j0, int j1, int j2, T v) {
                if (l > 0)
                    Gn[idx] = v;
                else if (k0 == 0)
                    dst[user(0, j0, j1, j2)] = v;
                else
                    a.Wk[idx] = v;
            };
            for (int ps = 0; ps < na; ps++) {
                tail_adj_phase(L, tab, A, ps, [&](int c, int step, int n, const auto& t) {
#pragma unroll
                    for (int k = 0; k < (int)(sizeof(t) / sizeof(T)); k++) {
                        if (k >= n) break;
                        const int idx = c + k * step;
                        int j0, j1, j2;
                        node_of(L, idx, j0, j1, j2);
                        if (((j0 | j1 | j2) & 1) == 0) continue;
                        const T v = A[idx] + t[k];
                        A[idx] = v;
                        put(idx, j0, j1, j2, v);
                    }
                });
                __syncthreads();
            }
            for (int c = threadIdx.x; c < L.Vc; c += kT) {
                int i[3];
                coarse_of(L, c, i[0], i[1], i[2]);
                const T v = G[c] - tail_restrict(L, tab, A, i);
                const int idx = 2 * (__mul24(__mul24(i[0], L.d[1].m) + i[1], L.d[2].m) + i[2]);
                put(idx, 2 * i[0], 2 * i[1], 2 * i[2], v);
            }
            __syncthreads();
        }
    } else {
        for (int l = 0; l < nlev; l++) {
            const TailLevel& L = lv[l];
            const T* const tab = tables(L);
            T* const A = lds + (L.cum - base);
            T* const G = A + L.g;
            const bool last = l + 1 == nlev;
            const TailLevel& N = lv[last ? l : l + 1];
            T* const An = lds + (N.cum - base);
            for (int c = threadIdx.x; c < L.Vc; c += kT) {
                int i[3];
                coarse_of(L, c, i[0], i[1], i[2]);
                const T h = G[c] + tail_restrict(L, tab, A, i);
                G[c] = h;
                if (last)
                    dst[user(nlev, i[0], i[1], i[2])] = h;
                else if (((i[0] | i[1] | i[2]) & 1) == 0)
                    An[N.g + __mul24(__mul24(i[0] >> 1, N.d[1].mc) + (i[1] >> 1), N.d[2].mc) + (i[2] >> 1)] = h;
                else
                    An[c] = h;
            }
            __syncthreads();
        }
        for (int ps = 0; ps < na; ps++) {
            for (int l = 0; l < nlev; l++) {
                const TailLevel& L = lv[l];
                T* const A = lds + (L.cum - base);
                tail_adj_phase(L, tables(L), A, ps, [&](int c, int step, int n, const auto& t) {
#pragma unroll
                    for (int k = 0; k < (int)(sizeof(t) / sizeof(T)); k++) {
                        if (k >= n) break;
                        const int idx = c + k * step;
                        int j0, j1, j2;
                        node_of(L, idx, j0, j1, j2);
                        if ((j0 | j1 | j2) & 1) dst[user(l, j0, j1, j2)] = A[idx] - t[k];
                    }
                });
            }
            __syncthreads();
        }
    }
}

extern __shared__ __align__(16) unsigned char tail_lds[];

template <typename T, bool kDec, bool kLdsTab>
__global__ void __launch_bounds__(kT) k_tail(TailArgs<T> a)
{
    __shared__ TailStatic sm;
    tail_body<T, kDec, kLdsTab>(a, a.src, a.dst, reinterpret_cast<T*>(tail_lds), sm);
}

template <typename T, bool kRec, bool kLdsTab>
__global__ void __launch_bounds__(kT) k_tail_adj(TailArgs<T> a)
{
    __shared__ TailStatic sm;
    tail_adj_body<T, kRec, kLdsTab>(a, reinterpret_cast<T*>(tail_lds), sm);
}

// One workgroup per entry of a batch; arguments in device memory.
template <typename T>
__global__ void __launch_bounds__(kT) k_tail_batch(const TailArgs<T>* __restrict__ args, const int* __restrict__ field,
                                                   const T* const* __restrict__ src, T* const* __restrict__ dst)
{
    __shared__ TailStatic sm;
    const int f = field[blockIdx.x];
    const TailArgs<T>& a = args[blockIdx.x];
    if (tail_tab_in_lds(a))
        tail_body<T, true, true>(a, src[f], dst[f], reinterpret_cast<T*>(tail_lds), sm);
    else
        tail_body<T, true, false>(a, src[f], dst[f], reinterpret_cast<T*>(tail_lds), sm);
}

// LDS beyond 64 KB has to be asked for once per kernel and device.
template <typename K>
hipError_t allow_lds(K kern, size_t bytes, bool (&done)[64])
{
    if (bytes <= 65536) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (done[dev]) return hipSuccess;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kTailLdsBytes);
    if (e == hipSuccess) done[dev] = true;
    return e;
}

template <typename T, bool kDec, bool kLdsTab>
hipError_t launch_tail_cfg(const TailArgs<T>& a, size_t bytes, hipStream_t st)
{
    static bool done[64] = {};
    const hipError_t e = allow_lds(k_tail<T, kDec, kLdsTab>, bytes, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_tail<T, kDec, kLdsTab>), dim3(1), dim3(kT), bytes, st, a);
    return hipGetLastError();
}

template <typename T, bool kRec, bool kLdsTab>
hipError_t launch_adj_cfg(const TailArgs<T>& a, size_t bytes, hipStream_t st)
{
    static bool done[64] = {};
    const hipError_t e = allow_lds(k_tail_adj<T, kRec, kLdsTab>, bytes, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_tail_adj<T, kRec, kLdsTab>), dim3(1), dim3(kT), bytes, st, a);
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_tail_adjoint(const TailArgs<T>& a, bool recompose, hipStream_t st)
{
    const size_t bytes = sizeof(T) * (size_t)tail_lds_elems(a);
    if (tail_tab_in_lds(a))
        return recompose ? launch_adj_cfg<T, true, true>(a, bytes, st) : launch_adj_cfg<T, false, true>(a, bytes, st);
    return recompose ? launch_adj_cfg<T, true, false>(a, bytes, st) : launch_adj_cfg<T, false, false>(a, bytes, st);
}

template <typename T>
hipError_t launch_tail_batch(const TailArgs<T>* dev_args, const int* field, const T* const* src, T* const* dst, int n,
                             int lds_elems, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    static bool done[64] = {};
    const size_t bytes = sizeof(T) * (size_t)lds_elems;
    const hipError_t e = allow_lds(k_tail_batch<T>, bytes, done);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_tail_batch<T>), dim3((unsigned)n), dim3(kT), bytes, st, dev_args, field, src, dst);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tail(const TailArgs<T>& a, bool decompose, hipStream_t st)
{
    const size_t bytes = sizeof(T) * (size_t)tail_lds_elems(a);
    if (tail_tab_in_lds(a))
        return decompose ? launch_tail_cfg<T, true, true>(a, bytes, st) : launch_tail_cfg<T, false, true>(a, bytes, st);
    return decompose ? launch_tail_cfg<T, true, false>(a, bytes, st) : launch_tail_cfg<T, false, false>(a, bytes, st);
}

template hipError_t launch_tail_adjoint<float>(const TailArgs<float>&, bool, hipStream_t);
template hipError_t launch_tail_adjoint<double>(const TailArgs<double>&, bool, hipStream_t);
template hipError_t launch_tail<float>(const TailArgs<float>&, bool, hipStream_t);
template hipError_t launch_tail<double>(const TailArgs<double>&, bool, hipStream_t);
template hipError_t launch_tail_batch<float>(const TailArgs<float>*, const int*, const float* const*, float* const*,
                                             int, int, hipStream_t);
template hipError_t launch_tail_batch<double>(const TailArgs<double>*, const int*, const double* const*,
                                              double* const*, int, int, hipStream_t);

}  // namespace mgr
