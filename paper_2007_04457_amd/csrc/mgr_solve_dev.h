// Device code of the partitioned Thomas solve (see mgr_solve.hip for the
// method): shared by the per-level kernels and the batched work-queue
// kernel.  Internal; included by .hip files only.
#pragma once
#include "mgr_internal.h"

namespace mgr {
namespace {

constexpr int kBlk = 256;
constexpr int kMaxSegWG = 16;  // strided single-launch form: S <= 16

// LDS position of staged element e: one pad element per 32
__device__ __forceinline__ int padded(int e) { return e + (e >> 5); }

struct FibreMap {
    int64_t n, inner, outer, nfib;
    int S;
};

// Interior [lo, lo + len) of segment s.
__device__ __forceinline__ void seg_range(const FibreMap& m, int s, int& lo, int& len)
{
    lo = s * kSeg + (s > 0 ? 1 : 0);
    const int hi = (s == m.S - 1) ? (int)m.n : (s + 1) * kSeg;
    len = hi - lo;
}

// Segment-local Thomas solve in registers with padded tables (L = forward
// multipliers, U = super-diagonal, IP = inverse pivots; zero past the
// segment so padded slots come out as 0).
// The roundings are fixed (explicit FMAs), so that every form gives the same
// values.
template <typename T>
__device__ __forceinline__ void seg_solve(T (&v)[kSlot], const T* L, const T* U, const T* IP)
{
#pragma unroll
    for (int q = 1; q < kSlot; q++) v[q] = fma(-L[q], v[q - 1], v[q]);
    T z = T(0);
#pragma unroll
    for (int q = kSlot - 1; q >= 0; q--) {
        z = fma(-U[q], z, v[q]) * IP[q];
        v[q] = z;
    }
}

// y at the last node of segment s (the fibre's first has kSeg nodes, the
// others one fewer; the last segment's end is next to no separator).
template <typename T>
__device__ __forceinline__ T seg_last(const T (&v)[kSlot], int s)
{
    return s == 0 ? v[kSeg - 1] : v[kSeg - 2];
}

// Separator elimination and the segments' final values with one fixed
// rounding (explicit FMAs), shared by every solve form so that they all give
// the same values: right-hand side of separator k from f there and the
// neighbouring segments' end values, its forward elimination, its back
// substitution, and z = y + alpha z_left + beta z_right in a segment.
template <typename T>
__device__ __forceinline__ T sep_rhs(T f, T sub, T ylast, T sup, T yfirst)
{
    return fma(-sup, yfirst, fma(-sub, ylast, f));
}
template <typename T>
__device__ __forceinline__ T sep_fwd(T rhs, T l, T g)
{
    return fma(-l, g, rhs);
}
template <typename T>
__device__ __forceinline__ T sep_bwd(T f, T u, T z, T ip)
{
    return fma(-u, z, f) * ip;
}
template <typename T>
__device__ __forceinline__ T seg_final(T y, T alpha, T zl, T beta, T zr)
{
    return fma(beta, zr, fma(alpha, zl, y));
}

// Tables of segments s0 .. s0 + ns - 1 to LDS: the segment tables (L, U, IP,
// alpha, beta) and the separators' (sub, sup, sl, sip, su), all loads of a turn
// ahead of its stores, so that one memory latency covers both.
template <typename T, int NT, int NS>
__device__ __forceinline__ void stage_tables(const SolveTables<T>& tb, int s0, int ns, int tid, int nthr,
                                             T (&tab)[5][NT], T (&septab)[5][NS])
{
    for (int e = tid; e < ns * kSlot; e += nthr) {
        const int g = s0 * kSlot + e, k = s0 + min(e, ns - 1);
        const T a[5] = {tb.L[g], tb.U[g], tb.IP[g], tb.A[g], tb.B[g]};
        const T b[5] = {tb.ssub[k], tb.ssup[k], tb.sl[k], tb.sip[k], tb.su[k]};
#pragma unroll
        for (int q = 0; q < 5; q++) tab[q][e] = a[q];
        if (e < ns)
#pragma unroll
            for (int q = 0; q < 5; q++) septab[q][e] = b[q];
    }
}

// The final values of a whole segment to put(q, value), q descending, in groups:
// a group's values before the first of them is stored.  Under a store's
// condition (slot in the segment) the table reads would each wait their own
// round trip to the LDS (plane solve, 33 slots: 4300 cycles, 2000 so); all
// reads ahead of all stores would need more registers than there are.
template <typename T, class Put>
__device__ __forceinline__ void seg_finals(T (&v)[kSlot], const T* ta, T zl, const T* tb, T zr, Put put)
{
    constexpr int G = 11;
    static_assert(kSlot % G == 0, "whole groups");
#pragma unroll
    for (int g = kSlot - G; g >= 0; g -= G) {
#pragma unroll
        for (int q = 0; q < G; q++) v[g + q] = seg_final(v[g + q], ta[g + q], zl, tb[g + q], zr);
#pragma unroll
        for (int q = G - 1; q >= 0; q--) put(g + q, v[g + q]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A separator whose neighbours' terms are below the working precision
// (SolveTables::dec).
template <typename T>
__device__ __forceinline__ T sep_alone(T f, T sub, T ylast, T sup, T yfirst, T ip)
{
    return sep_rhs(f, sub, ylast, sup, yfirst) * ip;
}

// Separator system of one fibre from the separator f values (in sep[], which
// receives z) and the segment-end values; coefficient tables per separator.
template <typename T>
__device__ __forceinline__ void sep_solve(int S, T* sep, int64_t sstride, const T* yfirst,
                                          const T* ylast, int64_t ystride, const T* ssub,
                                          const T* ssup, const T* sl, const T* sip,
                                          const T* su)
{
    T g = T(0);
    for (int k = 1; k < S; k++) {
        const T rhs = sep_rhs(sep[k * sstride], ssub[k], ylast[(k - 1) * ystride], ssup[k], yfirst[k * ystride]);
        g = (k == 1) ? rhs : sep_fwd(rhs, sl[k], g);
        sep[k * sstride] = g;
    }
    T z = T(0);
    for (int k = S - 1; k >= 1; k--) {
        z = (k == S - 1) ? sep[k * sstride] * sip[k] : sep_bwd(sep[k * sstride], su[k], z, sip[k]);
        sep[k * sstride] = z;
    }
}

// ---- strided dimensions, one launch ---------------------------------------
// A tile of FB neighbouring fibres (coalesced) x S segments; lane j of
// segment s handles fibre fib0 + j.  The per-level launch uses FB = 64 (one
// wave per segment); the batched kernel packs FB = 16 fibres x up to 16
// segments into 256 threads.
template <typename T>
struct StridedSmem {
    T tab[5][kMaxSegWG * kSlot];  // L, U, IP, alpha, beta
    T septab[5][kMaxSegWG];       // sub, sup, sl, sip, su at separators
    T end[2][kMaxSegWG * 64];     // y at the two ends of each segment [s][j]
    T sep[kMaxSegWG * 64];        // f, then z, at each separator [s][j]
};

// s: the lane's segment within the workgroup, of the ns segments s0 .. s0 +
// ns - 1 (a whole fibre, or a chunk of one whose separators do not couple:
// its two outer separators are then in zb, the chunk's own at zb[fib], the
// next one's at zb[nfib + fib]).  kAllSeg: every s < ns.
template <typename T, int FB, bool kAllSeg>
__device__ __forceinline__ void solve_strided_tile(const T* in, T* F, const FibreMap& m,
                                                   const SolveTables<T>& tb, int64_t fib0, int s,
                                                   int j, int nthr, int tid, StridedSmem<T>& sm,
                                                   int s0, int ns, const T* __restrict__ zb)
{
    const int S = m.S;
    const bool inseg = kAllSeg || s < ns;
    const int sc = kAllSeg ? s : (inseg ? s : ns - 1);
    const int64_t fib = fib0 + j;
    const bool active = inseg && fib < m.nfib;
    const int64_t fc = fib < m.nfib ? fib : m.nfib - 1;  // idle lanes read a valid fibre
    const int64_t base = (fc / m.inner) * m.n * m.inner + fc % m.inner;
    const bool outer_l = s == 0 && s0 > 0, outer_r = s == ns - 1 && s0 + ns < S;
    int lo, len;
    seg_range(m, s0 + sc, lo, len);
    // the fibre loads are issued first and the tables' after them, so that
    // one memory latency covers both (staging the tables first would wait
    // for their loads before the fibre loads were issued)
    T v[kSlot];
#pragma unroll
    for (int q = 0; q < kSlot; q++) v[q] = in[base + (int64_t)(lo + min(q, len - 1)) * m.inner];
    const T fsep = in[base + (int64_t)((s0 + sc) * kSeg) * m.inner];  // f at the segment's left separator
    T zol = T(0), zor = T(0);
    if (outer_l) zol = zb[fc];
    if (outer_r) zor = zb[m.nfib + fc];
    stage_tables(tb, s0, ns, tid, nthr, sm.tab, sm.septab);
    if (inseg) sm.sep[s * FB + j] = (s0 + s > 0) ? fsep : T(0);
    __syncthreads();  // tables staged
    seg_solve(v, &sm.tab[0][sc * kSlot], &sm.tab[1][sc * kSlot], &sm.tab[2][sc * kSlot]);
    if (inseg) {
        sm.end[0][s * FB + j] = v[0];
        sm.end[1][s * FB + j] = seg_last(v, s0 + s);
    }
    __syncthreads();
    T zl, zr;
    if (!tb.dec) {
        if (s == 0 && S > 1)
            sep_solve(S, &sm.sep[j], FB, &sm.end[0][j], &sm.end[1][j], FB, sm.septab[0], sm.septab[1],
                      sm.septab[2], sm.septab[3], sm.septab[4]);
        __syncthreads();
    }
    if (!active) return;
    // the separators left and right of the segment, read without a condition
    // (indices clamped to a separator there is)
    auto sep = [&](int k) {
        const int kc = min(max(k, ns > 1 ? 1 : 0), ns - 1), km = max(kc - 1, 0);
        const T z = sm.sep[kc * FB + j];
        const T w = sep_alone(z, sm.septab[0][kc], sm.end[1][km * FB + j], sm.septab[1][kc], sm.end[0][kc * FB + j],
                              sm.septab[3][kc]);
        return tb.dec ? w : z;
    };
    const T sl = sep(s), sr = sep(s + 1);
    zl = (s > 0) ? sl : zol;
    zr = (s < ns - 1) ? sr : zor;
    seg_finals(v, &sm.tab[3][s * kSlot], zl, &sm.tab[4][s * kSlot], zr, [&](int q, T x) {
        if (q < len) F[base + (int64_t)(lo + q) * m.inner] = x;
    });
    if (s0 + s > 0) F[base + (int64_t)((s0 + s) * kSeg) * m.inner] = zl;
}

// ---- long fibres whose separators do not couple ----------------------------
// The separators between chunks (every ns-th of a fibre), each from the 31
// rows on either side of it: with alpha and beta the segments' responses to
// it, z = sip (f + sum beta f over the segment before + sum alpha f over the
// segment after), which is the separator's row with the segments' end values
// written out as the inner products they are.  zb[(b - 1) * nfib + fib] for
// b = 1 .. chunks - 1.
__device__ __forceinline__ int chunk_bounds(const FibreMap& m, int ns) { return (m.S + ns - 1) / ns - 1; }

// Weight of row p - 31 + j around separator s at row p (1 at the separator).
template <typename T>
__device__ __forceinline__ T sep_weight(const SolveTables<T>& tb, int s, int j)
{
    if (j < 31) return tb.B[(s - 1) * kSlot + 1 + j - (s > 1 ? 1 : 0)];
    if (j == 31) return T(1);
    return tb.A[s * kSlot + j - 32];
}

// One separator of one fibre per lane (strided dimensions).
template <typename T>
__device__ __forceinline__ void sep_bounds_strided(const T* __restrict__ F, T* __restrict__ zb, const FibreMap& m,
                                                   const SolveTables<T>& tb, int ns, int bx, int b)
{
    const int64_t fib = (int64_t)bx * kBlk + threadIdx.x;
    if (fib >= m.nfib) return;
    const int64_t base = (fib / m.inner) * m.n * m.inner + fib % m.inner;
    const int s = (b + 1) * ns, p = s * kSeg;
    T acc = T(0);
    for (int j0 = 0; j0 < 63; j0 += 21) {
        T v[21];
#pragma unroll
        for (int q = 0; q < 21; q++) v[q] = F[base + (int64_t)min(p - 31 + j0 + q, (int)m.n - 1) * m.inner];
#pragma unroll
        for (int q = 0; q < 21; q++) acc = fma(sep_weight(tb, s, j0 + q), v[q], acc);
    }
    zb[(int64_t)b * m.nfib + fib] = acc * tb.sip[s];
}

// One separator of one contiguous fibre per wave: lane j takes row
// p - 31 + j, and the wave sums.  u: separator of the launch, fibres fastest.
template <typename T>
__device__ __forceinline__ void sep_bounds_rows(const T* __restrict__ F, T* __restrict__ zb, const FibreMap& m,
                                                const SolveTables<T>& tb, int ns, int64_t u)
{
    if (u >= m.nfib * chunk_bounds(m, ns)) return;
    const int b = (int)(u / m.nfib);
    const int64_t fib = u - b * m.nfib;
    const int s = (b + 1) * ns, p = s * kSeg, j = threadIdx.x & 63;
    T acc = T(0);
    if (j < 63) acc = sep_weight(tb, s, j) * F[fib * m.n + min(p - 31 + j, (int)m.n - 1)];
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) acc += __shfl_xor(acc, w);
    if (j == 0) zb[(int64_t)b * m.nfib + fib] = acc * tb.sip[s];
}

// Rows [row0, row0 + nrows) x segments [s0, s0 + ns) (nrows * ns <= kBlk,
// nrows * (ns * kSeg + 1) <= kSpan): the chunk's columns, from its own left
// separator on, are staged through LDS, solved and written back.
template <typename T, int kSpan, bool kLdsTab>
struct ChunkSmem {
    T f[kSpan + kSpan / 32 + 1];
    T end[2][kBlk];
    T tab[5][kLdsTab ? kMaxSegWG * kSlot : 1];
};
template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void solve_chunk_rows(T* __restrict__ F, const FibreMap& m, const SolveTables<T>& tb,
                                                 int64_t row0, int nrows, int s0, int ns, const T* __restrict__ zb,
                                                 ChunkSmem<T, kSpan, kLdsTab>& sm)
{
    const int tid = threadIdx.x, n = (int)m.n;
    const int c0 = s0 * kSeg;                                   // the chunk's first column
    const int c1 = (s0 + ns >= m.S) ? n : (s0 + ns) * kSeg;     // one past its last
    const int w = c1 - c0, span = nrows * w;
    // (row, segment) of the lane; segment fastest
    const int r = tid / ns, s = tid - r * ns;
    const bool active = r < nrows;
    const int rr = active ? r : 0;
    constexpr int NQ = (kSpan + kBlk - 1) / kBlk;
    T tmp[NQ];
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        const int e = min(q * kBlk + tid, span - 1);
        const int er = e / w;
        tmp[q] = F[(row0 + er) * n + c0 + (e - er * w)];
    }
    T zl = T(0), zr = T(0);
    const int64_t fib = row0 + rr;
    if (s == 0 && s0 > 0) zl = zb[fib];
    if (s == ns - 1 && s0 + ns < m.S) zr = zb[m.nfib + fib];
    if (kLdsTab)
        for (int e = tid; e < ns * kSlot; e += kBlk) {
            const int g = s0 * kSlot + e;
            sm.tab[0][e] = tb.L[g];
            sm.tab[1][e] = tb.U[g];
            sm.tab[2][e] = tb.IP[g];
            sm.tab[3][e] = tb.A[g];
            sm.tab[4][e] = tb.B[g];
        }
#pragma unroll
    for (int q = 0; q < NQ; q++)
        if (q * kBlk + tid < span) sm.f[padded(q * kBlk + tid)] = tmp[q];
    __syncthreads();
    const int so = kLdsTab ? s * kSlot : (s0 + s) * kSlot;
    const T* const tA = kLdsTab ? &sm.tab[3][so] : tb.A + so;
    const T* const tB = kLdsTab ? &sm.tab[4][so] : tb.B + so;
    int lo, len;
    seg_range(m, s0 + s, lo, len);
    const int e0 = rr * w - c0;  // staged index of column c is e0 + c
    T v[kSlot];
#pragma unroll
    for (int q = 0; q < kSlot; q++) v[q] = sm.f[padded(e0 + lo + min(q, len - 1))];
    seg_solve(v, kLdsTab ? &sm.tab[0][so] : tb.L + so, kLdsTab ? &sm.tab[1][so] : tb.U + so,
              kLdsTab ? &sm.tab[2][so] : tb.IP + so);
    sm.end[0][tid] = v[0];
    sm.end[1][tid] = seg_last(v, s0 + s);
    __syncthreads();
    auto sep = [&](int k) {  // separator left of local segment k, clamped to one there is
        const int kc = min(max(k, ns > 1 ? 1 : 0), ns - 1), t = min(tid - s + kc, kBlk - 1), tm = max(t - 1, 0);
        return sep_alone(sm.f[padded(e0 + (s0 + kc) * kSeg)], tb.ssub[s0 + kc], sm.end[1][tm], tb.ssup[s0 + kc],
                         sm.end[0][t], tb.sip[s0 + kc]);
    };
    const T sl = sep(s), sr = sep(s + 1);
    zl = (s > 0) ? sl : zl;
    zr = (s < ns - 1) ? sr : zr;
    __syncthreads();  // every lane has read its separators
    if (active) {
        // (slots past the segment: to its last node, before that node's value)
        seg_finals(v, tA, zl, tB, zr, [&](int q, T x) { sm.f[padded(e0 + lo + min(q, len - 1))] = x; });
        if (s0 + s > 0) sm.f[padded(e0 + (s0 + s) * kSeg)] = zl;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        const int e = q * kBlk + tid;
        const int er = e / w;
        if (e < span) F[(row0 + er) * n + c0 + (e - er * w)] = sm.f[padded(e)];
    }
}

// ---- contiguous dimension, one launch --------------------------------------
// ---- contiguous dimension: rows staged through LDS ------------------------
constexpr int kSpanMax = kBlk * kSlot;
// Elements a per-level rows workgroup stages: the same bytes for either type
// (FP64 stages half the elements), so both keep three workgroups per CU.
template <typename T>
constexpr int rows_span()
{
    return kSpanMax * 4 / (int)sizeof(T);
}

template <typename T, int kSpan, bool kLdsTab>
struct RowsSmem {
    T f[kSpan + kSpan / 32 + 1];
    T end[2][kBlk];
    T tab[5][kLdsTab ? kMaxSegWG * kSlot : 1];  // segment tables (S <= kMaxSegWG)
    T septab[5][kLdsTab ? kMaxSegWG : kBlk];    // sub, sup, sl, sip, su at separators
};

// Rows row0 .. row0 + nrows - 1 (nrows * S <= kBlk, nrows * n <= kSpan),
// in phases: the span's loads into registers (all in flight together,
// indices clamped into the span so the loads are unconditional), their LDS
// staging, the segment tables, the solve in LDS, and the span's stores.
template <typename T, int kSpan>
__device__ __forceinline__ void rows_load(const T* __restrict__ F, int64_t row0, int span, int n,
                                          T (&tmp)[(kSpan + kBlk - 1) / kBlk], int tid)
{
    // one descriptor over the span (past its end the loads read zero), one
    // 32-bit offset per load; the whole offset is in the per-lane operand,
    // which is what the hardware range check covers (the instruction's
    // scalar offset is added after the check)
    const __amdgpu_buffer_rsrc_t r = make_rsrc(F + row0 * n, (unsigned)span * (unsigned)sizeof(T));
    const unsigned o = (unsigned)tid * (unsigned)sizeof(T);
#pragma unroll
    for (int q = 0; q < (kSpan + kBlk - 1) / kBlk; q++) tmp[q] = buf_load<T>(r, o + (unsigned)(q * kBlk * sizeof(T)));
}

template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void rows_stage(const T (&tmp)[(kSpan + kBlk - 1) / kBlk], int span,
                                           RowsSmem<T, kSpan, kLdsTab>& sm)
{
    // padded(q kBlk + t) = q (kBlk + kBlk / 32) + padded(t): one address
    // register, the rest in the instructions' offsets
    T* const f = sm.f + padded((int)threadIdx.x);
#pragma unroll
    for (int q = 0; q < (kSpan + kBlk - 1) / kBlk; q++)
        if (q * kBlk + (int)threadIdx.x < span) f[q * (kBlk + kBlk / 32)] = tmp[q];
}

template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void rows_tables(const FibreMap& m, const SolveTables<T>& tb,
                                            RowsSmem<T, kSpan, kLdsTab>& sm)
{
    if constexpr (kLdsTab) {
        stage_tables(tb, 0, m.S, (int)threadIdx.x, kBlk, sm.tab, sm.septab);
        return;
    }
    // separator tables: the separator sweep is serial, so each of its steps
    // must find them in LDS rather than wait on a global load
    for (int e = threadIdx.x; e < m.S; e += kBlk) {
        sm.septab[0][e] = tb.ssub[e];
        sm.septab[1][e] = tb.ssup[e];
        sm.septab[2][e] = tb.sl[e];
        sm.septab[3][e] = tb.sip[e];
        sm.septab[4][e] = tb.su[e];
    }
}

// The solve of the staged rows, in LDS.  Starts after a barrier that
// follows the staging, ends with the solution in sm.f and a barrier.
// tid: threadIdx.x (a caller in a loop passes it through an opaque copy, so
// that the compiler does not hoist the per-slot LDS addresses out of the
// loop and keep them all in registers).
template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void rows_solve_lds(const FibreMap& m, const SolveTables<T>& tb, int nrows,
                                               RowsSmem<T, kSpan, kLdsTab>& sm, int tid)
{
    auto bar = [] { __syncthreads(); };
    const int n = (int)m.n;
    const int r = tid / m.S, s = tid % m.S;
    const bool active = r < nrows;
    const int rr = active ? r : 0;
    int lo, len;
    seg_range(m, s, lo, len);
    const int so = s * kSlot;
    const T* tL = kLdsTab ? &sm.tab[0][so] : tb.L + so;
    const T* tU = kLdsTab ? &sm.tab[1][so] : tb.U + so;
    const T* tI = kLdsTab ? &sm.tab[2][so] : tb.IP + so;
    const T* tA = kLdsTab ? &sm.tab[3][so] : tb.A + so;
    const T* tB = kLdsTab ? &sm.tab[4][so] : tb.B + so;
    T v[kSlot];
#pragma unroll
    for (int q = 0; q < kSlot; q++) v[q] = sm.f[padded(rr * n + lo + min(q, len - 1))];
    seg_solve(v, tL, tU, tI);
    sm.end[0][tid] = v[0];
    sm.end[1][tid] = seg_last(v, s);
    bar();
    if (!tb.dec) {
        if (active && s == 0 && m.S > 1) {
            // row r's separators live in sm.f at r*n + k*kSeg
            const int t0 = tid;
            T gg = T(0);
            for (int k = 1; k < m.S; k++) {
                const int e = padded(r * n + k * kSeg);
                const T rhs =
                    sep_rhs(sm.f[e], sm.septab[0][k], sm.end[1][t0 + k - 1], sm.septab[1][k], sm.end[0][t0 + k]);
                gg = (k == 1) ? rhs : sep_fwd(rhs, sm.septab[2][k], gg);
                sm.f[e] = gg;
            }
            T z = T(0);
            for (int k = m.S - 1; k >= 1; k--) {
                const int e = padded(r * n + k * kSeg);
                z = (k == m.S - 1) ? sm.f[e] * sm.septab[3][k] : sep_bwd(sm.f[e], sm.septab[4][k], z, sm.septab[3][k]);
                sm.f[e] = z;
            }
        }
        bar();
    }
    // read without a condition, indices clamped to a separator there is
    auto sep = [&](int k) {
        const int kc = min(max(k, m.S > 1 ? 1 : 0), m.S - 1), t = min(tid - s + kc, kBlk - 1), tm = max(t - 1, 0);
        const T z = sm.f[padded(rr * n + kc * kSeg)];
        const T w = sep_alone(z, sm.septab[0][kc], sm.end[1][tm], sm.septab[1][kc], sm.end[0][t], sm.septab[3][kc]);
        return tb.dec ? w : z;
    };
    const T sl = sep(s), sr = sep(s + 1);
    const T zl = (s > 0) ? sl : T(0), zr = (s < m.S - 1) ? sr : T(0);
    bar();  // every lane has read its separators
    if (active) {
        // slots past the segment go to its last node, before that node's own
        // value (a store each, without a condition)
        seg_finals(v, tA, zl, tB, zr, [&](int q, T x) { sm.f[padded(r * n + lo + min(q, len - 1))] = x; });
        if (s > 0) sm.f[padded(r * n + s * kSeg)] = zl;
    }
    bar();
}

template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void rows_store(T* __restrict__ F, int64_t row0, int span, int n,
                                           const RowsSmem<T, kSpan, kLdsTab>& sm)
{
    T* g = F + row0 * n;
    for (int e = threadIdx.x; e < span; e += kBlk) g[e] = sm.f[padded(e)];
}

template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void solve_rows_tile(T* __restrict__ F, const FibreMap& m,
                                                const SolveTables<T>& tb, int64_t row0, int nrows,
                                                RowsSmem<T, kSpan, kLdsTab>& sm)
{
    const int n = (int)m.n;
    const int span = nrows * n;
    {
        T tmp[(kSpan + kBlk - 1) / kBlk];
        rows_load<T, kSpan>(F, row0, span, n, tmp, (int)threadIdx.x);
        rows_tables(m, tb, sm);  // (one memory latency covers both)
        rows_stage<T, kSpan, kLdsTab>(tmp, span, sm);
    }
    __syncthreads();
    rows_solve_lds<T, kSpan, kLdsTab>(m, tb, nrows, sm, (int)threadIdx.x);
    rows_store(F, row0, span, n, sm);
}

// The span's stores with their LDS reads issued in batches (a loop of single
// read-then-store steps waits a full LDS round trip per element): one
// descriptor over the span, past whose end the stores are dropped, so the
// unrolled batches need no per-element branch; element indices past the span
// read its last element instead.
template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void rows_store_batched(T* __restrict__ F, int64_t row0, int span, int n,
                                                   const RowsSmem<T, kSpan, kLdsTab>& sm, int tid)
{
    constexpr int NQ = (kSpan + kBlk - 1) / kBlk;
    constexpr int CH = (sizeof(T) == 4) ? 11 : 9;  // values in flight per lane
    const __amdgpu_buffer_rsrc_t r = make_rsrc(F + row0 * n, (unsigned)span * (unsigned)sizeof(T));
    const unsigned o = (unsigned)tid * (unsigned)sizeof(T);
#pragma unroll
    for (int q0 = 0; q0 < NQ; q0 += CH) {
        T v[CH];
#pragma unroll
        for (int q = 0; q < CH; q++)
            if (q0 + q < NQ) v[q] = sm.f[padded(min((q0 + q) * kBlk + tid, span - 1))];
#pragma unroll
        for (int q = 0; q < CH; q++)
            if (q0 + q < NQ) buf_store(v[q], r, o + (unsigned)((q0 + q) * kBlk * sizeof(T)));
    }
}

// The per-level launch: each workgroup runs blocks blockIdx.x, + gridDim.x,
// ... (every block rpb rows, the last one fewer), with the loads of its next
// block issued right after the current block is staged, so that they are in
// flight during the solve and the stores.  A block past the last reads
// through an empty descriptor (no memory access), so the loads stay
// unconditional.
template <typename T, int kSpan, bool kLdsTab>
__device__ __forceinline__ void solve_rows_loop(T* __restrict__ F, const FibreMap& m, const SolveTables<T>& tb,
                                                int rpb, RowsSmem<T, kSpan, kLdsTab>& sm)
{
    const int n = (int)m.n;
    const int64_t nblk = (m.nfib + rpb - 1) / rpb;
    auto span_of = [&](int64_t b) {
        return b < nblk ? (int)min((int64_t)rpb, m.nfib - b * rpb) * n : 0;
    };
    T tmp[(kSpan + kBlk - 1) / kBlk];
    int64_t b = blockIdx.x;
    rows_load<T, kSpan>(F, b < nblk ? b * rpb : 0, span_of(b), n, tmp, (int)threadIdx.x);
    // after the first block's loads were issued: one memory latency covers both
    rows_tables(m, tb, sm);
    for (; b < nblk; b += gridDim.x) {
        const int span = span_of(b);
        rows_stage<T, kSpan, kLdsTab>(tmp, span, sm);
        // an opaque copy of the thread index: the per-load and per-slot
        // offsets derived from it are then formed inside the loop rather than
        // hoisted out of it and held in registers for its whole length
        int tid = (int)threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int64_t bn = b + gridDim.x;
        rows_load<T, kSpan>(F, bn < nblk ? bn * rpb : 0, span_of(bn), n, tmp, tid);
        __syncthreads();
        rows_solve_lds<T, kSpan, kLdsTab>(m, tb, span / n, sm, tid);
        rows_store_batched<T, kSpan, kLdsTab>(F, b * rpb, span, n, sm, tid);
        __syncthreads();  // every lane has read sm.f before the next block is staged
    }
}

// ---- long fibres: three launches through global memory ---------------------
// Phase 1 and 3 work item: strided dimensions use blockIdx.y as the segment
// and x over fibres; the contiguous dimension runs x over (row, segment).
__device__ __forceinline__ bool locate(const FibreMap& m, int bx, int by, int64_t& base, int64_t& fib, int& s)
{
    const int64_t gx = (int64_t)bx * kBlk + threadIdx.x;
    int64_t in, o;
    if (m.inner > 1) {
        if (gx >= m.nfib) return false;
        s = by;
        in = gx % m.inner;
        o = gx / m.inner;
    } else {
        if (gx >= m.nfib * m.S) return false;
        s = (int)(gx % m.S);
        o = gx / m.S;
        in = 0;
    }
    fib = o * m.inner + in;
    base = o * m.n * m.inner + in;
    return true;
}

__device__ __forceinline__ int64_t yb_index(const FibreMap& m, int64_t fib, int s)
{
    return 2 * ((m.inner > 1) ? (int64_t)s * m.nfib + fib : fib * m.S + s);
}

template <typename T>
__device__ __forceinline__ void load_solve(const T* F, const FibreMap& m, int64_t base, int s,
                                        const SolveTables<T>& tb, T (&v)[kSlot], int& lo, int& len)
{
    seg_range(m, s, lo, len);
#pragma unroll
    for (int q = 0; q < kSlot; q++) v[q] = F[base + (int64_t)(lo + min(q, len - 1)) * m.inner];
    seg_solve(v, tb.L + s * kSlot, tb.U + s * kSlot, tb.IP + s * kSlot);
}

template <typename T>
__device__ __forceinline__ void seg_ends_tile(const T* __restrict__ F, T* __restrict__ Yb, const FibreMap& m,
                                              const SolveTables<T>& tb, int bx, int by)
{
    int64_t base, fib;
    int s, lo, len;
    if (!locate(m, bx, by, base, fib, s)) return;
    T v[kSlot];
    load_solve(F, m, base, s, tb, v, lo, len);
    const int64_t yi = yb_index(m, fib, s);
    Yb[yi] = v[0];
    Yb[yi + 1] = seg_last(v, s);
}

template <typename T>
__device__ __forceinline__ void separators_tile(T* __restrict__ F, const T* __restrict__ Yb, const FibreMap& m,
                                                const SolveTables<T>& tb, int bx)
{
    const int64_t fib = (int64_t)bx * kBlk + threadIdx.x;
    if (fib >= m.nfib) return;
    const int64_t o = fib / m.inner, in = fib % m.inner;
    T* p = F + o * m.n * m.inner + in;
    const int64_t ys = (m.inner > 1) ? 2 * m.nfib : 2;
    const T* y0 = Yb + yb_index(m, fib, 0);
    if (tb.dec) {
        // (the batch's rows that are too long for its staging and too few for
        // chunks: the values of the kernels that keep such a row whole)
        const int64_t ps = (int64_t)kSeg * m.inner;
        for (int k = 1; k < m.S; k++)
            p[k * ps] = sep_alone(p[k * ps], tb.ssub[k], y0[1 + (k - 1) * ys], tb.ssup[k], y0[k * ys], tb.sip[k]);
        return;
    }
    sep_solve(m.S, p, (int64_t)kSeg * m.inner, y0, y0 + 1, ys, tb.ssub, tb.ssup, tb.sl, tb.sip, tb.su);
}

template <typename T>
__device__ __forceinline__ void seg_final_tile(T* __restrict__ F, const FibreMap& m, const SolveTables<T>& tb,
                                               int bx, int by)
{
    int64_t base, fib;
    int s, lo, len;
    if (!locate(m, bx, by, base, fib, s)) return;
    T v[kSlot];
    load_solve(F, m, base, s, tb, v, lo, len);
    const T zl = (s > 0) ? F[base + (int64_t)(s * kSeg) * m.inner] : T(0);
    const T zr = (s < m.S - 1) ? F[base + (int64_t)((s + 1) * kSeg) * m.inner] : T(0);
#pragma unroll
    for (int q = 0; q < kSlot; q++)
        if (q < len)
            F[base + (int64_t)(lo + q) * m.inner] = seg_final(v[q], tb.A[s * kSlot + q], zl, tb.B[s * kSlot + q], zr);
}

// ---- planes in LDS ------------------------------------------------------------
// Largest plane-solve workgroup: ten waves, so that the compiler may give a
// lane up to 168 registers (the FP64 kernel spilled at the 128 of 16 waves).
constexpr int kPlaneThreads = 640;

// Solve of nf fibres of n nodes in LDS along one dimension, one task per lane (S nf
// lanes): fibre f starts at P[f sf] (kSplit: at P[f % inner + (f / inner) so]),
// its node i is sd further on each.  Tables: [L, U, IP, A, B][segment][slot] and
// [sub, sup, sl, sip, su][separator], kMaxSegWG segments; end0, end1: kPlaneThreads
// elements.
template <bool kSplit, typename T>
__device__ __forceinline__ void plane_dim(T* P, T* end0, T* end1, const T* tab, const T* septab, int n, int S,
                                          int nf, int sd, int sf, int inner, int so, int tid, int dec)
{
    // task tid: segment s of fibre f
    const bool active = tid < S * nf;
    const int s = active ? tid / nf : 0, f = active ? tid % nf : 0;
    FibreMap m;
    m.n = n;
    m.S = S;
    int lo, len;
    seg_range(m, s, lo, len);
    // node lo + q, clamped to the segment's last
    T* const p = P + (kSplit ? f % inner + (f / inner) * so : f * sf);
    T* const p0 = p + __mul24(lo, sd);
    T v[kSlot];
#pragma unroll
    for (int q = 0; q < kSlot; q++) v[q] = p0[__mul24(min(q, len - 1), sd)];
    seg_solve(v, tab + 0 * kMaxSegWG * kSlot + s * kSlot, tab + 1 * kMaxSegWG * kSlot + s * kSlot,
              tab + 2 * kMaxSegWG * kSlot + s * kSlot);
    if (active) {
        end0[s * nf + f] = v[0];
        end1[s * nf + f] = seg_last(v, s);
    }
    __syncthreads();
    if (!dec) {
        if (active && s == 0 && S > 1)
            sep_solve(S, p, (int64_t)kSeg * sd, end0 + f, end1 + f, nf, septab + 0 * kMaxSegWG,
                      septab + 1 * kMaxSegWG, septab + 2 * kMaxSegWG, septab + 3 * kMaxSegWG, septab + 4 * kMaxSegWG);
        __syncthreads();
    }
    // read without a condition, indices clamped to a separator there is
    auto sep = [&](int k) {
        const int kc = min(max(k, S > 1 ? 1 : 0), S - 1), km = max(kc - 1, 0);
        const T z = p[(kc * kSeg) * sd];
        const T w = sep_alone(z, septab[0 * kMaxSegWG + kc], end1[km * nf + f], septab[1 * kMaxSegWG + kc],
                              end0[kc * nf + f], septab[3 * kMaxSegWG + kc]);
        return dec ? w : z;
    };
    const T sl = sep(s), sr = sep(s + 1);
    const T zl = (s > 0) ? sl : T(0), zr = (s < S - 1) ? sr : T(0);
    __syncthreads();  // every task has read its separators
    if (active) {
        // slots past the segment go to its last node, before that node's own
        // value (a store each, without a condition)
        seg_finals(v, tab + 3 * kMaxSegWG * kSlot + s * kSlot, zl, tab + 4 * kMaxSegWG * kSlot + s * kSlot, zr,
                   [&](int q, T x) { p0[__mul24(min(q, len - 1), sd)] = x; });
        if (s > 0) p[(s * kSeg) * sd] = zl;
    }
    __syncthreads();
}

}  // namespace
}  // namespace mgr
