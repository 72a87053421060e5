// Level steps of four-dimensional grids, plane by plane.
//
// A level grid of m0 x m1 x m2 x m3 nodes (any sizes; the coarse nodes of a
// dimension are its even positions and its last one) is worked on by one
// workgroup per plane (j0, j1) of its last two dimensions, in LDS:
//   decomposition   the plane's interpolant Q between the (up to four) planes
//                   of coarse (j0, j1) around it, at the coarse nodes of dims
//                   2 and 3; the coefficients u - Pi Q at every node that is
//                   not coarse in all four dimensions (Sec. II-A.1), written to
//                   their nodes; and the load-vector stencils (Sec. II-A.2,
//                   merged form) along dims 3 and 2 of the plane, written
//                   packed (m0, m1, mc2, mc3);
//   load vector     the same stencils on stored coefficients;
//   recomposition   coefficients plus Pi Q, Q from the corrected coarse values.
// The stencils along dims 1 and 0 follow on that quarter (25 inputs per output,
// all but the first read of each from the caches), a workgroup per coarse plane,
// which solves dims 3 and 2 of its plane in LDS before it stores it
// (k_mass_plane); the solves along dims 1 and 0 run on column tiles in LDS
// (k_solve_cols).  Sizes that do not fit those take the stencils and the solves
// one by one.  A correction is never added in a pass of its own: the next level
// step reads W + Z.
//
// Bound by memory at the finest step, by launches below it: three per level
// step of a decomposition.  40 x 50 x 60 x 70 FP64 nonuniform decomposed and recomposed in
// 478 us (62, 33 and 40 us the plane passes of the finest step), against 1925 us with a thread per node, 64-bit index divisions, up to
// sixteen corner reads per node and ten launches per level step.
#include <algorithm>

#include "mgr_solve_dev.h"

namespace mgr {
namespace {

// idx / n, exact for idx < 2^20 (r = 1 / n; the quotient of idx + 1/2 is at
// least 1 / (2 n) from a whole number).
__device__ __forceinline__ int fdiv(int idx, float r) { return (int)fmaf((float)idx, r, 0.5f * r); }

__device__ __forceinline__ bool fine_at(int j, int m) { return (j & 1) && j != m - 1; }
// Level index of coarse node i, coarse index of a coarse level index j.
__device__ __forceinline__ int level_of(int i, int m, int mc) { return i == mc - 1 ? m - 1 : 2 * i; }
__device__ __forceinline__ int coarse_of(int j, int m) { return j == m - 1 ? m >> 1 : j >> 1; }

// One of the up to four coarse-(j0, j1) planes around a plane.
struct Corner {
    int j0, j1;
};

template <typename T>
struct Corners {
    Corner c[4];
    T w[4];
    int n;
};
template <typename T>
__device__ __forceinline__ Corners<T> corners_of(const Plane4<T>& a, int j0, int j1)
{
    const bool f0 = fine_at(j0, a.m[0]), f1 = fine_at(j1, a.m[1]);
    Corners<T> r;
    r.n = (f0 ? 2 : 1) * (f1 ? 2 : 1);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const bool u1 = q & 1, u0 = q >> 1;  // (for two corners along dim 0, q = 0, 1 are them)
        const bool up0 = (f0 && f1) ? u0 : (f0 && u1), up1 = f1 && u1;
        r.c[q].j0 = f0 ? (up0 ? j0 + 1 : j0 - 1) : j0;
        r.c[q].j1 = f1 ? (up1 ? j1 + 1 : j1 - 1) : j1;
        const T w0 = f0 ? (up0 ? a.wh[0][j0] : a.wl[0][j0]) : T(1);
        const T w1 = f1 ? (up1 ? a.wh[1][j1] : a.wl[1][j1]) : T(1);
        r.w[q] = q < r.n ? w0 * w1 : T(0);
    }
    return r;
}

// Offset in the user's array of level index j along dimension d.
template <typename T>
__device__ __forceinline__ int64_t user_at(const Plane4<T>& a, int d, int j)
{
    return min((int64_t)j << a.k, a.n[d] - 1) * a.st[d];
}

// Interpolant along dims 2 and 3 at node (j2, j3) from the coarse plane Q.
// (weights: [dim 2: low, high; dim 3: low, high] in LDS).
template <typename T>
__device__ __forceinline__ T plane_interp(const Plane4<T>& a, const T* Q, const T* wt, int j2, int j3)
{
    const int m2 = a.m[2], m3 = a.m[3], mc3 = a.mc[3];
    const bool f2 = fine_at(j2, m2), f3 = fine_at(j3, m3);
    const int i2 = f2 ? j2 >> 1 : coarse_of(j2, m2), i3 = f3 ? j3 >> 1 : coarse_of(j3, m3);
    const int s2 = f2 ? mc3 : 0, s3 = f3 ? 1 : 0;
    const T* q = Q + i2 * mc3 + i3;
    const T l2 = wt[j2], h2 = wt[m2 + j2], l3 = wt[2 * m2 + j3], h3 = wt[2 * m2 + m3 + j3];
    const T lo = f3 ? lerp2(l3, q[0], h3, q[s3]) : q[0];
    const T hi = f3 ? lerp2(l3, q[s2], h3, q[s2 + s3]) : q[s2];
    return f2 ? lerp2(l2, lo, h2, hi) : lo;
}

extern __shared__ __align__(16) unsigned char plane4_lds[];

constexpr int kPlane4Threads = 512;

// kMode 0: decomposition, 1: load vector of stored coefficients, 2:
// recomposition.
template <typename T, int kMode>
__global__ void __launch_bounds__(kPlane4Threads) k_plane4(Plane4<T> a)
{
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int m1 = a.m[1], m2 = a.m[2], m3 = a.m[3], mc2 = a.mc[2], mc3 = a.mc[3];
    const int P = (int)blockIdx.x, j0 = P / m1, j1 = P - j0 * m1;
    const bool f0 = fine_at(j0, a.m[0]), f1 = fine_at(j1, a.m[1]);
    const bool coarse01 = !f0 && !f1;
    const int V = m2 * m3, Vc = mc2 * mc3;
    T* const U = reinterpret_cast<T*>(plane4_lds);  // the plane; then its coefficients (zero at coarse nodes)
    T* const wt = U + V;                            // weights of dims 2 and 3
    T* const Q = wt + 2 * (m2 + m3);                // coarse values between the corner planes
    T* const S = Q;                                 // (after Q) stencil along dim 3, m2 x mc3
    const float r3 = 1.0f / (float)m3, rc3 = 1.0f / (float)mc3;
    const int64_t up = user_at(a, 0, j0) + user_at(a, 1, j1);      // the plane in the user's array
    const int64_t pk = ((int64_t)j0 * m1 + j1) * V;                // and in the packed level grid
    auto node = [&](int e, int& j2, int& j3) {
        j2 = fdiv(e, r3);
        j3 = e - j2 * m3;
    };
    auto user = [&](int j2, int j3) { return up + user_at(a, 2, j2) + user_at(a, 3, j3); };
    const bool packed_in = kMode == 0 && a.k > 0;

    // ---- the plane's values and Q
    for (int e0 = 0; e0 < V; e0 += 4 * nthr) {
        T v[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int e = min(e0 + q * nthr + tid, V - 1);
            int j2, j3;
            node(e, j2, j3);
            v[q] = packed_in ? a.Wk[pk + e] + a.Z[pk + e] : a.in[a.k == 0 ? up + e : user(j2, j3)];
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int e = e0 + q * nthr + tid;
            if (e >= V) continue;
            if (kMode != 0 && coarse01) {
                int j2, j3;
                node(e, j2, j3);
                // coarse positions hold other classes: their coefficient is zero
                if (!fine_at(j2, m2) && !fine_at(j3, m3)) v[q] = T(0);
            }
            U[e] = v[q];
        }
    }
    if (kMode != 1) {
        for (int d = 2; d < 4; d++) {
            T* const w = wt + (d - 2) * 2 * m2;
            for (int j = tid; j < a.m[d]; j += nthr) {
                const bool f = fine_at(j, a.m[d]);
                w[j] = f ? a.wl[d][j] : T(1);
                w[a.m[d] + j] = f ? a.wh[d][j] : T(0);
            }
        }
        const Corners<T> co = corners_of(a, j0, j1);
        for (int c = tid; c < Vc; c += nthr) {
            const int i2 = fdiv(c, rc3), i3 = c - i2 * mc3;
            T g[4];
            if (kMode == 2) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int p0 = coarse_of(co.c[q].j0, a.m[0]), p1 = coarse_of(co.c[q].j1, a.m[1]);
                    const int64_t o = ((int64_t)p0 * a.mc[1] + p1) * Vc + c;
                    g[q] = q < co.n ? a.Wn[o] - a.Z[o] : T(0);
                }
            } else {
                const int j2 = level_of(i2, m2, mc2), j3 = level_of(i3, m3, mc3);
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    g[q] = T(0);
                    if (q < co.n) {
                        const int64_t o = ((int64_t)co.c[q].j0 * m1 + co.c[q].j1) * V + j2 * m3 + j3;
                        g[q] = packed_in ? a.Wk[o] + a.Z[o]
                                         : a.in[user_at(a, 0, co.c[q].j0) + user_at(a, 1, co.c[q].j1) + user_at(a, 2, j2) +
                                                user_at(a, 3, j3)];
                    }
                }
            }
            T s = co.w[0] * g[0];
#pragma unroll
            for (int q = 1; q < 4; q++) s = fma(co.w[q], g[q], s);
            Q[c] = s;
            // coarse nodes go on to the next level grid
            if (kMode == 0 && coarse01)
                a.Wn[((int64_t)coarse_of(j0, a.m[0]) * a.mc[1] + coarse_of(j1, a.m[1])) * Vc + c] = g[0];
        }
    }
    __syncthreads();

    if (kMode != 1) {
        for (int e = tid; e < V; e += nthr) {
            int j2, j3;
            node(e, j2, j3);
            const bool coarse = coarse01 && !fine_at(j2, m2) && !fine_at(j3, m3);
            const T p = plane_interp(a, Q, wt, j2, j3);
            if (kMode == 0) {
                const T c = coarse ? T(0) : U[e] - p;
                U[e] = c;
                if (!coarse) a.out[a.k == 0 ? up + e : user(j2, j3)] = c;
            } else {
                const T v = U[e] + p;
                a.out[(a.k == 0 ? up : pk) + e] = v;
            }
        }
        if (kMode == 2) return;
        __syncthreads();
    }

    // ---- stencils along dims 3 and 2
    for (int e = tid; e < m2 * mc3; e += nthr) {
        const int j2 = fdiv(e, rc3), i = e - j2 * mc3, f = level_of(i, m3, mc3);
        const T* u = U + j2 * m3;
        T s = T(0);
#pragma unroll
        for (int t = 0; t < 5; t++) {
            const int c = f - 2 + t;
            if (c >= 0 && c < m3) s = fma(a.K[3][5 * i + t], u[c], s);
        }
        S[e] = s;
    }
    __syncthreads();
    T* const F = a.F + ((int64_t)j0 * m1 + j1) * Vc;
    for (int e = tid; e < Vc; e += nthr) {
        const int i = fdiv(e, rc3), f = level_of(i, m2, mc2);
        const T* u = S + (e - i * mc3);
        T s = T(0);
#pragma unroll
        for (int t = 0; t < 5; t++) {
            const int c = f - 2 + t;
            if (c >= 0 && c < m2) s = fma(a.K[2][5 * i + t], u[c * mc3], s);
        }
        F[e] = s;
    }
}

// Stencils along dims 1 and 0 of in (m0, m1, R) at coarse (i0, i1), element r.
template <typename T>
__device__ __forceinline__ T mass01_at(const T* __restrict__ in, const Plane4<T>& a, int R, int i0, int i1, int r)
{
    const int m0 = a.m[0], m1 = a.m[1];
    const int f0 = level_of(i0, m0, a.mc[0]), f1 = level_of(i1, m1, a.mc[1]);
    // (all 25 loads at once, at clamped indices; outside the grid K is zero)
    T v[5][5];
#pragma unroll
    for (int s = 0; s < 5; s++)
#pragma unroll
        for (int t = 0; t < 5; t++) {
            const int c0 = min(max(f0 - 2 + s, 0), m0 - 1), c1 = min(max(f1 - 2 + t, 0), m1 - 1);
            v[s][t] = in[((int64_t)c0 * m1 + c1) * R + r];
        }
    T acc = T(0);
#pragma unroll
    for (int s = 0; s < 5; s++) {
        T t5 = T(0);
#pragma unroll
        for (int t = 0; t < 5; t++) {
            const bool in1 = f1 - 2 + t >= 0 && f1 - 2 + t < m1;
            t5 = fma(in1 ? a.K[1][5 * i1 + t] : T(0), v[s][t], t5);
        }
        const bool in0 = f0 - 2 + s >= 0 && f0 - 2 + s < m0;
        acc = fma(in0 ? a.K[0][5 * i0 + s] : T(0), t5, acc);
    }
    return acc;
}

// out (mc0, mc1, R), R contiguous; workgroup (x, i0 mc1 + i1).
template <typename T>
__global__ void __launch_bounds__(256) k_mass01(const T* __restrict__ in, T* __restrict__ out, Plane4<T> a, int R, int nx)
{
    const int b = (int)blockIdx.x / nx, r = ((int)blockIdx.x - b * nx) * 256 + (int)threadIdx.x;
    if (r >= R) return;
    const int i0 = b / a.mc[1], i1 = b - i0 * a.mc[1];
    out[(int64_t)b * R + r] = mass01_at(in, a, R, i0, i1, r);
}

// LDS of the plane solves: tables of two dimensions, segment ends, the nodes.
constexpr int kTab4 = 5 * kMaxSegWG * kSlot, kSep4 = 5 * kMaxSegWG;
template <typename T>
size_t solve4_bytes(int64_t nodes)
{
    return sizeof(T) * (size_t)(2 * kTab4 + 2 * kSep4 + 2 * kPlaneThreads + nodes);
}
template <typename T>
__device__ __forceinline__ void stage4(T* lds, const SolveTables<T> (&tb)[2], int tid, int nthr)
{
#pragma unroll
    for (int d = 0; d < 2; d++)
        stage_tables(tb[d], 0, tb[d].S, tid, nthr, *reinterpret_cast<T(*)[5][kMaxSegWG * kSlot]>(lds + d * kTab4),
                     *reinterpret_cast<T(*)[5][kMaxSegWG]>(lds + 2 * kTab4 + d * kSep4));
}

template <typename T>
struct Tables2 {
    SolveTables<T> tb[2];
};

// Stencils along dims 1 and 0 of one coarse plane, then the solves of its dims 3
// and 2 (tb[0], tb[1]): workgroup i0 mc1 + i1.
template <typename T>
__global__ void __launch_bounds__(kPlaneThreads)
k_mass_plane(const T* __restrict__ in, T* __restrict__ out, Plane4<T> a, Tables2<T> t)
{
    T* const lds = reinterpret_cast<T*>(plane4_lds);
    T* const sep = lds + 2 * kTab4;
    T* const end = sep + 2 * kSep4;
    T* const P = end + 2 * kPlaneThreads;
    const int tid = threadIdx.x, nthr = blockDim.x, b = (int)blockIdx.x;
    const int n2 = a.mc[2], n3 = a.mc[3], R = n2 * n3, i0 = b / a.mc[1], i1 = b - i0 * a.mc[1];
    stage4(lds, t.tb, tid, nthr);
    for (int r = tid; r < R; r += nthr) P[r] = mass01_at(in, a, R, i0, i1, r);
    __syncthreads();
#pragma unroll 1
    for (int d = 0; d < 2; d++)
        plane_dim<false>(P, end, end + kPlaneThreads, lds + d * kTab4, sep + d * kSep4, d ? n2 : n3, t.tb[d].S, d ? n3 : n2,
                         d ? n3 : 1, d ? 1 : n3, 1, 0, tid, t.tb[d].dec);
    for (int r = tid; r < R; r += nthr) out[(int64_t)b * R + r] = P[r];
}

// Solves along dims 1 and 0 (tb[0], tb[1]) of F (n0, n1, R): a workgroup takes
// kCols elements of R.
template <typename T>
constexpr int kCols = 64 / (int)sizeof(T);
template <typename T>
__global__ void __launch_bounds__(kPlaneThreads) k_solve_cols(T* F, int n0, int n1, int R, Tables2<T> t)
{
    constexpr int C = kCols<T>;
    T* const lds = reinterpret_cast<T*>(plane4_lds);
    T* const sep = lds + 2 * kTab4;
    T* const end = sep + 2 * kSep4;
    T* const P = end + 2 * kPlaneThreads;
    const int tid = threadIdx.x, nthr = blockDim.x, r0 = (int)blockIdx.x * C, V = n0 * n1 * C;
    // node (i0, i1, r) at P[(i0 n1 + i1) C + r]; columns past R repeat its last one
    // and are not stored
    for (int b0 = 0; b0 < V; b0 += 8 * nthr) {
        T v[8];
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const int e = min(b0 + q * nthr + tid, V - 1);
            v[q] = F[(int64_t)(e / C) * R + min(r0 + e % C, R - 1)];
        }
        if (b0 == 0) stage4(lds, t.tb, tid, nthr);
#pragma unroll
        for (int q = 0; q < 8; q++)
            if (b0 + q * nthr + tid < V) P[b0 + q * nthr + tid] = v[q];
    }
    __syncthreads();
#pragma unroll 1
    for (int d = 0; d < 2; d++)
        plane_dim<true>(P, end, end + kPlaneThreads, lds + d * kTab4, sep + d * kSep4, d ? n0 : n1, t.tb[d].S,
                        (d ? n1 : n0) * C, d ? n1 * C : C, 1, d ? n1 * C : C, d ? 0 : n1 * C, tid, t.tb[d].dec);
    for (int e = tid; e < V; e += nthr)
        if (r0 + e % C < R) F[(int64_t)(e / C) * R + r0 + e % C] = P[e];
}

// Two solves of n nodes each, of nfa and nfb fibres, as plane_dim's tasks: their
// lanes, or 0 where they do not fit.
template <typename T>
int solve4_lanes(const SolveTables<T>& ta, int64_t na, int64_t nfa, const SolveTables<T>& tb, int64_t nb, int64_t nfb,
                 int64_t nodes)
{
    if (ta.S < 1 || tb.S < 1 || ta.S > kMaxSegWG || tb.S > kMaxSegWG || na < 2 || nb < 2) return 0;
    const int64_t tasks = std::max<int64_t>(ta.S * nfa, tb.S * nfb);
    if (tasks > kPlaneThreads || solve4_bytes<T>(nodes) > (size_t)kPlane4Lds) return 0;
    return (int)((tasks + 63) / 64 * 64);
}

template <typename T>
size_t plane4_bytes(const Plane4<T>& a)
{
    return sizeof(T) * ((size_t)a.m[2] * a.m[3] + 2 * ((size_t)a.m[2] + a.m[3]) + (size_t)a.m[2] * a.mc[3]);
}

// LDS beyond 64 KB has to be asked for once per kernel and device.
template <typename K>
hipError_t allow_lds4(K kern, size_t bytes, bool (&done)[64])
{
    if (bytes <= 65536) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (done[dev]) return hipSuccess;
    e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kPlane4Lds);
    if (e == hipSuccess) done[dev] = true;
    return e;
}

template <typename T, int kMode>
hipError_t launch_mode(const Plane4<T>& a, hipStream_t st)
{
    const size_t bytes = plane4_bytes(a);
    static bool done[64] = {};
    const hipError_t e = allow_lds4(k_plane4<T, kMode>, bytes, done);
    if (e != hipSuccess) return e;
    // a few nodes a lane, so that the loads of a plane are in flight together
    const int V = a.m[2] * a.m[3];
    const unsigned thr = V <= 128 ? 64 : V <= 1024 ? 256 : kPlane4Threads;
    hipLaunchKernelGGL((k_plane4<T, kMode>), dim3((unsigned)(a.m[0] * a.m[1])), dim3(thr), bytes, st, a);
    return hipGetLastError();
}

}  // namespace

template <typename T>
bool plane4_fits(const Plane4<T>& a)
{
    // planes in LDS, and every launch's grid below 2^32 threads (the plane
    // solves take up to 1024 a plane)
    return plane4_bytes(a) <= (size_t)kPlane4Lds && (int64_t)a.m[0] * a.m[1] < ((int64_t)1 << 22) &&
           (int64_t)a.mc[0] * a.mc[1] * ((a.mc[2] * a.mc[3] + 255) / 256) < ((int64_t)1 << 24);
}

template <typename T>
hipError_t launch_plane4(const Plane4<T>& a, int mode, hipStream_t st)
{
    return mode == 0 ? launch_mode<T, 0>(a, st) : mode == 1 ? launch_mode<T, 1>(a, st) : launch_mode<T, 2>(a, st);
}

// Stencils along dims 1 and 0 alone.
template <typename T>
static hipError_t launch_mass01(const T* in, T* out, const Plane4<T>& a, hipStream_t st)
{
    const int R = a.mc[2] * a.mc[3], nx = (R + 255) / 256;
    hipLaunchKernelGGL(k_mass01<T>, dim3((unsigned)((int64_t)a.mc[0] * a.mc[1] * nx)), dim3(256), 0, st, in, out, a, R, nx);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_mass_plane(const T* in, T* out, const Plane4<T>& a, const SolveTables<T>& t3, const SolveTables<T>& t2,
                             hipStream_t st, bool* done_)
{
    const int64_t n2 = a.mc[2], n3 = a.mc[3];
    // (with more planes than CUs the stencils' own launch, of many more waves, is
    // faster: 546 planes of 31 x 36 FP64 16 + 20 us against 42 together; 12 of 8 x 9
    // 13 against 10)
    const int lanes = a.mc[0] * a.mc[1] > device_cu_count() ? 0 : solve4_lanes<T>(t3, n3, n2, t2, n2, n3, n2 * n3);
    *done_ = lanes > 0;
    if (lanes == 0) return launch_mass01<T>(in, out, a, st);
    static bool done[64] = {};
    const size_t bytes = solve4_bytes<T>(n2 * n3);
    const hipError_t e = allow_lds4(k_mass_plane<T>, bytes, done);
    if (e != hipSuccess) return e;
    // (two or three stencils a lane)
    const int64_t want = (n2 * n3 / 3 + 63) / 64 * 64;
    const unsigned thr = (unsigned)std::min<int64_t>(kPlaneThreads, std::max<int64_t>(lanes, want));
    Tables2<T> t;
    t.tb[0] = t3;
    t.tb[1] = t2;
    hipLaunchKernelGGL(k_mass_plane<T>, dim3((unsigned)(a.mc[0] * a.mc[1])), dim3(thr), bytes, st, in, out, a, t);
    return hipGetLastError();
}

template <typename T>
int solve_cols_lanes(const Plane4<T>& a, const SolveTables<T>& t1, const SolveTables<T>& t0)
{
    const int64_t n0 = a.mc[0], n1 = a.mc[1];
    if (n0 * n1 > device_cu_count()) return 0;
    return solve4_lanes<T>(t1, n1, n0 * kCols<T>, t0, n0, n1 * kCols<T>, n0 * n1 * kCols<T>);
}
template <typename T>
bool solve_cols_fits(const Plane4<T>& a, const SolveTables<T>& t1, const SolveTables<T>& t0)
{
    return solve_cols_lanes<T>(a, t1, t0) > 0;
}

template <typename T>
hipError_t launch_solve_cols(T* F, const Plane4<T>& a, const SolveTables<T>& t1, const SolveTables<T>& t0, hipStream_t st)
{
    const int64_t n0 = a.mc[0], n1 = a.mc[1], nodes = n0 * n1 * kCols<T>;
    const int lanes = solve_cols_lanes<T>(a, t1, t0);
    if (lanes == 0) return hipErrorNotSupported;
    static bool done[64] = {};
    const size_t bytes = solve4_bytes<T>(nodes);
    const hipError_t e = allow_lds4(k_solve_cols<T>, bytes, done);
    if (e != hipSuccess) return e;
    const int R = a.mc[2] * a.mc[3];
    const unsigned thr = (unsigned)std::min<int64_t>(kPlaneThreads, std::max<int64_t>(lanes, (nodes / 8 + 63) / 64 * 64));
    Tables2<T> t;
    t.tb[0] = t1;
    t.tb[1] = t0;
    hipLaunchKernelGGL(k_solve_cols<T>, dim3((unsigned)((R + kCols<T> - 1) / kCols<T>)), dim3(thr), bytes, st, F, (int)n0,
                       (int)n1, R, t);
    return hipGetLastError();
}

template bool plane4_fits<float>(const Plane4<float>&);
template bool plane4_fits<double>(const Plane4<double>&);
template hipError_t launch_plane4<float>(const Plane4<float>&, int, hipStream_t);
template hipError_t launch_plane4<double>(const Plane4<double>&, int, hipStream_t);
template hipError_t launch_mass_plane<float>(const float*, float*, const Plane4<float>&, const SolveTables<float>&,
                                             const SolveTables<float>&, hipStream_t, bool*);
template hipError_t launch_mass_plane<double>(const double*, double*, const Plane4<double>&, const SolveTables<double>&,
                                              const SolveTables<double>&, hipStream_t, bool*);
template hipError_t launch_solve_cols<float>(float*, const Plane4<float>&, const SolveTables<float>&,
                                             const SolveTables<float>&, hipStream_t);
template bool solve_cols_fits<float>(const Plane4<float>&, const SolveTables<float>&, const SolveTables<float>&);
template hipError_t launch_solve_cols<double>(double*, const Plane4<double>&, const SolveTables<double>&,
                                              const SolveTables<double>&, hipStream_t);
template bool solve_cols_fits<double>(const Plane4<double>&, const SolveTables<double>&, const SolveTables<double>&);

}  // namespace mgr
