// Class-packed layout of the refactored data (include/mgr.h,
// mgr_pack_classes): the paper stores and moves the coefficient classes
// separately and a reader may take only the coarsest ones (Sec. I; Sec. II-A,
// overall process).  Class 0 (the coarsest nodal values), then class 1, ...,
// class L, each a contiguous segment with its nodes in C order of their
// grid indices.
//
// Class c >= 1 holds the nodes of level grid c (stride 2^v, v = L - c) that are
// not on level grid c - 1, i.e. whose level indices j = i >> v are not all even;
// C order of the full grid restricted to them is C order of j, so
//     rank = lex(j) - #{all-even j' before j in C order},
// and the all-even count of a box (m0, m1, m2) before j is
//     E(j0) e1 e2 + [j0 even] (E(j1) e2 + [j1 even] E(j2)),
// with E(x) = (x + 1) / 2 even values in [0, x) and e_d = (m_d + 1) / 2.
// Class 0 is the coarsest grid itself: rank = lex(j).
//
// The work goes by rows (i0, i1).  With w the smaller 2-adic valuation of i0
// and i1, a row holds the classes of v = 0 .. w: at the columns of valuation v
// < w, every second node of the row's level-v grid, and at the remaining ones
// its whole level-w grid.  Each is a contiguous piece of its class segment, so
// a row needs one start per class and no division per node, and the three
// rows of four with w = 0 are plain copies.  A wave walks consecutive row
// pieces, stepping (i0, i1) instead of dividing.
//
// Bound by memory: 513^3 FP32 (1.08 GB moved) packed in 231 us, 4.7 TB/s,
// against 552 us with a thread per node and two 64-bit divisions each; it
// moves no byte twice (534 MB written to HBM).  The rest of the way to a
// linear copy's 6.1 TB/s is the rows' arbitrary alignment: 16-byte stores
// aligned to the destination measured the same, and so did an XCD-contiguous
// order of workgroups.
//
// A wave takes the classes of a row one after the other, so that this needs
// long rows and many of them (pack_by_rows); 1-D fields, whose only row holds
// every class, short rows and small arrays go by nodes instead, a thread each,
// its rank from the formula above.
#include <algorithm>

#include "mgr_internal.h"

namespace mgr {
namespace {

constexpr int kPackBlock = 256;

__device__ __forceinline__ int v2(int64_t i, int cap)
{
    return (i == 0) ? cap : min(cap, (int)__builtin_ctzll((unsigned long long)i));
}

// Start of the piece of row (i0, i1) that belongs to the class of valuation v
// (v <= w): packed position of its level-v node 0, with the piece's nodes
// counted as j2 >> 1 (v < w) or j2 (v = w).
__device__ __forceinline__ int64_t piece_start(int64_t i0, int64_t i1, int v, int w, const PackArgs& a)
{
    const int64_t m1 = ((a.n[1] - 1) >> v) + 1, m2 = ((a.n[2] - 1) >> v) + 1;
    const int64_t j0 = i0 >> v, j1 = i1 >> v;
    const int64_t lex = (j0 * m1 + j1) * m2;
    if (v >= a.L) return lex;  // class 0: the coarsest grid in C order
    const int64_t e1 = (m1 + 1) >> 1, e2 = (m2 + 1) >> 1;
    // (v < w: j0 and j1 are even and the piece's j2 odd, so j2 - E(j2) = j2 >> 1)
    const int64_t ev = ((j0 + 1) >> 1) * e1 * e2 + ((j0 & 1) ? 0 : ((j1 + 1) >> 1) * e2);
    return a.off[a.L - v] + lex - ev;
}

// Packed position of node (i0, i1, i2).
__device__ __forceinline__ int64_t packed_index(int64_t i0, int64_t i1, int64_t i2, const PackArgs& a)
{
    const int w = min(v2(i0, a.L), v2(i1, a.L)), v = min(w, v2(i2, a.L));
    return piece_start(i0, i1, v, w, a) + (v < w ? i2 >> (v + 1) : i2 >> v);
}

template <typename T, bool kPack>
__global__ void __launch_bounds__(kPackBlock) k_pack_nodes(const T* __restrict__ src, T* __restrict__ dst, PackArgs a)
{
    const int64_t total = a.n[0] * a.n[1] * a.n[2];
    const int64_t stride = (int64_t)gridDim.x * kPackBlock;
    for (int64_t idx = (int64_t)blockIdx.x * kPackBlock + threadIdx.x; idx < total; idx += stride) {
        const int64_t t = idx / a.n[2], i2 = idx - t * a.n[2];
        const int64_t i0 = t / a.n[1], i1 = t - i0 * a.n[1];
        const int64_t p = packed_index(i0, i1, i2, a);
        if (kPack)
            dst[p] = src[idx];
        else
            dst[idx] = src[p];
    }
}

// A wave takes `per` consecutive units (row, piece of seg columns), pieces
// fastest; kPackBatch elements in flight per lane.  Pos: the type of packed
// positions (32 bits where the array has fewer elements than that).
template <typename T, bool kPack, int kPackBatch, typename Pos>
__global__ void __launch_bounds__(kPackBlock)
    k_pack_rows(const T* __restrict__ src, T* __restrict__ dst, PackArgs a, int64_t seg, int64_t nseg, int64_t per)
{
    constexpr int kLanes = 64;
    const int lane = threadIdx.x % kLanes;
    const int64_t group = (int64_t)blockIdx.x * (kPackBlock / kLanes) + uni((int)(threadIdx.x / kLanes));
    const int64_t n1 = a.n[1], n2 = a.n[2];
    const int64_t units = a.n[0] * n1 * nseg;
    int64_t u = group * per;
    const int64_t end = min(u + per, units);
    if (u >= end) return;
    int64_t row = u / nseg, s = u - row * nseg;
    int64_t i0 = row / n1, i1 = row - i0 * n1;
    for (; u < end; u++) {
        const int w = min(v2(i0, a.L), v2(i1, a.L));
        // (a piece's columns count from its first, in 32 bits)
        const int64_t c0 = s * seg;
        const int n = (int)min(seg, n2 - c0);
        const int64_t rb = row * n2 + c0;
        if (w == 0) {
            const int64_t b0 = piece_start(i0, i1, 0, 0, a) + c0;
            const T* const x = src + (kPack ? rb : b0);
            T* const y = dst + (kPack ? b0 : rb);
            for (int i = lane; i < n; i += kLanes * kPackBatch) {
                T v[kPackBatch];
#pragma unroll
                for (int q = 0; q < kPackBatch; q++) v[q] = x[min(i + q * kLanes, n - 1)];
#pragma unroll
                for (int q = 0; q < kPackBatch; q++)
                    if (i + q * kLanes < n) y[i + q * kLanes] = v[q];
            }
        } else {
            // column c belongs to the class of valuation min(v2(c), w): its
            // packed position, the row's classes one after the other, then one
            // load and one store
            const T* const x = src + rb;
            T* const y = dst + rb;
            for (int i = lane; i < n; i += kLanes * kPackBatch) {
                Pos p[kPackBatch];
                int cv[kPackBatch];
                T t[kPackBatch];
#pragma unroll
                for (int q = 0; q < kPackBatch; q++) {
                    const int e = min(i + q * kLanes, n - 1);
                    cv[q] = min(v2(c0 + e, a.L), w);
                    if (kPack) t[q] = x[e];
                    p[q] = 0;
                }
                for (int v = 0; v <= w; v++) {
                    const int sh = v < w ? v + 1 : v;
                    const Pos b = (Pos)(piece_start(i0, i1, v, w, a) + (c0 >> sh));
                    const int low = (int)(c0 & (((int64_t)1 << sh) - 1));
#pragma unroll
                    for (int q = 0; q < kPackBatch; q++) {
                        const Pos o = b + (Pos)((low + min(i + q * kLanes, n - 1)) >> sh);
                        p[q] = (cv[q] == v) ? o : p[q];
                    }
                }
                if constexpr (!kPack) {
#pragma unroll
                    for (int q = 0; q < kPackBatch; q++) t[q] = src[p[q]];
                }
#pragma unroll
                for (int q = 0; q < kPackBatch; q++)
                    if (i + q * kLanes < n) {
                        if (kPack)
                            dst[p[q]] = t[q];
                        else
                            y[i + q * kLanes] = t[q];
                    }
            }
        }
        if (++s == nseg) {
            s = 0;
            row++;
            if (++i1 == n1) {
                i1 = 0;
                i0++;
            }
        }
    }
}

constexpr int64_t kPackSeg = 2304;  // columns of a row piece
inline int64_t pack_units(const PackArgs& a) { return a.n[0] * a.n[1] * ((a.n[2] + kPackSeg - 1) / kPackSeg); }

template <typename T, int kPackBatch>
hipError_t launch_pack_rows(const T* src, T* dst, const PackArgs& a, bool pack, hipStream_t st)
{
    // row pieces of a few thousand columns, and enough waves for several
    // rounds of the chip's wave slots where there are rows for them
    const int64_t rows = a.n[0] * a.n[1];
    const int64_t seg = std::min<int64_t>(a.n[2], kPackSeg), nseg = (a.n[2] + seg - 1) / seg;
    const int64_t units = rows * nseg;
    const int64_t groups = (int64_t)device_cu_count() * 128;
    const int64_t per = std::max<int64_t>(1, (units + groups - 1) / groups);
    const int64_t blocks = ((units + per - 1) / per + kPackBlock / 64 - 1) / (kPackBlock / 64);
    auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(kPackBlock), 0, st, src, dst, a, seg, nseg, per); };
    const bool small = rows * a.n[2] < ((int64_t)1 << 32);
    if (pack)
        small ? launch(k_pack_rows<T, true, kPackBatch, unsigned>) : launch(k_pack_rows<T, true, kPackBatch, int64_t>);
    else
        small ? launch(k_pack_rows<T, false, kPackBatch, unsigned>) : launch(k_pack_rows<T, false, kPackBatch, int64_t>);
    return hipGetLastError();
}

// By rows where a wave's chain of classes is short beside its columns and there
// are rows enough to fill the chip; by nodes otherwise.  FP32, by nodes and by
// rows: 4097 x 513 9.6, 8.6 us, 4097^2 58.5, 37.7, 257^3 56.9, 26.9, 262145 x 129 118,
// 96; but 2049 x 1025 9.6, 9.9, 513 x 4097 9.9, 17.5, 16385 x 129 9.9, 12.6, 513 x 513 x 65
// 57, 74, 2^20 x 3 10.5, 37, 1-D 2^16 8.4, 22.6 and 2^26 278, 359.
bool pack_by_rows(const PackArgs& a)
{
    if (a.n[0] * a.n[1] == 1) return false;
    const int64_t units = pack_units(a);
    return (a.n[2] > 192 && units >= 4096) || (a.n[2] > 128 && units >= 65536);
}

}  // namespace

template <typename T>
hipError_t launch_pack(const T* src, T* dst, const PackArgs& a, bool pack, hipStream_t st)
{
    const int64_t n = a.n[2];
    if (!pack_by_rows(a)) {
        const int64_t b = (a.n[0] * a.n[1] * n + kPackBlock - 1) / kPackBlock;
        const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(b, (int64_t)1 << 20)));
        if (pack)
            hipLaunchKernelGGL((k_pack_nodes<T, true>), grid, dim3(kPackBlock), 0, st, src, dst, a);
        else
            hipLaunchKernelGGL((k_pack_nodes<T, false>), grid, dim3(kPackBlock), 0, st, src, dst, a);
        return hipGetLastError();
    }
    // as many elements in flight as a row of 2^k + 1 takes whole (its odd last
    // element in a batch of its own cost a second memory latency per row: 292
    // against 257 us at 513^3, other things equal)
    if (n <= 192) return launch_pack_rows<T, 3>(src, dst, a, pack, st);
    if (n <= 320) return launch_pack_rows<T, 5>(src, dst, a, pack, st);
    return launch_pack_rows<T, 9>(src, dst, a, pack, st);
}

template hipError_t launch_pack<float>(const float*, float*, const PackArgs&, bool, hipStream_t);
template hipError_t launch_pack<double>(const double*, double*, const PackArgs&, bool, hipStream_t);

}  // namespace mgr
