// Quantisation of the refactored classes (include/mgr.h, mgr_quantize):
// the lossy-compression use of the refactoring quantises every coefficient
// class with its own bin width and keeps the integer codes (Sec. V).  The
// paper names the stage, not the quantiser; the one implemented is a uniform
// scalar quantiser per class:
//     code = round-half-even(y / b_c)   (in the data's precision, b_c rounded
//                                        to it first)
//     value = code * b_c
// with a quotient that is NaN or beyond +-(2^31 - 1) clamped (NaN to 0) and
// counted.
//
// Both layouts are handled.  In-place node order: the class of a node comes
// from the 2-adic valuations of its indices, and a work unit is one segment
// of one row, so the row's outer indices (and their valuation) are
// wave-uniform and no per-element division is needed.  Class-packed: the
// class of an element is the segment its position falls in.
#include <algorithm>
#include <type_traits>

#include "mgr_internal.h"

namespace mgr {
namespace {

constexpr int kQuantBlock = 256;

__device__ __forceinline__ int val2(int64_t i, int cap)
{
    return (i == 0) ? cap : min(cap, (int)__builtin_ctzll((unsigned long long)i));
}

__device__ __forceinline__ float div_round(float y, float b) { return rintf(y / b); }
__device__ __forceinline__ double div_round(double y, double b) { return rint(y / b); }

// Code of one value; *clamped counts a rounded quotient that is NaN or out of
// the int32 range that is kept symmetric.
template <typename T>
__device__ __forceinline__ int code_of(T y, T b, int* clamped)
{
    const double r = (double)div_round(y, b);
    if (r != r) {
        ++*clamped;
        return 0;
    }
    if (r > 2147483647.0) {
        ++*clamped;
        return 2147483647;
    }
    if (r < -2147483647.0) {
        ++*clamped;
        return -2147483647;
    }
    return (int)r;
}

// One atomic per wave with clamped codes for their count.
__device__ __forceinline__ void count_clamped(int c, unsigned long long* counter)
{
    if (!counter || !__any(c)) return;
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) c += __shfl_xor(c, w);
    if ((threadIdx.x & 63) == 0) atomicAdd(counter, (unsigned long long)c);
}

template <typename T, bool kQuant>
__global__ void __launch_bounds__(kQuantBlock)
    k_quant_inplace(const T* __restrict__ y, int* __restrict__ q, T* __restrict__ out, QuantArgs a,
                    unsigned long long* counter)
{
    // unit = (row, segment of seg columns); rows are (i0, i1) of the internal 3-D form
    const int L = a.L;
    const int64_t n1 = a.n[1], n2 = a.n[2];
    const int64_t rows = a.n[0] * n1;
    const int64_t units = rows * a.nseg;
    const int wave = uni((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int64_t wstride = (int64_t)gridDim.x * (kQuantBlock / 64);
    int clamped = 0;
    for (int64_t u = (int64_t)blockIdx.x * (kQuantBlock / 64) + wave; u < units; u += wstride) {
        const int64_t row = u / a.nseg;  // wave-uniform
        const int64_t s = u - row * a.nseg;
        const int64_t i0 = row / n1, i1 = row - i0 * n1;
        const int vrow = min(val2(i0, L), val2(i1, L));
        const int64_t c0 = s * a.seg, c1 = min(c0 + a.seg, n2);
        const int64_t base = row * n2;
        for (int64_t i2 = c0 + lane; i2 < c1; i2 += 64) {
            const int cls = L - min(vrow, val2(i2, L));
            const T b = (T)a.bins[cls];
            if (kQuant) {
                q[base + i2] = code_of(y[base + i2], b, &clamped);
            } else {
                out[base + i2] = (T)q[base + i2] * b;
            }
        }
    }
    if (kQuant) count_clamped(clamped, counter);
}

// Bound by memory: 513^3 FP32 (1.08 GB moved) quantised in 182 us, 5.9 TB/s,
// against 280 us with a class lookup per element and 4-byte accesses;
// dequantised in 181 (232).
//
// Class-packed: a workgroup takes kSpan consecutive elements.  Nearly every
// span lies inside one class, whose bin is then uniform; a span across a
// boundary steps every lane's class up from the first.  kVec elements move per
// access (one where the pointers are not 16-byte aligned), kBatch accesses in
// flight: four, or one where spans of four would leave the chip a single round
// of workgroups, all loading and then all storing (dequantised FP32, four and
// one: 2^23 + 1 elements 19.6, 12.9 us, 2^24 + 1 25.4, 20.7).
template <typename T>
constexpr int quant_vec()
{
    return 16 / (int)sizeof(T) < 4 ? 2 : 4;
}
constexpr int kQuantBatch = 4;
template <typename E, int N>
struct QuantVec {
    typedef E V __attribute__((ext_vector_type(N)));
};
template <typename E>
struct QuantVec<E, 1> {
    struct V {
        E x;
        __device__ E& operator[](int) { return x; }
    };
};

template <typename T, bool kQuant, int kVec, int kBatch>
__global__ void __launch_bounds__(kQuantBlock)
    k_quant_packed(const T* __restrict__ y, int* __restrict__ q, T* __restrict__ out, QuantArgs a,
                   unsigned long long* counter)
{
    using VT = typename QuantVec<T, kVec>::V;
    using VI = typename QuantVec<int, kVec>::V;
    constexpr int64_t kSpan = (int64_t)kQuantBlock * kVec * kBatch;
    const int64_t total = a.off[a.L + 1];
    int clamped = 0;
    for (int64_t e0 = (int64_t)blockIdx.x * kSpan; e0 < total; e0 += (int64_t)gridDim.x * kSpan) {
        // class of the span's first element: among the finest, which hold most; else
        // from the starts at or below it, one a lane
        const int lane = (int)threadIdx.x & 63;
        int cls = a.L;
        for (int k = 0; k < 4 && e0 < a.off[cls]; k++) cls--;
        if (e0 < a.off[cls]) cls = uni((int)__popcll(__ballot(lane < a.L && e0 >= a.off[min(lane, a.L)])) - 1);
        const int64_t e1 = min(e0 + kSpan, total);
        if (e1 <= a.off[cls + 1] && e1 - e0 == kSpan) {
            const T b = (T)a.bins[cls];
            const int64_t i0 = e0 + (int64_t)threadIdx.x * kVec;
            VT v[kBatch];
            VI c[kBatch];
#pragma unroll
            for (int k = 0; k < kBatch; k++) {
                const int64_t i = i0 + (int64_t)k * kQuantBlock * kVec;
                if (kQuant)
                    v[k] = *reinterpret_cast<const VT*>(y + i);
                else
                    c[k] = *reinterpret_cast<const VI*>(q + i);
            }
#pragma unroll
            for (int k = 0; k < kBatch; k++) {
                const int64_t i = i0 + (int64_t)k * kQuantBlock * kVec;
#pragma unroll
                for (int j = 0; j < kVec; j++) {
                    if (kQuant)
                        c[k][j] = code_of((T)v[k][j], b, &clamped);
                    else
                        v[k][j] = (T)c[k][j] * b;
                }
                if (kQuant)
                    *reinterpret_cast<VI*>(q + i) = c[k];
                else
                    *reinterpret_cast<VT*>(out + i) = v[k];
            }
        } else {
            int ci = cls;  // (a lane's elements ascend)
            for (int64_t i = e0 + threadIdx.x; i < e1; i += kQuantBlock) {
                while (i >= a.off[ci + 1]) ci++;
                const T b = (T)a.bins[ci];
                if (kQuant)
                    q[i] = code_of(y[i], b, &clamped);
                else
                    out[i] = (T)q[i] * b;
            }
        }
    }
    if (kQuant) count_clamped(clamped, counter);
}

__global__ void k_zero_u64(unsigned long long* p)
{
    if (threadIdx.x == 0) *p = 0ull;
}

}  // namespace

template <typename T>
hipError_t launch_quant(const T* y, int* q, T* out, QuantArgs a, bool quant, unsigned long long* counter,
                        hipStream_t st)
{
    // a grid of a few rounds of the chip's workgroup slots
    int64_t work;
    if (a.packed) {
        work = (a.off[a.L + 1] + kQuantBlock - 1) / kQuantBlock;
    } else {
        // segments of whole waves (64 columns), enough units to fill the chip
        const int64_t rows = a.n[0] * a.n[1];
        const int64_t want = (int64_t)device_cu_count() * 64;
        int64_t nseg = std::max<int64_t>(1, (want + rows - 1) / rows);
        int64_t seg = (a.n[2] + nseg - 1) / nseg;
        seg = std::max<int64_t>(64, (seg + 63) / 64 * 64);
        a.seg = seg;
        a.nseg = (a.n[2] + seg - 1) / seg;
        work = (rows * a.nseg + (kQuantBlock / 64) - 1) / (kQuantBlock / 64);
    }
    const int64_t cap = (int64_t)device_cu_count() * 32;
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min(work, cap));
    if (quant && counter) hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, st, counter);
    if (a.packed) {
        // wide accesses where codes and values are 16-byte aligned (as the
        // device's allocations are); the wide form's spans are kVec times as
        // long
        constexpr int kV = quant_vec<T>();
        const uintptr_t where = (uintptr_t)q | (uintptr_t)(quant ? (const void*)y : (const void*)out);
        const bool wide = where % 16 == 0;
        auto spans = [&](int batch) {
            const int64_t span = (int64_t)kQuantBlock * batch * (wide ? kV : 1);
            return (a.off[a.L + 1] + span - 1) / span;
        };
        auto launch = [&](auto batch) {
            constexpr int B = decltype(batch)::value;
            const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>(spans(B), (int64_t)1 << 22)));
            auto go = [&](auto kern) { hipLaunchKernelGGL(kern, grid, dim3(kQuantBlock), 0, st, y, q, out, a, counter); };
            if (quant)
                wide ? go(k_quant_packed<T, true, kV, B>) : go(k_quant_packed<T, true, 1, B>);
            else
                wide ? go(k_quant_packed<T, false, kV, B>) : go(k_quant_packed<T, false, 1, B>);
        };
        if (spans(kQuantBatch) < 8192)
            launch(std::integral_constant<int, 1>{});
        else
            launch(std::integral_constant<int, kQuantBatch>{});
    } else {
        if (quant)
            hipLaunchKernelGGL((k_quant_inplace<T, true>), dim3(blocks), dim3(kQuantBlock), 0, st, y, q, out, a,
                               counter);
        else
            hipLaunchKernelGGL((k_quant_inplace<T, false>), dim3(blocks), dim3(kQuantBlock), 0, st, y, q, out, a,
                               counter);
    }
    return hipGetLastError();
}

template hipError_t launch_quant<float>(const float*, int*, float*, QuantArgs, bool, unsigned long long*,
                                        hipStream_t);
template hipError_t launch_quant<double>(const double*, int*, double*, QuantArgs, bool, unsigned long long*,
                                         hipStream_t);

}  // namespace mgr
