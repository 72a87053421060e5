// Batched decomposition of many independent fields.
//
// The host lists every workgroup-sized piece of work of every field (the
// streaming level tiles and the correction-solve blocks of each level step)
// as an item, grouped into waves: wave (k, s) holds stage s of level step k
// of every field that has it (stage 0 the streaming pass, then the solves).
// One launch runs a wave's items of one type, one workgroup per item,
// whatever its field or shape; stream order between the waves carries every
// dependency (stage s of a field needs its stage s - 1, level step k + 1
// needs the last solve of step k), so no workgroup ever waits for another.
// The whole sequence (a few dozen launches for any number of fields) is
// what a HIP graph captures.
#include "mgr_solve_dev.h"
#include "mgr_stream_dev.h"

namespace mgr {
namespace {

template <typename T>
union BatchSmem {
    LevelSmem<T, true, true, true, false> lv3;
    LevelSmem<T, true, true, true, true> lv3w;
    LevelSmem<T, true, false, true> lv2;
    LevelSmem<T, false, false, true> lv1;
    StridedSmem<T> str;
    RowsSmem<T, kBatchRowSpan, true> rows_t;
    RowsSmem<T, kBatchRowSpan, false> rows_g;
    ChunkSmem<T, kBatchRowSpan + 64, true> chunk_t;
    ChunkSmem<T, kBatchRowSpan + 64, false> chunk_g;
};

// The queue kernel's LDS (dynamic, sized to BatchSmem<T> at launch).  There each
// item type runs in a function of its own (not inlined), so that its registers
// are allocated on its own: the kernel's register budget is then set by the
// largest item, and items above it spill inside themselves only.
extern __shared__ __align__(16) unsigned char batch_lds[];

// Copy of a wave-uniform struct in scalar registers (the item functions
// reach their arguments through generic pointers, whose loads land in vector
// registers).
template <class S>
__device__ __forceinline__ S load_uniform(const S* p)
{
    static_assert(sizeof(S) % 4 == 0, "whole dwords");
    S out;
    int* o = reinterpret_cast<int*>(&out);
    const int* q = reinterpret_cast<const int*>(p);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(S) / 4); i++) o[i] = __builtin_amdgcn_readfirstlane(q[i]);
    return out;
}

// kWide: the tile geometry the plan chose (3-D only; the 2-D and 1-D
// geometry does not depend on it).
template <typename T, bool kAct0, bool kAct1, bool kWide>
__device__ __attribute__((noinline)) void exec_stream(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    auto& sm = *reinterpret_cast<LevelSmem<T, kAct0, kAct1, true, kWide>*>(batch_lds);
    const BatchItem it = load_uniform(itp);
    StreamArgs<T> a = load_uniform(A->sargs + it.args);
    if (!a.A) a.A = load_uniform(A->src + it.field);
    a.C = load_uniform(A->dst + it.field);
    // unit column strides: FP32 column pairs move in single 8-byte accesses
    const bool unit = a.av.s[2] == 1 && a.cv.s[2] == 1;
    if constexpr (cols_per_lane<T>() == 2) {
        if (unit) {
            if (a.Z)
                stream_level_tile<T, kAct0, kAct1, true, true, true, kWide>(a, it.bx, sm);
            else
                stream_level_tile<T, kAct0, kAct1, true, false, true, kWide>(a, it.bx, sm);
            return;
        }
    }
    if (a.Z)
        stream_level_tile<T, kAct0, kAct1, true, true, false, kWide>(a, it.bx, sm);
    else
        stream_level_tile<T, kAct0, kAct1, true, false, false, kWide>(a, it.bx, sm);
}

template <typename T>
__device__ __forceinline__ FibreMap fibre_map(const BatchSolve<T>& b)
{
    FibreMap m;
    m.n = b.n;
    m.inner = b.inner;
    m.outer = b.outer;
    m.nfib = b.nfib;
    m.S = b.tb.S;
    return m;
}

template <typename T, bool kLdsTab>
__device__ __forceinline__ void rows_item(const BatchItem& it, const BatchSolve<T>& b,
                                          RowsSmem<T, kBatchRowSpan, kLdsTab>& sm)
{
    const FibreMap m = fibre_map(b);
    const int64_t row0 = (int64_t)it.bx * b.rows;
    const int nrows = (int)min((int64_t)b.rows, m.nfib - row0);
    solve_rows_tile<T, kBatchRowSpan, kLdsTab>(b.F, m, b.tb, row0, nrows, sm);
}

template <typename T>
__device__ __attribute__((noinline)) void exec_rows(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    const BatchSolve<T> b = load_uniform(A->solves + it.args);
    if (b.tb.S <= kMaxSegWG)
        rows_item<T, true>(it, b, *reinterpret_cast<RowsSmem<T, kBatchRowSpan, true>*>(batch_lds));
    else
        rows_item<T, false>(it, b, *reinterpret_cast<RowsSmem<T, kBatchRowSpan, false>*>(batch_lds));
}

template <typename T>
__device__ __forceinline__ void strided_item(const BatchItem& it, const BatchSolve<T>& b, StridedSmem<T>& sm)
{
    const FibreMap m = fibre_map(b);
    const int tid = threadIdx.x;
    auto run = [&](auto fb) {
        constexpr int FB = decltype(fb)::value;
        solve_strided_tile<T, FB, false>(b.F, b.F, m, b.tb, (int64_t)it.bx * FB, tid / FB, tid % FB, kThreads, tid, sm,
                                         0, m.S, nullptr);
    };
    switch (batch_strided_fibres(m.S)) {
        case 256: run(std::integral_constant<int, 256>{}); break;
        case 128: run(std::integral_constant<int, 128>{}); break;
        case 64: run(std::integral_constant<int, 64>{}); break;
        case 32: run(std::integral_constant<int, 32>{}); break;
        default: run(std::integral_constant<int, 16>{}); break;
    }
}

template <typename T>
__device__ __attribute__((noinline)) void exec_strided(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    const BatchSolve<T> b = load_uniform(A->solves + it.args);
    const FibreMap m = fibre_map(b);
    const int tid = threadIdx.x;
    solve_strided_tile<T, 16, false>(b.F, b.F, m, b.tb, (int64_t)it.bx * 16, tid / 16, tid % 16, kThreads, tid,
                                     *reinterpret_cast<StridedSmem<T>*>(batch_lds), 0, m.S, nullptr);
}

// Long fibres whose separators do not couple: the separators between chunks,
// and the chunks.
template <typename T>
__device__ __forceinline__ void sep_bounds_item(const BatchItem& it, const BatchSolve<T>& b)
{
    const FibreMap m = fibre_map(b);
    const int ns = solve_chunk_segs(m.S, m.inner, m.nfib);
    if (m.inner > 1)
        sep_bounds_strided(b.F, b.Yb, m, b.tb, ns, it.bx, it.by);
    else
        sep_bounds_rows(b.F, b.Yb, m, b.tb, ns, (int64_t)it.bx * (kBlk / 64) + (threadIdx.x >> 6));
}

template <typename T>
__device__ __attribute__((noinline)) void exec_sep_bounds(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    sep_bounds_item<T>(it, load_uniform(A->solves + it.args));
}

template <typename T, bool kLdsTab>
__device__ __forceinline__ void chunk_rows_item(const BatchItem& it, const BatchSolve<T>& b, int ns,
                                                ChunkSmem<T, kBatchRowSpan + 64, kLdsTab>& sm)
{
    const FibreMap m = fibre_map(b);
    const int s0 = it.by * ns, nsc = min(ns, m.S - s0);
    const int64_t row0 = (int64_t)it.bx * b.rows;
    const int nrows = (int)min((int64_t)b.rows, m.nfib - row0);
    const T* zb = b.Yb + ((int64_t)it.by - 1) * m.nfib;
    solve_chunk_rows<T, kBatchRowSpan + 64, kLdsTab>(b.F, m, b.tb, row0, nrows, s0, nsc, zb, sm);
}

template <typename T>
__device__ __attribute__((noinline)) void exec_chunk_rows(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    const BatchSolve<T> b = load_uniform(A->solves + it.args);
    const int ns = solve_chunk_segs(b.tb.S, b.inner, b.nfib);
    if (ns <= kMaxSegWG)
        chunk_rows_item<T, true>(it, b, ns, *reinterpret_cast<ChunkSmem<T, kBatchRowSpan + 64, true>*>(batch_lds));
    else
        chunk_rows_item<T, false>(it, b, ns, *reinterpret_cast<ChunkSmem<T, kBatchRowSpan + 64, false>*>(batch_lds));
}

template <typename T>
__device__ __forceinline__ void chunk_strided_item(const BatchItem& it, const BatchSolve<T>& b, StridedSmem<T>& sm)
{
    const FibreMap m = fibre_map(b);
    const int ns = solve_chunk_segs(m.S, m.inner, m.nfib), s0 = it.by * ns;
    const int tid = threadIdx.x;
    solve_strided_tile<T, 16, false>(b.F, b.F, m, b.tb, (int64_t)it.bx * 16, tid / 16, tid % 16, kThreads, tid, sm, s0,
                                     min(ns, m.S - s0), b.Yb + ((int64_t)it.by - 1) * m.nfib);
}

template <typename T>
__device__ __attribute__((noinline)) void exec_chunk_strided(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    const BatchSolve<T> b = load_uniform(A->solves + it.args);
    chunk_strided_item<T>(it, b, *reinterpret_cast<StridedSmem<T>*>(batch_lds));
}

template <typename T>
__device__ __forceinline__ void phase_item(const BatchItem& it, const BatchSolve<T>& b)
{
    const FibreMap m = fibre_map(b);
    if (it.type == BI_SEG_ENDS)
        seg_ends_tile(b.F, b.Yb, m, b.tb, it.bx, it.by);
    else if (it.type == BI_SEPARATORS)
        separators_tile(b.F, b.Yb, m, b.tb, it.bx);
    else
        seg_final_tile(b.F, m, b.tb, it.bx, it.by);
}

template <typename T>
__device__ __attribute__((noinline)) void exec_phase(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    phase_item<T>(it, load_uniform(A->solves + it.args));
}

template <typename T>
__device__ __forceinline__ void scatter_item(const BatchItem& it, const BatchScatter<T>& sc, T* dst)
{
    const int64_t idx = (int64_t)it.bx * kThreads + threadIdx.x;
    if (idx >= sc.n[0] * sc.n[1] * sc.n[2]) return;
    const int64_t j2 = idx % sc.n[2], j1 = (idx / sc.n[2]) % sc.n[1], j0 = idx / (sc.n[1] * sc.n[2]);
    dst[j0 * sc.ds[0] + j1 * sc.ds[1] + j2 * sc.ds[2]] = sc.W[idx] + sc.Z[idx];
}

template <typename T>
__device__ __attribute__((noinline)) void exec_scatter(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    const BatchItem it = load_uniform(itp);
    scatter_item<T>(it, load_uniform(A->scatters + it.args), load_uniform(A->dst + it.field));
}

// One launch per item type of a wave: its kernel holds that type alone, with
// its registers and LDS, and deals neighbouring items to one XCD (they share
// halo lines).  60 fields FP32 (445 MB): 910 us, against 1286 in launches of a
// kernel that reached every type through function calls (four waves a SIMD and
// 30 KB of LDS for all of them); 16 fields FP64 650 against 2320 (904 bytes of
// scratch there).  Types of a wave run one after the other: also with few items
// that is faster than together (4 fields 168 -> 130 and 620 -> 216 us).
template <typename T, bool kAct0, bool kAct1, bool kWide, bool kZ>
__global__ void __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && kWide && !kZ ? 4 : stream_min_waves<T, true, kZ>(), 8)))
k_batch_stream(BatchKernelArgs<T> A, int first)
{
    __shared__ LevelSmem<T, kAct0, kAct1, true, kWide> sm;
    const BatchItem it = A.items[first + remap_xcd((int)blockIdx.x, (int)gridDim.x)];
    StreamArgs<T> a = A.sargs[it.args];
    if (!kZ) a.A = A.src[it.field];
    a.C = A.dst[it.field];
    stream_level_tile<T, kAct0, kAct1, true, kZ, false, kWide>(a, it.bx, sm);
}

template <typename T, bool kLong>
__global__ void __launch_bounds__(kThreads) k_batch_rows(BatchKernelArgs<T> A, int first)
{
    __shared__ RowsSmem<T, kBatchRowSpan, !kLong> sm;
    const BatchItem it = A.items[first + remap_xcd((int)blockIdx.x, (int)gridDim.x)];
    rows_item<T, !kLong>(it, A.solves[it.args], sm);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_batch_strided(BatchKernelArgs<T> A, int first)
{
    __shared__ StridedSmem<T> sm;
    const BatchItem it = A.items[first + remap_xcd((int)blockIdx.x, (int)gridDim.x)];
    const BatchSolve<T> b = A.solves[it.args];
    strided_item<T>(it, b, sm);
}

template <typename T, bool kLong>
__global__ void __launch_bounds__(kThreads) k_batch_chunk_rows(BatchKernelArgs<T> A, int first)
{
    __shared__ ChunkSmem<T, kBatchRowSpan + 64, !kLong> sm;
    const BatchItem it = A.items[first + (int)blockIdx.x];
    const BatchSolve<T> b = A.solves[it.args];
    chunk_rows_item<T, !kLong>(it, b, solve_chunk_segs(b.tb.S, b.inner, b.nfib), sm);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_batch_chunk_strided(BatchKernelArgs<T> A, int first)
{
    __shared__ StridedSmem<T> sm;
    const BatchItem it = A.items[first + remap_xcd((int)blockIdx.x, (int)gridDim.x)];
    const BatchSolve<T> b = A.solves[it.args];
    chunk_strided_item<T>(it, b, sm);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_batch_sep_bounds(BatchKernelArgs<T> A, int first)
{
    const BatchItem it = A.items[first + (int)blockIdx.x];
    sep_bounds_item<T>(it, A.solves[it.args]);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_batch_phase(BatchKernelArgs<T> A, int first)
{
    const BatchItem it = A.items[first + (int)blockIdx.x];
    phase_item<T>(it, A.solves[it.args]);
}

template <typename T>
__global__ void __launch_bounds__(kThreads) k_batch_scatter(BatchKernelArgs<T> A, int first)
{
    const BatchItem it = A.items[first + (int)blockIdx.x];
    scatter_item<T>(it, A.scatters[it.args], A.dst[it.field]);
}

// Device side of the queue protocol (mgr_queue.h), run by a whole wave:
// every value it returns is wave-uniform (one lane does each atomic and the
// result is broadcast), so the loops and branches around it are uniform.
// The queue words are accessed with agent-scope atomics; polls are relaxed
// loads with a sleep between them.  An item and the items it depends on run
// on one XCD, under one L2: the producer's stores have reached that L2 when
// its counter moves (the caller waits for them), so no L2 write-back is
// needed.  The consumer must still drop its CU's L1, which may hold lines it
// read before the producer wrote them (a cache line can span the parts of
// two items); on this device only an agent-scope invalidation reaches the L1
// of a workgroup whose waves share one CU (a workgroup-scope one is a no-op
// there), and it also drops the XCD's clean L2 lines, never dirty ones.
struct DevQueueOps {
    __device__ static bool leader() { return (threadIdx.x & 63) == 0; }
    __device__ int load_relaxed(int* p) const
    {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __device__ void fence_acquire() const { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent"); }
    __device__ int fetch_add_relaxed(int* p, int v) const
    {
        int r = 0;
        if (leader()) r = __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return __builtin_amdgcn_readfirstlane(r);
    }
    // the caller has waited until every store of the item reached the L2
    __device__ void add_release(int* p, int v) const
    {
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        if (leader()) (void)__hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ void store_relaxed(int* p, int v) const
    {
        if (leader()) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ void cas_relaxed(int* p, int expect, int v) const
    {
        if (leader())
            (void)__hip_atomic_compare_exchange_strong(p, &expect, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ void pause() const { __builtin_amdgcn_s_sleep(2); }
};

template <typename T>
__device__ __forceinline__ void run_item(const BatchKernelArgs<T>* A, const BatchItem* itp)
{
    switch (itp->type) {
        case BI_STREAM3: exec_stream<T, true, true, false>(A, itp); break;
        case BI_STREAM3W: exec_stream<T, true, true, true>(A, itp); break;
        case BI_STREAM2: exec_stream<T, true, false, false>(A, itp); break;
        case BI_STREAM1: exec_stream<T, false, false, false>(A, itp); break;
        case BI_ROWS:
        case BI_ROWS_LONG: exec_rows<T>(A, itp); break;
        case BI_STRIDED: exec_strided<T>(A, itp); break;
        case BI_SCATTER: exec_scatter<T>(A, itp); break;
        case BI_SEP_BOUNDS: exec_sep_bounds<T>(A, itp); break;
        case BI_CHUNK_ROWS:
        case BI_CHUNK_ROWS_LONG: exec_chunk_rows<T>(A, itp); break;
        case BI_CHUNK_STRIDED: exec_chunk_strided<T>(A, itp); break;
        default: exec_phase<T>(A, itp); break;
    }
}

// The persistent form: every workgroup takes items from the queue of the XCD
// it runs on until that queue is empty (or the run is aborted), waiting for
// each item's dependency group first.  The grid size is free (a workgroup
// takes an item only while it runs; workgroups are dealt to every XCD).
// Wave 0 takes and finishes items as a whole wave (the branch on the wave
// index is uniform); the position is broadcast through LDS and read back as
// a uniform value, so the loop's exit and every branch around its barriers
// are uniform: with a per-thread index the compiler may restructure the loop
// so that the lanes of one wave take different paths around a barrier, and
// the wave never reconverges.  After an item every thread waits until its
// own memory operations have completed (its stores are then in the L2), the
// barrier then lets wave 0 mark the item finished; wave 0's cache
// invalidation after the wait precedes the barrier that starts the next item
// for every thread (all waves of a workgroup share one CU and its L1).
template <typename T>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8)))
k_batch_queue(const BatchKernelArgs<T>* __restrict__ A, QueueTables qt, QueueState qs, unsigned limit)
{
    __shared__ int s_item;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned xcc;
    asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
    const int q = (int)(xcc & 0xfu) % qt.nq;
    int last_dg = -1;  // wave 0's
    for (;;) {
        if (wave == 0) {
            const int t = queue_take(qt, qs, q, limit, last_dg, DevQueueOps{});
            if (DevQueueOps::leader()) s_item = t;
        }
        __syncthreads();
        const int i = __builtin_amdgcn_readfirstlane(s_item);
        if (i < 0) break;
        run_item(A, A->items + qt.order[i]);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);  // no memory operation moves below the wait
        __builtin_amdgcn_s_waitcnt(0);             // this wave's loads and stores completed
        __syncthreads();
        if (wave == 0) queue_finish(qt, qs, i, DevQueueOps{});
    }
}

__global__ void __launch_bounds__(256) k_zero_words(int* p, int n)
{
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < n; i += (int)(gridDim.x * 256)) p[i] = 0;
}

}  // namespace

int device_cu_count()
{
    static int cache[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cache[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cache[dev] = n;
    }
    return cache[dev];
}

template <typename T>
hipError_t launch_batch_items(const BatchKernelArgs<T>& a, int first, int n, int type, bool z, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)n), dim3(kThreads), 0, st, a, first);
        return hipGetLastError();
    };
    switch (type) {
        case BI_STREAM3:
            return z ? go(k_batch_stream<T, true, true, false, true>) : go(k_batch_stream<T, true, true, false, false>);
        case BI_STREAM3W:
            return z ? go(k_batch_stream<T, true, true, true, true>) : go(k_batch_stream<T, true, true, true, false>);
        case BI_STREAM2:
            return z ? go(k_batch_stream<T, true, false, false, true>) : go(k_batch_stream<T, true, false, false, false>);
        case BI_STREAM1:
            return z ? go(k_batch_stream<T, false, false, false, true>) : go(k_batch_stream<T, false, false, false, false>);
        case BI_ROWS: return go(k_batch_rows<T, false>);
        case BI_ROWS_LONG: return go(k_batch_rows<T, true>);
        case BI_STRIDED: return go(k_batch_strided<T>);
        case BI_CHUNK_ROWS: return go(k_batch_chunk_rows<T, false>);
        case BI_CHUNK_ROWS_LONG: return go(k_batch_chunk_rows<T, true>);
        case BI_CHUNK_STRIDED: return go(k_batch_chunk_strided<T>);
        case BI_SEP_BOUNDS: return go(k_batch_sep_bounds<T>);
        case BI_SEG_ENDS:
        case BI_SEPARATORS:
        case BI_SEG_FINAL: return go(k_batch_phase<T>);
        case BI_SCATTER: return go(k_batch_scatter<T>);
        default: return hipErrorInvalidValue;
    }
}

// Writes up to kPtrChunk pointers, passed by value, to dst.  A graph that
// captures the launch keeps the values in its kernel node, so each replay
// restores the pointers of the call that was captured, whatever calls ran
// in between.
__global__ void __launch_bounds__(64) k_set_ptrs(PtrChunk c, void** dst)
{
    for (int i = (int)threadIdx.x; i < c.n; i += 64) dst[c.first + i] = c.p[i];
}

hipError_t launch_set_ptrs(const PtrChunk& c, void** dst, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_ptrs, dim3(1), dim3(64), 0, st, c, dst);
    return hipGetLastError();
}

// The whole queue in one launch of `grid` workgroups, after zeroing the
// queue words (`words` ints from qs.next: next, abort, err, then done[]).
template <typename T>
hipError_t launch_batch_queue(const BatchKernelArgs<T>* dev_a, const QueueTables& qt, const QueueState& qs, int words,
                              int grid, unsigned limit, hipStream_t st)
{
    hipLaunchKernelGGL(k_zero_words, dim3((unsigned)std::min(64, (words + 255) / 256)), dim3(256), 0, st, qs.abort,
                       words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_batch_queue<T>, dim3((unsigned)grid), dim3(kThreads), sizeof(BatchSmem<T>), st, dev_a, qt, qs,
                       limit);
    return hipGetLastError();
}

// Workgroups of the queue kernel that the device holds at once.
template <typename T>
int batch_queue_slots()
{
    static int cache[2] = {0, 0};
    int& c = cache[sizeof(T) == 8 ? 1 : 0];
    if (c == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_batch_queue<T>, kThreads, sizeof(BatchSmem<T>)) !=
                hipSuccess ||
            n <= 0)
            n = 1;
        c = n * device_cu_count();
    }
    return c;
}

template hipError_t launch_batch_queue<float>(const BatchKernelArgs<float>*, const QueueTables&, const QueueState&, int,
                                              int, unsigned, hipStream_t);
template hipError_t launch_batch_queue<double>(const BatchKernelArgs<double>*, const QueueTables&, const QueueState&,
                                               int, int, unsigned, hipStream_t);
template int batch_queue_slots<float>();
template int batch_queue_slots<double>();
template hipError_t launch_batch_items<float>(const BatchKernelArgs<float>&, int, int, int, bool, hipStream_t);
template hipError_t launch_batch_items<double>(const BatchKernelArgs<double>&, int, int, int, bool, hipStream_t);

}  // namespace mgr
