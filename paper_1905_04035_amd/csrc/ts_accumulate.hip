// ts_accumulate: the paper's two accumulation rules (arXiv 1905.04035, Section 3,
// Algorithm 1 and Section 6, Algorithm 2) for the gradients one variable receives.
//
// The rule picks a branch on the host; the branches are
//   reduce            sum_kernel: dense tensors added in list order, one streaming pass
//   convert + reduce  the dense tensor (or sum_kernel's sum of several) becomes dense_in of
//                     ts_densify_multi, which converts the slice gradients and adds them
//   gather            every gradient as slices, laid end to end, in one launch: gather_kernel
//                     copies ids and value rows and writes ids 0 .. V-1 for a dense tensor
// This file sits on top of the public entry points; it shares no state with them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ts_densify.h"

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kMaxDense = 16;     // dense tensors summed by one launch
constexpr int kThreads = 256;             // of a work-group of sum_kernel
constexpr int64_t kMaxWgs = 1 << 22;      // work-groups per launch (a launch has less than 2^32 threads)

struct DenseList {
    int32_t m;
    const float* src[kMaxDense];
};

__device__ __forceinline__ f4 load_stream(const float* p, int64_t i)
{
    return __builtin_nontemporal_load(reinterpret_cast<const f4*>(p) + i);
}

// out[i] = ((src0[i] + src1[i]) + src2[i]) + ...   HBM-bound: (M + 1) * 4 bytes per element.
// A work-group takes U slabs of 4 KiB that lie one behind the other, from every source, and all
// loads of a thread are in flight before the first addition.  M = 0: any number of sources, one
// slab.  U = 4 where the registers hold it.  Three tensors of [32768, 1024]: 84.6 us = 6.3 TB/s; one
// slab per work-group 85.6, a grid-stride loop over 16384 work-groups, as this kernel used to be, 88.3;
// work-groups of 128 / 512 threads 86.5 / 89.6.
template <int M, int U>
__global__ __launch_bounds__(kThreads) void sum_kernel(DenseList l, float* out, int64_t n4, int64_t i_first)
{
    const int64_t i0 = i_first + (int64_t)blockIdx.x * (U * kThreads) + threadIdx.x;
    if constexpr (M == 0) {
        if (i0 >= n4) return;
        f4 acc = load_stream(l.src[0], i0);
        for (int j = 1; j < l.m; ++j) acc += load_stream(l.src[j], i0);
        __builtin_nontemporal_store(acc, reinterpret_cast<f4*>(out) + i0);
    } else {
        f4 x[M][U];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < M; ++j) {
                // threads past the end read the last element again: no load is conditional
                const int64_t i = i0 + u * kThreads;
                x[j][u] = load_stream(l.src[j], i < n4 ? i : n4 - 1);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 1; j < M; ++j) x[0][u] += x[j][u];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kThreads < n4) __builtin_nontemporal_store(x[0][u], reinterpret_cast<f4*>(out) + i0 + u * kThreads);
    }
}

// A gather lays all gradients end to end with one launch: every gradient is a run of value rows
// and a run of ids (copied, or 0 .. V-1 for a dense tensor), and a work-group of one wavefront
// takes 64 consecutive elements of one run (16 bytes of value rows or one id per lane).  HBM-bound:
// every byte is read once and written once.  Two slice gradients of 8192 rows and a dense
// [32768, 1024] one, 403 MB: 62.9 us = 6.40 TB/s; with work-groups of 128 / 256 / 512 threads 66.8 /
// 65.6 / 65.6 us (slots are given back in larger lots), and with two launches per gradient, as it was
// before, 72.5.
enum { RUN_ROWS = 0, RUN_IDS = 1, RUN_IOTA = 2 };

struct Run {
    const void* src;
    void* dst;
    int64_t n;              // elements: 16-byte vectors of value rows, or ids
    int32_t first_wg;
    int32_t kind;
};

constexpr int kGatherThreads = 64;
constexpr int kMaxRuns = 64;               // per launch; runs beyond it, or beyond kMaxWgs, go to further launches

struct RunTable {
    int32_t m;
    Run run[kMaxRuns];      // ascending first_wg
};

__global__ __launch_bounds__(kGatherThreads) void gather_kernel(RunTable t)
{
    const int b = (int)blockIdx.x;
    int lo = 0, hi = t.m - 1;           // the last run that begins at or before this work-group
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (t.run[mid].first_wg <= b) lo = mid;
        else hi = mid - 1;
    }
    const Run r = t.run[lo];
    const int64_t i = (int64_t)(b - r.first_wg) * kGatherThreads + threadIdx.x;
    if (i >= r.n) return;
    if (r.kind == RUN_ROWS)
        __builtin_nontemporal_store(load_stream((const float*)r.src, i), (f4*)r.dst + i);
    else
        ((int32_t*)r.dst)[i] = r.kind == RUN_IDS ? ((const int32_t*)r.src)[i] : (int32_t)((int64_t)(uintptr_t)r.src + i);
}

int launch_sum(const DenseList& l, float* out, int64_t n4, hipStream_t stream)
{
    constexpr int U = 4;
    for (int64_t at = 0; at < n4;) {
        const int64_t per_wg = (l.m <= 4 ? U : 1) * kThreads;
        const int64_t wgs = (n4 - at + per_wg - 1) / per_wg;
        const dim3 grid((unsigned)(wgs < kMaxWgs ? wgs : kMaxWgs));
        if (l.m == 1) hipLaunchKernelGGL((sum_kernel<1, U>), grid, dim3(kThreads), 0, stream, l, out, n4, at);
        else if (l.m == 2) hipLaunchKernelGGL((sum_kernel<2, U>), grid, dim3(kThreads), 0, stream, l, out, n4, at);
        else if (l.m == 3) hipLaunchKernelGGL((sum_kernel<3, U>), grid, dim3(kThreads), 0, stream, l, out, n4, at);
        else if (l.m == 4) hipLaunchKernelGGL((sum_kernel<4, U>), grid, dim3(kThreads), 0, stream, l, out, n4, at);
        else hipLaunchKernelGGL((sum_kernel<0, 1>), grid, dim3(kThreads), 0, stream, l, out, n4, at);
        at += (int64_t)grid.x * per_wg;
    }
    return hipGetLastError() == hipSuccess ? TS_OK : TS_ERR_HIP;
}

bool overlap(const void* a, int64_t a_bytes, const void* b, int64_t b_bytes)
{
    return (uintptr_t)a < (uintptr_t)b + (uintptr_t)b_bytes && (uintptr_t)b < (uintptr_t)a + (uintptr_t)a_bytes;
}

// Collects runs and launches when the table or the grid is full, or (in_order) run by run.
struct Gather {
    RunTable t;
    int64_t wgs;
    hipStream_t stream;
    bool in_order;

    Gather(hipStream_t s, bool order) : wgs(0), stream(s), in_order(order) { t.m = 0; }
    void flush()
    {
        if (t.m > 0) hipLaunchKernelGGL(gather_kernel, dim3((unsigned)wgs), dim3(kGatherThreads), 0, stream, t);
        t.m = 0;
        wgs = 0;
    }
    // src of RUN_IOTA: the first number, as an address
    void add(int kind, const void* src, void* dst, int64_t n)
    {
        const int64_t dst_bytes = kind == RUN_ROWS ? 16 : 4, src_bytes = kind == RUN_IOTA ? 1 : dst_bytes;
        for (int64_t a = 0, len; a < n; a += len) {
            len = n - a < kMaxWgs * kGatherThreads ? n - a : kMaxWgs * kGatherThreads;
            const int64_t need = (len + kGatherThreads - 1) / kGatherThreads;
            if (t.m == kMaxRuns || wgs + need > kMaxWgs || in_order) flush();
            t.run[t.m++] = Run{(const void*)((uintptr_t)src + (uintptr_t)(a * src_bytes)), (char*)dst + a * dst_bytes, len, (int32_t)wgs, kind};
            wgs += need;
        }
    }
};

int strategy_of(const ts_grad* grads, int32_t m, int32_t rule)
{
    if (m < 2) return TS_ACC_PASS_THROUGH;
    bool all_dense = true, any_dense = false;
    for (int i = 0; i < m; ++i) {
        if (grads[i].kind == TS_GRAD_DENSE) any_dense = true;
        else all_dense = false;
    }
    if (all_dense) return TS_ACC_REDUCE;
    if (rule == TS_RULE_PROPOSED && any_dense) return TS_ACC_DENSIFY_REDUCE;
    return TS_ACC_GATHER;
}

int check_list(const ts_grad* grads, int32_t m, int32_t rule)
{
    if (!grads) return TS_ERR_NULL;
    if (m < 1 || (rule != TS_RULE_TF && rule != TS_RULE_PROPOSED)) return TS_ERR_SHAPE;
    for (int i = 0; i < m; ++i) {
        const ts_grad& g = grads[i];
        if (g.kind != TS_GRAD_DENSE && g.kind != TS_GRAD_SLICES) return TS_ERR_SHAPE;
        if (g.kind == TS_GRAD_SLICES && g.n < 0) return TS_ERR_SHAPE;
        const bool empty = g.kind == TS_GRAD_SLICES && g.n == 0;
        if (!empty && !g.values) return TS_ERR_NULL;
        if (g.kind == TS_GRAD_SLICES && g.n > 0 && !g.ids) return TS_ERR_NULL;
        if ((uintptr_t)g.values & 15u) return TS_ERR_ALIGN;
    }
    return TS_OK;
}

}  // namespace

extern "C" {

int ts_accumulate_strategy(const ts_grad* grads, int32_t m, int32_t rule, int32_t* strategy_out)
{
    if (!strategy_out) return TS_ERR_NULL;
    const int rc = check_list(grads, m, rule);
    if (rc != TS_OK) return rc;
    *strategy_out = strategy_of(grads, m, rule);
    return TS_OK;
}

int ts_accumulate(const ts_grad* grads, int32_t m, int32_t rule, int32_t d, int32_t V, float* dense_out,
                  int32_t* ids_out, float* rows_out, int64_t slice_capacity, int64_t* n_slices_out,
                  int32_t* strategy_out, void* stream_v)
{
    int rc = check_list(grads, m, rule);
    if (rc != TS_OK) return rc;
    if (V <= 0 || d <= 0 || (d % 4) != 0) return TS_ERR_SHAPE;
    hipStream_t stream = (hipStream_t)stream_v;
    const int st = strategy_of(grads, m, rule);
    if (strategy_out) *strategy_out = st;
    const int64_t vd4 = (int64_t)V * d / 4;

    const bool dense_result = st == TS_ACC_REDUCE || st == TS_ACC_DENSIFY_REDUCE ||
                              (st == TS_ACC_PASS_THROUGH && grads[0].kind == TS_GRAD_DENSE);
    if (dense_result) {
        if (!dense_out) return TS_ERR_NULL;
        if ((uintptr_t)dense_out & 15u) return TS_ERR_ALIGN;
        // the dense tensors, in list order
        DenseList l;
        l.m = 0;
        for (int i = 0; i < m; ++i)
            if (grads[i].kind == TS_GRAD_DENSE) {
                if (l.m == kMaxDense) return TS_ERR_SHAPE;
                l.src[l.m++] = grads[i].values;
            }
        for (int j = l.m; j < kMaxDense; ++j) l.src[j] = nullptr;
        if (st != TS_ACC_DENSIFY_REDUCE) {
            if (l.m == 1 && l.src[0] == dense_out) return TS_OK;       // passed through in place
            return launch_sum(l, dense_out, vd4, stream);
        }
        // Algorithm 2, added branch: one dense tensor is the dense operand of the conversion as
        // it is; several are summed into dense_out first and the conversion adds in place
        const float* dense_in = l.src[0];
        if (l.m > 1) {
            rc = launch_sum(l, dense_out, vd4, stream);
            if (rc != TS_OK) return rc;
            dense_in = dense_out;
        }
        const int32_t* ids_k[TS_MAX_SHARDS];
        const void* rows_k[TS_MAX_SHARDS];
        int64_t n_k[TS_MAX_SHARDS];
        int k = 0;
        for (int i = 0; i < m; ++i)
            if (grads[i].kind == TS_GRAD_SLICES) {
                if (k == TS_MAX_SHARDS) return TS_ERR_SHAPE;
                ids_k[k] = grads[i].ids;
                rows_k[k] = grads[i].values;
                n_k[k] = grads[i].n;
                ++k;
            }
        return ts_densify_multi(ids_k, rows_k, n_k, k, TS_ROW_FP32, d, V, dense_in, dense_out, stream);
    }

    // slices result: gather, or one slices gradient passed through
    int64_t total = 0;
    for (int i = 0; i < m; ++i) {
        total += grads[i].kind == TS_GRAD_DENSE ? (int64_t)V : grads[i].n;
        if (total >= ((int64_t)1 << 31)) return TS_ERR_OVERFLOW;
    }
    if (!n_slices_out) return TS_ERR_NULL;
    if (total > slice_capacity) return TS_ERR_CAPACITY;
    if (total > 0 && (!ids_out || !rows_out)) return TS_ERR_NULL;
    if ((uintptr_t)rows_out & 15u) return TS_ERR_ALIGN;
    *n_slices_out = total;
    // An input that lies in an output, but not where it is copied to (ids in the place of a later gradient's
    // ids, say), is read before later runs are written over it: the runs are then launched one by one.
    bool in_order = false;
    int64_t at = 0;
    for (int i = 0; i < m; ++i) {
        const bool dense = grads[i].kind == TS_GRAD_DENSE;
        const int64_t n = dense ? (int64_t)V : grads[i].n;
        const auto in_outputs = [&](const void* src, int64_t bytes, const void* dst) {
            return src != dst && (overlap(src, bytes, ids_out, total * 4) || overlap(src, bytes, rows_out, total * d * 4));
        };
        if (n > 0 && !dense) in_order = in_order || in_outputs(grads[i].ids, n * 4, ids_out + at);
        if (n > 0) in_order = in_order || in_outputs(grads[i].values, n * d * 4, rows_out + at * d);
        at += n;
    }
    Gather g(stream, in_order);
    at = 0;
    for (int i = 0; i < m; ++i) {
        const bool dense = grads[i].kind == TS_GRAD_DENSE;
        const int64_t n = dense ? (int64_t)V : grads[i].n;
        if (n == 0) continue;
        g.add(dense ? RUN_IOTA : RUN_IDS, dense ? nullptr : grads[i].ids, ids_out + at, n);
        g.add(RUN_ROWS, grads[i].values, rows_out + at * d, n * d / 4);
        at += n;
    }
    g.flush();
    return hipGetLastError() == hipSuccess ? TS_OK : TS_ERR_HIP;
}

}  // extern "C"
