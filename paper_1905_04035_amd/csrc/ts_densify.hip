// ts_densify: densify an assumed-sparse gradient and add the dense one, on gfx950.
//
// The result is the one defined by arXiv 1905.04035, Section 4 (Listing 1: an
// IndexedSlices gradient becomes a dense tensor) and Section 6 (Algorithm 2, added
// branch: every gradient becomes dense, then they are summed):
//
//     dense_out[v,:] = dense_in[v,:] + sum_{t : ids[t] == v} rows[t,:]
//
// Two launches per call (three when the pairs need more than one sort slice, one for the smallest calls:
// small_kernel), all on the caller's stream, no host synchronisation, no allocation:
//
//   sort_kernel     stable counting sort of the pairs by id.  Work-group (g, s) owns `part`
//                   consecutive ids (128 .. 2048) and slice s of the pairs; its 16
//                   wavefronts load their sub-slices into registers, list the pairs the
//                   work-group owns in LDS, count them into LDS-private tables, an
//                   exclusive scan turns the counts into offsets, and a walk over the
//                   lists hands every owned pair its final position.
//                   A part's first position is the number of pairs with a smaller id,
//                   which the work-group counts itself while it scans, so parts never
//                   wait for one another.  With one slice (up to 57344 pairs) this is a
//                   single launch; with more, a counting launch (count_kernel: one LDS
//                   table per work-group, no lists) fills a [slice][id] table first.
//                   The sort leaves one 32-byte record per sorted pair.
//   reduce_kernel   the HBM-bound kernel.  First the work-groups that add value rows: each
//                   takes four (C = 8: eight) consecutive pieces of C sorted positions (one per wavefront)
//                   and one block of 256 columns.  The pieces of a row with more than C
//                   pairs are added up through LDS by the wavefront that holds the row's
//                   last piece in the work-group.  A row that spans several work-groups
//                   leaves one fp32 share per work-group in scratch; arrival counters tell
//                   the work-group that brings the last share, which adds the shares in a
//                   fixed tree order, adds dense_in and writes the row.  Then work-groups
//                   that take one output row (1024 columns of it, if it is wider) per
//                   wavefront, 16 bytes per lane, streaming:
//                   they copy the rows that received no pair.  Rows with at most C pairs:
//                   in a call with few pairs or narrow rows the wavefront in whose piece such
//                   a row starts finishes it (dense_in + sum straight to dense_out); else
//                   the wavefront that would copy the row adds up its few value rows
//                   instead, and the pieces pass over them; there, with pieces of 16
//                   positions or fewer, one wavefront walks the pieces of a group by itself
//                   and keeps their sums in registers (no LDS, no barrier).  Same order of
//                   additions, same bits in every form.
//
// The sort is a chain of latencies and instructions that moves almost nothing, so a sort of up to six
// slices also carries work-groups that copy dense rows [0, X) and keep HBM busy, before it
// is known which of them receive pairs (the reduce kernel, which runs later, overwrites
// those).  The reduce kernel copies the untouched rows of [X, V).
//
// No floating-point atomics anywhere: the position of every pair, the cut points and
// the order of every addition depend on the ids and the sizes (pairs, columns, vocabulary,
// row type) alone, so results are reproducible bit for bit.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <string.h>
#include <type_traits>

#include "ts_densify.h"
#include "ts_densify_tools.h"

// Built-in workspace of ts_densify_static, the entry point for callers that cannot allocate.
// One copy per GPU, held from the moment the library is loaded on it until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress: kernels and
// memory calls are given the device address that call returns (static_scratch() below).
static __device__ __align__(256) unsigned char scratch[TS_STATIC_SCRATCH_BYTES];

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// One sorted pair, as the sort leaves it for the reduce kernel: where its value row is, and
// everything the reduce kernel needs to know about the output row it belongs to.
struct alignas(32) SortedPair {
    uint64_t row_addr;
    int32_t id;
    int32_t pos;        // position of the pair in the input (concatenation order)
    int32_t count;      // pairs of this id
    int32_t row_start;  // sorted position of the id's first pair
    int32_t pad[2];
};
static_assert(sizeof(SortedPair) == 32, "two 16-byte accesses per record");

constexpr int kMaxPart = 2048;     // most ids one sort work-group owns (LDS: 88 KiB of tables and 68 KiB of lists)
constexpr int kMinPart = 128;
constexpr int kColBlock = 256;     // fp32 columns per wavefront item (64 lanes x 4)
constexpr int kMaxSlices = 64;
constexpr int kSliceTokens = 16384;
constexpr int kRangeSliceTokens = 8192;     // slices of a sort that owns few parts of the ids
constexpr int kFusedSortMax = 57344;   // up to here one launch sorts everything (measured against two launches)
constexpr int kPieceSmallMax = 96256;  // up to here pieces of 16 positions, above 32 (bf16 rows read 16 bytes
                                       // per lane: always 16) -- measured: equal up to 25600 pairs, 16 ahead by
                                       // 1-4 % from 51200 to 131072, 32 ahead by 1 % from 200000; the limit is set
                                       // where a call's workspace (more pieces, more shares) still fits the built-in one

// ------------------------------------------------------------------ device helpers
__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

// Lanes of m below this one, plus more.
__device__ __forceinline__ uint32_t lanes_below(uint64_t m, uint32_t more = 0u)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, more));
}

__device__ __forceinline__ uint32_t bcast(uint32_t x, int lane) { return __builtin_amdgcn_readlane(x, lane); }

__device__ __forceinline__ uint64_t bcast64(uint64_t x, int lane)
{
    uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, lane);
    uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Waits until every vector memory operation of the wavefront has completed (vmcnt = 0, the
// other counters left alone).  The builtin, not an asm statement: the compiler takes note of it.
__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Sums across the wavefront with the data-parallel-primitive moves of the vector unit (one
// instruction and a few cycles per step; a shuffle through the LDS crossbar is an LDS instruction with
// its latency, and six of them in a row stand in the sort work-groups' chain).  A wavefront is four
// rows of 16 lanes.  dpp_or_zero: the value of the lane that CTRL names, 0 where there is none or
// where the row is not in ROW_MASK.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xf, true);
}

__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x, int)
{
    x += dpp_or_zero<0x111, 0xf>(x);        // lane - 1 of the row
    x += dpp_or_zero<0x112, 0xf>(x);        // lane - 2
    x += dpp_or_zero<0x114, 0xf>(x);        // lane - 4
    x += dpp_or_zero<0x118, 0xf>(x);        // lane - 8: every row holds its own inclusive scan
    x += dpp_or_zero<0x142, 0xa>(x);        // rows 1 and 3 add the last lane of the row before them
    x += dpp_or_zero<0x143, 0xc>(x);        // rows 2 and 3 add lane 31, the sum of rows 0 and 1
    return x;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x)
{
    return __builtin_amdgcn_readlane(wave_inclusive_scan(x, 0), 63);
}

// Value rows: 4 * NV consecutive columns per lane.  load() brings them as they lie in memory
// (Raw: what stays in registers while the load is in flight), widen() makes fp32 of them.  (The
// address arrives as an integer: say that it is global memory, or the compiler falls back to
// flat loads.)
template <typename RowT, int NV>
struct RowLoad;

template <>
struct RowLoad<float, 1> {
    typedef f4 Raw;
    static __device__ __forceinline__ Raw load(uint64_t row_addr, int col)
    {
        typedef const f4 __attribute__((address_space(1))) * global_f4;
        return __builtin_nontemporal_load(reinterpret_cast<global_f4>(row_addr + (uint64_t)col * 4u));
    }
    static __device__ __forceinline__ void widen(Raw b, f4 (&out)[1]) { out[0] = b; }
};

__device__ __forceinline__ f4 widen_bf16x4(uint32_t lo, uint32_t hi)
{
    f4 r;
    r.x = __uint_as_float(lo << 16);
    r.y = __uint_as_float(lo & 0xFFFF0000u);
    r.z = __uint_as_float(hi << 16);
    r.w = __uint_as_float(hi & 0xFFFF0000u);
    return r;
}

template <>
struct RowLoad<uint16_t, 1> {
    typedef u2 Raw;
    static __device__ __forceinline__ Raw load(uint64_t row_addr, int col)
    {
        typedef const u2 __attribute__((address_space(1))) * global_u2;
        return __builtin_nontemporal_load(reinterpret_cast<global_u2>(row_addr + (uint64_t)col * 2u));
    }
    static __device__ __forceinline__ void widen(Raw b, f4 (&out)[1]) { out[0] = widen_bf16x4(b.x, b.y); }
};

// bf16 rows with d % 8 == 0: one 16-byte load brings eight columns
template <>
struct RowLoad<uint16_t, 2> {
    typedef u4 Raw;
    static __device__ __forceinline__ Raw load(uint64_t row_addr, int col)
    {
        typedef const u4 __attribute__((address_space(1))) * global_u4;
        return __builtin_nontemporal_load(reinterpret_cast<global_u4>(row_addr + (uint64_t)col * 2u));
    }
    static __device__ __forceinline__ void widen(Raw b, f4 (&out)[2])
    {
        out[0] = widen_bf16x4(b.x, b.y);
        out[1] = widen_bf16x4(b.z, b.w);
    }
};


// A partial row that another work-group of the same launch will read: a 16-byte store at
// agent scope, i.e. written through to memory, so that once it has been acknowledged nothing
// of it sits dirty in this work-group's L2 slice.  (The compiler offers that scope for
// 4-byte atomic stores only, and four of those per lane turn every 16-byte store into four
// strided partial writes; hence the instruction is spelled out.)
__device__ __forceinline__ void store_f4_through(float* p, f4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}

// The matching loads: at agent scope, so they are answered from memory and not from a line
// that this L2 slice or this compute unit's cache may still hold from an earlier call.  Eight
// 16-byte loads and the wait for them in ONE statement, so that the compiler never sees a
// loaded register before its data is there.  All eight addresses must be readable.
__device__ __forceinline__ void load8_through(f4 (&x)[8], const float* const (&addr)[8])
{
    asm volatile(
        "global_load_dwordx4 %0, %8, off sc1\n\t"
        "global_load_dwordx4 %1, %9, off sc1\n\t"
        "global_load_dwordx4 %2, %10, off sc1\n\t"
        "global_load_dwordx4 %3, %11, off sc1\n\t"
        "global_load_dwordx4 %4, %12, off sc1\n\t"
        "global_load_dwordx4 %5, %13, off sc1\n\t"
        "global_load_dwordx4 %6, %14, off sc1\n\t"
        "global_load_dwordx4 %7, %15, off sc1\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(x[4]), "=&v"(x[5]), "=&v"(x[6]), "=&v"(x[7])
        : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "v"(addr[4]), "v"(addr[5]), "v"(addr[6]), "v"(addr[7])
        : "memory");
}

// Streaming accesses for data that is touched once per call (value rows, dense_in,
// dense_out): the nontemporal hint keeps them from displacing the sort's arrays and the
// partial rows in the caches, and measures about 8 % faster on a plain [V, d] copy.
__device__ __forceinline__ f4 load_f4_stream(const float* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const f4*>(p));
}
__device__ __forceinline__ void store_f4_stream(float* p, f4 v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<f4*>(p));
}

// What happens to a finished output row on its way to memory.  EPI_NONE: stored as it is
// (untouched rows are bit copies of dense_in).  EPI_SCALE: every element multiplied by one
// fp32 factor (an average over k contributions is scale = 1/k).  EPI_SCALE_BF16: the same,
// then rounded to bf16 (nearest, ties to even), which halves the bytes written.
enum { EPI_NONE = 0, EPI_SCALE = 1, EPI_SCALE_BF16 = 2 };

__device__ __forceinline__ uint32_t bf16_rne(float x)
{
    const uint32_t b = __float_as_uint(x);
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) return (b >> 16) | 0x0040u;      // NaN stays NaN (quiet)
    return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}

// Stores four consecutive output elements starting at element index idx of the output.
template <int EPI>
__device__ __forceinline__ void store_out(void* out, size_t idx, f4 v, float scale)
{
    if (EPI == EPI_NONE) {
        store_f4_stream(reinterpret_cast<float*>(out) + idx, v);
    } else if (EPI == EPI_SCALE) {
        store_f4_stream(reinterpret_cast<float*>(out) + idx, v * scale);
    } else {
        v = v * scale;
        u2 b;
        b.x = bf16_rne(v.x) | (bf16_rne(v.y) << 16);
        b.y = bf16_rne(v.z) | (bf16_rne(v.w) << 16);
        __builtin_nontemporal_store(b, reinterpret_cast<u2*>(reinterpret_cast<uint16_t*>(out) + idx));
    }
}

// A work-group of the sort launches copies the elements [e, e + 2048 * kSortWaves) that lie below e_end, from dense_in to
// the output: the copies beside the sort take whole rows, one behind the other, so where a row ends does not matter
// here.  All loads are issued before the first store.  At every step the work-group's wavefronts move 1 KiB each of one
// stretch of 16 KiB.  Bound by HBM.  us where every wavefront moves 8 KiB of its own / so:
//   192 such work-groups by themselves, 50.3 MB        10.3 /  9.6
//   256 of them, 67.1 MB                               12.6 / 11.9
//   calls: V = 32768, d = 512, 8192 pairs              28.4 / 27.7      (without a dense operand level)
//          V = 32768, d = 1024, 16384 pairs            58.4 / 57.7
// The loads are conditional: the same loads for every lane with the index clamped take 1.3 us more at d = 1024 (they
// disturb the sort beside them).
constexpr int kBlindElems = 2048;
constexpr int kSortWaves = 16;     // wavefronts per sort work-group

template <int EPI>
__device__ __forceinline__ void copy_flat(const float* dense_in, void* dense_out, int64_t e, int64_t e_end, int w, int lane,
                                          float scale)
{
    constexpr int U = kBlindElems / kColBlock;
    if (e >= e_end) return;
    const int rest = (int)min(e_end - e, (int64_t)kBlindElems * kSortWaves);
    f4 x[U];
    if (dense_in) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = (u * kSortWaves + w) * kColBlock + lane * 4;
            x[u] = (f4)(0.0f);
            if (i < rest) x[u] = load_f4_stream(dense_in + e + i);
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = (f4)(0.0f);
    }
    // With an epilogue every value is transformed before the first store is issued: a
    // multiply placed between two stores makes the compiler wait for the earlier store
    // (the empty asm statements keep it from moving the arithmetic down to the stores).
    u2 packed[U];
    if constexpr (EPI != EPI_NONE) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            x[u] = x[u] * scale;
            if constexpr (EPI == EPI_SCALE_BF16) {
                packed[u].x = bf16_rne(x[u].x) | (bf16_rne(x[u].y) << 16);
                packed[u].y = bf16_rne(x[u].z) | (bf16_rne(x[u].w) << 16);
                asm volatile("" : "+v"(packed[u]));
            } else {
                asm volatile("" : "+v"(x[u]));
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = (u * kSortWaves + w) * kColBlock + lane * 4;
        if (i < rest) {
            if constexpr (EPI == EPI_SCALE_BF16)
                __builtin_nontemporal_store(packed[u], reinterpret_cast<u2*>(reinterpret_cast<uint16_t*>(dense_out) + e + i));
            else
                store_f4_stream(reinterpret_cast<float*>(dense_out) + e + i, x[u]);
        }
    }
}

// One wavefront copies columns [c0, c0 + 1024) of dense row v (the reduce kernel's copy of a row
// that received no pair).  A lane past the row's last column reads the row's last four columns
// again and stores nothing: no load depends on the lane, so the four loads stay back to back.
template <int EPI>
__device__ __forceinline__ void copy_chunk(const float* dense_in, void* dense_out, int v, int c0, int d, int lane,
                                           float scale)
{
    f4 x[4];
    if (dense_in) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            x[u] = load_f4_stream(dense_in + (size_t)v * d + min(c0 + u * kColBlock + lane * 4, d - 4));
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = (f4)(0.0f);
    }
    // every value is transformed before the first store is issued, as in copy_flat
    u2 packed[4];
    if constexpr (EPI != EPI_NONE) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            x[u] = x[u] * scale;
            if constexpr (EPI == EPI_SCALE_BF16) {
                packed[u].x = bf16_rne(x[u].x) | (bf16_rne(x[u].y) << 16);
                packed[u].y = bf16_rne(x[u].z) | (bf16_rne(x[u].w) << 16);
                asm volatile("" : "+v"(packed[u]));
            } else {
                asm volatile("" : "+v"(x[u]));
            }
        }
    }
    // One wait for all loads: the stores sit in blocks of their own (not every lane stores), and the
    // compiler would wait at each of them for everything before it, the store before it included.
    // (In the copies beside the sort, copy_flat, that chain of stores is left as it is: there it
    // measured 0.7-1 us faster per launch, the sort's own loads wait less behind gentler copies.)
    wait_vm_all();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int col = c0 + u * kColBlock + lane * 4;
        if (col < d) {
            const size_t idx = (size_t)v * d + col;
            if constexpr (EPI == EPI_SCALE_BF16)
                __builtin_nontemporal_store(packed[u], reinterpret_cast<u2*>(reinterpret_cast<uint16_t*>(dense_out) + idx));
            else
                store_f4_stream(reinterpret_cast<float*>(dense_out) + idx, x[u]);
        }
    }
}

// Narrow rows: one wavefront takes the R = 1024 / d (at most 64) rows from v0 on, which lie one behind
// the other, and copies those that received no pair.  The lane's four elements at u * 256 + 4 * lane
// belong to row elem * row_magic >> 20 (row_magic = ceil(2^20 / d): exact for elements below 1024 and d
// below 1028).  One row per wavefront moves 4 d bytes for a chain of two latencies and leaves lanes
// idle below 256 columns: V = 100000, 8000 pairs 46.9 -> 40.1 us at d = 256, 29.8 -> 20.3 at d = 64; V = 130000,
// d = 256, 100000 pairs 113.3 -> 102.4.  A lane without anything to copy reads the first untouched row again.
template <int EPI>
__device__ __forceinline__ void copy_narrow(const int32_t* count, const float* dense_in, void* dense_out, int v0,
                                            int rows, uint32_t row_magic, int d, int lane, float scale)
{
    const bool untouched = lane < rows && count[v0 + min(lane, rows - 1)] == 0;
    const uint64_t todo = ballot64(untouched);
    if (!todo) return;
    const size_t base = (size_t)v0 * d;
    const int first = (int)__builtin_ctzll(todo) * d, end = rows * d;
    f4 x[4];
    int at[4];
    bool go[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = u * kColBlock + lane * 4;
        const uint32_t r = ((uint32_t)i * row_magic) >> 20;
        go[u] = i < end && ((todo >> (r & 63u)) & 1ull);
        at[u] = go[u] ? i : first;
    }
    if (dense_in) {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = load_f4_stream(dense_in + base + at[u]);
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = (f4)(0.0f);
    }
    wait_vm_all();          // one wait for all loads, as in copy_chunk
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (go[u]) store_out<EPI>(dense_out, base + at[u], x[u], scale);
}

// ------------------------------------------------------------------ shard table
struct ShardTable {
    int32_t k;
    int32_t off[TS_MAX_SHARDS + 1];          // first global pair index of each shard
    const int32_t* ids[TS_MAX_SHARDS];
    const char* rows[TS_MAX_SHARDS];
};

// A wavefront's view of the shard table: lane j holds where shard j begins and its two arrays, moved back
// by that much, so that pair idx has its id at ids + 4 idx and its value row at rows + idx row_bytes.  One
// load per array for all shards (a walk over the table, entry by entry, is a chain of scalar loads).  Pairs
// [a, b) of the wavefront lie in shards j0 .. j1, mostly one and the same.
struct ShardView {
    int32_t off_l;
    uint64_t ids_l, rows_l;
    int32_t j0, j1;
    uint64_t ids0, rows0;       // of shard j0
};

__device__ __forceinline__ ShardView view_shards(const ShardTable& sh, int a, int b, int row_bytes, int lane)
{
    ShardView v;
    v.off_l = 0;
    v.j0 = v.j1 = 0;
    v.ids_l = v.ids0 = (uint64_t)(uintptr_t)sh.ids[0];
    v.rows_l = v.rows0 = (uint64_t)(uintptr_t)sh.rows[0];
    if (sh.k > 1) {
        const int j = min(lane, sh.k - 1);
        v.off_l = sh.off[j];
        v.ids_l = (uint64_t)(uintptr_t)sh.ids[j] - (uint64_t)(uint32_t)v.off_l * 4u;
        v.rows_l = (uint64_t)(uintptr_t)sh.rows[j] - (uint64_t)(uint32_t)v.off_l * (uint64_t)(uint32_t)row_bytes;
        // the last shard that begins at or before a, and the last one that begins before b
        v.j0 = (int)__popcll(ballot64(lane < sh.k && v.off_l <= a)) - 1;
        v.j1 = max((int)__popcll(ballot64(lane < sh.k && v.off_l < b)) - 1, v.j0);
        v.ids0 = bcast64(v.ids_l, v.j0);
        v.rows0 = bcast64(v.rows_l, v.j0);
    }
    return v;
}

// The array (ids_l or rows_l) of the shard that pair idx lies in, where the wavefront's pairs lie in several.
__device__ __forceinline__ uint64_t shard_base(const ShardView& v, uint64_t base0, uint64_t base_l, int idx)
{
    uint64_t base = base0;
    for (int j = v.j0 + 1; j <= v.j1; ++j) {
        const uint64_t next = bcast64(base_l, j);
        if (idx >= (int)bcast((uint32_t)v.off_l, j)) base = next;
    }
    return base;
}

__device__ __forceinline__ int32_t load_id(uint64_t base, int idx)
{
    typedef const int32_t __attribute__((address_space(1))) * global_i32;
    return *reinterpret_cast<global_i32>(base + (uint64_t)(uint32_t)idx * 4u);
}

// ------------------------------------------------------------------ sort
struct SortParams {
    int32_t n, V, G, S, SL;
    // The rows of the call are ids id_base .. id_base + V - 1 of a vocabulary of V_total ids
    // (the whole vocabulary: id_base = 0, V_total = V).  Ids of the vocabulary outside the
    // call's range belong to another owner: skipped, but not counted as bad.
    int32_t id_base, V_total;
    int32_t part;       // ids owned by one work-group (power of two)
    int32_t list_cap;   // entries in a wavefront's list of owned pairs
    uint32_t list_full; // a list with more entries may not hold another 4 tiles' pairs
    int32_t row_bytes;
    int32_t* count;
    int32_t* row_start;
    SortedPair* sorted;
    uint32_t* tot;      // [S][G * part]   pairs per (slice, id), 16 bits each (WIDE: 32)
    uint32_t* below;    // [S][G]          pairs of the slice with a valid id below the part
    uint32_t* bad;      // [S]             pairs of the slice with an id outside [0, V)
    int32_t* n_valid;
    int32_t* n_bad;
    int32_t* arrive;    // arrival counters of the reduce kernel, cleared here (arrive_vec 16-byte words)
    int32_t arrive_vec;
    // Work-groups past the sorting ones copy the elements [copy_e0, copy_e1) (whole rows) to the output
    // without knowing yet which rows receive pairs (the reduce kernel, which runs after,
    // overwrites those).  It keeps HBM busy while the latency-bound sort runs.
    const float* copy_in;
    void* copy_out;
    int64_t copy_e0, copy_e1;
    float scale;
};

enum { SORT_FUSED = 0, SORT_SCATTER = 2 };

// Wavefront w of copying work-group cw of a sort launch.
template <int EPI>
__device__ __forceinline__ void blind_copy(const SortParams& p, int cw, int w, int lane)
{
    const int64_t e = p.copy_e0 + (int64_t)cw * (kSortWaves * kBlindElems);
    copy_flat<EPI>(p.copy_in, p.copy_out, e, p.copy_e1, w, lane, p.scale);
}

// One wavefront walks its sub-slice [a, b) in rounds of kRoundTiles tiles of 64 pairs.  All ids of a round are
// loaded before any is used, so a round costs one memory latency.
constexpr int kRoundTiles = 16;
constexpr int kRoundPairs = kRoundTiles * 64;

__device__ __forceinline__ void load_round(const ShardView& v, int a0, int b, int lane, int32_t (&idr)[kRoundTiles])
{
    // lanes past the end re-read the last pair, so that every load is unconditional and all of them are
    // in flight together; such lanes are masked where ids are used
    if (v.j0 == v.j1) {
#pragma unroll
        for (int u = 0; u < kRoundTiles; ++u) idr[u] = load_id(v.ids0, min(a0 + u * 64 + lane, b - 1));
    } else {
#pragma unroll
        for (int u = 0; u < kRoundTiles; ++u) {
            const int idx = min(a0 + u * 64 + lane, b - 1);
            idr[u] = load_id(shard_base(v, v.ids0, v.ids_l, idx), idx);
        }
    }
}

// Which of the pairs that it looks at a work-group counts besides the ones it owns: those with id - off
// below `below` (unsigned).  Part 0, below which there is no id, counts the ids inside the vocabulary
// (what is left are the bad ones); every other part the ids of the call that lie below the part.
struct Tally {
    uint32_t off, below;
};

__device__ __forceinline__ Tally tally_of(int g, int lo, int id_base, int V_total)
{
    Tally t;
    t.off = g == 0 ? 0u : (uint32_t)id_base;
    t.below = g == 0 ? (uint32_t)V_total : (uint32_t)lo;
    return t;
}

// No id: below no tally's limit and in no part (ids are below 2^31).
constexpr int32_t kNoId = -1;

// Lanes past the sub-slice's end hold no id.
__device__ __forceinline__ void mask_tail(int32_t (&idr)[kRoundTiles], int a0, int b, int lane)
{
    if (a0 + kRoundPairs > b) {
#pragma unroll
        for (int u = 0; u < kRoundTiles; ++u) idr[u] = a0 + u * 64 + lane < b ? idr[u] : kNoId;
    }
}

// Appends the pairs of a round that this work-group owns to the wavefront's list, in input order
// (tiles in order, lanes in order).  An entry is (id - lo) << 21 | position of the pair in the
// wavefront's sub-slice (ids per part <= 2^11, pairs per sub-slice <= 2^21).  Every work-group looks at every
// pair of its slice but owns few of them: counting and ranking walk the short list.  first = id_base + lo.
// A wavefront issues one instruction at a time whatever its kind, and 16 of them share a compute unit here,
// so the pass is bound by its instruction count; the tally is kept per lane (a compare and an add-with-carry;
// a ballot, a population count and a scalar add cost more) and added up over the wavefront at the end.
constexpr int kLdsBytes = 160 * 1024;       // LDS of a compute unit, the most a work-group can have
constexpr int kListPosBits = 21;
constexpr int kGroupTiles = 4;              // tiles that are listed between two looks at how full the list is (room)

// (SPARSE: most tiles hold no owned pair)
template <bool TALLY, bool SPARSE>
__device__ __forceinline__ void list_tile(int32_t id, uint32_t pos, uint32_t first, uint32_t span, const Tally& t, uint32_t* list,
                                          uint32_t& nown, uint32_t& tally)
{
    const uint32_t idg = (uint32_t)id;
    const uint32_t rel = idg - first;
    const bool own = rel < span;
    const uint64_t m = ballot64(own);
    if (TALLY) tally += idg - t.off < t.below ? 1u : 0u;
    if (!SPARSE || m) {
        if (own) list[lanes_below(m, nown)] = (rel << kListPosBits) | pos;
        nown += (uint32_t)__popcll(m);
    }
}

template <bool TALLY, typename Room>
__device__ __forceinline__ void list_round(const int32_t (&idr)[kRoundTiles], int a0, int b, uint32_t pos0, int lane, uint32_t first,
                                           uint32_t span, const Tally& t, uint32_t* list, uint32_t& nown, uint32_t& tally, Room&& room)
{
    const uint32_t pos_l = pos0 + (uint32_t)lane;
#pragma unroll
    for (int v = 0; v < kRoundTiles; v += kGroupTiles) {
        if (a0 + v * 64 < b) {
            room();
#pragma unroll
            for (int u = v; u < v + kGroupTiles; ++u)
                list_tile<TALLY, true>(idr[u], pos_l + (uint32_t)(u * 64), first, span, t, list, nown, tally);
        }
    }
}

// The sort is bound by its chain of latencies and, in the listing and in the work-groups that own the hottest ids, by its
// instructions.  So the shard table is looked up by lanes, the tables hold 16 bits, the lists a whole round, a round's ids
// are loaded while the one before is listed, one tally is kept instead of two, and only ids that really meet in 64 list
// entries are ranked in a loop.  us of the launch (counting + scattering) before all of these / with them:
//   16384 pairs, d = 1024, in place                     9.5        /  8.2
//   51200 pairs, 95 MB of copies beside                22.3        / 20.0
//   80011 pairs in 8 shards of several lengths  10.1 + 14.0        /  7.0 + 10.6
//   131072 pairs                                 7.1 + 12.3        /  5.4 +  9.9
//   262144 pairs, 38 % on one id                 8.5 + 22.8        /  7.6 + 17.5
//
// The tables of pairs per (wavefront, id) in LDS.  Two ids share a word as long as the pairs of a slice fit
// 16 bits: half the LDS to clear and to scan, and a work-group of 2048 ids has room for lists that hold a
// whole round.  Larger slices (calls of more than 4 million pairs): a word per id (WIDE).
constexpr int kNarrowSlice = 65536 - 1024;

template <bool WIDE>
__device__ __forceinline__ uint32_t tab_word(uint32_t rel) { return WIDE ? rel : rel >> 1; }
template <bool WIDE>
__device__ __forceinline__ uint32_t tab_shift(uint32_t rel) { return WIDE ? 0u : (rel & 1u) << 4; }
template <bool WIDE>
__device__ __forceinline__ uint32_t tab_get(uint32_t word, uint32_t shift) { return WIDE ? word : (word >> shift) & 0xFFFFu; }

// Adds the pairs of a tile (or of 64 list entries; a lane without one holds no id of the part) to a table.
// The pairs of the first lane's id are counted by that lane alone: a hot id would otherwise be one LDS
// atomic per pair, all on one address.
template <bool WIDE>
__device__ __forceinline__ void count_ids(uint32_t* tab, uint32_t rel, int ll, int lane)
{
    const uint32_t rl = bcast(rel, ll);
    const uint64_t sm = ballot64(rel == rl);
    if (lane == ll) atomicAdd(&tab[tab_word<WIDE>(rl)], (uint32_t)__popcll(sm) << tab_shift<WIDE>(rl));
    if (rel != rl && rel != 0xFFFFFFFFu) atomicAdd(&tab[tab_word<WIDE>(rel)], 1u << tab_shift<WIDE>(rel));
}

template <bool WIDE>
__device__ __forceinline__ void count_listed(uint32_t* tab, const uint32_t* list, uint32_t nown, int lane)
{
    for (uint32_t e0 = 0; e0 < nown; e0 += 64)
        count_ids<WIDE>(tab, e0 + lane < nown ? list[e0 + lane] >> kListPosBits : 0xFFFFFFFFu, 0, lane);
}

// The numbers that 64 list entries take from a table of their wavefront (what the table holds for an id is the number of
// its next pair; a lane without an entry passes rel of an id of the part and own = false).  The entries of the first one's id
// take theirs together (a hot id would be 64 LDS atomics on one address, one after the other: of 51200 pairs, 14 % on
// one id, its work-group ended 2 us later), the others with one LDS atomic each.  Entries of one id take theirs in no order
// that could be relied on, so what the table holds afterwards is read back: an id is among the 64 several times if and
// only if one of its entries finds more there than its own number and one.  The entries of such ids, and only those, are
// numbered again, by lane.
template <bool WIDE>
__device__ __forceinline__ uint32_t number_entries(uint32_t* tab, uint32_t rel, bool own, int lane)
{
    uint32_t* const word = tab + tab_word<WIDE>(rel);
    const uint32_t shift = tab_shift<WIDE>(rel);
    const uint32_t relx = own ? rel : 0xFFFFFFFFu;
    const uint32_t rel0 = bcast(relx, 0);
    const uint64_t sm0 = ballot64(relx == rel0);
    // (no short circuits: they become branches, which cost a call with a dominating id half a per cent)
    const bool first = lane == 0;
    const bool takes = first | (own & (rel != rel0));
    const uint32_t add = first ? (uint32_t)__popcll(sm0) : 1u;
    uint32_t number = 0, after = 1;
    if (takes) {
        number = tab_get<WIDE>(__hip_atomic_fetch_add(word, add << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP), shift);
        // every lane's addition comes before any lane's look (no instruction: LDS operations of a wavefront are carried
        // out in order, this keeps the compiler from another one)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        after = tab_get<WIDE>(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP), shift);
    }
    const uint32_t number0 = bcast(number, 0);
    uint64_t m = ballot64(after != number + 1u) & ~sm0;
    if (relx == rel0) number = number0 + lanes_below(sm0);
    while (m) {
        const uint32_t rl = bcast(rel, (int)__builtin_ctzll(m));
        const uint64_t sm = ballot64(relx == rl);
        if (relx == rl) number = after - (uint32_t)__popcll(sm) + lanes_below(sm);
        m &= ~sm;
    }
    return number;
}

// Every pair of a wavefront's list takes the next position of its id: put(position, address of the value row, id within the part,
// index of the pair, the id's count and first position).  The list keeps the pairs in input order and wavefronts own consecutive
// sub-slices (this one's begins at pair a), so the sort is stable.  id_pos: where the slice's pairs of an id begin (SLICES).
template <bool WIDE, bool SLICES, typename Put>
__device__ __forceinline__ void rank_listed(uint32_t* tab, const uint32_t* list, uint32_t nown, const u2* id_info, const uint32_t* id_pos,
                                            const ShardView& v, int a, int row_bytes, int lane, Put&& put)
{
    for (uint32_t e0 = 0; e0 < nown; e0 += 64) {
        const bool own = e0 + lane < nown;
        const uint32_t ent = own ? list[e0 + lane] : 0u;
        const uint32_t rel = ent >> kListPosBits;       // (a lane without an entry looks where id 0 of the part stands)
        const int idx = a + (int)(ent & ((1u << kListPosBits) - 1u));
        const u2 info = id_info[rel];
        const uint32_t pos = SLICES ? id_pos[rel] : info.y;
        const uint32_t number = number_entries<WIDE>(tab, rel, own, lane);
        const uint64_t rows = v.j0 == v.j1 ? v.rows0 : shard_base(v, v.rows0, v.rows_l, idx);
        if (own) put(pos + number, rows + (uint64_t)(uint32_t)idx * (uint64_t)(uint32_t)row_bytes, rel, idx, info);
    }
}

__device__ __forceinline__ void write_record(SortedPair* at, uint64_t row_addr, uint32_t id, int idx, u2 info)
{
    u4* const rec = reinterpret_cast<u4*>(at);
    u4 r0, r1;
    r0.x = (uint32_t)row_addr;
    r0.y = (uint32_t)(row_addr >> 32);
    r0.z = id;
    r0.w = (uint32_t)idx;
    r1.x = info.x;
    r1.y = info.y;
    r1.z = 0u;
    r1.w = 0u;
    rec[0] = r0;
    rec[1] = r1;
}

// The counting launch of a sort that takes several slices: work-group (g, s) counts the pairs of
// slice s per id of part g (p.tot: 16 bits each, WIDE 32), those with a valid id below the part (p.below) and
// those with an id outside the vocabulary (p.bad).  One LDS table for the whole work-group: the order
// of the pairs does not matter here.  It also clears the arrival counters of the reduce kernel,
// and the work-groups past the counting ones copy dense rows like those of sort_kernel.
template <bool WIDE, int EPI>
__global__ __launch_bounds__(1024) void count_kernel(SortParams p, ShardTable sh)
{
    extern __shared__ __align__(16) uint32_t tab[];     // [part] counts
    __shared__ uint32_t red[kSortWaves];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nsort = p.G * p.S;
    // what the sort's chain begins with, asked for in one go with the sizes above (else one more latency behind them)
    asm volatile("" ::"s"(p.n), "s"(p.V), "s"(p.SL), "s"(p.id_base), "s"(p.part), "s"(sh.k), "s"(sh.ids[0]), "s"(sh.rows[0]));
    if ((int)blockIdx.x >= nsort) {
        blind_copy<EPI>(p, (int)blockIdx.x - nsort, w, lane);
        return;
    }
    const int g = (int)blockIdx.x % p.G;
    const int sl = (int)blockIdx.x / p.G;
    const int part = p.part;
    const int lo = g * part;
    const uint32_t span = (uint32_t)min(part, p.V - lo);
    const uint32_t first = (uint32_t)p.id_base + (uint32_t)lo;
    const Tally t = tally_of(g, lo, p.id_base, p.V_total);

    const int t0 = sl * p.SL;
    const int t1 = (int)min((int64_t)p.n, (int64_t)t0 + p.SL);
    const int L = p.SL / kSortWaves;
    const int a = (int)min((int64_t)t1, (int64_t)t0 + (int64_t)w * L);
    const int b = (int)min((int64_t)t1, (int64_t)a + L);
    const int rounds = (b - a + kRoundPairs - 1) / kRoundPairs;
    const ShardView v = view_shards(sh, a, b, 0, lane);

    int32_t idr[kRoundTiles];
    if (rounds > 0) load_round(v, a, b, lane, idr);
    {
        u4* const z = reinterpret_cast<u4*>(p.arrive);
        for (int i = (int)blockIdx.x * 1024 + tid; i < p.arrive_vec; i += nsort * 1024) z[i] = (u4)(0u);
    }
    const int words = WIDE ? part : part / 2;
    for (int i = tid; i < words; i += 1024) tab[i] = 0u;
    __syncthreads();

    uint32_t tally = 0;
    for (int r = 0; r < rounds; ++r) {
        const int a0 = a + r * kRoundPairs;
        if (r > 0) load_round(v, a0, b, lane, idr);
        mask_tail(idr, a0, b, lane);
#pragma unroll
        for (int u = 0; u < kRoundTiles; ++u) {
            const uint32_t idg = (uint32_t)idr[u];
            const uint32_t rel = idg - first;
            const uint64_t m = ballot64(rel < span);
            tally += idg - t.off < t.below ? 1u : 0u;
            // many owned pairs in a tile: a hot id among them, most likely
            if (__popcll(m) > 12) {
                count_ids<WIDE>(tab, rel < span ? rel : 0xFFFFFFFFu, (int)__builtin_ctzll(m), lane);
            } else if (rel < span) {
                atomicAdd(&tab[tab_word<WIDE>(rel)], 1u << tab_shift<WIDE>(rel));
            }
        }
    }
    tally = wave_sum(tally);
    if (lane == 0) red[w] = tally;
    __syncthreads();
    const size_t GW = (size_t)p.G * words;
    for (int i = tid; i < words; i += 1024) p.tot[(size_t)sl * GW + (size_t)g * words + i] = tab[i];
    if (w == 0) {
        const uint32_t all = wave_sum(lane < kSortWaves ? red[lane] : 0u);
        if (lane == 0) {
            p.below[sl * p.G + g] = g == 0 ? 0u : all;
            if (g == 0) p.bad[sl] = (uint32_t)(t1 - t0) - all;
        }
    }
}

// DEEP (a one-launch sort of more than one round): the ids of a round are loaded while the round before it is
// listed.
template <int MODE, bool WIDE, bool DEEP, int EPI>
__global__ __launch_bounds__(1024) void sort_kernel(SortParams p, ShardTable sh)
{
    // [kSortWaves][words] counts, then per-id totals, starts and (with several slices) first positions of
    // the slice's pairs, then [kSortWaves][list_cap] lists of owned pairs
    extern __shared__ __align__(16) uint32_t cnt[];
    __shared__ uint32_t red[2 * kSortWaves];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nsort = p.G * p.S;
    // what the sort's chain begins with, asked for in one go with the sizes above (else one more latency behind them)
    asm volatile("" ::"s"(p.n), "s"(p.V), "s"(p.SL), "s"(p.id_base), "s"(p.part), "s"(sh.k), "s"(sh.ids[0]), "s"(sh.rows[0]));
    if ((int)blockIdx.x >= nsort) {
        blind_copy<EPI>(p, (int)blockIdx.x - nsort, w, lane);
        return;
    }
    constexpr int E = WIDE ? 1 : 2;         // ids per word of a table
    const int g = (int)blockIdx.x % p.G;
    const int sl = (int)blockIdx.x / p.G;
    const int part = p.part;
    const int words = part / E;
    const int lo = g * part;
    const uint32_t span = (uint32_t)min(part, p.V - lo);
    const uint32_t first = (uint32_t)p.id_base + (uint32_t)lo;
    uint32_t* const mycnt = cnt + w * words;
    u2* const id_info = reinterpret_cast<u2*>(cnt + kSortWaves * words);       // pairs of the id, its first sorted position
    uint32_t* const id_pos = reinterpret_cast<uint32_t*>(id_info + part);      // several slices: where this slice's begin
    uint32_t* const list = id_pos + (MODE == SORT_SCATTER ? part : 0) + w * p.list_cap;

    const int t0 = sl * p.SL;
    const int t1 = (int)min((int64_t)p.n, (int64_t)t0 + p.SL);
    const int L = p.SL / kSortWaves;
    const int a = (int)min((int64_t)t1, (int64_t)t0 + (int64_t)w * L);
    const int b = (int)min((int64_t)t1, (int64_t)a + L);
    const int rounds = (b - a + kRoundPairs - 1) / kRoundPairs;
    const ShardView v = view_shards(sh, a, b, p.row_bytes, lane);

    int32_t idr[kRoundTiles];
    if (rounds > 0) load_round(v, a, b, lane, idr);

    if (MODE == SORT_FUSED) {
        // the first launch of a call clears the arrival counters of the reduce kernel
        u4* const z = reinterpret_cast<u4*>(p.arrive);
        for (int i = (int)blockIdx.x * 1024 + tid; i < p.arrive_vec; i += nsort * 1024) z[i] = (u4)(0u);
    }

    uint32_t base = 0, nbad = 0;            // first sorted position of the part; bad ids
    // Everything the counting launch has left, asked for here and looked at behind the listing, so that the latency runs
    // beside it.  Per slice (lane s2 speaks for slice s2, at most 64 slices): the pairs below the part and the bad ids.  Per
    // id: its count in all slices and in the slices before this one, the first sixteen here; none beyond the last slice.
    // us of the call looked at here / behind the listing / that, with the loads beyond the last slice:
    //   V = 131072, d = 64, 200000 pairs                     72.7 / 67.9 / 69.5
    //   V = 32768, d = 64, 60000 pairs                       27.8 / 27.3 / 28.0
    //   80011 pairs in eight shards, averaged to bf16        80.8 / 80.2 / 80.6
    const size_t GW = (size_t)p.G * words;
    uint32_t bl = 0, bd = 0, tot[16];
    if (MODE == SORT_SCATTER) {
        bl = p.below[min(lane, p.S - 1) * p.G + g];
        bd = p.bad[min(lane, p.S - 1)];
#pragma unroll
        for (int q = 0; q < 16; ++q) tot[q] = q < p.S ? p.tot[(size_t)q * GW + (size_t)g * words + min(tid, words - 1)] : 0u;
    }
    // every wavefront clears its own table of counts, so none has to wait for the others before it
    // starts to list and count (the tables meet at the barrier before the scan)
    {
        u4* const c4 = reinterpret_cast<u4*>(mycnt);
        for (int i = lane; i < words / 4; i += 64) c4[i] = (u4)(0u);
    }

    // pass 1: list the owned pairs, count them per (wavefront, id); tally the others.  A list that might not
    // hold another four tiles' pairs (list_full: more entries than that; never, if it holds the whole sub-slice)
    // is counted and started again, and the sub-slice walked again for the ranking.
    const Tally t = tally_of(g, lo, p.id_base, p.V_total);
    uint32_t tally = 0, nown = 0;
    bool flushed = false;
    auto pass1 = [&](int32_t (&ids)[kRoundTiles], int rd) {
        const int a0 = a + rd * kRoundPairs;
        mask_tail(ids, a0, b, lane);
        list_round<MODE == SORT_FUSED>(ids, a0, b, (uint32_t)(rd * kRoundPairs), lane, first, span, t, list, nown, tally, [&] {
            if (nown > p.list_full) {
                count_listed<WIDE>(mycnt, list, nown, lane);
                nown = 0;
                flushed = true;
            }
        });
    };
    if constexpr (DEEP) {
        // every load is unconditional (beyond the last round it reads the last pair again): a load that may or may
        // not have been issued would be waited for with the ids of the round at hand
        int32_t other[kRoundTiles];
        for (int rd = 0; rd < rounds; rd += 2) {
            load_round(v, a + (rd + 1) * kRoundPairs, b, lane, other);
            pass1(idr, rd);
            load_round(v, a + (rd + 2) * kRoundPairs, b, lane, idr);
            if (rd + 1 < rounds) pass1(other, rd + 1);
        }
    } else {
        for (int rd = 0; rd < rounds; ++rd) {
            if (rd > 0) load_round(v, a + rd * kRoundPairs, b, lane, idr);
            pass1(idr, rd);
        }
    }
    count_listed<WIDE>(mycnt, list, nown, lane);
    if (MODE == SORT_SCATTER) {
        if (tid < words) {
            uint32_t total[E], pre[E];
#pragma unroll
            for (int e = 0; e < E; ++e) total[e] = pre[e] = 0u;
            for (int sb = 0; sb < p.S; sb += 16) {
                if (sb > 0) {
#pragma unroll
                    for (int q = 0; q < 16; ++q) tot[q] = sb + q < p.S ? p.tot[(size_t)(sb + q) * GW + (size_t)g * words + tid] : 0u;
                }
#pragma unroll
                for (int q = 0; q < 16; ++q)
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const uint32_t c = tab_get<WIDE>(tot[q], 16u * e);
                        total[e] += c;
                        if (sb + q < sl) pre[e] += c;
                    }
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                id_info[tid * E + e].x = total[e];
                id_pos[tid * E + e] = pre[e];
            }
        }
        base = wave_sum(lane < p.S ? bl : 0u);
        nbad = wave_sum(lane < p.S ? bd : 0u);
    }
    if (MODE == SORT_FUSED) {
        tally = wave_sum(tally);
        if (lane == 0) red[w] = tally;
    }
    __syncthreads();
    if (MODE == SORT_FUSED) {
        // the wavefronts' tallies, one per lane, added up across the wavefront
        const uint32_t all = wave_sum(lane < kSortWaves ? red[lane] : 0u);
        base = g == 0 ? 0u : all;
        nbad = (uint32_t)p.n - all;
    }
    if (sl == 0 && g == 0 && tid == 0) *p.n_bad = (int32_t)nbad;

    // The ids of the part in one sweep: thread tid speaks for the ids of word tid.  Totals over the
    // wavefronts (and slices), exclusive scan into first positions, and per wavefront the pairs of the id that
    // earlier wavefronts hold, packed as the counts are.  Each id's count and first position are kept where the
    // ranking pass reads them.
    {
        typedef uint32_t vec __attribute__((ext_vector_type(E)));
        const int i = tid * E;
        const bool idt = tid < words;
        uint32_t c[kSortWaves];
        vec total = (vec)(0u), pre = (vec)(0u);
        if (idt) {
            uint32_t sum = 0;
#pragma unroll
            for (int ww = 0; ww < kSortWaves; ++ww) {
                c[ww] = cnt[ww * words + tid];
                sum += c[ww];
            }
            if (MODE == SORT_SCATTER) {
                // over all slices, fetched at the start of the kernel
#pragma unroll
                for (int e = 0; e < E; ++e) total[e] = id_info[i + e].x;
                pre = *reinterpret_cast<const vec*>(id_pos + i);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) total[e] = tab_get<WIDE>(sum, 16u * e);
            }
        }
        uint32_t mine = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) mine += total[e];
        const uint32_t incl = wave_inclusive_scan(mine, lane);
        if (lane == 63) red[kSortWaves + w] = incl;
        __syncthreads();
        // what the wavefronts before this one hold: their sums, one per lane, added up
        const uint32_t woff = wave_sum(lane < w ? red[kSortWaves + lane] : 0u);
        uint32_t rs = base + woff + incl - mine;        // first sorted position of this thread's first id
        if (idt) {
            vec start;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                start[e] = rs;
                if (sl == 0 && (uint32_t)(i + e) < span) {
                    p.count[lo + i + e] = (int32_t)total[e];
                    p.row_start[lo + i + e] = (int32_t)rs;
                    if (lo + i + e == p.V - 1) {
                        p.row_start[p.V] = (int32_t)(rs + total[e]);
                        *p.n_valid = (int32_t)(rs + total[e]);
                    }
                }
                rs += total[e];
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                u2 info;
                info.x = total[e];
                info.y = start[e];
                id_info[i + e] = info;
            }
            if (MODE == SORT_SCATTER) *reinterpret_cast<vec*>(id_pos + i) = start + pre;
            uint32_t o = 0;
#pragma unroll
            for (int ww = 0; ww < kSortWaves; ++ww) {
                cnt[ww * words + tid] = o;
                o += c[ww];
            }
        }
        __syncthreads();
    }

    // pass 2
    const auto rank = [&] {
        rank_listed<WIDE, MODE == SORT_SCATTER>(mycnt, list, nown, id_info, id_pos, v, a, p.row_bytes, lane,
                                                [&](uint32_t pos, uint64_t row_addr, uint32_t rel, int idx, u2 info) {
            write_record(p.sorted + pos, row_addr, (uint32_t)lo + rel, idx, info);
        });
    };
    if (!flushed) {
        rank();
        return;
    }
    // the list did not hold all owned pairs: the sub-slice once more, round by round
    for (int rd = 0; rd < rounds; ++rd) {
        const int a0 = a + rd * kRoundPairs;
        load_round(v, a0, b, lane, idr);
        mask_tail(idr, a0, b, lane);
        nown = 0;
        list_round<false>(idr, a0, b, (uint32_t)(rd * kRoundPairs), lane, first, span, t, list, nown, tally, [] {});
        rank();
    }
}

// ------------------------------------------------------------------ reduce
struct ReduceParams {
    // the first 64 bytes: all that a wavefront which copies a row needs
    int32_t V, d, C, ncb;
    int32_t n_piece_groups;     // work-groups that sum pieces: (groups of pieces) x column blocks
    int32_t row0;               // the work-groups after them take the rows from here on, one per wavefront
    int32_t short_max;          // rows with at most this many pairs are added up row by row (0 or C)
    int32_t copy_row0;          // untouched rows below this one have been copied by the sort launches
    const int32_t* count;
    const float* dense_in;
    void* dense_out;
    float scale;
    int32_t copy_untouched;     // 0: rows without pairs are left as they are (in place, no epilogue)
    int32_t row_chunks;         // a wavefront of those work-groups takes 1024 columns of a row: chunks per row;
                                // negative: it takes -row_chunks narrow rows, and only copies
    // the rest
    const int32_t* row_start;
    const SortedPair* sorted;
    const int32_t* n_valid;
    int32_t n;                  // pairs in the call (records beyond n_valid hold nothing)
    int32_t nslots;             // 2 * groups
    float* partial;             // [2 * groups][d]: slot 2g holds group g's share of a row that began before it,
                                // slot 2g + 1 its share of a row that begins in it and goes on beyond it
    int32_t* arrive;            // [levels][2 * groups][ncb] arrival counters, all zero when the launch starts
    int32_t logC, logG;         // log2 C; log2 of the sorted positions of a group of pieces
    uint32_t row_magic;         // ceil(2^20 / d), where row_chunks < 0
    int32_t part_owned;         // the call owns a range of the ids: most groups of pieces may be empty
};

// Pieces per work-group of the reduce kernel, one per wavefront: 64 sorted positions with pieces of 8
// or 16, 128 with pieces of 32.
constexpr __host__ __device__ int group_pieces(int C) { return C <= 8 ? 8 : 4; }

// Fixed-order combine of a row that spans several work-groups, inside the launch that made
// the shares (a share: what one work-group's pieces hold of the row, already added up in
// piece order).  The shares of a row form a tree with a fan-in of 16: share j of a level belongs
// to group j / 16, and a group's sum is itself share j / 16 of the next level, until one
// group holds the whole row.  Every wavefront that has stored a share counts itself in at
// the share's group; the one that finds all the others there adds the group's shares in a
// fixed order (a batch at a time as a balanced tree, the batches in order), stores the sum
// in the slot of the group's first share and moves up a level; at the top dense_in is
// added and the output row is written.  Which wavefront does the adding depends on timing,
// what it adds and in which order does not.
//
// Ordering without a release fence (which writes the whole L2 back and costs more than the
// rest of the kernel) and without an acquire fence (which empties this L2 slice for
// everybody): shares are stored through to memory (store_f4_through); a wavefront counts
// itself in only after those stores have been acknowledged; the wavefront that sees the
// full count reads the shares from memory (load8_through), past its caches.
constexpr int kFanIn = 16;
constexpr int kLogFanIn = 4;

// A share this wavefront has stored: that of group k (of pieces) of the cut row `id`, whose
// c pairs start at sorted position s.
struct CutRef {
    int32_t k, id, s, c;
};

// k0: the group in which the row begins.
__device__ __forceinline__ size_t share_slot(int k0, int group_in_row)
{
    return group_in_row == 0 ? (size_t)(2 * k0 + 1) : (size_t)2 * (size_t)(k0 + group_in_row);
}

__device__ __forceinline__ int32_t* arrival_counter(const ReduceParams& p, int level, size_t first_slot, int cb)
{
    return p.arrive + ((size_t)level * p.nslots + first_slot) * p.ncb + cb;
}

// Counts a level-0 share in.  The caller has made sure that the share's stores are
// acknowledged.  Returns (in lane 0) how many shares of the group had arrived before.
__device__ __forceinline__ int announce_share(const ReduceParams& p, const CutRef& r, int cb, int lane)
{
    const int k0 = r.s >> p.logG;
    const int g = (r.k - k0) >> kLogFanIn;
    int arrived = 0;
    if (lane == 0)
        arrived = __hip_atomic_fetch_add(arrival_counter(p, 0, share_slot(k0, g << kLogFanIn), cb), 1, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    return arrived;
}

// arrived0: what announce_share returned for this share.  If the share was its group's
// last, adds the group up and climbs the tree for as long as it is the last to arrive.
template <int NV, int EPI>
__device__ __forceinline__ void combine_if_last(const ReduceParams& p, const CutRef& r, int cb, int col, bool colok,
                                                int lane, int arrived0)
{
    constexpr int kBatch = 8 / NV;                  // shares loaded together: eight 16-byte loads
    const int k0 = r.s >> p.logG;                                     // the row's first group of pieces
    int Pl = ((r.s + r.c - 1) >> p.logG) - k0 + 1;                    // shares at this level (groups at level 0)
    int j = r.k - k0;                                                 // this wavefront's share
    int shift = 0;                                                    // a share of this level spans 16^level groups
    int arrived = __builtin_amdgcn_readfirstlane(arrived0);
    for (int level = 0;; ++level) {
        const int g = j >> kLogFanIn;
        const int m = min(kFanIn, Pl - (g << kLogFanIn));             // shares in this group
        const size_t first_slot = share_slot(k0, (g << kLogFanIn) << shift);
        const bool top = Pl <= kFanIn;
        if (level > 0) {
            // the group sum stored below has to be in memory before it is counted in
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            int x = 0;
            if (lane == 0)
                x = __hip_atomic_fetch_add(arrival_counter(p, level, first_slot, cb), 1, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
            arrived = __builtin_amdgcn_readfirstlane(x);
        }
        if (arrived != m - 1) return;
        f4 dn[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            dn[q] = (f4)(0.0f);
            if (top && colok && p.dense_in) dn[q] = load_f4_stream(p.dense_in + (size_t)r.id * p.d + col + 4 * q);
        }
        f4 tot[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) tot[q] = (f4)(0.0f);
        // lanes past the row's last column read column 0 and drop it; shares past the group's
        // last read the last one again and drop it: every load is to an address that exists
        const int safe_col = colok ? col : 0;
        for (int i0 = 0; i0 < m; i0 += kBatch) {
            f4 x[8];                    // share u of the batch, vector q: x[u * NV + q]
            const float* addr[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int i = min(i0 + t / NV, m - 1);
                addr[t] = p.partial + share_slot(k0, ((g << kLogFanIn) + i) << shift) * p.d + safe_col + 4 * (t % NV);
            }
            load8_through(x, addr);
#pragma unroll
            for (int t = 0; t < 8; ++t) x[t] = (i0 + t / NV < m && colok) ? x[t] : (f4)(0.0f);
#pragma unroll
            for (int w = 1; w < kBatch; w <<= 1)
#pragma unroll
                for (int u = 0; u + w < kBatch; u += 2 * w)
#pragma unroll
                    for (int q = 0; q < NV; ++q) x[u * NV + q] += x[(u + w) * NV + q];
#pragma unroll
            for (int q = 0; q < NV; ++q) tot[q] += x[q];
        }
        if (top) {
            if (colok) {
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    if constexpr (EPI == EPI_NONE)
                        store_f4_stream(reinterpret_cast<float*>(p.dense_out) + (size_t)r.id * p.d + col + 4 * q,
                                        tot[q] + dn[q]);
                    else
                        store_out<EPI>(p.dense_out, (size_t)r.id * p.d + col + 4 * q, tot[q] + dn[q], p.scale);
                }
            }
            return;
        }
        if (colok) {
#pragma unroll
            for (int q = 0; q < NV; ++q) store_f4_through(p.partial + first_slot * p.d + col + 4 * q, tot[q]);
        }
        j = g;
        Pl = (Pl + kFanIn - 1) >> kLogFanIn;
        shift += kLogFanIn;
    }
}

// Columns [c0, c0 + 1024) of one output row v, by one wavefront, when rows with at most short_max
// (> 0) pairs are added up row by row.  A row that received no pair is copied from dense_in, unless
// that has been done or is not wanted; of a row that received at most short_max pairs, the
// value rows are added up in sorted order and dense_in last.  (Longer rows belong to the
// pieces.)  dense_in is asked for before the row's count is known whenever it will most
// likely be needed: all but the few long rows need it then.
template <typename RowT, int EPI>
__device__ __forceinline__ void short_row(const ReduceParams& p, int v, int c0, int lane)
{
    const bool copy = p.copy_untouched && v >= p.copy_row0;    // what to do if the row received no pair
    const bool early = copy;                                   // then only a long row makes the early load useless
    constexpr int RB = sizeof(RowT) == 4 ? 4 : 8;      // value rows in flight together (16 KiB; 8 KiB measured 2 % slower
                                                       // where short rows have up to 32 pairs)
    typedef typename RowLoad<RowT, 1>::Raw Raw;
    const int d = p.d;
    f4 dn[4];
    // a lane past the row's last column reads the last four columns again (and stores nothing), so
    // that no load depends on the lane
    auto load_dense = [&](int c0) {
        if (p.dense_in) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                dn[u] = load_f4_stream(p.dense_in + (size_t)v * d + min(c0 + u * kColBlock + lane * 4, d - 4));
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) dn[u] = (f4)(0.0f);
        }
    };
    if (early) load_dense(c0);
    const int c = p.count[v];
    if (c > p.short_max || (c == 0 && !copy)) return;
    uint64_t addr = 0;
    if (lane < c) addr = p.sorted[p.row_start[v] + lane].row_addr;
    if (!early) load_dense(c0);
    if (c > 0) {
        f4 acc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[u] = (f4)(0.0f);
        for (int j0 = 0; j0 < c; j0 += RB) {
            Raw raw[RB][4];
#pragma unroll
            for (int t = 0; t < RB; ++t) {
                const uint64_t ra = bcast64(addr, min(j0 + t, c - 1));
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int col = min(c0 + u * kColBlock + lane * 4, d - 4);
                    raw[t][u] = Raw{};
                    if (j0 + t < c) raw[t][u] = RowLoad<RowT, 1>::load(ra, col);
                }
            }
#pragma unroll
            for (int t = 0; t < RB; ++t) {
                if (j0 + t < c) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        f4 r[1];
                        RowLoad<RowT, 1>::widen(raw[t][u], r);
                        acc[u] = acc[u] + r[0];
                    }
                }
            }
        }
        // dense_in has been in flight all along; the output row takes its place
#pragma unroll
        for (int u = 0; u < 4; ++u) dn[u] = acc[u] + dn[u];
    }
    // one wait for all that is still on its way, then the stores back to back
    wait_vm_all();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int col = c0 + u * kColBlock + lane * 4;
        if (col < d) store_out<EPI>(p.dense_out, (size_t)v * d + col, dn[u], p.scale);
    }
}

// Where short rows are added up row by row, the long rows are added up by wavefronts that
// work alone: one wavefront takes a whole group of pieces (64 sorted positions)
// and one block of columns, walks the pieces one after the other and keeps in registers
// what the work-group form keeps in LDS.  The sums are the same, in the same order: a piece's
// pairs in sorted order, the pieces of the group in order; a row that lies inside the group is
// finished there, of any other the group's sum becomes a share.  No barrier, no LDS, and a
// wavefront that has to wait for its share to be acknowledged, or to combine shares, holds up
// nobody but itself.  For groups of at most 64 sorted positions (C <= 16): one per lane.
template <typename RowT, int NV, int EPI>
__device__ __forceinline__ void group_wave(const ReduceParams& p, int kg, int cb, int lane)
{
    typedef typename RowLoad<RowT, NV>::Raw Raw;
    constexpr int BATCH = 16;                   // value rows in flight together
    constexpr int NW = 1;                       // windows of 64 sorted positions
    const int C = p.C;
    const int G = 1 << p.logG;                   // sorted positions of the group (at most 64)
    const int gpos0 = kg << p.logG;
    const int col = (cb * kColBlock + lane * 4) * NV;
    const bool colok = col < p.d;
    const bool have_dense = p.dense_in != nullptr;

    // lane j of window w looks at sorted position gpos0 + 64 w + j; records are read before
    // n_valid is known, what lies at or beyond it is ignored
    u4 r0[NW], r1[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int jr = w * 64 + lane;
        r0[w] = (u4)(0u);
        r1[w] = (u4)(0u);
        if (jr < G && gpos0 + jr < p.n) {
            const u4* rec = reinterpret_cast<const u4*>(p.sorted + gpos0 + jr);
            r0[w] = rec[0];
            r1[w] = rec[1];
        }
    }
    const int nvalid = *p.n_valid;
    int32_t id[NW], c[NW], s[NW];
    uint64_t addr[NW];
    uint64_t L[NW], RS[NW], RE[NW];             // positions of long rows; where such a row starts; where it ends
    uint64_t INSIDE[NW];                        // positions of rows that start inside the group
    bool any = false;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int jr = w * 64 + lane;
        const int wpos = gpos0 + jr;
        const bool inwin = jr < G && wpos < p.n && wpos < nvalid;
        id[w] = inwin ? (int32_t)r0[w].z : -1;
        c[w] = inwin ? (int32_t)r1[w].x : 0;
        s[w] = inwin ? (int32_t)r1[w].y : 0;
        addr[w] = inwin ? (((uint64_t)r0[w].y << 32) | r0[w].x) : 0ull;
        const bool lng = inwin && c[w] > C;
        L[w] = ballot64(lng);
        RS[w] = ballot64(lng && wpos == s[w]);
        RE[w] = ballot64(lng && wpos == s[w] + c[w] - 1);
        INSIDE[w] = ballot64(lng && s[w] >= gpos0);
        any = any || L[w] != 0;
    }
    if (!any) return;
    const uint64_t PS = ballot64((lane & (C - 1)) == 0);            // first and last position of a piece
    const uint64_t PE = ballot64((lane & (C - 1)) == C - 1);        // (C divides 64)

    f4 acc[NV], tot[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q] = tot[q] = (f4)(0.0f);
    bool segfirst = true;       // the piece at hand is the first of its row within the group
    CutRef ref[2];
    ref[0].k = ref[1].k = -1;
    int nref = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        uint64_t rem = L[w];
        while (rem) {
            // the next BATCH positions of long rows: all loads are issued before the first is used
            int jj[BATCH];
            Raw raw[BATCH];
            f4 dn[2][NV];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < NV; ++q) dn[t][q] = (f4)(0.0f);
            static_assert(BATCH == 16, "two slots, one per 8 positions");
            // dense_in of a row that is finished here: one slot and one load instruction per half of
            // the batch, issued behind the half's value rows.  A long row has more than 8 pairs, so
            // no two of them end within 8 positions of long rows.  (Several conditional loads into
            // one slot, or a slot chosen at run time, make the compiler load into a spare register
            // and move the value afterwards, with a wait for it and for all loads before it.)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint64_t half = 0;
#pragma unroll
                for (int uu = 0; uu < 8; ++uu) {
                    const int u = 8 * h + uu;
                    jj[u] = -1;
                    raw[u] = Raw{};
                    if (rem) {
                        const int j = (int)__builtin_ctzll(rem);
                        rem &= rem - 1ull;
                        half |= 1ull << j;
                        jj[u] = j;
                        if (colok) raw[u] = RowLoad<RowT, NV>::load(bcast64(addr[w], j), col);
                    }
                }
                const uint64_t ends = half & RE[w] & INSIDE[w];
                if (have_dense && ends && colok) {
                    const int vj = (int)bcast((uint32_t)id[w], (int)__builtin_ctzll(ends));
#pragma unroll
                    for (int q = 0; q < NV; ++q) dn[h][q] = load_f4_stream(p.dense_in + (size_t)vj * p.d + col + 4 * q);
                }
            }
            // one wait for the whole batch: the compiler waits for all of it at the first use anyway, and
            // would then wait again at every later position, which after a row's store means for that store
            wait_vm_all();
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int j = jj[u];
                if (j >= 0) {
                    const bool rs = (RS[w] >> j) & 1ull, re = (RE[w] >> j) & 1ull;
                    const bool ps = (PS >> j) & 1ull, pe = (PE >> j) & 1ull;
                    const bool fresh = rs || ps;
                    if (fresh) segfirst = rs || (w == 0 && j == 0);
                    f4 r[NV];
                    RowLoad<RowT, NV>::widen(raw[u], r);
#pragma unroll
                    for (int q = 0; q < NV; ++q) acc[q] = (fresh ? (f4)(0.0f) : acc[q]) + r[q];
                    if (re || pe) {
                        // the row's pairs in this piece are in: the pieces of the group in order
#pragma unroll
                        for (int q = 0; q < NV; ++q) tot[q] = segfirst ? acc[q] : tot[q] + acc[q];
                        segfirst = false;
                        const bool gend = w * 64 + j == G - 1;
                        if (re || gend) {
                            const int sj = (int)bcast((uint32_t)s[w], j);
                            const int cj = (int)bcast((uint32_t)c[w], j);
                            const int idj = (int)bcast((uint32_t)id[w], j);
                            if (re && sj >= gpos0) {
                                // the row lies inside the group
                                f4 dj[NV];
#pragma unroll
                                for (int q = 0; q < NV; ++q) dj[q] = have_dense ? dn[u >> 3][q] : (f4)(0.0f);
                                if (colok) {
#pragma unroll
                                    for (int q = 0; q < NV; ++q)
                                        store_out<EPI>(p.dense_out, (size_t)idj * p.d + col + 4 * q, tot[q] + dj[q], p.scale);
                                }
                            } else {
                                // the group's share of a row that began before it or goes on beyond it
                                const int kg0 = sj >> p.logG;
                                const size_t slot = share_slot(kg0, kg - kg0);
                                if (colok) {
#pragma unroll
                                    for (int q = 0; q < NV; ++q) store_f4_through(p.partial + slot * p.d + col + 4 * q, tot[q]);
                                }
                                CutRef x;
                                x.k = kg;
                                x.id = idj;
                                x.s = sj;
                                x.c = cj;
                                if (nref == 0) ref[0] = x; else ref[1] = x;
                                ++nref;
                            }
                        }
                    }
                }
            }
        }
    }
    if (nref == 0) return;
    // shares are counted in once their stores are acknowledged; whoever brings the last share
    // of a group of shares adds the group up
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int answer[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) answer[t] = ref[t].k >= 0 ? announce_share(p, ref[t], cb, lane) : 0;
#pragma unroll
    for (int t = 0; t < 2; ++t)
        if (ref[t].k >= 0) combine_if_last<NV, EPI>(p, ref[t], cb, col, colok, lane, answer[t]);
}

// NV: 16-byte fp32 vectors per lane (a wavefront of a piece covers 256 * NV columns); BATCH:
// sorted positions whose rows are loaded together.
//
// Output rows with more than C pairs are added up by pieces.  A work-group takes GP
// consecutive pieces of C sorted positions, one per wavefront, and one block of columns.  A
// wavefront adds up the pairs of such a row that lie in its piece and leaves the sum in LDS.
// After one barrier the wavefront that holds a row's last piece within the work-group adds
// the work-group's pieces of that row in piece order; if the row lies inside the work-group it
// is finished there and then, otherwise the sum goes to scratch as the work-group's share of
// the row, and the shares are combined as described above.
//
// Output rows with at most C pairs, SHORT = 0: the wavefront in whose piece such a row
// starts adds it up completely (its window is two pieces long for that) and writes
// dense_in + sum; the work-groups after those of the pieces copy the rows without pairs, one
// per wavefront.  SHORT = 1 or 2: those work-groups take every row that is not long, one per
// wavefront (short_row), and the pieces pass over the positions of short rows; with
// SHORT = 1 (pieces of at most 16 positions) the long rows go to wavefronts that work alone
// (group_wave) instead of the work-groups described here.  The order of additions, and so
// every bit of the result, is the same in all three.
template <typename RowT, int NV, int BATCH, int EPI, int SHORT, int GP>
__global__ __launch_bounds__(64 * GP) void reduce_kernel(ReduceParams p)
{
    // SHORT: 0 short rows in the pieces; 1 row by row, long rows by lone wavefronts (group_wave);
    // 2 row by row, long rows by the work-groups below
    // [wavefront][0: of a row that began before the piece, 1: of a row that begins in it][vector][lane]
    __shared__ f4 chain[SHORT == 1 ? 1 : GP][2][NV][64];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    if ((int)blockIdx.x >= p.n_piece_groups) {
        // one wavefront per row and chunk of 1024 columns (wider rows: several wavefronts, so that
        // no wavefront has to work through its row chunk after chunk)
        const int item = ((int)blockIdx.x - p.n_piece_groups) * GP + wave;
        if constexpr (!SHORT) {
            if (p.row_chunks < 0) {
                const int v0 = p.row0 - item * p.row_chunks;
                if (v0 < p.V)
                    copy_narrow<EPI>(p.count, p.dense_in, p.dense_out, v0, min(-p.row_chunks, p.V - v0), p.row_magic, p.d,
                                     lane, p.scale);
                return;
            }
        }
        int v = p.row0 + item, c0 = 0;
        if (p.row_chunks > 1) {
            const int r = item / p.row_chunks;
            v = p.row0 + r;
            c0 = (item - r * p.row_chunks) * 4 * kColBlock;
        }
        if constexpr (!SHORT) {
            // the pieces add up every row that received pairs: copy the row if it received none
            if (v < p.V && p.count[v] == 0) copy_chunk<EPI>(p.dense_in, p.dense_out, v, c0, p.d, lane, p.scale);
        } else {
            if (v < p.V) short_row<RowT, EPI>(p, v, c0, lane);
        }
        return;
    }

    if constexpr (SHORT == 1) {
        // Four wavefronts, four consecutive groups of pieces, one block of columns.  Work-groups b, b + 8,
        // b + 16, ... run on the same XCD (one of eight, each with an L2 of its own): the column blocks of
        // one quadruple of groups go to work-groups of one XCD, which then reads the quadruple's records
        // from memory once.  Quadruples beyond a multiple of eight keep the plain order.  (Measured: 0.6-1.2 %
        // of the call at 50-130 thousand pairs; the same mapping for the work-group form of the pieces
        // changed nothing or cost 0.5 %, and giving an XCD 16 consecutive rows in the row work-groups
        // cost 1.5-4 us: consecutive rows are better spread over the XCDs, as they are.)
        const int b = (int)blockIdx.x;
        const int nq = p.n_piece_groups / p.ncb;
        int kq, cb;
        if (b < (nq & ~7) * p.ncb) {
            const int i = b >> 3;
            const int q = i / p.ncb;
            cb = i - q * p.ncb;
            kq = q * 8 + (b & 7);
        } else {
            kq = b / p.ncb;
            cb = b - kq * p.ncb;
        }
        const int kg = kq * 4 + wave;
        if (p.part_owned && (kg << p.logG) >= *p.n_valid) return;
        if (kg < p.nslots / 2) group_wave<RowT, NV, EPI>(p, kg, cb, lane);
        return;
    }

    // ---- piece k: sorted positions [pos0, pos0 + C), columns [cb*256*NV, (cb+1)*256*NV)
    const int kg = (int)blockIdx.x / p.ncb;
    // a range's groups beyond its pairs, most of them: out before the records are asked for (one eighth of
    // 32768 ids, 131072 pairs: 41.3 -> 39.1 us; where all pairs are owned the question would be one latency more)
    if (p.part_owned && (kg << p.logG) >= *p.n_valid) return;
    const int cb = (int)blockIdx.x - kg * p.ncb;
    const int k = kg * GP + wave;
    const int col = (cb * kColBlock + lane * 4) * NV;
    const bool colok = col < p.d;
    const int C = p.C;
    const int pos0 = k * C;

    // lane j looks at sorted position pos0 + j; the window is two pieces long because
    // an output row with at most C pairs that starts in this piece is finished here (unless
    // such rows are added up row by row: then the piece itself is all there is to look at).  The records are read before n_valid is known (one
    // memory latency instead of two); what lies at or beyond n_valid is ignored.
    const int wpos = pos0 + lane;
    const bool inarr = lane < (SHORT ? C : 2 * C) && wpos < p.n;
    u4 r0 = (u4)(0u), r1 = (u4)(0u);
    if (inarr) {
        const u4* rec = reinterpret_cast<const u4*>(p.sorted + wpos);
        r0 = rec[0];
        r1 = rec[1];
    }
    const int nvalid = *p.n_valid;
    const bool inwin = inarr && wpos < nvalid;
    const int32_t id = inwin ? (int32_t)r0.z : -1;
    const int32_t c = inwin ? (int32_t)r1.x : 0;
    const int32_t s = inwin ? (int32_t)r1.y : 0;
    const uint64_t addr = inwin ? (((uint64_t)r0.y << 32) | r0.x) : 0ull;
    const bool whole = c <= C;       // output row small enough to be summed by one wavefront
    const bool active = inwin && (whole ? (!SHORT && s >= pos0 && s < pos0 + C) : (lane < C));
    const bool first = active && (wpos == s || (!whole && lane == 0));
    const bool last = active && (wpos == s + c - 1 || (!whole && lane == C - 1));
    const uint64_t A = ballot64(active);
    const uint64_t F = ballot64(first);
    const uint64_t Lm = ballot64(last);
    const uint64_t W = ballot64(whole);
    const uint64_t H = ballot64(s >= pos0);      // the row of this position begins in this piece
    const bool have_dense = p.dense_in != nullptr;

    if (A != 0) {
        typedef typename RowLoad<RowT, NV>::Raw Raw;
        f4 acc[NV];
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q] = (f4)(0.0f);
        // The active positions are consecutive, or (when short rows are added up elsewhere) lie in
        // two runs: the end of one long row and the beginning of another.
        uint64_t rem = A;
        while (rem) {
            const int a = (int)__builtin_ctzll(rem);
            int b = 64 - __builtin_clzll(rem);
            if constexpr (SHORT) {
                const uint64_t gap = ~(rem >> a);
                b = a + (gap ? (int)__builtin_ctzll(gap) : 64 - a);
            }
            rem &= b < 64 ? ~0ull << b : 0ull;
            for (int base = a; base < b; base += BATCH) {
                // all loads of a batch are issued before the first is used
                Raw raw[BATCH];
                f4 dn[BATCH][NV];
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int j = base + u;
                    raw[u] = Raw{};
#pragma unroll
                    for (int q = 0; q < NV; ++q) dn[u][q] = (f4)(0.0f);
                    if (j < b) {
                        if (colok) raw[u] = RowLoad<RowT, NV>::load(bcast64(addr, j), col);
                        if (have_dense && (((Lm & W) >> j) & 1ull)) {
                            const int vj = (int)bcast((uint32_t)id, j);
                            if (colok) {
#pragma unroll
                                for (int q = 0; q < NV; ++q)
                                    dn[u][q] = load_f4_stream(p.dense_in + (size_t)vj * p.d + col + 4 * q);
                            }
                        }
                    }
                }
                // (where only long rows are left to the pieces, the compiler's code waits before every
                // position for all memory operations, a finished row's store included: one wait instead)
                if constexpr (SHORT != 0) wait_vm_all();
#pragma unroll
                for (int u = 0; u < BATCH; ++u) {
                    const int j = base + u;
                    if (j < b) {
                        const bool fresh = (F >> j) & 1ull;
                        f4 r[NV];
                        RowLoad<RowT, NV>::widen(raw[u], r);
#pragma unroll
                        for (int q = 0; q < NV; ++q) acc[q] = (fresh ? (f4)(0.0f) : acc[q]) + r[q];
                        if ((Lm >> j) & 1ull) {
                            if ((W >> j) & 1ull) {
                                const int vj = (int)bcast((uint32_t)id, j);
                                if (colok) {
#pragma unroll
                                    for (int q = 0; q < NV; ++q)
                                        store_out<EPI>(p.dense_out, (size_t)vj * p.d + col + 4 * q, acc[q] + dn[u][q], p.scale);
                                }
                            } else {
                                const int portion = (int)((H >> j) & 1ull);
#pragma unroll
                                for (int q = 0; q < NV; ++q) chain[wave][portion][q][lane] = acc[q];
                            }
                        }
                    }
                }
            }
        }
    }
    __syncthreads();

    // The cut rows that pass through this piece (at most two: one that ends in it or covers
    // it, one that begins in it).  The wavefront with the row's last piece inside the
    // work-group adds the work-group's pieces of the row, in piece order.
    uint64_t cuts = Lm & ~W;
    const int g_first = kg * GP, g_last = g_first + GP - 1;
    CutRef ref[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        ref[t].k = -1;
        if (cuts) {
            const int j = __builtin_ctzll(cuts);
            cuts &= cuts - 1;
            const int idj = (int)bcast((uint32_t)id, j);
            const int sj = (int)bcast((uint32_t)s, j);
            const int cj = (int)bcast((uint32_t)c, j);
            const int piece_first = sj >> p.logC, piece_last = (sj + cj - 1) >> p.logC;
            if (k == min(piece_last, g_last)) {
                const bool inside = piece_first >= g_first && piece_last <= g_last;
                f4 dn[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) {
                    dn[q] = (f4)(0.0f);
                    if (inside && have_dense && colok) dn[q] = load_f4_stream(p.dense_in + (size_t)idj * p.d + col + 4 * q);
                }
                const int x0 = max(piece_first, g_first);
                f4 tot[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) tot[q] = chain[x0 - g_first][x0 == piece_first ? 1 : 0][q][lane];
                for (int x = x0 + 1; x <= k; ++x) {
#pragma unroll
                    for (int q = 0; q < NV; ++q) tot[q] += chain[x - g_first][0][q][lane];
                }
                if (inside) {
                    if (colok) {
#pragma unroll
                        for (int q = 0; q < NV; ++q) {
                            if constexpr (EPI == EPI_NONE)
                                store_f4_stream(reinterpret_cast<float*>(p.dense_out) + (size_t)idj * p.d + col + 4 * q,
                                                tot[q] + dn[q]);
                            else
                                store_out<EPI>(p.dense_out, (size_t)idj * p.d + col + 4 * q, tot[q] + dn[q], p.scale);
                        }
                    }
                } else {
                    // the work-group's share of a row that goes beyond it
                    const int kg0 = sj >> p.logG;
                    const size_t slot = share_slot(kg0, kg - kg0);
                    if (colok) {
#pragma unroll
                        for (int q = 0; q < NV; ++q) store_f4_through(p.partial + slot * p.d + col + 4 * q, tot[q]);
                    }
                    ref[t].k = kg;
                    ref[t].id = idj;
                    ref[t].s = sj;
                    ref[t].c = cj;
                }
            }
        }
    }
    if (ref[0].k < 0 && ref[1].k < 0) return;
    // shares are counted in once their stores are acknowledged; whoever brings the last share
    // of a group of shares adds the group up
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int answer[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) answer[t] = ref[t].k >= 0 ? announce_share(p, ref[t], cb, lane) : 0;
#pragma unroll
    for (int t = 0; t < 2; ++t)
        if (ref[t].k >= 0) combine_if_last<NV, EPI>(p, ref[t], cb, col, colok, lane, answer[t]);
}

// ------------------------------------------------------------------ small calls: one launch
// A call with few pairs and a small output is as long as its chain of latencies: two launches of 5 us each with one
// and a half between them.  small_kernel does it in one: V = 1000, d = 64, 2048 pairs with uniform ids 10.1 -> 7.2 us per call (more
// at small_call).  Work-group (g, cb) owns `part` consecutive ids and a block of 4 * lanes columns.  It sorts the pairs of
// its ids as sort_kernel does (all pairs are looked at, its own listed, counted, scanned and ranked; dense_in of its rows is on
// its way meanwhile), keeps the sorted pairs in LDS and adds up its own rows: longer rows by pieces of C sorted positions,
// whose sums, and the shares of groups of pieces, meet in LDS; rows of at most C pairs, and rows without pairs, by the lanes of one
// row.  Same order of additions as in the other kernels, same bits.
// Where ids crowd into one part its longer rows bound the call: a compute unit takes in value rows at 25 to 50 bytes a
// nanosecond.  So a block is as narrow as it takes for every piece to have lanes of its own, with all loads in flight at
// once (small_lanes).  256 columns per block, pieces in up to four turns and their shares added by the lanes of one row / now, all
// pairs on one id: d = 64, 2048 pairs 17.4 / 12.6 us, d = 1024, 512 pairs 20.1 / 9.8.
constexpr int kSmallWaves = kSortWaves;
constexpr int kSmallTiles = 2;              // of 64 pairs per wavefront
constexpr int kSmallMax = kSmallWaves * kSmallTiles * 64;
constexpr int kSmallSums = kSmallWaves * 64 * 2;
constexpr int kSmallRows = 4;               // rows per lane at most
constexpr int kSmallLanes = 16;             // lanes of a row at most
constexpr int kSmallPiece = 8;              // pieces are no shorter
constexpr int kSmallPart = 32;              // ids of a work-group, unless that makes too many of them
constexpr int kSmallPartMax = 1024;         // (two to a thread in the scan, with a wavefront's counts in 2 KiB)
constexpr int kXcds = 8;
static_assert(kSmallWaves * 64 / kSmallLanes >= kSmallMax / 64, "every group of pieces has lanes of its own");
static_assert(kSmallMax / 64 <= kFanIn * kFanIn, "two levels of sums of shares");

// The lanes of a row in small_kernel, four columns each: no more than leave lanes to every piece of n pairs.
int small_lanes(int64_t n, int32_t d)
{
    int lanes = 1;
    while (lanes < kSmallLanes && lanes * 4 < d && 2 * lanes * n <= kSmallWaves * 64 * kSmallPiece) lanes *= 2;
    return lanes;
}

struct SmallParams {
    int32_t n, V, G, stride, id_base, V_total, part, row_bytes, d;
    int32_t C, lanes, rounds, combine_batch;    // lanes of a row; rounds of rows; shares that are added as a balanced tree
    int32_t* count;
    int32_t* row_start;
    SortedPair* sorted;
    int32_t* n_valid;
    int32_t* n_bad;
    const float* dense_in;
    void* dense_out;
    int32_t copy_untouched;
    float scale;
};

// LDS: the counts per (wavefront, id), per id its pairs and first position, per sorted pair the address of its value row
// its id within the part, the lists of owned pairs or the pieces' sums, and the shares of long rows.
constexpr size_t small_lds(int n, int part, int lanes)
{
    return (size_t)kSmallWaves * part * 2 + (size_t)part * 8 + (size_t)((n + 7) / 8 * 8) * 10 + kSmallSums * 16 +
           (size_t)(n / 64 + 2) * 2 * lanes * 16;
}
static_assert(kSmallMax * 4 <= kSmallSums * 16, "the lists fit in the place of the sums");

template <typename RowT, int EPI>
__global__ __launch_bounds__(64 * kSmallWaves) void small_kernel(SmallParams p, ShardTable sh)
{
    extern __shared__ __align__(16) uint32_t lds[];
    __shared__ uint32_t red[2 * kSmallWaves];
    typedef typename RowLoad<RowT, 1>::Raw Raw;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = (int)blockIdx.x % p.stride;
    const int cb = (int)blockIdx.x / p.stride;
    if (g >= p.G) return;
    const int part = p.part;
    const int words = part / 2;
    const int lo = g * part;
    const uint32_t span = (uint32_t)min(part, p.V - lo);
    const uint32_t first = (uint32_t)p.id_base + (uint32_t)lo;
    const int L = ((p.n + kSmallWaves * 64 - 1) / (kSmallWaves * 64)) * 64;
    uint32_t* const mycnt = lds + w * words;
    u2* const id_info = reinterpret_cast<u2*>(lds + kSmallWaves * words);       // pairs of the id, its first sorted position
    uint64_t* const row_addr = reinterpret_cast<uint64_t*>(id_info + part);
    uint16_t* const pair_rel = reinterpret_cast<uint16_t*>(row_addr + (p.n + 7) / 8 * 8);
    // the lists of owned pairs, and later in their place the pieces' sums: [piece][0: of a row that began before it, 1: of
    // a row that begins in it][lane of the row]
    f4* const chain = reinterpret_cast<f4*>(pair_rel + (p.n + 7) / 8 * 8);
    // shares of long rows: two per group of 64 positions, as in the reduce kernel (share_slot, from the part's first group on)
    f4* const share = chain + kSmallSums;
    uint32_t* const list = reinterpret_cast<uint32_t*>(chain) + w * L;

    const int a = min(p.n, w * L), b = min(p.n, a + L);
    const ShardView v = view_shards(sh, a, b, p.row_bytes, lane);
    int32_t idr[kSmallTiles];
    if (a < b) {
#pragma unroll
        for (int u = 0; u < kSmallTiles; ++u) {
            if (u * 64 < L) {
                const int idx = min(a + u * 64 + lane, b - 1);
                idr[u] = load_id(v.j0 == v.j1 ? v.ids0 : shard_base(v, v.ids0, v.ids_l, idx), idx);
            }
        }
    }
    // the lanes of a row; a lane past the row's last column reads the last columns again and stores nothing
    const int sub = lane / p.lanes, sl = lane - sub * p.lanes, per_wave = 64 / p.lanes;
    const int col = (cb * p.lanes + sl) * 4;
    const bool colok = col < p.d;
    const int colr = min(col, p.d - 4);
    f4 dn[kSmallRows];
#pragma unroll
    for (int it = 0; it < kSmallRows; ++it) {
        dn[it] = (f4)(0.0f);
        const int r = (it * kSmallWaves + w) * per_wave + sub;
        if (it < p.rounds && p.dense_in && p.copy_untouched && r < (int)span)
            dn[it] = load_f4_stream(p.dense_in + (size_t)(lo + r) * p.d + colr);
    }
    for (int i = lane; i < words; i += 64) mycnt[i] = 0u;

    const Tally t = tally_of(g, lo, p.id_base, p.V_total);
    uint32_t tally = 0, nown = 0;
#pragma unroll
    for (int u = 0; u < kSmallTiles; ++u) {
        if (a + u * 64 < b)
            list_tile<true, false>(a + u * 64 + lane < b ? idr[u] : kNoId, (uint32_t)(u * 64 + lane), first, span, t, list, nown, tally);
    }
    count_listed<false>(mycnt, list, nown, lane);
    tally = wave_sum(tally);
    if (lane == 0) red[w] = tally;
    __syncthreads();
    const uint32_t all = wave_sum(lane < kSmallWaves ? red[lane] : 0u);
    const uint32_t base = g == 0 ? 0u : all;        // first sorted position of the part
    if (g == 0 && cb == 0 && tid == 0) *p.n_bad = (int32_t)((uint32_t)p.n - all);
    // The scan of sort_kernel for one slice and two ids to a word, what the ranking waits for first (one function for both
    // kernels: V = 1000, d = 64, 2048 pairs 6.60 -> 6.69 us, 80011 pairs averaged to bf16 79.8 -> 80.1).
    {
        const bool idt = tid < words;
        uint32_t c[kSmallWaves], sum = 0;
        if (idt) {
#pragma unroll
            for (int ww = 0; ww < kSmallWaves; ++ww) {
                c[ww] = lds[ww * words + tid];
                sum += c[ww];
            }
        }
        const uint32_t t0 = sum & 0xFFFFu, t1 = sum >> 16;
        const uint32_t incl = wave_inclusive_scan(t0 + t1, lane);
        if (lane == 63) red[kSmallWaves + w] = incl;
        __syncthreads();
        const uint32_t woff = wave_sum(lane < w ? red[kSmallWaves + lane] : 0u);
        const uint32_t s0 = base + woff + incl - t0 - t1, s1 = s0 + t0;
        if (idt) {
            u4 info;
            info.x = t0;
            info.y = s0;
            info.z = t1;
            info.w = s1;
            *reinterpret_cast<u4*>(id_info + 2 * tid) = info;
            uint32_t o = 0;
#pragma unroll
            for (int ww = 0; ww < kSmallWaves; ++ww) {
                lds[ww * words + tid] = o;
                o += c[ww];
            }
            if (cb == 0) {
                const int i = lo + 2 * tid;
                if (2 * tid < (int)span) {
                    p.count[i] = (int32_t)t0;
                    p.row_start[i] = (int32_t)s0;
                    if (i == p.V - 1) {
                        p.row_start[p.V] = (int32_t)s1;
                        *p.n_valid = (int32_t)s1;
                    }
                }
                if (2 * tid + 1 < (int)span) {
                    p.count[i + 1] = (int32_t)t1;
                    p.row_start[i + 1] = (int32_t)s1;
                    if (i + 1 == p.V - 1) {
                        p.row_start[p.V] = (int32_t)(s1 + t1);
                        *p.n_valid = (int32_t)(s1 + t1);
                    }
                }
            }
        }
        __syncthreads();
    }
    rank_listed<false, false>(mycnt, list, nown, id_info, nullptr, v, a, p.row_bytes, lane,
                              [&](uint32_t pos, uint64_t addr, uint32_t rel, int idx, u2 info) {
        row_addr[pos - base] = addr;
        pair_rel[pos - base] = (uint16_t)rel;
        if (cb == 0) write_record(p.sorted + pos, addr, (uint32_t)lo + rel, idx, info);
    });
    __syncthreads();

    const uint32_t off = (uint32_t)colr * (uint32_t)sizeof(RowT);
    const auto load_pair = [&](int lp) {
        typedef const Raw __attribute__((address_space(1))) * global_raw;
        return __builtin_nontemporal_load(reinterpret_cast<global_raw>(row_addr[lp] + off));
    };
    // Longer rows: a piece to the lanes of one row (small_lanes sees to it that there are enough).  A piece holds a part of a
    // long row that began before it, and of one that begins in it.
    const int own_end = (int)(id_info[span - 1].x + id_info[span - 1].y);       // one behind the part's last position
    const int k_first = (int)base >> 6, k_last = own_end > (int)base ? (own_end - 1) >> 6 : k_first - 1;
    const int slot = w * per_wave + sub;
    const int logC = 31 - __builtin_clz((unsigned)p.C), log_pieces = 6 - logC;
    {
        const int q0 = k_first << log_pieces, piece = q0 + slot;        // the part's first piece, and the one at hand
        const int group = piece >> log_pieces, g_first = group << log_pieces, g_last = g_first + (1 << log_pieces) - 1;
        const int begin = max(piece << logC, (int)base), end = min((piece + 1) << logC, own_end);
        // the row that has the piece's first position, and the one that has its last
        int rel[2] = {0, 0}, s[2] = {0, 0}, c[2] = {0, 0};
        f4 d0[2], acc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            d0[t] = acc[t] = (f4)(0.0f);
            if (begin < end) {
                rel[t] = pair_rel[(t == 0 ? begin : end - 1) - (int)base];
                const u2 info = id_info[rel[t]];
                s[t] = (int)info.y;
                c[t] = (int)info.x > p.C && (t == 0 || rel[1] != rel[0]) ? (int)info.x : 0;
            }
            if (c[t] && p.dense_in && s[t] >= group << 6 && (s[t] + c[t] - 1) >> logC == piece)
                d0[t] = load_f4_stream(p.dense_in + (size_t)(lo + rel[t]) * p.d + colr);
        }
        if (c[0] | c[1]) {
            // the first one's positions end before end0, the last one's begin at begin1
            const int end0 = c[0] ? min(end, s[0] + c[0]) : begin, begin1 = c[1] ? max(begin, s[1]) : end;
            for (int at = begin; at < end; at += 8) {
                Raw raw[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    raw[u] = Raw{};
                    if (at + u < end0 || (at + u >= begin1 && at + u < end)) raw[u] = load_pair(at + u - (int)base);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    f4 x[1];
                    RowLoad<RowT, 1>::widen(raw[u], x);
                    if (at + u < end0) acc[0] = acc[0] + x[0];
                    if (at + u >= begin1 && at + u < end) acc[1] = acc[1] + x[0];
                }
            }
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (c[t]) chain[(slot * 2 + (s[t] >= piece << logC ? 1 : 0)) * p.lanes + sl] = acc[t];
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (c[t]) {
                const int piece_first = s[t] >> logC, piece_last = (s[t] + c[t] - 1) >> logC;
                if (piece == min(piece_last, g_last)) {
                    const int x0 = max(piece_first, g_first);
                    f4 tot = chain[((x0 - q0) * 2 + (x0 == piece_first ? 1 : 0)) * p.lanes + sl];
                    for (int x = x0 + 1; x <= piece; ++x) tot = tot + chain[(x - q0) * 2 * p.lanes + sl];
                    if (piece_first >= g_first && piece_last <= g_last) {
                        if (colok) store_out<EPI>(p.dense_out, (size_t)(lo + rel[t]) * p.d + col, tot + d0[t], p.scale);
                    } else {
                        share[(share_slot(s[t] >> 6, group - (s[t] >> 6)) - 2 * k_first) * p.lanes + sl] = tot;
                    }
                }
            }
        }
    }

    // Rows that span several groups: their shares are added as combine_if_last adds them, sixteen at a time, sixteen number q by
    // the lanes of its first share's group (the first one by those of the second share's: the group in which a row begins
    // belongs to others, too).  What these lanes need is asked for here, behind the loads of the short rows.
    int j = 0, Pl = 0, slot0 = 0, crel = 0;
    f4 cd = (f4)(0.0f);
    {
        const int k = k_first + 1 + slot;
        if (k <= k_last) {
            crel = pair_rel[(k << 6) - (int)base];
            const u2 info = id_info[crel];
            const int k0 = (int)info.y >> 6;
            if ((int)info.x > p.C && k0 < k) {
                j = k - k0;
                Pl = ((int)(info.y + info.x - 1) >> 6) - k0 + 1;
                slot0 = 2 * (k0 - k_first);
                if (j == 1 && p.dense_in) cd = load_f4_stream(p.dense_in + (size_t)(lo + crel) * p.d + colr);
            }
        }
    }

    // rows without pairs and of at most C pairs
#pragma unroll
    for (int it = 0; it < kSmallRows; ++it) {
        const int r = (it * kSmallWaves + w) * per_wave + sub;
        if (it < p.rounds && r < (int)span) {
            const u2 info = id_info[r];
            const int c = (int)info.x, lp = (int)(info.y - base);
            if (c <= p.C && (c > 0 || p.copy_untouched)) {
                f4 out[1] = {dn[it]};
                if (c > 0) {
                    if (!p.copy_untouched && p.dense_in) dn[it] = load_f4_stream(p.dense_in + (size_t)(lo + r) * p.d + colr);
                    f4 acc[1] = {(f4)(0.0f)};
                    for (int j0 = 0; j0 < c; j0 += 8) {
                        Raw raw[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            raw[u] = Raw{};
                            if (j0 + u < c) raw[u] = load_pair(lp + j0 + u);
                        }
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            f4 x[1];
                            RowLoad<RowT, 1>::widen(raw[u], x);
                            if (j0 + u < c) acc[0] = acc[0] + x[0];
                        }
                    }
                    out[0] = acc[0] + dn[it];
                }
                if (colok) store_out<EPI>(p.dense_out, (size_t)(lo + r) * p.d + col, out[0], p.scale);
            }
        }
    }

    if (k_first >= k_last) return;          // (the same for the whole work-group)
    __syncthreads();
    const auto add_shares = [&](int from, int shift, int m) {
        f4 tot = (f4)(0.0f);
        for (int i0 = 0; i0 < m; i0 += 8) {
            f4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int at = (from + min(i0 + u, m - 1)) << shift;
                x[u] = share[(at == 0 ? slot0 + 1 : slot0 + 2 * at) * p.lanes + sl];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = i0 + u < m ? x[u] : (f4)(0.0f);
            const f4 h0 = (x[0] + x[1]) + (x[2] + x[3]), h1 = (x[4] + x[5]) + (x[6] + x[7]);
            tot = p.combine_batch > 4 ? tot + (h0 + h1) : (tot + h0) + h1;
        }
        return tot;
    };
    const int from = j == 1 ? 0 : j;
    const bool adds = j == 1 || (j > 0 && j % kFanIn == 0);
    f4 tot = (f4)(0.0f);
    if (adds) tot = add_shares(from, 0, min(kFanIn, Pl - from));
    if (k_last - k_first >= kFanIn) {       // (the same for the whole work-group)
        if (adds) share[(from == 0 ? slot0 + 1 : slot0 + 2 * from) * p.lanes + sl] = tot;
        __syncthreads();
        if (j == 1 && Pl > kFanIn) tot = add_shares(0, kLogFanIn, (Pl + kFanIn - 1) / kFanIn);
    }
    if (j == 1 && colok) store_out<EPI>(p.dense_out, (size_t)(lo + crel) * p.d + col, tot + cd, p.scale);
}

// ------------------------------------------------------------------ unique ids (introspection)
__global__ __launch_bounds__(1024) void unique_kernel(const int32_t* count, int V, int32_t* out,
                                                      int32_t* n_out)
{
    __shared__ uint32_t wsum[kSortWaves];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = tid >> 6;
    uint32_t base = 0;
    for (int v0 = 0; v0 < V; v0 += 1024) {
        const int v = v0 + tid;
        const bool flag = v < V && count[v] > 0;
        const uint64_t m = ballot64(flag);
        if (lane == 0) wsum[w] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t woff = 0, tot = 0;
        for (int ww = 0; ww < kSortWaves; ++ww) {
            if (ww < w) woff += wsum[ww];
            tot += wsum[ww];
        }
        if (flag) out[base + woff + lanes_below(m)] = v;
        base += tot;
        __syncthreads();
    }
    if (tid == 0) *n_out = (int32_t)base;
}

// ------------------------------------------------------------------ host side
struct Plan {
    bool wide_tab;              // tables of the sort: a word per id
    uint32_t list_full;
    size_t sort_lds;
    int32_t S, SL, G, part, list_cap, C, NB, NBG, levels, ncb;   // NB pieces in NBG groups; levels of the combine tree; 256-column blocks of a row
    size_t off_nvalid, off_nbad, off_arrive, arrive_bytes, off_count, off_row_start, off_sorted, off_tot,
        off_below, off_bad, off_partial, total;
};

int g_piece_override = 0;
int32_t g_short_rows = -1;       // -1: choose; 0: the pieces take the short rows along; 1: row by row
int64_t g_overlap_sort = -1;            // dense bytes (read + write) copied beside each sort launch; -1 = default
int32_t g_part_override = 0;
void* g_ws = nullptr;
int64_t g_ws_bytes = 0;
Plan g_last_plan;
void* g_last_ws = nullptr;              // the workspace the most recent call used (bound, or the built-in one)
int32_t g_last_V = 0;
int32_t g_last_info[8] = {0, 0, 0, 0, 0, 0, 0, 0};
bool g_have_last = false;

constexpr int kMaxProfile = 4096;
hipEvent_t g_ev[2 * kMaxProfile];
int g_ev_made = 0;
int g_prof_cap = 0;
int g_prof_used = 0;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Calls with at least this many pairs add up their short rows row by row, the others in the pieces.
// Row by row a wavefront has one output row's few value rows in flight, all columns of them, after
// three loads that depend on each other; in the pieces it has up to sixteen pairs of 256 (bf16: eight of 512)
// columns in flight (half as many when the limits below were measured), and every block of columns repeats the bookkeeping.  So the wider the rows and
// the more pairs, the better the first does.  Measured on V = 8192 .. 131072, Zipf ids: narrower than
// 256 columns it never pays (half-empty wavefronts), at 256 from about 400 thousand pairs (2 %), at 512
// from 65 to 100 thousand, at 1024 from 25 thousand (bf16 rows, 6-13 % by 50 thousand) or 40-50
// thousand (fp32 rows, 0.5-5 %), and from there on the limit halves when the width doubles (d = 4096:
// 8 to 16 thousand; 3-10 % beyond); below those it loses up to 30 % on narrow rows and small V.
// A dense operand of half a gigabyte or more (V = 131072 at d = 1024): row by row at any number of pairs
// (2-5 % measured from 8192 pairs on; the launch is so long that what row-by-row costs at its start and
// end no longer counts).
int64_t short_rows_from(int32_t d, int32_t V, bool bf16)
{
    if (d < 256) return INT64_MAX;
    if (d < 512) return 393216;
    if (d < 1024) return 65536;
    if ((int64_t)V * d >= ((int64_t)128 << 20)) return 0;
    return (int64_t)(bf16 ? 24576 : 40960) * 1024 / d;
}

int piece_tokens_for(int64_t n, bool wide_bf16)
{
    if (g_piece_override) return g_piece_override;
    return (wide_bf16 || n <= kPieceSmallMax) ? 16 : 32;
}

// Few pairs: pieces of 8 positions instead of 16 (a workspace of the same size: groups of pieces are 64 positions
// either way).  A piece's window is then 16 positions, and all its value rows are in flight at once: the launch of
// a call with few pairs is as long as a wavefront's chain of batches.  But work-groups of eight wavefronts (and twice
// as many of them) suit a launch that mostly copies or mostly gathers less.  fp32 rows, us with 8 / 16: V = 4000, d = 256,
// 2000 pairs 13.1 / 14.9, 20000 pairs 24.0 / 22.9; V = 1000, d = 272, 8000 pairs 18.9 / 19.6, 12000 pairs 24.0 / 22.6; V = 3000, d = 256,
// 16000 pairs 19.3 / 20.0, 17500 pairs 23.2 / 22.2 (uniform ids 21.1 / 18.4); V = 9000, d = 512, 9200 pairs 21.1 / 21.0; V = 32768, d = 256,
// 17500 pairs 24.1 / 24.8 (uniform ids 23.2 / 24.9); V = 16000, d = 512, 8000 pairs 23.8 / 25.5; V = 32768, d = 512, 8192 pairs
// 30.1 / 28.0.  bf16 rows (half the bytes per row, half the work-groups), V = 32768: d = 512, 12000 pairs 30.7 / 33.9, 24000
// pairs 38.5 / 41.3; d = 1024, 24000 pairs 63.9 / 63.3; d = 256, 100000 pairs 49.7 / 45.6.  The limits on the vocabulary cost
// calls in place that touch little of a large one (fp32, V = 74365, d = 256, 3280 pairs 13.8 / 15.5; bf16, V = 131072, d = 512, 5000 pairs
// 17.3 / 18.8), but out of place 8 loses there: fp32 29.7 / 28.6 and, d = 512, 98.0 / 90.3; bf16 rows to a bf16 result, V = 108448, d = 512,
// 4325 pairs 64.6 / 60.6.
// The length of the pieces fixes the order of additions, so it goes by the pairs, the width, the row type and the
// whole vocabulary alone: what only spreads the work (in place or not, short rows in the pieces or row by
// row, the range that a call owns) must not change a bit.  In these limits no call goes row by row unless forced to.
bool pieces_of_8(int64_t n, int32_t d, int32_t V_total, int32_t row_dtype, bool wide)
{
    const int64_t cols = (d + kColBlock - 1) / kColBlock * kColBlock;      // a piece has a wavefront per block
    if (wide) return d <= 512 && n <= 32768 && (int64_t)V_total * d <= 20 << 20;
    // 8 << 19: 256 work-groups.  A few more are a second round, which only a launch with something to copy hides.
    return row_dtype == TS_ROW_FP32 && n * cols <= ((int64_t)V_total * d < 5 << 20 ? 8 : 9) << 19 && (int64_t)V_total * d <= 12 << 20;
}

// Twice as many value rows in flight per wavefront (32-64 registers more, so fewer wavefronts): not
// where narrow rows come in large numbers, and not where the launch has nothing to copy beside a large
// gather.  us with 16 / 8 fp32 rows in flight, V = 32768: d = 1024, 16384 pairs 58.5 / 59.7, without a dense
// operand 38.1 / 39.2, 25000 pairs 70.0 / 71.5; d = 512, 8192 pairs 28.0 / 29.7; in place d = 1024, 4000 pairs 16.7 / 17.5,
// 16384 pairs 32.4 / 31.8; d = 64, 47000 pairs 31.3 / 31.4, 50000 33.0 / 31.7, 65000 34.0 / 31.0; d = 128, 47000 31.5 / 31.9, 50000
// 34.5 / 33.0; d = 192, 55000 39.5 / 39.1, 80000 41.8 / 40.7, but V = 100000 43.7 / 44.8, 71.2 / 70.7.  bf16 rows, 8 / 4 in flight: d = 1024, 12000 pairs 52.7 / 55.4; d = 64, 65000 33.3 / 33.9, 80000 38.4 / 35.4.
// Many pairs per row is a gather too, but the limit depends on the form.  fp32 rows in pieces of 16, 2.2 / 3.5 / 5 / 7 pairs
// per row: d = 1024, 20000 pairs 41.0 / 41.5, 37.2 / 36.6, 37.6 / 36.2, 36.1 / 35.8; 33000 pairs, where rows are left
// to copy, 58.3 / 61.8, 53.7 / 54.4, 53.0 / 52.6; d = 256, 80000 pairs 45.9 / 47.0, 45.3 / 45.9, 44.3 / 43.1, 45.8 / 45.1.  In pieces
// of 32, 4.2 / 7 / 16 / 25: d = 256, 140000 pairs 72.3 / 75.6, 59.4 / 61.7, 60.8 / 61.1, 62.2 / 62.7; d = 384 at 5 / 16 / 25 / 50 83.3 / 84.8,
// 79.0 / 79.5, 81.8 / 81.1, 86.1 / 85.1.  bf16 rows, 4.2 / 7 / 10 / 16 / 50: d = 256, 140000 pairs 62.9 / 64.2, 49.9 / 50.7,
// 49.9 / 49.7, 50.6 / 49.3, 61.3 / 59.0; d = 384 72.1 / 76.4, 58.9 / 62.4, 57.3 / 59.6, 56.8 / 58.0, 65.9 / 65.5.
// A launch that writes bf16 is mostly rows without pairs, in half the bytes: fewer wavefronts lose there.  fp32 rows to a bf16
// result, V = 100000, 8000 pairs: d = 768 with a dense operand 90.8 / 79.1, without 50.0 / 41.0, d = 512 60.6 / 54.6; V = 33801,
// d = 768 37.2 / 33.9, d = 512 26.9 / 26.6.  bf16 rows: d = 768 with one, V = 33801 34.1 / 35.2, V = 100000 81.3 / 79.3, without one 43.4 / 39.2,
// d = 512 without one 32.4 / 34.8.
// A range is taken to own its share of the pairs: one eighth of 32768 ids, d = 1024, 131072 fp32 pairs 38.2 / 40.7 us, with the
// hottest id in it 53.5 / 55.3, with all hot ids in it 126.8 / 125.0; bf16 rows 36.6 / 37.7, 46.5 / 48.0, 94.2 / 94.0.
bool deep_batches(int64_t n, int32_t d, int32_t V, int32_t row_dtype, int32_t C, bool in_place, bool to_bf16, bool dense)
{
    if (to_bf16 && (row_dtype == TS_ROW_FP32 || (V > 65536 && (d > 512 || dense)))) return false;
    if (d < kColBlock && n > (row_dtype == TS_ROW_FP32 && d <= 128 ? 49152 : 65536)) return false;
    if (n * d <= 8 << 20) return true;
    if (in_place) return false;
    return n <= (row_dtype == TS_ROW_BF16 ? 8 : C >= 32 ? 16 : 4) * (int64_t)V;
}

// The lists of owned pairs: a wavefront's whole share where the LDS has room for it beside the tables, at least the
// 1024 pairs of a round.
void set_lists(Plan* pl)
{
    const int64_t share = pl->SL / kSortWaves;
    const int64_t tables = ((int64_t)kSortWaves * pl->part / (pl->wide_tab ? 1 : 2) + (pl->S > 1 ? 3 : 2) * (int64_t)pl->part) * 4;
    const int64_t room = (kLdsBytes - 256 - tables) / (kSortWaves * 4) / 64 * 64;
    pl->list_cap = (int32_t)(share < room ? share : room);
    pl->list_full = share <= room ? 0xFFFFFFFFu : (uint32_t)(pl->list_cap - kGroupTiles * 64);
    pl->sort_lds = (size_t)tables + (size_t)kSortWaves * pl->list_cap * 4;
}

// bound: size the arrays that depend on how the sort is split (slices, parts) for the largest
// split any call of at most n pairs and at most V rows can choose, so that the total never
// shrinks when n or V grows.
// group: sorted positions of a group of pieces (0: as many as go with C).  range_cus: of a call that owns
// a range of the vocabulary, the compute units of the GPU (0: slices as for a whole vocabulary).
void make_plan(int64_t n, int32_t d, int32_t V, int32_t C, Plan* pl, bool bound = false, int32_t group = 0,
               int32_t range_cus = 0)
{
    if (group == 0) group = C * group_pieces(C);
    if (n <= kFusedSortMax) {
        pl->S = 1;
        pl->SL = (int32_t)align_up((size_t)(n > 0 ? n : 1), 1024);
    } else {
        int64_t SL = kSliceTokens;
        int64_t S = (n + SL - 1) / SL;
        if (S > kMaxSlices) {
            SL = (int64_t)align_up((size_t)((n + kMaxSlices - 1) / kMaxSlices), 1024);
            S = (n + SL - 1) / SL;
        }
        pl->S = (int32_t)S;
        pl->SL = (int32_t)SL;
    }
    // ids per sort work-group: smaller parts shorten the sort (fewer owned pairs per
    // work-group), but every sorting work-group holds a compute unit that could copy; about 64 work-groups per slice measured best
    // (with several slices every part looks at every slice, and that dominates: the largest
    // parts that still give every compute unit a work-group)
    int part = (pl->S > 1 && (int64_t)((V + kMaxPart - 1) / kMaxPart) * pl->S >= 256) ? kMaxPart : 1024;
    while (pl->S == 1 && part > kMinPart && (int64_t)((V + part - 1) / part) < 64) part >>= 1;
    if (g_part_override) part = g_part_override;
    // the tables hold 16 bits per (wavefront, id) where the pairs of a slice fit, else 32
    pl->wide_tab = pl->SL > kNarrowSlice;
    if (pl->wide_tab && part > 1024) part = 1024;
    pl->part = part;
    set_lists(pl);
    pl->G = (V + part - 1) / part;
    pl->C = C;
    pl->NB = (int32_t)((n + pl->C - 1) / pl->C);
    // a work-group of the reduce kernel takes a group of pieces; the shares of a row that spans several
    // work-groups are added up in a tree with a fan-in of 16: levels needed for a row that spans them all
    pl->NBG = (int32_t)((n + group - 1) / group);
    pl->levels = 1;
    for (int64_t reach = kFanIn; reach < pl->NBG; reach *= kFanIn) ++pl->levels;
    pl->ncb = (d + kColBlock - 1) / kColBlock;
    size_t o = 0;
    pl->off_nvalid = o;
    pl->off_nbad = o + 4;
    o = 256;
    pl->off_arrive = o;
    pl->arrive_bytes = align_up((size_t)pl->levels * 2 * pl->NBG * pl->ncb * 4, 256);
    o += pl->arrive_bytes;
    pl->off_count = o;
    o = align_up(o + (size_t)V * 4, 256);
    pl->off_row_start = o;
    o = align_up(o + ((size_t)V + 1) * 4, 256);
    pl->off_sorted = o;
    o = align_up(o + (size_t)n * sizeof(SortedPair), 256);
    size_t S_tab = pl->S > 1 ? (size_t)pl->S : 0, ids_tab = (size_t)pl->G * pl->part, G_tab = (size_t)pl->G;
    if (bound && n > kFusedSortMax) {
        const size_t s16 = (size_t)((n + kSliceTokens - 1) / kSliceTokens);
        S_tab = s16 < (size_t)kMaxSlices ? s16 : (size_t)kMaxSlices;
        ids_tab = align_up((size_t)V, kMaxPart);
        G_tab = ((size_t)V + 63) / 64;
    }
    pl->off_tot = o;
    if (S_tab) o = align_up(o + S_tab * ids_tab * 4, 256);
    pl->off_below = o;
    if (S_tab) o = align_up(o + S_tab * G_tab * 4, 256);
    pl->off_bad = o;
    if (S_tab) o = align_up(o + S_tab * 4, 256);
    pl->off_partial = o;
    o = align_up(o + (size_t)2 * pl->NBG * (size_t)d * 4, 256);
    pl->total = o;
    const int64_t S = (n + kRangeSliceTokens - 1) / kRangeSliceTokens;
    if (pl->S > 1 && S > pl->S && S <= kMaxSlices && S * pl->G <= range_cus) {
        // A range has few parts, so slices of 16384 pairs leave most compute units without a work-group while
        // the others look at every pair of their slice: smaller slices, as long as every work-group still
        // has a compute unit.  The tables are done with before the first share of a long row is stored, so they
        // may take that place too: the workspace stays what it was, and a call whose tables don't fit keeps
        // its slices.  (32768 ids, d = 1024, 131072 pairs, with slices of 16384 / 8192 / 4096: 4097 rows 39.1 / 37.8 /
        // 37.6 us, 8192 rows 50.5 / 49.5 / 49.3; 4097 rows at d = 64, 200000 pairs 34.7 / 33.3 / 34.7.  A quarter of 100000
        // ids has 25 parts: 10 slices instead of 8 cost 40.0 -> 44.2, more work-groups than compute units.)
        const size_t below = align_up(pl->off_tot + (size_t)S * ids_tab * 4, 256);
        const size_t bad = align_up(below + (size_t)S * G_tab * 4, 256);
        if (bad + (size_t)S * 4 <= pl->total) {
            pl->S = (int32_t)S;
            pl->SL = kRangeSliceTokens;
            pl->off_below = below;
            pl->off_bad = bad;
            set_lists(pl);
        }
    }
}

int check_hip(hipError_t e) { return e == hipSuccess ? TS_OK : TS_ERR_HIP; }

// Compute units of the current GPU (asked once per device; 0 if the question fails, which
// only switches a tuning rule off).
int compute_units()
{
    static int cached[64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = -1;
        cached[dev] = n;
    }
    return cached[dev] > 0 ? cached[dev] : 0;
}

// Device address of the built-in workspace on the current GPU: every GPU holds its own copy
// of the array at its own address, looked up once per device and kept.
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TS_ERR_HIP;
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return TS_ERR_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return TS_OK;
}

// The three kinds of launches, one instantiation per epilogue (the epilogue is a template
// argument so that the plain path keeps its code).
template <int EPI>
void launch_count(dim3 grid, const Plan& pl, hipStream_t stream, const SortParams& sp, const ShardTable& sh)
{
    const size_t lds = (size_t)pl.part * (pl.wide_tab ? 4 : 2);
    if (pl.wide_tab)
        hipLaunchKernelGGL((count_kernel<true, EPI>), grid, dim3(1024), lds, stream, sp, sh);
    else
        hipLaunchKernelGGL((count_kernel<false, EPI>), grid, dim3(1024), lds, stream, sp, sh);
}

template <int EPI>
void launch_sort_scatter(dim3 grid, const Plan& pl, hipStream_t stream, const SortParams& sp, const ShardTable& sh)
{
    if (pl.wide_tab)
        hipLaunchKernelGGL((sort_kernel<SORT_SCATTER, true, false, EPI>), grid, dim3(1024), pl.sort_lds, stream, sp, sh);
    else
        hipLaunchKernelGGL((sort_kernel<SORT_SCATTER, false, false, EPI>), grid, dim3(1024), pl.sort_lds, stream, sp, sh);
}

template <int EPI>
void launch_sort_fused(dim3 grid, const Plan& pl, hipStream_t stream, const SortParams& sp, const ShardTable& sh)
{
    static_assert(kFusedSortMax <= kNarrowSlice, "16 bits per id");
    if (pl.SL <= kSortWaves * kRoundPairs)
        hipLaunchKernelGGL((sort_kernel<SORT_FUSED, false, false, EPI>), grid, dim3(1024), pl.sort_lds, stream, sp, sh);
    else
        hipLaunchKernelGGL((sort_kernel<SORT_FUSED, false, true, EPI>), grid, dim3(1024), pl.sort_lds, stream, sp, sh);
}

// With events (benchmarks only) the launch goes through the variant that stamps them with the
// kernel's own begin and end, so that their difference is the kernel's duration.
template <typename Kernel>
void launch_timed(Kernel kernel, unsigned grid, int threads, hipStream_t stream, hipEvent_t begin, hipEvent_t end,
                  const ReduceParams& rp)
{
    if (begin)
        hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, begin, end, 0, rp);
    else
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, stream, rp);
}

// DEEP: sixteen (bf16 rows read 16 bytes per lane: eight) value rows in flight per wavefront, else half.
template <int EPI, int SHORT, int GP, bool DEEP>
void launch_reduce_as(unsigned grid, bool wide, int32_t row_dtype, hipStream_t stream, hipEvent_t begin,
                      hipEvent_t end, const ReduceParams& rp)
{
    if (wide)
        launch_timed(reduce_kernel<uint16_t, 2, DEEP ? 8 : 4, EPI, SHORT, GP>, grid, 64 * GP, stream, begin, end, rp);
    else if (row_dtype == TS_ROW_BF16)
        launch_timed(reduce_kernel<uint16_t, 1, 8, EPI, SHORT, GP>, grid, 64 * GP, stream, begin, end, rp);
    else
        launch_timed(reduce_kernel<float, 1, DEEP ? 16 : 8, EPI, SHORT, GP>, grid, 64 * GP, stream, begin, end, rp);
}

template <int EPI>
void launch_reduce(unsigned grid, bool wide, bool deep, int32_t row_dtype, hipStream_t stream, hipEvent_t begin,
                   hipEvent_t end, const ReduceParams& rp)
{
    // short rows row by row: long rows by lone wavefronts where a group of pieces fits the lanes of one
    if (rp.short_max > 0 && rp.logG > 6)
        launch_reduce_as<EPI, 2, 4, false>(grid, wide, row_dtype, stream, begin, end, rp);
    else if (rp.short_max > 0)
        launch_reduce_as<EPI, 1, 4, false>(grid, wide, row_dtype, stream, begin, end, rp);
    else if (rp.logG - rp.logC == 3)
        launch_reduce_as<EPI, 0, 8, true>(grid, wide, row_dtype, stream, begin, end, rp);
    else if (deep)
        launch_reduce_as<EPI, 0, 4, true>(grid, wide, row_dtype, stream, begin, end, rp);
    else
        launch_reduce_as<EPI, 0, 4, false>(grid, wide, row_dtype, stream, begin, end, rp);
}

#define TS_DISPATCH_EPI(epi, fn, ...)                              \
    do {                                                           \
        if ((epi) == EPI_NONE) fn<EPI_NONE>(__VA_ARGS__);          \
        else if ((epi) == EPI_SCALE) fn<EPI_SCALE>(__VA_ARGS__);   \
        else fn<EPI_SCALE_BF16>(__VA_ARGS__);                      \
    } while (0)

void remember(const Plan& pl, void* ws, int32_t V, int32_t copied_beside, int32_t form)
{
    g_last_plan = pl;
    g_last_ws = ws;
    g_last_V = V;
    g_last_info[0] = pl.C;
    g_last_info[1] = copied_beside;
    g_last_info[2] = V;
    g_last_info[3] = pl.S;
    g_last_info[4] = pl.part;
    g_last_info[5] = pl.NB;
    g_last_info[6] = pl.levels;
    g_last_info[7] = form;
    g_have_last = true;
}

// Calls that small_kernel takes: those that it makes shorter where ids are spread, and not longer, but for some that crowd at the
// vocabulary's begin, than two launches.  All pairs may crowd into one work-group's part, on one id or in the order of their
// frequency; a part is the longer the larger the output is, so the limit on the output falls with the pairs.  us with two
// launches / one, input sets of 100 MB in turn:
//                                   uniform ids    Zipf 1.1       0.9 on one id   32 ids        Zipf 1.1, hottest first
//   within  V = 1000, d = 64, 2048    10.1 /  7.4                  14.1 / 13.0     15.8 / 15.2   13.9 / 13.1
//           V = 6144, d = 64, 2048    10.2 /  7.2                  14.4 / 13.5     15.7 / 15.2   13.6 / 13.2
//           V = 13312, d = 64, 2048   10.1 /  6.9    11.9 /  9.2   14.2 / 13.8     15.7 / 15.4   13.5 / 13.2
//           V = 26000, d = 64, 1048   11.0 /  8.1    12.8 /  9.5   13.3 / 11.6     13.9 / 12.2   12.7 / 12.7
//           V = 40960, d = 64, 660    11.3 /  9.1    12.8 /  9.7   13.3 / 11.4     12.6 / 11.2   12.4 / 13.0
//           V = 13600, d = 128, 1000  11.1 /  8.1    12.6 /  9.5   13.1 / 11.8     13.0 / 11.8   12.6 / 11.8
//           V = 8192, d = 256, 512    11.9 /  7.4    13.1 /  8.9   12.9 / 10.6     12.7 / 11.7   12.6 / 11.1
//           V = 2048, d = 1024, 512   12.1 /  8.1    13.2 /  9.6   13.4 / 11.4     12.9 / 11.9   12.9 / 11.8
//   beyond  V = 20480, d = 64, 2048   10.5 /  8.8    12.2 / 10.4   14.4 / 14.8     15.8 / 15.9   13.6 / 14.7
//           V = 40960, d = 64, 2048   11.5 / 12.5    13.1 / 13.3   15.1 / 17.2     15.9 / 17.4   13.9 / 18.0
//           V = 20480, d = 128, 1000  11.7 / 10.3    13.1 / 11.1   13.7 / 13.4     13.2 / 12.8   13.0 / 14.7
//           V = 5120, d = 512, 512    12.2 /  9.8    13.6 / 10.7   13.6 / 12.4     13.0 / 13.0   12.8 / 13.9
//           V = 1000, d = 64, 2304    10.0 /  7.7                  14.2 / 13.7     16.9 / 16.6   14.3 / 13.4
//           V = 1000, d = 64, 3072    10.7 /  8.9                  14.8 / 15.6     18.0 / 19.3   15.3 / 14.8
//           V = 1000, d = 128, 2048   10.1 /  8.1                  14.3 / 14.1     15.8 / 16.5   13.8 / 13.5
// (Zipf 1.5, hottest first, is what loses most within: V = 13312, d = 64, 2048 pairs 14.2 / 14.9.  Wide rows would bear
// more pairs: d = 256, 1024 pairs with 32 ids 12.9 / 12.5.  A setting that says how to split the work over the launches is for
// the two-launch form.)
constexpr int64_t kSmallPairLanes = 32768;      // pairs times lanes of a whole row, 64 at most
constexpr int64_t kSmallElems = 5 << 19;
constexpr int64_t kSmallPairElems = 13ll << 27, kSmallPairElemsWide = 8ll << 27;      // (wide: rows of more than 32 lanes)

bool small_call(int64_t n, int32_t d, int32_t V)
{
    if (g_piece_override || g_part_override || g_short_rows >= 0 || g_overlap_sort >= 0) return false;
    int64_t lanes = 1;
    while (lanes < 64 && lanes * 4 < d) lanes *= 2;
    const int64_t elems = (int64_t)V * d;
    return n >= 1 && n <= kSmallMax && n * lanes <= kSmallPairLanes && elems <= kSmallElems && n * elems <= (lanes <= 32 ? kSmallPairElems : kSmallPairElemsWide);
}

template <int EPI>
void launch_small(unsigned grid, size_t lds, int32_t row_dtype, hipStream_t stream, hipEvent_t begin, hipEvent_t end,
                  const SmallParams& q, const ShardTable& sh)
{
    const dim3 threads(64 * kSmallWaves);
    if (row_dtype == TS_ROW_BF16) {
        if (begin) hipExtLaunchKernelGGL((small_kernel<uint16_t, EPI>), dim3(grid), threads, lds, stream, begin, end, 0, q, sh);
        else hipLaunchKernelGGL((small_kernel<uint16_t, EPI>), dim3(grid), threads, lds, stream, q, sh);
    } else {
        if (begin) hipExtLaunchKernelGGL((small_kernel<float, EPI>), dim3(grid), threads, lds, stream, begin, end, 0, q, sh);
        else hipLaunchKernelGGL((small_kernel<float, EPI>), dim3(grid), threads, lds, stream, q, sh);
    }
}

int densify_small(const ShardTable& sh, Plan& pl, int32_t row_dtype, int32_t d, int32_t V, int32_t id_base, int32_t V_total,
                  const float* dense_in, void* dense_out, int epi, float scale, hipStream_t stream, char* ws, bool in_place, bool wide)
{
    SmallParams q;
    q.n = sh.off[sh.k];
    q.V = V;
    q.id_base = id_base;
    q.V_total = V_total;
    q.row_bytes = d * (row_dtype == TS_ROW_BF16 ? 2 : 4);
    q.d = d;
    q.C = pl.C;
    q.lanes = small_lanes(q.n, d);
    q.combine_batch = wide ? 4 : 8;
    const int ncb = (d + 4 * q.lanes - 1) / (4 * q.lanes);
    // kSmallPart ids to a work-group, or as many as it takes for every one to have a compute unit of its own
    const int rows = kSmallWaves * (64 / q.lanes);              // of a work-group in one round
    const int64_t cus = compute_units() > 0 ? compute_units() : 256;
    q.part = rows < kSmallPart ? rows : kSmallPart;
    // (blocks of columns that share lines of 128 bytes: those of a part on one XCD, with one L2; V = 6000, d = 64, 2048 pairs, nine
    // tenths of them on one id 14.3 -> 13.4 us)
    const bool share_lines = ncb > 1 && q.lanes * 16 < 128;
    for (;; q.part *= 2) {
        q.G = (V + q.part - 1) / q.part;
        q.stride = share_lines ? (q.G + kXcds - 1) / kXcds * kXcds : q.G;
        if (q.part >= kSmallPartMax || q.part >= rows * kSmallRows || (int64_t)q.stride * ncb <= cus) break;
    }
    q.rounds = (q.part + rows - 1) / rows;
    q.count = (int32_t*)(ws + pl.off_count);
    q.row_start = (int32_t*)(ws + pl.off_row_start);
    q.sorted = (SortedPair*)(ws + pl.off_sorted);
    q.n_valid = (int32_t*)(ws + pl.off_nvalid);
    q.n_bad = (int32_t*)(ws + pl.off_nbad);
    q.dense_in = dense_in;
    q.dense_out = dense_out;
    q.copy_untouched = !(in_place && epi == EPI_NONE);
    q.scale = scale;
    const bool prof = g_prof_used < g_prof_cap;
    hipEvent_t ev_begin = prof ? g_ev[2 * g_prof_used] : nullptr, ev_end = prof ? g_ev[2 * g_prof_used + 1] : nullptr;
    TS_DISPATCH_EPI(epi, launch_small, (unsigned)(q.stride * ncb), small_lds(q.n, q.part, q.lanes), row_dtype, stream, ev_begin, ev_end, q, sh);
    if (prof) ++g_prof_used;
    if (hipGetLastError() != hipSuccess) return TS_ERR_HIP;
    pl.part = q.part;
    remember(pl, ws, V, 0, (in_place ? 1 : 0) | 3 << 1);
    return TS_OK;
}

// V rows are produced: ids id_base .. id_base + V - 1 of a vocabulary of V_total ids.
int densify_impl(const ShardTable& sh, int64_t n, int32_t row_dtype, int32_t d, int32_t V, int32_t id_base,
                 int32_t V_total, const float* dense_in, void* dense_out, int epi, float scale, void* stream_v,
                 void* ws_v, int64_t ws_bytes)
{
    const bool wide = row_dtype == TS_ROW_BF16 && (d % 8) == 0;     // 16-byte loads of bf16 rows
    const bool in_place = (const void*)dense_in == (const void*)dense_out;
    // Output rows with at most C pairs: with many pairs in the call they are added up row by row, by the
    // wavefronts that would otherwise copy the row; with few, the pieces take them along.
    // What counts is the pairs that the call will own: of a range, about its share of the vocabulary.  (One
    // eighth of 32768 ids, 131072 bf16 pairs, d = 1024: with short rows in the pieces 37.7 us, by row 42.)
    const bool range = V < V_total;
    const int64_t n_own = range ? (int64_t)((double)n * V / V_total) : n;
    const bool by_row = g_short_rows < 0 ? n_own >= short_rows_from(d, V, row_dtype == TS_ROW_BF16) : g_short_rows == 1;
    // The groups of pieces, and with them the workspace, go by all pairs.
    int32_t C = piece_tokens_for(n, wide);
    const int32_t group = C * group_pieces(C);
    if (!g_piece_override && group == 64 && pieces_of_8(n, d, V_total, row_dtype, wide)) C = 8;
    const bool deep = deep_batches(n_own, d, V, row_dtype, C, in_place, epi == EPI_SCALE_BF16, dense_in != nullptr);
    Plan pl;
    make_plan(n, d, V, C, &pl, false, group, range ? compute_units() : 0);
    if (!ws_v || (int64_t)pl.total > ws_bytes) return TS_ERR_WORKSPACE;
    if ((int64_t)pl.NB * pl.ncb + (int64_t)V * ((d + 4 * kColBlock - 1) / (4 * kColBlock)) >= ((int64_t)1 << 31) - 8)
        return TS_ERR_OVERFLOW;
    hipStream_t stream = (hipStream_t)stream_v;
    char* ws = (char*)ws_v;

    if (small_call(n, d, V)) return densify_small(sh, pl, row_dtype, d, V, id_base, V_total, dense_in, dense_out, epi, scale, stream, ws, in_place, wide);

    SortParams sp;
    sp.n = (int32_t)n;
    sp.V = V;
    sp.id_base = id_base;
    sp.V_total = V_total;
    sp.G = pl.G;
    sp.S = pl.S;
    sp.SL = pl.SL;
    sp.part = pl.part;
    sp.row_bytes = d * (row_dtype == TS_ROW_BF16 ? 2 : 4);
    sp.count = (int32_t*)(ws + pl.off_count);
    sp.row_start = (int32_t*)(ws + pl.off_row_start);
    sp.sorted = (SortedPair*)(ws + pl.off_sorted);
    sp.tot = (uint32_t*)(ws + pl.off_tot);
    sp.below = (uint32_t*)(ws + pl.off_below);
    sp.bad = (uint32_t*)(ws + pl.off_bad);
    sp.n_valid = (int32_t*)(ws + pl.off_nvalid);
    sp.n_bad = (int32_t*)(ws + pl.off_nbad);
    sp.arrive = (int32_t*)(ws + pl.off_arrive);
    sp.arrive_vec = (int32_t)(pl.arrive_bytes / 16);

    // In place, the plain path leaves untouched rows alone.  With an epilogue they still have
    // to be scaled, by the item that reads them; only the copy made before the pairs are
    // sorted must go, because the reduce kernel would read scaled values.
    const bool skip_untouched = in_place && epi == EPI_NONE;
    // Rows copied by the sort launches: about as many bytes as HBM moves while a sort runs.  One slice: 32 MiB plus 1 MiB
    // per 1024 pairs up to 16384 pairs, 1.25 MiB per 1024 pairs beyond (the wavefronts then walk their shares in several
    // rounds; 2.5 MiB copies too many rows that receive pairs: V = 32768, d = 1024, 40000 pairs 84.9 us with 1.25, 86.5 with
    // 2.5, d = 512 48.4 and 51.5).  Where shards begin inside the shares of three or more wavefronts, these look their ids'
    // shards up and the sort is longer: 2.5 MiB there.  V = 32768, d = 1024, even shards, us with 1.25 / 2.5: 57000 pairs in 2 / 3 /
    // 4 / 8 shards 99.3 / 101.5, 99.9 / 101.4, 102.5 / 101.9, 105.6 / 101.7; d = 512, 40000 pairs in 2 / 3 / 8 47.1 / 50.2, 48.0 / 50.0,
    // 53.1 / 52.3.  Where the copies read nothing, any such shard counts: without a dense operand, in two shards, V = 68359, d = 1024,
    // 49901 pairs 99.2 / 96.1, V = 118817, d = 512, 49917 pairs 65.1 / 63.1, V = 33232, d = 512, 43556 pairs level.  (Right in the mean
    // only: 40219 pairs in two shards, V = 42517, d = 256 37.1 / 35.9.  Not for fewer pairs, beside which the copies are made one per
    // compute unit, below: V = 60000, d = 512, 6000 pairs in 3 shards 43.8, with more 47.2; 16000 in 16 level.)
    // A sort of a few slices leaves compute units idle, and a smaller blind copy beside each of its two launches still
    // pays (+4 % at 3-4 slices); a sort of many slices keeps the whole GPU busy by itself (a copying work-group beside every
    // sorting one lengthens the sort by more than the copy is worth), and with that many pairs a large share of the rows
    // copied blindly would be overwritten: no blind copy then.
    int32_t cut_shares = 0;
    for (int32_t j = 1, last = -1; n > 16384 && j < sh.k; ++j) {
        const int32_t share = pl.SL / kSortWaves, at = sh.off[j];
        if (at >= n || at % share == 0 || at / share == last) continue;
        last = at / share;
        ++cut_shares;
    }
    const bool cut = cut_shares >= (dense_in ? 3 : 1);
    const int64_t budget_single = n <= 16384 ? (32ll << 20) + (n / 1024 << 20)
                                             : (48ll << 20) + (n - 16384) / 1024 * ((cut ? 10ll : 5ll) << 18);
    const int64_t slices = (n + kSliceTokens - 1) / kSliceTokens;      // a range may have more, smaller ones
    const int64_t budget_multi = slices <= 4 ? (32ll << 20) : (slices <= 6 ? (16ll << 20) : 0);
    const int64_t budget = g_overlap_sort >= 0 ? g_overlap_sort
                                               : (pl.S == 1 ? budget_single : budget_multi);
    // The budget counts the bytes that a copied row really moves: without a dense operand it is only
    // written, and a bf16 result is half as long (V = 33801, d = 1024, without a dense operand: 4987 pairs
    // 33.0 -> 32.0 us, 16384 pairs 42.8 -> 40.5; two or three times the rows per work-group 32.4-32.8 / 41.2-43.9).
    // A bf16 result without one counts as an fp32 one beside a short sort: half the bytes again per work-group would
    // make three times as many of them as compute units (V = 20000 / 33801, d = 1024, 12000 pairs 28.8 -> 27.0 us, 31.6 -> 28.8;
    // 40000 pairs, a long sort, 57.4 with all of them, 59.9 with half).
    int64_t elem_bytes = (dense_in ? 4 : 0) + (epi == EPI_SCALE_BF16 ? 2 : 4);
    if (elem_bytes < 4 && n <= 22528 && g_overlap_sort < 0) elem_bytes = 4;
    const int64_t wg_elems = (int64_t)kBlindElems * kSortWaves;
    int64_t copy_wgs = in_place ? 0 : budget / (elem_bytes * wg_elems);
    // A work-group of these launches holds a compute unit (1024 threads, most of the LDS).  Where the default budget comes
    // to a little less than one work-group per compute unit in all, make it exactly one (fewer leave compute units idle:
    // V = 32768, d = 1024, 2048-12800 pairs 1-2 %); where it comes to more, too (a few more leave a second round of
    // stragglers), unless the sort is a long one or the copies read nothing.  us with more / exactly one: V = 32768, 18500 pairs, d = 1024
    // 64.1 / 62.0, d = 256 27.6 / 26.2; V = 60000, d = 512, 5000 pairs 47.3 / 44.7, without a dense operand 24.1 / 27.0; V = 60000,
    // d = 512, 21000 pairs 32.0 / 31.2; V = 131072, 26000 pairs 54.6 / 55.5.
    if (pl.S == 1 && g_overlap_sort < 0 && copy_wgs > 0) {
        const int64_t cus = compute_units();
        const int64_t all = pl.G + copy_wgs;
        const bool long_sort = n > 22528 || cut || !dense_in;
        if (cus > pl.G && 4 * all >= 3 * cus && (all < cus || !long_sort)) copy_wgs = cus - pl.G;
    }
    // Beside a sliced sort that leaves compute units idle: no more of them than that.  (More wait for the sort's, and the
    // two launches end late; where the sort fills the GPU anyway that costs nothing and copies are worth 1-5 %.)  us with
    // the budget / the idle ones: V = 41900, d = 256, 65536 pairs 49.8 / 44.8, uniform ids 53.6 / 46.8; d = 512, 97000 pairs 92.2 / 86.9;
    // V = 60000, d = 512, 58000 pairs 84.5 / 80.3, bf16 rows 77.8 / 73.0.  An fp32 result without a dense operand is written at
    // the same rate wherever it is: V = 33801, d = 512, 58000 pairs 51.9 / 54.9 (a bf16 one 53.0 / 50.0).
    if (pl.S > 1 && g_overlap_sort < 0 && (dense_in || epi == EPI_SCALE_BF16)) {
        const int64_t idle = (int64_t)compute_units() - (int64_t)pl.G * pl.S;
        if (idle > 0 && copy_wgs > idle) copy_wgs = idle;
    }
    const int64_t rows_per_launch = copy_wgs * wg_elems / d;
    int32_t copy_done = 0;
    auto sort_grid = [&](SortParams& q) {
        const int32_t row1 = (int32_t)(copy_done + rows_per_launch < V ? copy_done + rows_per_launch : V);
        q.copy_e0 = (int64_t)copy_done * d;
        q.copy_e1 = (int64_t)row1 * d;
        copy_done = row1;
        return dim3((unsigned)(pl.G * pl.S + (q.copy_e1 - q.copy_e0 + wg_elems - 1) / wg_elems));
    };
    sp.copy_in = dense_in;
    sp.copy_out = dense_out;
    sp.scale = scale;
    sp.list_cap = pl.list_cap;
    sp.list_full = pl.list_full;
    if (pl.S == 1) {
        const dim3 g1 = sort_grid(sp);
        TS_DISPATCH_EPI(epi, launch_sort_fused, g1, pl, stream, sp, sh);
    } else {
        const dim3 g1 = sort_grid(sp);
        TS_DISPATCH_EPI(epi, launch_count, g1, pl, stream, sp, sh);
        const dim3 g2 = sort_grid(sp);
        TS_DISPATCH_EPI(epi, launch_sort_scatter, g2, pl, stream, sp, sh);
    }
    if (hipGetLastError() != hipSuccess) return TS_ERR_HIP;

    ReduceParams rp;
    rp.V = V;
    rp.d = d;
    rp.C = pl.C;
    rp.ncb = wide ? (d + 2 * kColBlock - 1) / (2 * kColBlock) : pl.ncb;
    rp.n_piece_groups = pl.NBG * rp.ncb;
    rp.count = sp.count;
    rp.sorted = sp.sorted;
    rp.n = (int32_t)n;
    rp.n_valid = sp.n_valid;
    rp.dense_in = dense_in;
    rp.dense_out = dense_out;
    rp.scale = scale;
    rp.partial = (float*)(ws + pl.off_partial);
    rp.arrive = sp.arrive;
    rp.nslots = 2 * pl.NBG;
    rp.part_owned = range && pl.S > 1;      // few pairs: few groups, and the question costs more (16.4 -> 16.8 us)
    rp.logC = __builtin_ctz((unsigned)pl.C);
    rp.logG = group == 128 ? 7 : 6;
    const int gp = group / pl.C;
    rp.copy_row0 = copy_done;
    rp.copy_untouched = skip_untouched ? 0 : 1;
    rp.row_start = sp.row_start;
    rp.short_max = by_row ? pl.C : 0;
    // with pieces of at most 16 positions, the long rows by wavefronts that work alone, four groups
    // of pieces to a work-group
    if (rp.short_max > 0 && rp.logG <= 6) rp.n_piece_groups = (pl.NBG + 3) / 4 * rp.ncb;
    // after the work-groups of the pieces, one wavefront for every output row that may need one
    rp.row0 = rp.short_max > 0 ? 0 : (skip_untouched ? V : copy_done);
    // rows of at most 512 columns that are only copied: as many as make up 1024 columns per wavefront (below)
    const int32_t wave_rows = rp.short_max == 0 && d <= 512 ? (1024 / d < 64 ? 1024 / d : 64) : 1;
    const int32_t chunks = (d + 4 * kColBlock - 1) / (4 * kColBlock);
    rp.row_chunks = wave_rows > 1 ? -wave_rows : chunks;
    rp.row_magic = (uint32_t)(((1 << 20) + d - 1) / d);
    const int64_t row_items = ((int64_t)(V - rp.row0) + wave_rows - 1) / wave_rows * chunks;
    const int wg_waves = rp.short_max > 0 ? 4 : gp;
    const unsigned rgrid = (unsigned)(rp.n_piece_groups + (row_items + wg_waves - 1) / wg_waves);

    const bool prof = g_prof_used < g_prof_cap && rgrid > 0;
    hipEvent_t ev_begin = prof ? g_ev[2 * g_prof_used] : nullptr;
    hipEvent_t ev_end = prof ? g_ev[2 * g_prof_used + 1] : nullptr;
    if (rgrid > 0) TS_DISPATCH_EPI(epi, launch_reduce, rgrid, wide, deep, row_dtype, stream, ev_begin, ev_end, rp);
    if (prof) ++g_prof_used;
    if (hipGetLastError() != hipSuccess) return TS_ERR_HIP;

    // bit 0: in place; bits 1-2: how short rows were added up (0 in the pieces, 1 row by row with the long
    // rows by lone wavefronts, 2 row by row with the long rows by work-groups); bit 3: the deep batches
    const bool deep_form = rp.short_max == 0 && (gp == 8 || deep) && (wide || row_dtype == TS_ROW_FP32);
    remember(pl, ws, V, copy_done, (in_place ? 1 : 0) | ((rp.short_max == 0 ? 0 : (rp.logG <= 6 ? 1 : 2)) << 1) | (deep_form ? 8 : 0));
    return TS_OK;
}

int validate_common(int64_t n_total, int32_t d, int32_t V, const float* dense_in, const void* dense_out)
{
    if (!dense_out) return TS_ERR_NULL;
    if (n_total < 0 || V <= 0 || d <= 0 || (d % 4) != 0) return TS_ERR_SHAPE;
    if (n_total >= ((int64_t)1 << 31)) return TS_ERR_OVERFLOW;
    if (((uintptr_t)dense_out & 15u) || ((uintptr_t)dense_in & 15u)) return TS_ERR_ALIGN;
    return TS_OK;
}

int densify_shards(const int32_t* const* ids_k, const void* const* rows_k, const int64_t* n_k, int32_t k,
                   int32_t row_dtype, int32_t d, int32_t V, const float* dense_in, void* dense_out, int epi,
                   float scale, void* stream, int32_t v_begin = 0, int32_t v_end = -1, void* ws = nullptr,
                   int64_t ws_bytes = -1)
{
    if (ws_bytes < 0) {         // the bound workspace
        ws = g_ws;
        ws_bytes = g_ws_bytes;
    }
    if (v_end < 0) v_end = V;
    if (V <= 0 || v_begin < 0 || v_begin >= v_end || v_end > V) return TS_ERR_SHAPE;
    if (k < 1 || k > TS_MAX_SHARDS) return TS_ERR_SHAPE;
    if (row_dtype != TS_ROW_FP32 && row_dtype != TS_ROW_BF16) return TS_ERR_SHAPE;
    if (!ids_k || !rows_k || !n_k) return TS_ERR_NULL;
    int64_t n_total = 0;
    for (int j = 0; j < k; ++j) {
        if (n_k[j] < 0) return TS_ERR_SHAPE;
        n_total += n_k[j];
        if (n_total >= ((int64_t)1 << 31)) return TS_ERR_OVERFLOW;
    }
    int rc = validate_common(n_total, d, v_end - v_begin, dense_in, dense_out);
    if (rc != TS_OK) return rc;
    ShardTable sh;
    memset(&sh, 0, sizeof sh);
    sh.k = k;
    int64_t off = 0;
    for (int j = 0; j < k; ++j) {
        if (n_k[j] > 0 && (!ids_k[j] || !rows_k[j])) return TS_ERR_NULL;
        if ((uintptr_t)rows_k[j] & 15u) return TS_ERR_ALIGN;
        if ((uintptr_t)ids_k[j] & 3u) return TS_ERR_ALIGN;
        sh.off[j] = (int32_t)off;
        sh.ids[j] = ids_k[j];
        sh.rows[j] = (const char*)rows_k[j];
        off += n_k[j];
    }
    for (int j = k; j <= TS_MAX_SHARDS; ++j) sh.off[j] = (int32_t)off;
    return densify_impl(sh, n_total, row_dtype, d, v_end - v_begin, v_begin, V, dense_in, dense_out, epi, scale, stream,
                        ws, ws_bytes);
}

}  // namespace

// ------------------------------------------------------------------ C ABI
extern "C" {

int ts_densify(const int32_t* ids, const float* rows, int64_t n, int32_t d, int32_t V,
               const float* dense_in, float* dense_out, void* stream)
{
    const void* r = rows;
    return densify_shards(&ids, &r, &n, 1, TS_ROW_FP32, d, V, dense_in, dense_out, EPI_NONE, 1.0f, stream);
}

int ts_densify_static(const int32_t* ids, const float* rows, int64_t n, int32_t d, int32_t V,
                      const float* dense_in, float* dense_out, void* stream)
{
    // the size check comes first: a call that does not fit touches nothing, not even the device
    if (n < 0 || V <= 0 || d <= 0 || (d % 4) != 0) return TS_ERR_SHAPE;
    if (n >= ((int64_t)1 << 31)) return TS_ERR_OVERFLOW;
    Plan pl;
    make_plan(n, d, V, piece_tokens_for(n, false), &pl);
    if ((int64_t)pl.total > (int64_t)TS_STATIC_SCRATCH_BYTES) return TS_ERR_CAPACITY;
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != TS_OK) return rc;
    const void* r = rows;
    return densify_shards(&ids, &r, &n, 1, TS_ROW_FP32, d, V, dense_in, dense_out, EPI_NONE, 1.0f, stream, 0, -1, ws,
                          (int64_t)TS_STATIC_SCRATCH_BYTES);
}

int ts_densify_bf16(const int32_t* ids, const uint16_t* rows, int64_t n, int32_t d, int32_t V,
                    const float* dense_in, float* dense_out, void* stream)
{
    const void* r = rows;
    return densify_shards(&ids, &r, &n, 1, TS_ROW_BF16, d, V, dense_in, dense_out, EPI_NONE, 1.0f, stream);
}

int ts_densify_multi(const int32_t* const* ids_k, const void* const* rows_k, const int64_t* n_k,
                     int32_t k, int32_t row_dtype, int32_t d, int32_t V, const float* dense_in,
                     float* dense_out, void* stream)
{
    return densify_shards(ids_k, rows_k, n_k, k, row_dtype, d, V, dense_in, dense_out, EPI_NONE, 1.0f, stream);
}

int ts_densify_scaled(const int32_t* const* ids_k, const void* const* rows_k, const int64_t* n_k,
                      int32_t k, int32_t row_dtype, int32_t d, int32_t V, const float* dense_in,
                      void* out, int32_t out_dtype, float scale, void* stream)
{
    if (out_dtype != TS_OUT_FP32 && out_dtype != TS_OUT_BF16) return TS_ERR_SHAPE;
    if (!(scale - scale == 0.0f)) return TS_ERR_SHAPE;                  // infinite or NaN
    if (out_dtype == TS_OUT_BF16 && out && (const void*)dense_in == out) return TS_ERR_SHAPE;
    const int epi = out_dtype == TS_OUT_BF16 ? EPI_SCALE_BF16 : (scale == 1.0f ? EPI_NONE : EPI_SCALE);
    return densify_shards(ids_k, rows_k, n_k, k, row_dtype, d, V, dense_in, out, epi, scale, stream);
}

int ts_densify_range(const int32_t* const* ids_k, const void* const* rows_k, const int64_t* n_k,
                     int32_t k, int32_t row_dtype, int32_t d, int32_t V, int32_t v_begin, int32_t v_end,
                     const float* dense_in, float* dense_out, void* stream)
{
    if (v_end < 0) return TS_ERR_SHAPE;
    return densify_shards(ids_k, rows_k, n_k, k, row_dtype, d, V, dense_in, dense_out, EPI_NONE, 1.0f, stream,
                          v_begin, v_end);
}

int ts_fusion_place(int64_t capacity_bytes, int64_t used_bytes, int32_t d, int32_t V, int32_t out_dtype,
                    int64_t* offset_bytes, int64_t* used_after_bytes)
{
    if (!offset_bytes || !used_after_bytes) return TS_ERR_NULL;
    if (capacity_bytes < 0 || used_bytes < 0 || d <= 0 || V <= 0) return TS_ERR_SHAPE;
    if (out_dtype != TS_OUT_FP32 && out_dtype != TS_OUT_BF16) return TS_ERR_SHAPE;
    int64_t bytes, start, end;
    if (__builtin_mul_overflow((int64_t)V, (int64_t)d, &bytes) ||
        __builtin_mul_overflow(bytes, (int64_t)(out_dtype == TS_OUT_BF16 ? 2 : 4), &bytes) ||
        __builtin_add_overflow(used_bytes, (int64_t)255, &start))
        return TS_ERR_OVERFLOW;
    start = start / 256 * 256;
    if (__builtin_add_overflow(start, bytes, &end)) return TS_ERR_OVERFLOW;
    if (end > capacity_bytes) return TS_ERR_CAPACITY;
    *offset_bytes = start;
    *used_after_bytes = end;
    return TS_OK;
}

int ts_buffer_bytes(int64_t k, int64_t N, int32_t d, int32_t V, int32_t row_dtype, int64_t* gathered_bytes,
                    int64_t* dense_bytes)
{
    if (!gathered_bytes || !dense_bytes) return TS_ERR_NULL;
    if (k < 0 || N < 0 || d <= 0 || V <= 0) return TS_ERR_SHAPE;
    if (row_dtype != TS_ROW_FP32 && row_dtype != TS_ROW_BF16) return TS_ERR_SHAPE;
    const int64_t elem = row_dtype == TS_ROW_BF16 ? 2 : 4;
    int64_t per_slice, kn, g, dn;
    if (__builtin_mul_overflow(elem, (int64_t)d, &per_slice) || __builtin_add_overflow(per_slice, (int64_t)4, &per_slice) ||
        __builtin_mul_overflow(k, N, &kn) || __builtin_mul_overflow(kn, per_slice, &g) ||
        __builtin_mul_overflow((int64_t)4 * V, (int64_t)d, &dn))
        return TS_ERR_OVERFLOW;
    *gathered_bytes = g;
    *dense_bytes = dn;
    return TS_OK;
}

int ts_workspace_bytes(int64_t n_total, int32_t d, int32_t V, int64_t* bytes)
{
    if (!bytes) return TS_ERR_NULL;
    if (n_total < 0 || V <= 0 || d <= 0 || (d % 4) != 0) return TS_ERR_SHAPE;
    if (n_total >= ((int64_t)1 << 31)) return TS_ERR_OVERFLOW;
    // the smallest pieces a call of this size can use: the most pieces, the largest workspace
    Plan a;
    make_plan(n_total, d, V, piece_tokens_for(n_total, true), &a, true);
    *bytes = (int64_t)a.total;
    return TS_OK;
}

int ts_call_workspace_bytes(int64_t n_total, int32_t row_dtype, int32_t d, int32_t V, int64_t* bytes)
{
    if (!bytes) return TS_ERR_NULL;
    if (n_total < 0 || V <= 0 || d <= 0 || (d % 4) != 0) return TS_ERR_SHAPE;
    if (row_dtype != TS_ROW_FP32 && row_dtype != TS_ROW_BF16) return TS_ERR_SHAPE;
    if (n_total >= ((int64_t)1 << 31)) return TS_ERR_OVERFLOW;
    Plan a;
    make_plan(n_total, d, V, piece_tokens_for(n_total, row_dtype == TS_ROW_BF16 && (d % 8) == 0), &a);
    *bytes = (int64_t)a.total;
    return TS_OK;
}

int ts_bind_workspace(void* ws, int64_t bytes)
{
    if (!ws) {
        g_ws = nullptr;
        g_ws_bytes = 0;
        g_have_last = false;
        return TS_OK;
    }
    if (bytes <= 0) return TS_ERR_SHAPE;
    if ((uintptr_t)ws & 255u) return TS_ERR_ALIGN;
    g_ws = ws;
    g_ws_bytes = bytes;
    g_have_last = false;
    return TS_OK;
}

int ts_last_views(const int32_t** count, const int32_t** row_start, const void** sorted,
                  const int32_t** n_valid, const int32_t** n_bad_ids)
{
    if (!g_last_ws || !g_have_last) return TS_ERR_WORKSPACE;
    const char* ws = (const char*)g_last_ws;
    if (count) *count = (const int32_t*)(ws + g_last_plan.off_count);
    if (row_start) *row_start = (const int32_t*)(ws + g_last_plan.off_row_start);
    if (sorted) *sorted = (const void*)(ws + g_last_plan.off_sorted);
    if (n_valid) *n_valid = (const int32_t*)(ws + g_last_plan.off_nvalid);
    if (n_bad_ids) *n_bad_ids = (const int32_t*)(ws + g_last_plan.off_nbad);
    return TS_OK;
}

int ts_read_views(int32_t* count_out, int32_t* row_start_out, int64_t rows_capacity, void* sorted_out,
                  int64_t sorted_capacity, int32_t* n_valid_out, int32_t* n_bad_ids_out, void* stream)
{
    if (!g_last_ws || !g_have_last) return TS_ERR_WORKSPACE;
    if (sorted_out && sorted_capacity < 0) return TS_ERR_SHAPE;
    // the lengths of count and row_start come from the last call, not from this caller
    if ((count_out || row_start_out) && rows_capacity < (int64_t)g_last_V) return TS_ERR_CAPACITY;
    if (hipStreamSynchronize((hipStream_t)stream) != hipSuccess) return TS_ERR_HIP;
    const char* ws = (const char*)g_last_ws;
    int32_t n_valid = 0, n_bad = 0;
    if (hipMemcpy(&n_valid, ws + g_last_plan.off_nvalid, 4, hipMemcpyDeviceToHost) != hipSuccess) return TS_ERR_HIP;
    if (hipMemcpy(&n_bad, ws + g_last_plan.off_nbad, 4, hipMemcpyDeviceToHost) != hipSuccess) return TS_ERR_HIP;
    if (sorted_out && (int64_t)n_valid > sorted_capacity) return TS_ERR_CAPACITY;
    if (n_valid_out) *n_valid_out = n_valid;
    if (n_bad_ids_out) *n_bad_ids_out = n_bad;
    if (count_out && hipMemcpy(count_out, ws + g_last_plan.off_count, (size_t)g_last_V * 4, hipMemcpyDeviceToHost) != hipSuccess)
        return TS_ERR_HIP;
    if (row_start_out && hipMemcpy(row_start_out, ws + g_last_plan.off_row_start, ((size_t)g_last_V + 1) * 4,
                                   hipMemcpyDeviceToHost) != hipSuccess)
        return TS_ERR_HIP;
    if (sorted_out) {
        if (n_valid > 0 && hipMemcpy(sorted_out, ws + g_last_plan.off_sorted, (size_t)n_valid * sizeof(SortedPair),
                                     hipMemcpyDeviceToHost) != hipSuccess)
            return TS_ERR_HIP;
    }
    return TS_OK;
}

int ts_last_launch_info(int32_t* info)
{
    if (!info) return TS_ERR_NULL;
    if (!g_have_last) return TS_ERR_WORKSPACE;
    for (int i = 0; i < 8; ++i) info[i] = g_last_info[i];
    return TS_OK;
}

int ts_unique_ids(int32_t* unique_ids_out, int32_t* n_unique_out, void* stream)
{
    if (!unique_ids_out || !n_unique_out) return TS_ERR_NULL;
    if (!g_last_ws || !g_have_last) return TS_ERR_WORKSPACE;
    const int32_t* count = (const int32_t*)((const char*)g_last_ws + g_last_plan.off_count);
    hipLaunchKernelGGL(unique_kernel, dim3(1), dim3(1024), 0, (hipStream_t)stream, count, g_last_V,
                       unique_ids_out, n_unique_out);
    return check_hip(hipGetLastError());
}

int ts_profile_begin(int32_t capacity)
{
    if (capacity < 0 || capacity > kMaxProfile) return TS_ERR_SHAPE;
    while (g_ev_made < 2 * capacity) {
        if (hipEventCreate(&g_ev[g_ev_made]) != hipSuccess) return TS_ERR_HIP;
        ++g_ev_made;
    }
    g_prof_cap = capacity;
    g_prof_used = 0;
    return TS_OK;
}

int ts_profile_end(float* ms_out, int32_t capacity, int32_t* n_out)
{
    if (!ms_out || !n_out) return TS_ERR_NULL;
    int m = g_prof_used < capacity ? g_prof_used : capacity;
    if (m < 0) m = 0;
    for (int i = 0; i < m; ++i) {
        if (hipEventSynchronize(g_ev[2 * i + 1]) != hipSuccess) return TS_ERR_HIP;
        if (hipEventElapsedTime(&ms_out[i], g_ev[2 * i], g_ev[2 * i + 1]) != hipSuccess) return TS_ERR_HIP;
    }
    *n_out = m;
    g_prof_cap = 0;
    g_prof_used = 0;
    return TS_OK;
}

int ts_set_overlap_bytes(int64_t sort_bytes)
{
    if (sort_bytes < -1) return TS_ERR_SHAPE;
    g_overlap_sort = sort_bytes;
    return TS_OK;
}

int ts_set_sort_part(int32_t part)
{
    if (part != 0 && part != 64 && part != 128 && part != 256 && part != 512 && part != 1024 && part != kMaxPart)
        return TS_ERR_SHAPE;
    g_part_override = part;
    return TS_OK;
}

int ts_set_short_rows(int32_t mode)
{
    if (mode < -1 || mode > 1) return TS_ERR_SHAPE;
    g_short_rows = mode;
    return TS_OK;
}

int ts_set_piece_tokens(int32_t piece_tokens)
{
    if (piece_tokens != 0 && piece_tokens != 8 && piece_tokens != 16 && piece_tokens != 32) return TS_ERR_SHAPE;
    g_piece_override = piece_tokens;
    return TS_OK;
}

const char* ts_status_string(int status)
{
    switch (status) {
        case TS_OK: return "ok";
        case TS_ERR_NULL: return "a required pointer is NULL";
        case TS_ERR_SHAPE: return "bad shape or argument value";
        case TS_ERR_ALIGN: return "pointer not aligned";
        case TS_ERR_WORKSPACE: return "workspace not bound or too small";
        case TS_ERR_HIP: return "HIP runtime error";
        case TS_ERR_OVERFLOW: return "size overflow";
        case TS_ERR_CAPACITY: return "output buffer too small";
        default: return "unknown status";
    }
}

}  // extern "C"
