// Host-side internals shared by the translation units of the library: the
// plan object, the device primitives (scan, stable radix sort) and argument
// validation helpers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "cogdl.h"

namespace cogdl {

// Work unit: edges [beg, end) of one row, reduced either straight into the
// output (part < 0) or into partial-sum slot `part`.
// Layout int4 {row, beg, end, part}.

// Column slices of a sliced plan: one per XCD of the MI355X.
constexpr int kSlices = 8;

struct Plan {
    int32_t n_rows = 0;
    int64_t nnz = 0;
    int32_t group_size = 0;
    int32_t max_feat = 0;
    int32_t max_heads = 0;
    cogdl_balance mode_req = COGDL_BALANCE_AUTO;
    int device = 0;

    int64_t cap_units = 0;     // >= sum_i max(1, ceil(d_i / G))
    int64_t cap_split = 0;     // >= number of rows with d_i > G
    int64_t cap_partials = 0;  // >= sum over split rows of ceil(d_i / G)

    void *base = nullptr;
    size_t bytes = 0;

    int4 *units = nullptr;        // [cap_units] execution order
    int4 *units_tmp = nullptr;    // [cap_units] row order (build scratch)
    int4 *split_rows = nullptr;   // [cap_split] {row, first partial slot, #slots, degree}
    int4 *part_units = nullptr;   // [cap_partials] {row, beg, end, split index}
    int32_t *row_units = nullptr; // [n_rows + 1] units of each row; [n_rows] = #units
    int32_t *n_parts = nullptr;   // #partial slots
    int32_t *n_split = nullptr;   // #split rows
    uint32_t *block_sums = nullptr; // 8 sums of each workgroup of the count pass
    int32_t *counters = nullptr;  // [8]: 0 close-degree rows, 1 chosen mode,
                                  //      2 units longer than kTinyUnit, 3 zero,
                                  //      5 1 when the last build's totals exceeded the
                                  //        capacities (the plan was left empty)
                                  //      6 which row counts the build used
    uint32_t *sort_keys = nullptr;   // [4 * cap_units]: keys, 2 ping buffers, sorted keys
    uint32_t *sort_vals = nullptr;   // [3 * cap_units]: order, then 2 ping buffers
    void *sort_ws = nullptr;
    size_t sort_ws_bytes = 0;
    float *partials = nullptr;    // [cap_partials * max_feat]
    int32_t *parg = nullptr;      // [cap_partials * max_feat] edge ids of partial maxima
    float *gstats = nullptr;      // [cap_partials * max_heads * 2] per-group (m, z)
    float *rstats = nullptr;      // [cap_split * max_heads * 2] per-split-row (m, z)

    // Sliced plans (cogdl_plan_create_sliced): in neighbour-group mode a row
    // with more than slice_min edges is cut at the boundaries of kSlices equal
    // column ranges (then into groups of at most group_size edges), and the
    // units form kSlices lists, slice s in list s and every other unit in list
    // row % kSlices, so that each list's gathers stay inside one column range.
    int32_t sliced = 0;
    int32_t n_cols = 0;
    int32_t slice_min = 0;
    int32_t key_bits = 0;         // bits of the in-list sort key (group_size - size)
    void *base2 = nullptr;        // second allocation (sliced plans)
    int32_t *lists_tbl = nullptr; // [3 * kSlices]: list starts, ends of the long units, list ends
    int32_t *alt_units = nullptr; // [n_rows + 1]: the unsliced counts, used when the sliced
                                  //   ones exceed the capacities
    int32_t *row_cuts = nullptr;  // [n_rows][kSlices - 1]: the inner cuts of each sliced row
    unsigned long long *totals = nullptr;  // [3]: sliced units, partial slots, split rows

    const int32_t *n_units_dev() const { return row_units + n_rows; }
    const int32_t *n_big_dev() const { return counters + 2; }
    const int32_t *zero_dev() const { return counters + 3; }
    const int32_t *n_split_dev() const { return n_split; }
    const int32_t *n_parts_dev() const { return n_parts; }
};

// Units of at most this many edges run in the narrow-sub-group path.
constexpr int kTinyUnit = 8;

// The unit ranges a launch walks (see unit_walk): the long units, the tiny
// units or all of them; one range, or one per list for a sliced plan.
struct UnitRange {
    const int32_t *lo;
    const int32_t *hi;
    int lists;
};

inline UnitRange long_units(const Plan &P)
{
    if (P.sliced) return {P.lists_tbl, P.lists_tbl + kSlices, kSlices};
    return {P.zero_dev(), P.n_big_dev(), 1};
}

inline UnitRange tiny_units(const Plan &P)
{
    if (P.sliced) return {P.lists_tbl + kSlices, P.lists_tbl + 2 * kSlices, kSlices};
    return {P.n_big_dev(), P.n_units_dev(), 1};
}

inline UnitRange all_units(const Plan &P)
{
    if (P.sliced) return {P.lists_tbl, P.lists_tbl + 2 * kSlices, kSlices};
    return {P.zero_dev(), P.n_units_dev(), 1};
}

template <typename Args>
inline void set_units(Args &a, const UnitRange &r)
{
    a.u_lo = r.lo;
    a.u_hi = r.hi;
    a.lists = r.lists;
}

// A grid of `blocks` workgroups adjusted for `lists` lists: a multiple of it.
inline int64_t list_grid(int64_t blocks, int lists)
{
    if (lists <= 1) return blocks > 0 ? blocks : 1;
    const int64_t b = blocks / lists * lists;
    return b < lists ? lists : b;
}

const Plan *plan_of(const cogdl_plan *h);

// Workgroups of `block` threads of `kernel` with `shm` bytes of dynamic LDS that fit on
// the device at once (all compute units), at most `most` a compute unit when given;
// cached per kernel, shm and most.
int resident_blocks(const void *kernel, int block, size_t shm = 0, int most = 0);

// Workgroups a compute unit of the gathers over tables past the Infinity Cache (256 MB):
// with the fourth one the rows in flight evict more of what the L2s would serve.  SpMM
// with rows of 512 bytes and more, 122M edges x 256 bf16: 5.30 ms, with three 5.12 (60M
// fp32 rows of 512 bytes 0.96 and 0.94; rows of 256 bytes 1.27 and 1.32, so not there).
// Aggregation on given scores with a sliced plan, 122M edges: 4 x 64 bf16 7.68 and 7.44,
// 4 x 32 bf16 4.35 and 4.22, 8 x 16 fp32 7.40 and 7.30; with a plain one 9.33 and 9.33 (of a
// training step's forward and backward, 26 ms at 4 x 64, that is within the noise); on
// projected scores, rows of 512 bytes and more on 8 lanes or more a head: 4 x 64 bf16 plain
// 7.62 and 7.37, 8 x 64 17.0 and 16.5 (1 x 128, 256 bytes, 3.22 and 3.41; 4 x 32, 4 lanes a
// head, sliced, 2.64 and 2.86).  Tables the caches hold want every wavefront, and so do
// calls without a plan, which wait for their longest row: sums on 600k rows and 3M edges
// of 256 fp32 1.18 and 1.31, 2.4M and 12M 3.91 and 4.26, the aggregation on 1.2M and 6M
// at 4 x 64 bf16 2.69 and 2.90.
constexpr uint64_t kCachedTable = 256ull << 20;
constexpr int kFarTableBlocks = 3;

// Y[row] = sum of the partial rows of every split row of the plan (F columns),
// divided by the row's degree when `mean`, then act(. + bias) when given.
cogdl_status sum_reduce_launch(const char *name, const Plan &P, int64_t F, void *Y, int ydt,
                               bool mean, const float *bias, int act, hipStream_t s);

// Kernel tracing hooks (no-ops unless cogdl_trace_enable was called).
int trace_begin(const char *name, hipStream_t s);
void trace_end(int slot, hipStream_t s);

// ---------------------------------------------------------- primitives

// An extra 32-bit array carried through a radix sort: read from `in`,
// written in sorted order to `out`; `ping` is 2 * n elements of scratch.
// For the first payload only, `in` may be nullptr with `rowptr` set: the
// values are then the CSR rows of the elements (element e = edge e of the
// rowptr of n_rows rows), found by the sort itself instead of read.
struct RadixPayload {
    const uint32_t *in = nullptr;
    uint32_t *out = nullptr;
    uint32_t *ping = nullptr;
    const int32_t *rowptr = nullptr;
    int64_t n_rows = 0;
};

// Stable LSD radix sort of (key, value) pairs on the low `bits` bits of the
// keys.  vals_in == nullptr means values 0..n-1.  Results land in keys_out /
// vals_out (keys_out may be nullptr when the sorted keys are not needed); up
// to two payload arrays move with the keys.  ping: 2 * n keys and 2 * n
// values of scratch.  Digits are at most 8 bits wide, the key bits spread
// evenly over the fewest passes that allows.
size_t radix_workspace_bytes(int64_t n);
hipError_t radix_sort_pairs(const uint32_t *keys_in, const uint32_t *vals_in, uint32_t *keys_out,
                            uint32_t *vals_out, int64_t n, int bits, uint32_t *ping_keys,
                            uint32_t *ping_vals, void *ws, hipStream_t s,
                            RadixPayload pay0 = RadixPayload(), RadixPayload pay1 = RadixPayload());

// Fill n int32 with a value (a kernel, so it is safe inside graph capture).
hipError_t fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);

// ---------------------------------------------------------- validation

inline bool dtype_ok(int d) { return d == COGDL_F32 || d == COGDL_BF16 || d == COGDL_F16; }
inline int dtype_bytes(int d) { return d == COGDL_F32 ? 4 : 2; }

inline int bits_for(uint64_t max_value)
{
    int b = 0;
    while (b < 32 && (max_value >> b) != 0) ++b;
    return b;
}

inline int next_pow2(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

inline int log2i(int v)
{
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

// Launch geometry of the SpMM gather kernels for one row of `width` elements: VEC
// elements per lane, S lanes per edge row, CH chunks per lane and the number of feature
// slabs.
struct RowMap {
    int vec = 1;
    int S = 64;
    int log2S = 6;
    int ch = 1;
    int slab = 0;      // elements per slab
    int n_slabs = 1;
};

// 16-byte vectors at any alignment and any width of at least one vector (the kernel
// moves a row's last vector back to the row's end).  Rows of
// 41 bf16 classes take 6 lanes of 8 instead of 41 element lanes of 64.  Ragged rows
// of 8 to 32 elements keep one element per lane (16 or 32 lanes): on 45M edges their
// vectors measured slower (25 bf16: 1.88 against 1.73 ms, 11 fp32 1.60 against 1.41;
// 33 bf16 2.08 against 2.81, 7 fp32 1.38 against 1.52), rows off the 64-byte grid
// costing more requests as vectors than as lanes.
RowMap span_map(int64_t width, int elem_bytes);
RowMap element_map(int64_t width);      // one element per lane

// Geometry of k_gat for H heads of D features: 16-byte vectors at any alignment (one
// element per lane for heads narrower than a vector), L slots per head (k_gat), S lanes
// per edge row, CH slots per lane, and lm = log2 of the lanes of a head that share a
// batch's scores.  With `share` (scores or records to share; not on given weights) L is
// the head's vectors rounded up to a power of two wherever that needs no more lanes
// (always for a power of two of heads), at least so many that S >= 8: a chunk of column
// indices, one per lane, then fills a batch of 8 edges.  Given weights gain nothing from
// the padding and lose by it: 16 heads of 3 fp32 on 4 lanes each instead of 3, 20M edges
// 1525 us against 780.  Sub-groups of 8 lanes keep their tiny units: on 2 lanes those of
// 64 bf16 given weights on 2.5M edges took 76 us against 62.
struct HeadMap {
    int vec = 1;
    int L = 1;
    int S = 64;
    int log2S = 6;
    int ch = 1;
    int lm = 0;
    int n_slabs = 1;
    bool tiny = false;     // tiny units on S / 4 lanes, four slots a lane
};

HeadMap head_map(int H, int D, int elem_bytes, bool share);

}  // namespace cogdl

// Launch a kernel between the tracing events; return COGDL_ERR_LAUNCH from the
// enclosing function if the launch fails.
#define COGDL_LAUNCH(name, kern, grid, block, stream, ...)            \
    do {                                                             \
        const int _slot = ::cogdl::trace_begin(name, stream);        \
        kern<<<(grid), (block), 0, (stream)>>>(__VA_ARGS__);         \
        const hipError_t _e = hipGetLastError();                     \
        ::cogdl::trace_end(_slot, stream);                           \
        if (_e != hipSuccess) return COGDL_ERR_LAUNCH;               \
    } while (0)

// The same with `shm` bytes of dynamic LDS per workgroup.
#define COGDL_LAUNCH_SHM(name, kern, grid, block, shm, stream, ...)   \
    do {                                                             \
        const int _slot = ::cogdl::trace_begin(name, stream);        \
        kern<<<(grid), (block), (shm), (stream)>>>(__VA_ARGS__);     \
        const hipError_t _e = hipGetLastError();                     \
        ::cogdl::trace_end(_slot, stream);                           \
        if (_e != hipSuccess) return COGDL_ERR_LAUNCH;               \
    } while (0)

// Same for functions returning hipError_t.
#define COGDL_LAUNCH_HIP(name, kern, grid, block, stream, ...)        \
    do {                                                             \
        const int _slot = ::cogdl::trace_begin(name, stream);        \
        kern<<<(grid), (block), 0, (stream)>>>(__VA_ARGS__);         \
        const hipError_t _e = hipGetLastError();                     \
        ::cogdl::trace_end(_slot, stream);                           \
        if (_e != hipSuccess) return _e;                             \
    } while (0)

#define COGDL_HIP_TRY(expr)                                  \
    do {                                                     \
        hipError_t _e = (expr);                              \
        if (_e != hipSuccess) return COGDL_ERR_LAUNCH;       \
    } while (0)
