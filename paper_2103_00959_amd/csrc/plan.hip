// The data-aware workload balancer of section 2.2 (the "workload balance
// abstraction" listing): a preprocessing pass, run on the device, that
//   1. counts the rows whose degree is close to the average degree and picks
//      the row-split backend when at least 90% of them are, the neighbour-group
//      backend otherwise;
//   2. cuts each row into work units (one per row for row split; slices of at
//      most group_size edges for neighbour groups) and numbers the partial-sum
//      slots of rows cut into several units;
//   3. orders the units longest first (a stable sort, so equal lengths keep
//      row order) so that wavefronts sharing a workgroup get equal work and
//      the heaviest units start first.
// Every count stays on the device: no host synchronization, nothing read back
// (a column-sliced plan reads its unit totals back once, at creation, to size
// itself).
//
// Column-sliced plans (an MI355X addition, cogdl_plan_create_sliced): in
// neighbour-group mode a row with more than slice_min edges is also cut at the
// boundaries of kSlices equal column ranges, and the units form kSlices lists
// (range s in list s, every other unit in list row % kSlices), sorted by
// (list, length), each walked by the workgroups of one XCD.
#include <new>

#include "common.hpp"
#include "internal.hpp"

struct cogdl_plan {
    cogdl::Plan p;
};

namespace cogdl {
namespace {

constexpr int kPlanBlock = 256;

// Cuts of row [beg, end) (end > beg) at the column-range boundaries: cut[s]
// is the lower bound of column s * width in the row (a binary search over
// the whole row), and a running maximum keeps the cuts ordered for any column
// order: on sorted rows they are the exact boundaries, and any ordered cuts
// partition the row.  The seven searches advance in lockstep, so their loads
// are independent and a long row waits out one memory latency per halving
// instead of one per probe of each search in turn.
__device__ __forceinline__ void slice_cuts(const int32_t *__restrict__ col, int beg, int end, int64_t width,
                                           int (&cut)[kSlices + 1])
{
    int lo[kSlices - 1], hi[kSlices - 1];
#pragma unroll
    for (int s = 0; s < kSlices - 1; ++s) {
        lo[s] = beg;
        hi[s] = end;
    }
    int steps = 0;
    for (int n = end - beg; n > 0; n >>= 1) ++steps;
    for (int t = 0; t < steps; ++t) {
#pragma unroll
        for (int s = 0; s < kSlices - 1; ++s) {
            const int mid = lo[s] + ((hi[s] - lo[s]) >> 1);
            const int32_t v = col[mid < end ? mid : end - 1];
            const bool open = lo[s] < hi[s];
            const bool below = (int64_t)v < (int64_t)(s + 1) * width;
            lo[s] = (open && below) ? mid + 1 : lo[s];
            hi[s] = (open && !below) ? mid : hi[s];
        }
    }
    cut[0] = beg;
#pragma unroll
    for (int s = 0; s < kSlices - 1; ++s) cut[s + 1] = lo[s] > cut[s] ? lo[s] : cut[s];
    cut[kSlices] = end;
}

// Sums of a workgroup's rows, 8 per workgroup: the rows whose degree is close to the
// average, and the units, partial slots and split rows of the sliced (1-3; of a plain
// plan: the only) and of the unsliced neighbour groups (4-6).  k_plan_totals puts the
// sums over the workgroups before each one in 1-3.
constexpr int kPlanSums = 8;

// Per-row unit counts of the neighbour-group backend (the mode is not known yet), and
// the pad keys of the sort.  A sliced row (more than slice_min edges) gives ceil(len /
// G) units per nonempty slice, its cuts stored for k_plan_emit; alt_units keeps the
// unsliced count, which the build falls back to when the sliced totals exceed the
// plan's capacities.  With `mode` given no row is sliced when it is row split.
template <bool SLICED>
__global__ __launch_bounds__(kPlanBlock) void k_plan_counts(
    const int32_t *__restrict__ rowptr, const int32_t *__restrict__ col, int32_t n_rows, int64_t nnz, int32_t G,
    int64_t width, int32_t slice_min, const int32_t *__restrict__ mode, int32_t *__restrict__ row_units,
    int32_t *__restrict__ alt_units, int32_t *__restrict__ row_cuts, uint32_t *__restrict__ sums,
    uint32_t *__restrict__ keys, int64_t n_keys, uint32_t pad)
{
    for (int64_t k = (int64_t)blockIdx.x * kPlanBlock + threadIdx.x; k < n_keys; k += (int64_t)gridDim.x * kPlanBlock)
        keys[k] = pad;
    if (SLICED && mode && *mode == COGDL_BALANCE_ROW_SPLIT) slice_min = INT32_MAX;
    const int i = blockIdx.x * kPlanBlock + threadIdx.x;
    uint32_t v[7] = {0, 0, 0, 0, 0, 0, 0};
    if (i < n_rows) {
        const int beg = rowptr[i], end = rowptr[i + 1];
        const int d = end - beg;
        v[0] = (2 * (int64_t)d * n_rows >= nnz && (int64_t)d * n_rows <= 2 * nnz) ? 1u : 0u;
        const int alt = d > G ? ceil_div(d, G) : 1;
        int u = alt;
        if (SLICED && d > slice_min) {
            int cut[kSlices + 1];
            slice_cuts(col, beg, end, width, cut);
            u = 0;
            for (int s = 0; s < kSlices; ++s) u += ceil_div(cut[s + 1] - cut[s], G);
#pragma unroll
            for (int s = 1; s < kSlices; ++s) row_cuts[(int64_t)i * (kSlices - 1) + s - 1] = cut[s];
        }
        row_units[i] = u;
        if (SLICED) alt_units[i] = alt;
        v[1] = (uint32_t)u;
        v[2] = u > 1 ? (uint32_t)u : 0u;
        v[3] = u > 1 ? 1u : 0u;
        v[4] = (uint32_t)alt;
        v[5] = alt > 1 ? (uint32_t)alt : 0u;
        v[6] = alt > 1 ? 1u : 0u;
    }
    __shared__ uint32_t wsum[7][kPlanBlock / kWave];
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        v[c] = group_reduce(v[c], kWave, [](uint32_t a, uint32_t b) { return a + b; });
        if (lane_id() == 0) wsum[c][threadIdx.x / kWave] = v[c];
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        uint32_t s = 0;
#pragma unroll
        for (int w = 0; w < kPlanBlock / kWave; ++w) s += wsum[threadIdx.x][w];
        sums[(int64_t)blockIdx.x * kPlanSums + threadIdx.x] = s;
    }
}

// One workgroup: the totals, the mode (row split when at least 90% of the rows are close
// to the average), which counts the build uses (counters[6]: 0 the sliced ones, 1 the
// unsliced ones, 2 one unit per row), and each workgroup's first unit, partial slot and
// split row, in a fixed order.  The totals must fit the capacities the plan was
// allocated with.  They do whenever rowptr[n_rows] is the nnz given at creation; a
// rowptr with more edges would make the emit pass write past the plan's arrays, so
// instead the totals are set to zero (an empty plan, no unit runs) and counters[5] = 1,
// which cogdl_plan_query reports as COGDL_ERR_PLAN.
constexpr int kTotalsBlock = 1024;

__global__ __launch_bounds__(kTotalsBlock) void k_plan_totals(uint32_t *__restrict__ sums, int64_t n_blocks,
                                                              int32_t n_rows, int req, int sliced,
                                                              int64_t cap_units, int64_t cap_partials,
                                                              int64_t cap_split, unsigned long long *__restrict__ totals,
                                                              int32_t *__restrict__ n_units,
                                                              int32_t *__restrict__ n_parts,
                                                              int32_t *__restrict__ n_split,
                                                              int32_t *__restrict__ counters)
{
    constexpr int kWaves = kTotalsBlock / kWave;
    __shared__ unsigned long long part[7][kWaves];
    __shared__ int set_sh;
    unsigned long long t[7] = {0, 0, 0, 0, 0, 0, 0};
    for (int64_t b = threadIdx.x; b < n_blocks; b += kTotalsBlock) {
        const uint4 lo = *reinterpret_cast<const uint4 *>(sums + b * kPlanSums);
        const uint4 hi = *reinterpret_cast<const uint4 *>(sums + b * kPlanSums + 4);
        t[0] += lo.x; t[1] += lo.y; t[2] += lo.z; t[3] += lo.w;
        t[4] += hi.x; t[5] += hi.y; t[6] += hi.z;
    }
#pragma unroll
    for (int c = 0; c < 7; ++c) {
        for (int off = kWave / 2; off > 0; off >>= 1) t[c] += __shfl_xor(t[c], off);
        if (lane_id() == 0) part[c][threadIdx.x / kWave] = t[c];
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        unsigned long long sum = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) sum += part[threadIdx.x][w];
        part[threadIdx.x][0] = sum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < 7; ++c) t[c] = part[c][0];
        const int mode = req != COGDL_BALANCE_AUTO ? req
                         : 10ull * t[0] >= 9ull * (unsigned long long)n_rows ? (int)COGDL_BALANCE_ROW_SPLIT
                                                                              : (int)COGDL_BALANCE_NEIGHBOR_GROUP;
        const bool rows = mode == COGDL_BALANCE_ROW_SPLIT;
        if (rows) {
            t[1] = (unsigned long long)n_rows;
            t[2] = t[3] = 0;
        }
        if (totals) {
            totals[0] = t[1];
            totals[1] = t[2];
            totals[2] = t[3];
        }
        const auto fits = [&](int c) {
            return t[c] <= (unsigned long long)cap_units && t[c + 1] <= (unsigned long long)cap_partials &&
                   t[c + 2] <= (unsigned long long)cap_split;
        };
        int set = rows ? 2 : 0;
        int c = 1;
        if (!rows && sliced && !fits(1)) {
            set = 1;
            c = 4;
        }
        const bool ok = fits(c) && t[c] <= (unsigned long long)INT32_MAX && t[c + 1] <= (unsigned long long)INT32_MAX;
        *n_units = ok ? (int32_t)t[c] : 0;
        *n_parts = ok ? (int32_t)t[c + 1] : 0;
        *n_split = ok ? (int32_t)t[c + 2] : 0;
        counters[0] = (int32_t)t[0];
        counters[1] = mode;
        counters[2] = 0;
        counters[3] = 0;
        counters[5] = ok ? 0 : 1;
        counters[6] = set;
        set_sh = ok ? set : -1;
    }
    __syncthreads();
    const int set = set_sh;
    if (set < 0) return;
    int carry[3] = {0, 0, 0};
    for (int64_t b0 = 0; b0 < n_blocks; b0 += kTotalsBlock) {
        const int64_t b = b0 + threadIdx.x;
        const bool in = b < n_blocks;
        int x[3] = {0, 0, 0}, total[3];
        if (in && set == 2) {
            const int64_t left = n_rows - b * kPlanBlock;
            x[0] = (int)(left < kPlanBlock ? left : kPlanBlock);
        } else if (in) {
#pragma unroll
            for (int c = 0; c < 3; ++c) x[c] = (int)sums[b * kPlanSums + (set == 1 ? 4 : 1) + c];
        }
        block_exclusive_scans<3, kWaves>(x, total);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (in) sums[b * kPlanSums + 1 + c] = (uint32_t)(carry[c] + x[c]);
            carry[c] += total[c];
        }
    }
}

// The units of each row, in row order, with their sort keys: plain plans G - size
// (neighbour groups; 0 for row split); sliced plans (list << kb) | that, slice s of a
// sliced row in list s, every other unit in list row % kSlices.
template <bool SLICED>
__global__ __launch_bounds__(kPlanBlock) void k_plan_emit(
    const int32_t *__restrict__ rowptr, int32_t n_rows, int32_t G, int kb, int32_t slice_min,
    const int32_t *__restrict__ row_cuts, const int32_t *__restrict__ counters, const uint32_t *__restrict__ sums,
    const int32_t *__restrict__ row_units, const int32_t *__restrict__ alt_units, int4 *__restrict__ units_tmp,
    uint32_t *__restrict__ keys, int4 *__restrict__ split_rows, int4 *__restrict__ part_units)
{
    if (counters[5] != 0) return;
    const int i = blockIdx.x * kPlanBlock + threadIdx.x;
    const bool live = i < n_rows;
    const bool ng = counters[1] == COGDL_BALANCE_NEIGHBOR_GROUP;
    const int set = counters[6];
    const int nu = !live ? 0 : set == 2 ? 1 : (SLICED && set == 1) ? alt_units[i] : row_units[i];
    const uint32_t *first = sums + (int64_t)blockIdx.x * kPlanSums + 1;
    int at[3] = {nu, nu > 1 ? nu : 0, nu > 1 ? 1 : 0}, all[3];
    block_exclusive_scans<3>(at, all);
    if (!live) return;
    const int u0 = (int)first[0] + at[0], p0 = (int)first[1] + at[1], sidx = (int)first[2] + at[2];
    const int beg = rowptr[i], end = rowptr[i + 1];
    const int d = end - beg;
    const bool sliced_row = SLICED && set == 0 && d > slice_min;
    const uint32_t home = SLICED ? (uint32_t)(i % kSlices) << kb : 0u;
    int cut[SLICED ? kSlices + 1 : 1];
    if constexpr (SLICED) {
        if (sliced_row) {
            // the cuts the count pass found (the same for the same columns)
            cut[0] = beg;
#pragma unroll
            for (int s = 1; s < kSlices; ++s) cut[s] = row_cuts[(int64_t)i * (kSlices - 1) + s - 1];
            cut[kSlices] = end;
        }
    }
    if (nu == 1) {
        uint32_t list = home;
        if constexpr (SLICED) {
            if (sliced_row)
                for (int s = 0; s < kSlices; ++s)
                    if (cut[s + 1] > cut[s]) list = (uint32_t)s << kb;
        }
        units_tmp[u0] = make_int4(i, beg, end, -1);
        keys[u0] = list | (ng ? (uint32_t)(G - (d < G ? d : G)) : 0u);
        return;
    }
    split_rows[sidx] = make_int4(i, p0, nu, d);
    if constexpr (SLICED) {
        if (sliced_row) {
            int g = 0;
            for (int s = 0; s < kSlices; ++s) {
                for (int b = cut[s]; b < cut[s + 1]; b += G) {
                    const int e = (cut[s + 1] - b > G) ? b + G : cut[s + 1];
                    if (g < nu) {
                        units_tmp[u0 + g] = make_int4(i, b, e, p0 + g);
                        part_units[p0 + g] = make_int4(i, b, e, sidx);
                        keys[u0 + g] = ((uint32_t)s << kb) | (uint32_t)(G - (e - b));
                    }
                    ++g;
                }
            }
            return;
        }
    }
    for (int g = 0; g < nu; ++g) {
        const int b = beg + g * G;
        const int e = (end - b > G) ? b + G : end;
        units_tmp[u0 + g] = make_int4(i, b, e, p0 + g);
        part_units[p0 + g] = make_int4(i, b, e, sidx);
        keys[u0 + g] = home | (uint32_t)(G - (e - b));
    }
}

// First index of sorted[0, n) not below key, by a 64-way search of one wavefront.
__device__ __forceinline__ int32_t wave_lower_bound(const uint32_t *__restrict__ sorted, int32_t n, uint32_t key)
{
    int32_t lo = 0, hi = n;              // the answer is in [lo, hi]
    while (lo < hi) {
        const int32_t step = (hi - lo + kWave - 1) / kWave;
        const int64_t p = (int64_t)lo + (int64_t)lane_id() * step;
        // the probes below the key are a prefix of the lanes
        const int below = __popcll(__ballot(p < hi && sorted[p] < key));
        if (below == 0) return lo;
        const int64_t last = (int64_t)lo + (int64_t)(below - 1) * step;
        lo = (int32_t)last + 1;
        hi = (int32_t)(last + step < hi ? last + step : hi);
    }
    return lo;
}

// The units in sorted order, and (workgroup 0) where the sorted units split.  They are
// sorted by G - size (ascending), so the tiny ones (size <= T) form the tail of each
// list.  Plain plans: counters[2] = number of units longer than T (all of them in
// row-split mode, whose keys are all 0).  Sliced plans: for list x its first unit, the
// end of its long units (keys below (x << kb) | (G - T)) and its end; counters[2] =
// the long units of all lists.
constexpr int kFinishBlock = 1024;

__global__ __launch_bounds__(kFinishBlock) void k_plan_finish(const int4 *__restrict__ units_tmp,
                                                              const uint32_t *__restrict__ order,
                                                              const uint32_t *__restrict__ sorted,
                                                              const int32_t *__restrict__ n_units, int64_t cap,
                                                              int32_t G, int32_t T, int sliced, int kb,
                                                              int32_t *__restrict__ tbl,
                                                              int32_t *__restrict__ counters,
                                                              int4 *__restrict__ units)
{
    const int32_t n = *n_units;
    for (int64_t i = (int64_t)blockIdx.x * kFinishBlock + threadIdx.x; i < n && i < cap;
         i += (int64_t)gridDim.x * kFinishBlock)
        units[i] = units_tmp[order[i]];
    if (blockIdx.x != 0) return;
    __shared__ int32_t bound[2 * kSlices];
    const uint32_t big = G > T ? (uint32_t)(G - T) : 0u;
    const int w = threadIdx.x / kWave;
    if (!sliced) {
        if (w == 0) {
            const int32_t b = G > T ? wave_lower_bound(sorted, n, big) : n;
            if (lane_id() == 0) counters[2] = b;
        }
        return;
    }
    static_assert(kFinishBlock / kWave == 2 * kSlices, "a wavefront per bound");
    const uint32_t base = (uint32_t)(w / 2) << kb;
    const int32_t b = wave_lower_bound(sorted, n, w % 2 ? base | big : base);
    if (lane_id() == 0) bound[w] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t longs = 0;
        for (int x = 0; x < kSlices; ++x) {
            const int32_t lo = bound[2 * x], hi = x + 1 < kSlices ? bound[2 * x + 2] : n;
            const int32_t mid = G > T ? bound[2 * x + 1] : hi;
            tbl[x] = lo;
            tbl[kSlices + x] = mid;
            tbl[2 * kSlices + x] = hi;
            longs += mid - lo;
        }
        counters[2] = longs;
    }
}

__global__ void k_plan_export(const int4 *__restrict__ units, const int32_t *__restrict__ n_units,
                              int64_t capacity, int4 *__restrict__ out)
{
    const int64_t n = *n_units < capacity ? *n_units : capacity;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = units[i];
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// The row counts and totals of a rowptr (keys: the sort's keys to pad, or none).
// Searching the cuts of long rows costs more than the rest of the count, and a row-split
// plan has no use for them.  Where the mean degree is slice_min or more, the rows to cut
// can be most rows of a balanced graph, so the mode is found first, by a plain count and
// its totals (a rebuild of 200k rows of 300: 244 us with every cut searched, 79 now, 106
// before the counting passes were merged); it costs a skewed graph two launches, 11 us.
// Below, row split leaves few rows to cut in vain.
cogdl_status plan_count(Plan &P, const int32_t *rowptr, const int32_t *col, uint32_t *keys, int64_t n_keys,
                        uint32_t pad, hipStream_t s)
{
    const int n = P.n_rows;
    const unsigned blocks = (unsigned)((n + kPlanBlock - 1) / kPlanBlock);
    const auto totals = [&](int sliced) -> cogdl_status {
        COGDL_LAUNCH("plan_totals", k_plan_totals, 1, kTotalsBlock, s, P.block_sums, (int64_t)blocks, n,
                     (int)P.mode_req, sliced, P.cap_units, P.cap_partials, P.cap_split, sliced ? P.totals : nullptr,
                     P.row_units + n, P.n_parts, P.n_split, P.counters);
        return COGDL_OK;
    };
    const bool mode_first = P.sliced && P.mode_req == COGDL_BALANCE_AUTO && P.nnz >= (int64_t)P.slice_min * n;
    if (!P.sliced || mode_first) {
        COGDL_LAUNCH("plan_counts", k_plan_counts<false>, blocks, kPlanBlock, s, rowptr, nullptr, n, P.nnz,
                     P.group_size, 1, 0, nullptr, P.row_units, nullptr, nullptr, P.block_sums, keys, n_keys, pad);
        const cogdl_status st = totals(0);
        if (!P.sliced || st != COGDL_OK) return st;
        n_keys = 0;                               // padded
    }
    const int64_t width = ((int64_t)P.n_cols + kSlices - 1) / kSlices;
    // (a row-split plan asked for by the caller is never sliced)
    const int32_t slice_min = P.mode_req == COGDL_BALANCE_ROW_SPLIT ? INT32_MAX : P.slice_min;
    COGDL_LAUNCH("plan_counts", k_plan_counts<true>, blocks, kPlanBlock, s, rowptr, col, n, P.nnz, P.group_size,
                 width > 0 ? width : 1, slice_min, mode_first ? P.counters + 1 : nullptr, P.row_units, P.alt_units,
                 P.row_cuts, P.block_sums, keys, n_keys, pad);
    return totals(1);
}

// Counts, totals, units in row order, the sort by length, the sorted units: five
// launches beside the sort's three per pass (a build was 20 launches and is now 11 at
// 12 key bits; skewed graphs of 170k rows and 2.5M nonzeros, 2.4M and 100M: column-sliced
// 111 -> 70 and 361 -> 284 us, plain 79 -> 58 and 189 -> 151 us).
cogdl_status plan_build(Plan &P, const int32_t *rowptr, const int32_t *col, hipStream_t s)
{
    const int n = P.n_rows;
    const int32_t G = P.group_size;
    const int kb = P.sliced ? P.key_bits : 0;
    // Pad keys sort after every real unit; the sort covers the capacity.
    const uint32_t pad = P.sliced ? (((uint32_t)(kSlices - 1) << kb) | (uint32_t)(G + 1))
                                  : (uint32_t)G + 1u;
    if (n == 0) {
        COGDL_HIP_TRY(fill_i32(P.counters, 8, 0, s));
        COGDL_HIP_TRY(fill_i32(P.row_units, 1, 0, s));
        COGDL_HIP_TRY(fill_i32(P.n_parts, 1, 0, s));
        COGDL_HIP_TRY(fill_i32(P.n_split, 1, 0, s));
        if (P.sliced) COGDL_HIP_TRY(fill_i32(P.lists_tbl, 3 * kSlices, 0, s));
        return COGDL_OK;
    }
    const unsigned blocks = (unsigned)((n + kPlanBlock - 1) / kPlanBlock);
    const cogdl_status st = plan_count(P, rowptr, col, P.sort_keys, P.cap_units, pad, s);
    if (st != COGDL_OK) return st;
    if (P.sliced)
        COGDL_LAUNCH("plan_emit", k_plan_emit<true>, blocks, kPlanBlock, s, rowptr, n, G, kb, P.slice_min,
                     P.row_cuts, P.counters, P.block_sums, P.row_units, P.alt_units, P.units_tmp, P.sort_keys,
                     P.split_rows, P.part_units);
    else
        COGDL_LAUNCH("plan_emit", k_plan_emit<false>, blocks, kPlanBlock, s, rowptr, n, G, 0, 0, nullptr,
                     P.counters, P.block_sums, P.row_units, nullptr, P.units_tmp, P.sort_keys, P.split_rows,
                     P.part_units);
    uint32_t *order = P.sort_vals;                    // [cap]: final order
    uint32_t *ping_k = P.sort_keys + P.cap_units;     // [2 * cap] ping buffers
    uint32_t *ping_v = P.sort_vals + P.cap_units;
    uint32_t *sorted = P.sort_keys + 3 * P.cap_units; // [cap] keys in execution order
    const int bits = bits_for(pad);
    COGDL_HIP_TRY(radix_sort_pairs(P.sort_keys, nullptr, sorted, order, P.cap_units, bits, ping_k,
                                   ping_v, P.sort_ws, s));
    const int64_t gb = (P.cap_units + kFinishBlock - 1) / kFinishBlock;
    COGDL_LAUNCH("plan_finish", k_plan_finish, (unsigned)(gb < 2048 ? gb : 2048), kFinishBlock, s, P.units_tmp,
                 order, sorted, P.n_units_dev(), P.cap_units, G, kTinyUnit, (int)P.sliced, kb, P.lists_tbl,
                 P.counters, P.units);
    return COGDL_OK;
}

}  // namespace
}  // namespace cogdl

using cogdl::Plan;

extern "C" {

const char *cogdl_status_string(cogdl_status s)
{
    switch (s) {
    case COGDL_OK: return "ok";
    case COGDL_ERR_INVALID: return "invalid argument";
    case COGDL_ERR_DTYPE: return "unsupported dtype";
    case COGDL_ERR_PLAN: return "plan does not match the call";
    case COGDL_ERR_NOMEM: return "device allocation failed";
    case COGDL_ERR_LAUNCH: return "kernel launch or HIP call failed";
    case COGDL_ERR_TOO_LARGE: return "size exceeds a limit of the call (int32 indices, or the static scratch of the allocation-free transpose)";
    }
    return "unknown status";
}

int32_t cogdl_version(void) { return 100; }

}  // extern "C"

namespace cogdl {
namespace {

cogdl_status plan_args(int32_t n_rows, int64_t nnz, const int32_t *rowptr, int32_t max_feat,
                       int32_t max_heads, cogdl_balance mode, int32_t group_size)
{
    if (n_rows < 0 || nnz < 0 || max_feat < 1 || max_heads < 0 || max_heads > COGDL_MAX_HEADS ||
        group_size < 0 || (n_rows > 0 && !rowptr) ||
        (mode != COGDL_BALANCE_AUTO && mode != COGDL_BALANCE_ROW_SPLIT &&
         mode != COGDL_BALANCE_NEIGHBOR_GROUP))
        return COGDL_ERR_INVALID;
    if (nnz > COGDL_MAX_NNZ || n_rows == INT32_MAX) return COGDL_ERR_TOO_LARGE;
    if (n_rows == 0 && nnz != 0) return COGDL_ERR_INVALID;
    return COGDL_OK;
}

int32_t default_group(int32_t group_size, int64_t nnz)
{
    int32_t G = group_size;
    if (G == 0) {
        G = 256;
        while (G < 4096 && (int64_t)G * 2 * 16384 <= nnz) G *= 2;
    }
    return G;
}

// The per-row arrays, counters and workgroup sums: in the main allocation of
// a plain plan, in base2 of a sliced one (which also holds the unsliced
// counts and the list table), allocated first so that the creation can size
// the rest from the sliced totals.
size_t row_layout(Plan &P, char *b, bool assign)
{
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    const size_t rows = 4 * ((size_t)P.n_rows + 1);
    const size_t o_row_units = take(rows);
    const size_t o_counters = take(4 * 16);
    const size_t o_sums = take(4 * kPlanSums * (((size_t)P.n_rows + kPlanBlock - 1) / kPlanBlock + 1));
    size_t o_alt = 0, o_tbl = 0, o_cuts = 0, o_tot = 0;
    if (P.sliced) {
        o_alt = take(rows);
        o_tbl = take(4 * 3 * kSlices);
        o_cuts = take(4 * (kSlices - 1) * (size_t)P.n_rows);
        o_tot = take(8 * 3);
    }
    if (assign) {
        P.row_units = reinterpret_cast<int32_t *>(b + o_row_units);
        P.counters = reinterpret_cast<int32_t *>(b + o_counters);
        P.n_parts = P.counters + 8;
        P.n_split = P.counters + 9;
        P.block_sums = reinterpret_cast<uint32_t *>(b + o_sums);
        if (P.sliced) {
            P.alt_units = reinterpret_cast<int32_t *>(b + o_alt);
            P.lists_tbl = reinterpret_cast<int32_t *>(b + o_tbl);
            P.row_cuts = reinterpret_cast<int32_t *>(b + o_cuts);
            P.totals = reinterpret_cast<unsigned long long *>(b + o_tot);
        }
    }
    return off;
}

// The main allocation, sized by the capacities (with the row arrays unless the
// plan is sliced).
cogdl_status plan_alloc(Plan &P)
{
    const int64_t pstride = (P.max_feat + 7) / 8 * 8;
    size_t off = P.sliced ? 0 : row_layout(P, nullptr, false);
    auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
    const size_t o_units = take(sizeof(int4) * P.cap_units);
    const size_t o_units_tmp = take(sizeof(int4) * P.cap_units);
    const size_t o_split = take(sizeof(int4) * P.cap_split);
    const size_t o_part_units = take(sizeof(int4) * P.cap_partials);
    const size_t o_keys = take(4 * 4 * (size_t)P.cap_units);
    const size_t o_vals = take(4 * 3 * (size_t)P.cap_units);
    P.sort_ws_bytes = radix_workspace_bytes(P.cap_units);
    const size_t o_sort_ws = take(P.sort_ws_bytes);
    const size_t o_partials = take(sizeof(float) * (size_t)P.cap_partials * pstride);
    const size_t o_parg = take(sizeof(int32_t) * (size_t)P.cap_partials * pstride);
    const size_t o_gstats = take(sizeof(float) * 2 * (size_t)P.cap_partials * P.max_heads);
    const size_t o_rstats = take(sizeof(float) * 2 * (size_t)P.cap_split * P.max_heads);
    P.bytes = off;
    if (hipMalloc(&P.base, P.bytes) != hipSuccess) {
        (void)hipGetLastError();
        P.base = nullptr;
        return COGDL_ERR_NOMEM;
    }
    char *b = static_cast<char *>(P.base);
    if (!P.sliced) row_layout(P, b, true);
    P.units = reinterpret_cast<int4 *>(b + o_units);
    P.units_tmp = reinterpret_cast<int4 *>(b + o_units_tmp);
    P.split_rows = reinterpret_cast<int4 *>(b + o_split);
    P.part_units = reinterpret_cast<int4 *>(b + o_part_units);
    P.sort_keys = reinterpret_cast<uint32_t *>(b + o_keys);
    P.sort_vals = reinterpret_cast<uint32_t *>(b + o_vals);
    P.sort_ws = b + o_sort_ws;
    P.partials = reinterpret_cast<float *>(b + o_partials);
    P.parg = reinterpret_cast<int32_t *>(b + o_parg);
    P.gstats = reinterpret_cast<float *>(b + o_gstats);
    P.rstats = reinterpret_cast<float *>(b + o_rstats);
    return COGDL_OK;
}

void plan_free(cogdl_plan *h)
{
    (void)hipDeviceSynchronize();
    if (h->p.base) (void)hipFree(h->p.base);
    if (h->p.base2) (void)hipFree(h->p.base2);
    delete h;
}

}  // namespace
}  // namespace cogdl

extern "C" {

cogdl_status cogdl_plan_create(int32_t n_rows, int64_t nnz, const int32_t *rowptr, int32_t max_feat,
                               int32_t max_heads, cogdl_balance mode, int32_t group_size,
                               hipStream_t stream, cogdl_plan **out)
{
    if (!out) return COGDL_ERR_INVALID;
    const cogdl_status va = cogdl::plan_args(n_rows, nnz, rowptr, max_feat, max_heads, mode, group_size);
    if (va != COGDL_OK) return va;
    const int32_t G = cogdl::default_group(group_size, nnz);

    cogdl_plan *h = new (std::nothrow) cogdl_plan;
    if (!h) return COGDL_ERR_NOMEM;
    Plan &P = h->p;
    P.n_rows = n_rows;
    P.nnz = nnz;
    P.group_size = G;
    P.max_feat = max_feat;
    P.max_heads = max_heads;
    P.mode_req = mode;
    if (hipGetDevice(&P.device) != hipSuccess) { delete h; return COGDL_ERR_LAUNCH; }
    P.cap_units = (int64_t)n_rows + nnz / G + 1;
    P.cap_split = nnz / G + 1;
    P.cap_partials = 2 * (nnz / G) + 2;
    if (cogdl::plan_alloc(P) != COGDL_OK) { delete h; return COGDL_ERR_NOMEM; }

    cogdl_status st = cogdl::plan_build(P, rowptr, nullptr, stream);
    if (st != COGDL_OK) {
        cogdl::plan_free(h);
        return st;
    }
    *out = h;
    return COGDL_OK;
}

cogdl_status cogdl_plan_create_sliced(int32_t n_rows, int64_t nnz, const int32_t *rowptr,
                                      const int32_t *col, int32_t n_cols, int32_t max_feat,
                                      int32_t max_heads, cogdl_balance mode, int32_t group_size,
                                      int32_t slice_min, hipStream_t stream, cogdl_plan **out)
{
    if (!out) return COGDL_ERR_INVALID;
    const cogdl_status va = cogdl::plan_args(n_rows, nnz, rowptr, max_feat, max_heads, mode, group_size);
    if (va != COGDL_OK) return va;
    if (n_cols < 0 || slice_min < 0 || (nnz > 0 && (!col || n_cols < 1)) || group_size > (1 << 24))
        return COGDL_ERR_INVALID;
    const int32_t G = cogdl::default_group(group_size, nnz);

    cogdl_plan *h = new (std::nothrow) cogdl_plan;
    if (!h) return COGDL_ERR_NOMEM;
    Plan &P = h->p;
    P.n_rows = n_rows;
    P.nnz = nnz;
    P.group_size = G;
    P.max_feat = max_feat;
    P.max_heads = max_heads;
    P.mode_req = mode;
    P.sliced = 1;
    P.n_cols = n_cols;
    P.slice_min = slice_min > 0 ? slice_min : COGDL_DEFAULT_SLICE_MIN;
    P.key_bits = cogdl::bits_for((uint64_t)G + 1);
    if (hipGetDevice(&P.device) != hipSuccess) { delete h; return COGDL_ERR_LAUNCH; }
    const size_t rows_bytes = cogdl::row_layout(P, nullptr, false);
    if (hipMalloc(&P.base2, rows_bytes) != hipSuccess) {
        (void)hipGetLastError();
        delete h;
        return COGDL_ERR_NOMEM;
    }
    cogdl::row_layout(P, static_cast<char *>(P.base2), true);
    // Capacities: the unsliced bounds, raised to the sliced totals of this
    // graph (counted here, the one host read-back of the plan); a rebuild on
    // a graph whose sliced totals exceed them falls back to unsliced units.
    P.cap_units = (int64_t)n_rows + nnz / G + 1;
    P.cap_split = nnz / G + 1;
    P.cap_partials = 2 * (nnz / G) + 2;
    if (n_rows > 0) {
        unsigned long long tot[3] = {0, 0, 0};
        cogdl_status st = cogdl::plan_count(P, rowptr, col, nullptr, 0, 0, stream);
        if (st == COGDL_OK &&
            (hipMemcpyAsync(&tot[0], P.totals, sizeof(tot), hipMemcpyDeviceToHost, stream) != hipSuccess ||
             hipStreamSynchronize(stream) != hipSuccess))
            st = COGDL_ERR_LAUNCH;
        if (st != COGDL_OK) {
            cogdl::plan_free(h);
            return st;
        }
        if ((int64_t)tot[0] + 1 > P.cap_units) P.cap_units = (int64_t)tot[0] + 1;
        if ((int64_t)tot[1] + 2 > P.cap_partials) P.cap_partials = (int64_t)tot[1] + 2;
        if ((int64_t)tot[2] + 1 > P.cap_split) P.cap_split = (int64_t)tot[2] + 1;
    }
    if (cogdl::plan_alloc(P) != COGDL_OK) {
        cogdl::plan_free(h);
        return COGDL_ERR_NOMEM;
    }
    P.bytes += rows_bytes;                 // both allocations, as cogdl_plan_query reports them
    cogdl_status st = cogdl::plan_build(P, rowptr, col, stream);
    if (st != COGDL_OK) {
        cogdl::plan_free(h);
        return st;
    }
    *out = h;
    return COGDL_OK;
}

cogdl_status cogdl_plan_rebuild(cogdl_plan *plan, const int32_t *rowptr, hipStream_t stream)
{
    if (!plan || plan->p.sliced || (plan->p.n_rows > 0 && !rowptr)) return COGDL_ERR_INVALID;
    return cogdl::plan_build(plan->p, rowptr, nullptr, stream);
}

cogdl_status cogdl_plan_rebuild_sliced(cogdl_plan *plan, const int32_t *rowptr, const int32_t *col,
                                       hipStream_t stream)
{
    if (!plan || !plan->p.sliced || (plan->p.n_rows > 0 && !rowptr) || (plan->p.nnz > 0 && !col))
        return COGDL_ERR_INVALID;
    return cogdl::plan_build(plan->p, rowptr, col, stream);
}

cogdl_status cogdl_plan_destroy(cogdl_plan *plan)
{
    if (!plan) return COGDL_OK;
    cogdl_status st = COGDL_OK;
    if (hipDeviceSynchronize() != hipSuccess) st = COGDL_ERR_LAUNCH;
    if (hipFree(plan->p.base) != hipSuccess) st = COGDL_ERR_LAUNCH;
    if (plan->p.base2 && hipFree(plan->p.base2) != hipSuccess) st = COGDL_ERR_LAUNCH;
    delete plan;
    return st;
}

cogdl_status cogdl_plan_query(const cogdl_plan *plan, hipStream_t stream, cogdl_plan_info *info)
{
    if (!plan || !info) return COGDL_ERR_INVALID;
    const Plan &P = plan->p;
    int32_t v[6] = {0, 0, 0, 0, 0, 0};
    COGDL_HIP_TRY(hipMemcpyAsync(&v[0], P.n_units_dev(), 4, hipMemcpyDeviceToHost, stream));
    COGDL_HIP_TRY(hipMemcpyAsync(&v[1], P.n_split_dev(), 4, hipMemcpyDeviceToHost, stream));
    COGDL_HIP_TRY(hipMemcpyAsync(&v[2], P.n_parts_dev(), 4, hipMemcpyDeviceToHost, stream));
    COGDL_HIP_TRY(hipMemcpyAsync(&v[3], P.counters + 1, 4, hipMemcpyDeviceToHost, stream));
    COGDL_HIP_TRY(hipMemcpyAsync(&v[4], P.counters + 2, 4, hipMemcpyDeviceToHost, stream));
    COGDL_HIP_TRY(hipMemcpyAsync(&v[5], P.counters + 5, 4, hipMemcpyDeviceToHost, stream));
    COGDL_HIP_TRY(hipStreamSynchronize(stream));
    info->n_rows = P.n_rows;
    info->nnz = P.nnz;
    info->group_size = P.group_size;
    info->max_feat = P.max_feat;
    info->max_heads = P.max_heads;
    info->n_units = v[0];
    info->n_long_units = v[4];
    info->n_split_rows = v[1];
    info->n_partials = v[2];
    info->mode = P.n_rows == 0 ? (P.mode_req == COGDL_BALANCE_AUTO ? COGDL_BALANCE_ROW_SPLIT
                                                                     : (int32_t)P.mode_req)
                               : v[3];
    info->device_bytes = (int64_t)P.bytes;
    // the last build's rowptr held more edges than the plan was created for:
    // the plan was left empty (see k_plan_totals)
    return (P.n_rows > 0 && v[5] != 0) ? COGDL_ERR_PLAN : COGDL_OK;
}

cogdl_status cogdl_plan_units(const cogdl_plan *plan, int32_t *units, int64_t capacity,
                              hipStream_t stream)
{
    if (!plan || capacity < 0 || (capacity > 0 && !units)) return COGDL_ERR_INVALID;
    if (capacity == 0) return COGDL_OK;
    const Plan &P = plan->p;
    const int64_t cap = capacity < P.cap_units ? capacity : P.cap_units;
    const int64_t gb = (cap + 255) / 256;
    COGDL_LAUNCH("plan_export", cogdl::k_plan_export, (unsigned)(gb < 4096 ? gb : 4096), 256,
                 stream, P.units, P.n_units_dev(), cap, reinterpret_cast<int4 *>(units));
    return COGDL_OK;
}

}  // extern "C"

namespace cogdl {
const Plan *plan_of(const cogdl_plan *h) { return h ? &h->p : nullptr; }
}  // namespace cogdl
