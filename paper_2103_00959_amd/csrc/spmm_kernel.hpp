// The gather kernel of the generalized SpMM (section 2.2, Eq. 1), shared by
// the translation units that instantiate its variants: spmm.hip (sum of
// products, the hot path) and gspmm.hip (max, and the add / subtract
// messages).  See spmm.hip for the mapping onto gfx950.
#pragma once

#include "common.hpp"
#include "internal.hpp"

namespace cogdl {

constexpr int kSpmmBlock = 256;

struct SpmmArgs {
    const int4 *units;          // nullptr: one unit per row in row order
    const int32_t *u_lo;        // with units: this launch runs units [*u_lo, *u_hi)
    const int32_t *u_hi;        // (lists > 1: list x is [u_lo[x], u_hi[x]), see unit_walk)
    int32_t lists = 1;
    int32_t n_rows;
    const int32_t *rowptr;
    const int32_t *col;
    const float *val;           // nullptr: all ones
    const void *X;
    void *Y;
    int32_t *arg;               // max: edge id of each output maximum (nullable)
    float *partials;
    int32_t *parg;              // max: edge id of each partial maximum
    int64_t pstride;
    int64_t F;
    uint64_t x_bytes;           // size of X, bounds the buffer gathers
    int32_t slab;
    int32_t log2S;
    int32_t mean;               // sum / mean: divide whole rows by their degree
    float bsign;                // ADDOP: message x + bsign * val (+1 add, -1 subtract)
    const float *bias;          // epilogue: Y = act(reduced + bias), bias nullable
    int32_t act;
};

// Descriptor {row, first edge, end edge, partial slot} of unit u (an empty
// unit past the end, so prefetching one unit ahead needs no branch around it).
__device__ __forceinline__ int4 fetch_unit(const SpmmArgs &a, int64_t u, int64_t hi)
{
    if (u >= hi) return make_int4(0, 0, 0, -1);
    if (a.units) return a.units[u];
    const int r = (int)u;
    return make_int4(r, a.rowptr[r], a.rowptr[r + 1], -1);
}

// Stores N edge ids (16-byte stores when N is a multiple of four).
typedef int32_t i32x4_u __attribute__((ext_vector_type(4), aligned(4)));

template <int N>
__device__ __forceinline__ void store_ids(int32_t *__restrict__ p, int64_t i, const int32_t (&v)[N])
{
    if constexpr (N % 4 == 0) {
#pragma unroll
        for (int e = 0; e < N; e += 4)
            *reinterpret_cast<i32x4_u *>(p + i + e) = i32x4_u{v[e], v[e + 1], v[e + 2], v[e + 3]};
    } else {
#pragma unroll
        for (int e = 0; e < N; ++e) p[i + e] = v[e];
    }
}

// The message of edge k is val[k] * x (ADDOP = false; copy is val = 1) or
// x + bsign * val[k] (ADDOP = true: add, subtract).
// MAXR = false: sum of the messages (mean scales whole rows by 1 / degree);
// MAXR = true: maximum of the messages, each rounded once to fp32, edges
// taken in CSR order, the first edge kept unconditionally and a later one
// only if strictly greater, so the recorded edge is the first that attains
// the maximum.
template <typename TX, typename TY, int VEC, int CH, bool BUF, bool MAXR, bool ADDOP>
__global__ __launch_bounds__(kSpmmBlock) void k_spmm(SpmmArgs a)
{
    constexpr int U = (VEC == 1 ? 16 : 8) / CH;
    constexpr int AC = MAXR ? CH : 1;
    constexpr int AV = MAXR ? VEC : 1;
    const int log2S = a.log2S;
    const int S = 1 << log2S;
    const int lane = lane_id();
    const int lig = lane & (S - 1);
    const int gbase = lane & ~(S - 1);
    const UnitWalk walk = unit_walk(a.units != nullptr, a.u_lo, a.u_hi, a.lists, a.n_rows,
                                    kSpmmBlock >> log2S, threadIdx.x >> log2S);
    const int64_t stride = walk.step;
    const int64_t hi = walk.end;

    const int64_t f0 = (int64_t)blockIdx.y * a.slab;
    const int64_t f_end = (f0 + a.slab < a.F) ? f0 + a.slab : a.F;
    int64_t fe[CH];
    bool act[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        fe[c] = f0 + (int64_t)(c * S + lig) * VEC;
        act[c] = fe[c] < f_end;
        // A row that is no whole number of vectors ends with one moved back to its last
        // VEC features: the overlapped ones are summed twice, in the same order, and
        // stored twice with the same bits, so no lane needs a tail.  Against one element
        // per lane, which rows off 16-byte boundaries ran before: 64.3M edges of 41 bf16
        // classes 1.71 -> 1.25 ms, mean and max over 2.5M edges of 300 bf16 0.70 -> 0.56 ms.
        if (act[c] && fe[c] + VEC > a.F) fe[c] = a.F - VEC;
    }
    const RowGather<TX, VEC, BUF> X(a.X, a.x_bytes);
    const int32_t *__restrict__ col = a.col;
    const float *__restrict__ val = a.val;

    // Resident grid: sub-group i of a list runs its units i, i + stride, ...;
    // the units are sorted by length, so neighbouring sub-groups get equal work.
    // The loop is software-pipelined: the next unit's descriptor is fetched
    // when a unit starts and its first index chunk before the current output
    // is stored, so short units do not pay three dependent memory trips each.
    int64_t u = walk.first;
    if (u >= hi) return;
    int4 d = fetch_unit(a, u, hi);
    int c_cur = 0;
    float v_cur = 0.f;
    if (d.z > d.y) {
        // index loads are clamped to the unit's last edge instead of masked:
        // no branch, and lanes past the end are never read back
        const int k = d.y + lig < d.z - 1 ? d.y + lig : d.z - 1;
        c_cur = col[k];
        v_cur = val ? val[k] : 1.f;
    }
    for (;;) {
        const int64_t un = u + stride;
        const int4 dn = fetch_unit(a, un, hi);
        const int row = d.x, beg = d.y, end = d.z, part = d.w;
        float acc[CH][VEC];
        int32_t am[AC][AV];
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[c][e] = 0.f;
#pragma unroll
        for (int c = 0; c < AC; ++c)
#pragma unroll
            for (int e = 0; e < AV; ++e) am[c][e] = -1;

        const int last = end - 1;
        for (int k0 = beg; k0 < end; k0 += S) {
            const int n = (end - k0 < S) ? end - k0 : S;
            const int k = k0 + S + lig < last ? k0 + S + lig : last;
            const int c_nxt = col[k];
            const float v_nxt = val ? val[k] : 1.f;
            for (int j = 0; j < n; j += U) {
                int cc[U];
                float vv[U];
                bool ok[U];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    ok[t] = j + t < n;
                    const int src = gbase + (ok[t] ? j + t : j);
                    cc[t] = lane_bcast(c_cur, src);
                    vv[t] = lane_bcast(v_cur, src);
                    // a masked slot must add nothing: its gathered x is 0, so its w is too
                    if constexpr (ADDOP) vv[t] = ok[t] ? vv[t] * a.bsign : 0.f;
                }
                float xv[U][CH][VEC];
#pragma unroll
                for (int t = 0; t < U; ++t)
#pragma unroll
                    for (int c = 0; c < CH; ++c)
                        X.load((int64_t)cc[t] * a.F + fe[c], ok[t] && act[c], xv[t][c]);
                if constexpr (MAXR) {
#pragma unroll
                    for (int t = 0; t < U; ++t)
#pragma unroll
                        for (int c = 0; c < CH; ++c)
#pragma unroll
                            for (int e = 0; e < VEC; ++e) {
                                const float p = ADDOP ? xv[t][c][e] + vv[t] : vv[t] * xv[t][c][e];
                                const bool take = ok[t] && (am[c][e] < 0 || p > acc[c][e]);
                                acc[c][e] = take ? p : acc[c][e];
                                am[c][e] = take ? k0 + j + t : am[c][e];
                            }
                } else {
#pragma unroll
                    for (int t = 0; t < U; ++t)
#pragma unroll
                        for (int c = 0; c < CH; ++c)
#pragma unroll
                            for (int e = 0; e < VEC; ++e) {
                                if constexpr (ADDOP) acc[c][e] += xv[t][c][e] + vv[t];
                                else acc[c][e] = fmaf(vv[t], xv[t][c][e], acc[c][e]);
                            }
                }
            }
            c_cur = c_nxt;
            v_cur = v_nxt;
        }

        // first index chunk of the next unit, issued before this unit's stores
        if (dn.z > dn.y) {
            const int k = dn.y + lig < dn.z - 1 ? dn.y + lig : dn.z - 1;
            c_cur = col[k];
            v_cur = val ? val[k] : 1.f;
        }
        if (part < 0) {
            TY *__restrict__ Y = static_cast<TY *>(a.Y);
            if (!MAXR && a.mean && end > beg) {
                const float r = 1.f / (float)(end - beg);
#pragma unroll
                for (int c = 0; c < CH; ++c)
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[c][e] *= r;
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (!act[c]) continue;
                epilogue<VEC>(acc[c], a.bias, a.act, fe[c]);
                store_out<TY, VEC>(Y, (int64_t)row * a.F + fe[c], acc[c]);
                if constexpr (MAXR) {
                    if (a.arg) store_ids<VEC>(a.arg, (int64_t)row * a.F + fe[c], am[c]);
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                if (!act[c]) continue;
                store_vec<float, VEC>(a.partials, (int64_t)part * a.pstride + fe[c], acc[c]);
                if constexpr (MAXR)
                    store_ids<VEC>(a.parg, (int64_t)part * a.pstride + fe[c], am[c]);
            }
        }
        if (un >= hi) break;
        u = un;
        d = dn;
    }
}

// Sum of products for rows of at most four vectors (LQ = 1, 2 or 4 lanes): a group of
// S = 8 lanes per unit takes 8 / LQ edges side by side (lane = edge slot * LQ + vector
// of the row) and adds the slots' sums across lanes at the unit's end.  One LQ-lane
// group per unit instead would have LQ of every 8 gather slots filled (a chunk of
// indices is one per lane).  R chunks of 8 edges per step: R * LQ gathers in flight a
// lane.  Bound by the rate of random lines (about 70 G/s): 45M edges, both directions,
// 8 / 16 / 32 bf16 features 6.9 / 3.4 / 2.0 -> 1.2 / 1.3 / 1.5 ms, 2M edges
// 0.53 / 0.28 / 0.16 -> 0.065 / 0.071 / 0.097 ms.
template <typename TX, typename TY, int VEC, int LQ, int R>
__global__ __launch_bounds__(kSpmmBlock) void k_spmm_narrow(SpmmArgs a)
{
    constexpr int S = 8, EP = S / LQ, U = LQ * R;
    const int lane = lane_id();
    const int lig = lane & (S - 1);
    const int gbase = lane & ~(S - 1);
    const int q = lig & (LQ - 1), slot = lig / LQ;
    const UnitWalk walk = unit_walk(a.units != nullptr, a.u_lo, a.u_hi, a.lists, a.n_rows, kSpmmBlock / S,
                                    threadIdx.x / S);
    const int64_t stride = walk.step;
    const int64_t hi = walk.end;
    int64_t fe = (int64_t)q * VEC;
    const bool act = fe < a.F;
    if (act && fe + VEC > a.F) fe = a.F - VEC;       // the row's last vector (see k_spmm)
    const RowGather<TX, VEC, true> X(a.X, a.x_bytes);
    const uint32_t row_bytes = (uint32_t)a.F * (uint32_t)sizeof(TX);
    const uint32_t lane_off = act ? (uint32_t)fe * (uint32_t)sizeof(TX) : 0u;
    const uint32_t lane_min = act ? 0u : kMaskedOffset;
    const auto fetch_index = [&](int k, int end, uint32_t (&o)[R], float (&v)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int kc = k + r * S + lig < end ? k + r * S + lig : end - 1;
            o[r] = (uint32_t)a.col[kc];
            v[r] = a.val ? a.val[kc] : 1.f;
        }
    };
    int64_t u = walk.first;
    if (u >= hi) return;
    int4 d = fetch_unit(a, u, hi);
    uint32_t o_cur[R];
    float v_cur[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { o_cur[r] = 0u; v_cur[r] = 0.f; }
    if (d.z > d.y) fetch_index(d.y, d.z, o_cur, v_cur);
    for (;;) {
        const int64_t un = u + stride;
        const int4 dn = fetch_unit(a, un, hi);
        const int row = d.x, beg = d.y, end = d.z, part = d.w;
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
        for (int k0 = beg; k0 < end; k0 += R * S) {
            // row offsets of the chunk (edges past the unit: past the buffer, weight 0)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool in = k0 + r * S + lig < end;
                o_cur[r] = in ? o_cur[r] * row_bytes : kMaskedOffset;
                v_cur[r] = in ? v_cur[r] : 0.f;
            }
            uint32_t o_nxt[R];
            float v_nxt[R];
            fetch_index(k0 + R * S, end, o_nxt, v_nxt);
            float xv[U][VEC], vv[U];
#pragma unroll
            for (int t = 0; t < U; ++t) {
                const int src = gbase + (t % LQ) * EP + slot;
                const uint32_t off = (uint32_t)lane_bcast((int)o_cur[t / LQ], src) + lane_off;
                vv[t] = lane_bcast(v_cur[t / LQ], src);
                X.load_off(off > lane_min ? off : lane_min, xv[t]);
            }
#pragma unroll
            for (int t = 0; t < U; ++t)
#pragma unroll
                for (int e = 0; e < VEC; ++e) acc[e] = fmaf(vv[t], xv[t][e], acc[e]);
#pragma unroll
            for (int r = 0; r < R; ++r) { o_cur[r] = o_nxt[r]; v_cur[r] = v_nxt[r]; }
        }
        if (dn.z > dn.y) fetch_index(dn.y, dn.z, o_cur, v_cur);
        // the edge slots' sums: lanes with the same vector of the row
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if constexpr (LQ == 1) acc[e] += bfly_partner<1>(acc[e]);
            if constexpr (LQ <= 2) acc[e] += bfly_partner<2>(acc[e]);
            acc[e] += __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(acc[e]), 0x101F));   // lane ^ 4
        }
        if (slot == 0 && act) {
            if (part < 0) {
                if (a.mean && end > beg) {
                    const float r = 1.f / (float)(end - beg);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] *= r;
                }
                epilogue<VEC>(acc, a.bias, a.act, fe);
                store_out<TY, VEC>(static_cast<TY *>(a.Y), (int64_t)row * a.F + fe, acc);
            } else {
                store_vec<float, VEC>(a.partials, (int64_t)part * a.pstride + fe, acc);
            }
        }
        if (un >= hi) break;
        u = un;
        d = dn;
    }
}

// Sum of products with a wavefront per unit, for graphs of few units (unit_per_wave): there
// a call takes as long as its longest unit, a chain of batches of gathers, one memory
// latency each, so the wavefront's 64 / 2^log2S edge slots (lane = slot * 2^log2S +
// vector of the row) take the unit's edges side by side, up to 8 gathers in flight a lane
// (as many as the unit still has edges for), and their sums are added across lanes at the
// end.  Rows of one slab and one chunk per lane.  Short units are bound by the trips to
// descriptor, indices and rows, so the first two are fetched ahead: 50k rows of 5 edges,
// 64 / 128 bf16, 31 / 30 us with every trip in turn, 23 / 20 now; 12k rows and 100k edges
// without a plan, 256 bf16, 66 and 54, 10k and 1M 152 and 125.
// NARROW: fewer than 8 lanes a row, whose steps of 8 edges a slot can pass the chunk's end.
template <typename TX, typename TY, int VEC, bool NARROW>
__global__ __launch_bounds__(kSpmmBlock) void k_spmm_wave(SpmmArgs a)
{
    constexpr int U = 8;
    const int lane = lane_id();
    const int LQ = 1 << a.log2S, EP = kWave >> a.log2S;
    const int q = lane & (LQ - 1), slot = lane >> a.log2S;
    const UnitWalk walk = unit_walk(a.units != nullptr, a.u_lo, a.u_hi, a.lists, a.n_rows, kSpmmBlock / kWave,
                                    threadIdx.x / kWave);
    const int64_t hi = walk.end;
    int64_t fe = (int64_t)q * VEC;
    const bool act = fe < a.F;
    if (act && fe + VEC > a.F) fe = a.F - VEC;       // the row's last vector (see k_spmm)
    const RowGather<TX, VEC, true> X(a.X, a.x_bytes);
    const uint32_t row_bytes = (uint32_t)a.F * (uint32_t)sizeof(TX);
    const uint32_t lane_off = act ? (uint32_t)fe * (uint32_t)sizeof(TX) : 0u;
    const uint32_t lane_min = act ? 0u : kMaskedOffset;
    // (software-pipelined as k_spmm: descriptors a unit ahead, indices a chunk ahead)
    int64_t u = walk.first;
    if (u >= hi) return;
    int4 d = fetch_unit(a, u, hi);
    uint32_t c_nxt = 0u;
    float v_nxt = 0.f;
    const auto fetch_index = [&](int k0, int end) {
        const int k = k0 + lane < end ? k0 + lane : end - 1;
        c_nxt = (uint32_t)a.col[k];
        v_nxt = a.val ? a.val[k] : 1.f;
    };
    if (d.z > d.y) fetch_index(d.y, d.z);
    for (;;) {
        const int64_t un = u + walk.step;
        const int4 dn = fetch_unit(a, un, hi);
        const int row = d.x, beg = d.y, end = d.z, part = d.w;
        float acc[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
        for (int k0 = beg; k0 < end; k0 += kWave) {
            const int n = (end - k0 < kWave) ? end - k0 : kWave;
            // row offset and weight of edge k0 + lane (past the unit: past the buffer, 0)
            const uint32_t o_cur = lane < n ? c_nxt * row_bytes : kMaskedOffset;
            const float v_cur = lane < n ? v_nxt : 0.f;
            if (k0 + kWave < end) fetch_index(k0 + kWave, end);
            // UU EP edges from edge j of the chunk on
            const auto batch = [&](auto uu, int j) {
                constexpr int UU = decltype(uu)::value;
                // (16-bit rows stay packed until used: 8 vectors in 32 registers)
                constexpr bool PACKED = sizeof(TX) == 2 && VEC == 8;
                float xv[PACKED ? 1 : UU][VEC], vv[UU];
                uint4 xw[PACKED ? UU : 1];
#pragma unroll
                for (int t = 0; t < UU; ++t) {
                    const int src = j + t * EP + slot;
                    const bool inside = !NARROW || src < kWave;
                    const uint32_t o = (uint32_t)lane_bcast((int)o_cur, src);
                    const uint32_t off = (inside ? o : kMaskedOffset) + lane_off;
                    const float v = lane_bcast(v_cur, src);
                    vv[t] = inside ? v : 0.f;
                    if constexpr (PACKED) xw[t] = X.load_raw16_off(off > lane_min ? off : lane_min);
                    else X.load_off(off > lane_min ? off : lane_min, xv[t]);
                }
#pragma unroll
                for (int t = 0; t < UU; ++t) {
                    float (&x)[VEC] = xv[PACKED ? 0 : t];
                    if constexpr (PACKED) RowGather<TX, VEC, true>::unpack16(xw[t].x, xw[t].y, xw[t].z, xw[t].w, x);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] = fmaf(vv[t], x[e], acc[e]);
                }
            };
            for (int j = 0; j < n; j += U * EP) {
                if (n - j > 4 * EP) batch(std::integral_constant<int, 8>{}, j);
                else if (n - j > 2 * EP) batch(std::integral_constant<int, 4>{}, j);
                else batch(std::integral_constant<int, 2>{}, j);
            }
        }
        if (dn.z > dn.y) fetch_index(dn.y, dn.z);
        for (int off = LQ; off < kWave; off <<= 1)
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e] += lane_xor(acc[e], off);
        if (slot == 0 && act) {
            if (part < 0) {
                if (a.mean && end > beg) {
                    const float r = 1.f / (float)(end - beg);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) acc[e] *= r;
                }
                epilogue<VEC>(acc, a.bias, a.act, fe);
                store_out<TY, VEC>(static_cast<TY *>(a.Y), (int64_t)row * a.F + fe, acc);
            } else {
                store_vec<float, VEC>(a.partials, (int64_t)part * a.pstride + fe, acc);
            }
        }
        if (un >= hi) break;
        u = un;
        d = dn;
    }
}

using SpmmKernel = void (*)(SpmmArgs);

template <typename TX, typename TY>
SpmmKernel wave_pick_v(int vec, bool narrow)
{
    constexpr int V = (int)(16 / sizeof(TX));
    if (vec == 1) return narrow ? k_spmm_wave<TX, TY, 1, true> : k_spmm_wave<TX, TY, 1, false>;
    return narrow ? k_spmm_wave<TX, TY, V, true> : k_spmm_wave<TX, TY, V, false>;
}

// S: lanes a row (at most 32).
inline SpmmKernel wave_pick(int xdt, int ydt, int vec, int S)
{
    const auto pick_y = [&](auto tx) -> SpmmKernel {
        using TX = decltype(tx);
        if (ydt == COGDL_F32) return wave_pick_v<TX, float>(vec, S < 8);
        if (ydt == COGDL_BF16) return wave_pick_v<TX, bf16_t>(vec, S < 8);
        return wave_pick_v<TX, f16_t>(vec, S < 8);
    };
    if (xdt == COGDL_F32) return pick_y(float{});
    if (xdt == COGDL_BF16) return pick_y(bf16_t{});
    return pick_y(f16_t{});
}

template <typename TX, typename TY>
SpmmKernel narrow_pick_lq(int vec, int lq)
{
    constexpr int V = (int)(16 / sizeof(TX));
    if (vec == 1) {
        if (lq == 1) return k_spmm_narrow<TX, TY, 1, 1, 2>;
        if (lq == 2) return k_spmm_narrow<TX, TY, 1, 2, 2>;
        return k_spmm_narrow<TX, TY, 1, 4, 1>;
    }
    if (lq == 1) return k_spmm_narrow<TX, TY, V, 1, 2>;
    if (lq == 2) return k_spmm_narrow<TX, TY, V, 2, 2>;
    return k_spmm_narrow<TX, TY, V, 4, 1>;
}

// The kernel for rows on lq = 1, 2 or 4 lanes.
inline SpmmKernel narrow_pick(int xdt, int ydt, int vec, int lq)
{
    const auto pick_y = [&](auto tx) -> SpmmKernel {
        using TX = decltype(tx);
        if (ydt == COGDL_F32) return narrow_pick_lq<TX, float>(vec, lq);
        if (ydt == COGDL_BF16) return narrow_pick_lq<TX, bf16_t>(vec, lq);
        return narrow_pick_lq<TX, f16_t>(vec, lq);
    };
    if (xdt == COGDL_F32) return pick_y(float{});
    if (xdt == COGDL_BF16) return pick_y(bf16_t{});
    return pick_y(f16_t{});
}

// Kernel for (VEC, CH) of one variant.  Max outputs keep the input format or
// widen it to fp32 (each output is one fp32 message rounded once); the caller
// rejects other pairs.
template <typename TX, typename TY, bool BUF, bool MAXR, bool ADDOP>
SpmmKernel spmm_pick_vec(int vec, int ch)
{
    constexpr int V = (int)(16 / sizeof(TX));
    if (vec == 1) {
        if (ch == 1) return k_spmm<TX, TY, 1, 1, BUF, MAXR, ADDOP>;
        if (ch == 2) return k_spmm<TX, TY, 1, 2, BUF, MAXR, ADDOP>;
        return k_spmm<TX, TY, 1, 4, BUF, MAXR, ADDOP>;
    }
    if (ch == 1) return k_spmm<TX, TY, V, 1, BUF, MAXR, ADDOP>;
    if (ch == 2) return k_spmm<TX, TY, V, 2, BUF, MAXR, ADDOP>;
    return k_spmm<TX, TY, V, 4, BUF, MAXR, ADDOP>;
}

template <typename TX, bool BUF, bool MAXR, bool ADDOP>
SpmmKernel spmm_pick_y(int ydt, int vec, int ch)
{
    if (ydt == COGDL_F32) return spmm_pick_vec<TX, float, BUF, MAXR, ADDOP>(vec, ch);
    if constexpr (MAXR) {
        return spmm_pick_vec<TX, TX, BUF, MAXR, ADDOP>(vec, ch);
    } else {
        if (ydt == COGDL_BF16) return spmm_pick_vec<TX, bf16_t, BUF, MAXR, ADDOP>(vec, ch);
        return spmm_pick_vec<TX, f16_t, BUF, MAXR, ADDOP>(vec, ch);
    }
}

template <bool MAXR, bool ADDOP>
SpmmKernel spmm_pick(int xdt, int ydt, int vec, int ch, bool buf)
{
    if (buf) {
        if (xdt == COGDL_F32) return spmm_pick_y<float, true, MAXR, ADDOP>(ydt, vec, ch);
        if (xdt == COGDL_BF16) return spmm_pick_y<bf16_t, true, MAXR, ADDOP>(ydt, vec, ch);
        return spmm_pick_y<f16_t, true, MAXR, ADDOP>(ydt, vec, ch);
    }
    if (xdt == COGDL_F32) return spmm_pick_y<float, false, MAXR, ADDOP>(ydt, vec, ch);
    if (xdt == COGDL_BF16) return spmm_pick_y<bf16_t, false, MAXR, ADDOP>(ydt, vec, ch);
    return spmm_pick_y<f16_t, false, MAXR, ADDOP>(ydt, vec, ch);
}

// The variants instantiated in gspmm.hip (max of products, sum and max of
// x + bsign * val); the sum of products is instantiated in spmm.hip.
SpmmKernel gspmm_pick(bool maxr, bool addop, int xdt, int ydt, int vec, int ch, bool buf);

}  // namespace cogdl
