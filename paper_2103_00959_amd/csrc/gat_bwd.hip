// Backward pass of the attention path of section 2.2, and the dot-product
// SDDMM that carries the gradient to the attention matrix.
//
// For the loss gradient dY of Y[i,h,:] = sum_k alpha[k,h] X[col[k],h,:]:
//   dalpha[k,h] = <dY[i,h,:], X[j,h,:]>          SDDMM  A (.) (dY_h X_h^T)
//   c[i,h]      = sum_{k in row i} alpha[k,h] dalpha[k,h]
//   dscore[k,h] = f * alpha[k,h] * (dalpha[k,h] - c[i,h]),  f = 1 if the
//                 pre-activation s_dst[i,h] + s_src[j,h] > 0 else the slope
//   ds_dst[i,h] = sum_{k in row i} dscore[k,h]
//   ds_src[j,h] = sum_{k: col[k] = j} dscore[k,h]
//   dX[j,h,:]   = sum_{k: col[k] = j} alpha[k,h] dY[i,h,:]
//
// Pass 1 runs on the CSR units.  With the SpMM lane map (S lanes x VEC
// features of a row, the L = D / VEC lanes of a head side by side) each lane
// multiplies its dY elements into every gathered neighbour row and a
// reduction over the head's lanes completes the dot product, so the gathered
// rows are read once, as in the forward aggregation.  The lanes fold the row
// sum c as they go and park dalpha and u = f alpha of every edge (each value
// by a fixed lane: in LDS for a whole row that fits, else in memory); once c
// is complete, the same lanes read their own parked values back and write
// dscore and ds_dst.  A neighbour group of a split row leaves its share of c
// in the plan, and two small kernels finish those rows once every group is
// done.  dalpha and dscore are optional outputs: a layer's backward needs
// only ds_dst, ds_src and dX, and its kernels then park in LDS and the
// records alone.
//
// The pairs (alpha, dscore) of an edge's heads end side by side in the
// caller's edge workspace, 8 H bytes per edge in CSR order.  Pass 2 is the
// aggregation kernel run on the CSC (rows = source nodes), reaching each
// edge's pair through perm: one random 8H-byte record per edge instead of
// two 4H-byte rows in two arrays, each of which costs a cache line.  It sums
// dscore per head along the way: dX and ds_src in one sweep over dY.
#include "gat_kernel.hpp"

namespace cogdl {
namespace {

constexpr int kBlock = kGatBlock;

struct BwdArgs {
    const int4 *units;          // nullptr: one unit per row in row order
    const int32_t *u_lo;        // units [*u_lo, *u_hi), or per list (see unit_walk)
    const int32_t *u_hi;
    int32_t lists = 1;
    int32_t n_rows;
    const int32_t *rowptr;
    const int32_t *col;
    int32_t H;
    int32_t D;
    int64_t W;                  // H * D
    const float *s_dst;
    const float *s_src;
    float slope;
    const float *alpha;         // forward weights [nnz][H]; nullptr: rebuilt from row_stats, or the SDDMM alone
    const float *row_stats;     // per row the forward's (m, 1/z) of each head, 2H floats (or nullptr)
    const void *X;              // gathered operand, n_cols x W
    uint64_t x_bytes;
    const void *P;              // row operand (dY), n_rows x W
    float *dalpha;              // [nnz][H], or nullptr (not written)
    float *dscore;              // [nnz][H], or nullptr (not written)
    float2 *rec;                // [nnz][H] parked pairs (see park_edge), then (alpha, dscore)
    int32_t park_cap;           // LDS floats per sub-group for whole rows' parked values (0: none)
    float *ds_dst;              // [n_rows][H]
    float *gstats;              // split rows: per partial slot c[max_heads], sum[max_heads]
    int32_t sstride;            // 2 * max_heads
    const int4 *part_units;     // {row, beg, end, split index} per partial slot
    const int32_t *n_parts;
    const int4 *split_rows;     // {row, first slot, #slots, degree}
    const int32_t *n_split;
    int32_t log2S;
    int32_t log2L;              // lanes per head (k_bwd_rows)
    int32_t HG;                 // heads per slab (k_bwd_rows)
};

__device__ __forceinline__ int4 fetch_bwd_unit(const BwdArgs &a, int64_t u, int64_t hi)
{
    if (u >= hi) return make_int4(0, 0, 0, -1);
    if (a.units) return a.units[u];
    const int r = (int)u;
    return make_int4(r, a.rowptr[r], a.rowptr[r + 1], -1);
}

// The score gradient of edge k and head h is f * alpha * (dalpha - c), with f
// the LeakyReLU slope at the pre-activation t and c the row's sum of alpha *
// dalpha.  Pass 1 parks u = f * alpha and dalpha, as ParkMode below lays
// out (c is not known yet); once c is known, dscore = u (dalpha - c), and the
// edge's record ends as (alpha, dscore).
__device__ __forceinline__ float park_value(float t, float slope, float al)
{
    return (t > 0.f ? 1.f : slope) * al;
}

__device__ __forceinline__ float parked_grad(float u, float da, float c) { return u * (da - c); }

// a + b rounded on its own: a sum of stored values is not fused with the
// multiply that produced b (so every kernel variant forms ds_dst from exactly
// the dscore values it writes).
__device__ __forceinline__ float add_stored(float a, float b)
{
#pragma clang fp contract(off)
    return a + b;
}

// How pass 1 parks what the fix-up needs (c is not known yet):
//   kParkSep:   alpha given, dalpha and dscore both written.  dalpha is in its
//               output, so u alone parks: in dscore for a split row, in the LDS
//               slot li for a whole row that fits its sub-group's share, else
//               beside alpha in the record (alpha, u).
//   kParkPair:  alpha given, an output left out: the pair (dalpha, u) parks in
//               LDS (slots 2 li, 2 li + 1) or in the record.
//   kParkStats: alpha rebuilt from the row's softmax state: the pair
//               (dalpha, v) parks, v = alpha on the LeakyReLU's positive branch
//               and -alpha on the other (alpha >= 0 here), so alpha = |v| and u
//               = f alpha come back with the same bits.
enum ParkMode { kParkSep, kParkPair, kParkStats };

// Fix-up of one parked edge-head: dscore from alpha, the parked u and
// dalpha, into the record and the dscore output (when there is one).
template <int PK>
__device__ __forceinline__ float finish_edge(const BwdArgs &a, int64_t i, float al, float u, float da, float c)
{
    const float g = parked_grad(u, da, c);
    if (PK == kParkSep || a.dscore) a.dscore[i] = g;
    a.rec[i] = make_float2(al, g);
    return g;
}

template <int PK>
__device__ __forceinline__ void park_edge(const BwdArgs &a, int64_t i, bool split, float al, float da, float u,
                                          float *lds, int li)
{
    if constexpr (PK == kParkSep) {
        if (split) a.dscore[i] = u;
        else if (lds) lds[li] = u;
        else a.rec[i] = make_float2(al, u);
    } else {
        const float v = PK == kParkStats ? (u == al ? al : -al) : u;
        if (lds) {
            lds[2 * li] = da;
            lds[2 * li + 1] = v;
        } else {
            a.rec[i] = make_float2(da, v);
        }
    }
}

// (alpha, u) from a kParkStats value v.
__device__ __forceinline__ float2 unpark_stats(float v, float slope)
{
    const float al = fabsf(v);
    return make_float2(al, signbit(v) ? slope * al : al);
}

// LDS floats of a rows workgroup for whole rows' parked values, shared by its sub-groups.
constexpr int kRowParkFloats = 4096;

// Pass 1, feature-parallel: one S-lane sub-group per unit, each head on L = 2^log2L
// adjacent lanes (L a power of two, at least D / VEC), lane q of a head holding its
// features [q VEC, (q + 1) VEC).  A head that is no whole number of vectors (RAG) ends
// with a vector moved back to its last VEC features, whose first ones, already held by
// the lane before, are masked to zero in both operands.  Heads past the lanes of a
// wavefront go to further slabs (grid y, HG heads each).
//
// Every edge k of a unit is owned by lane q = (k - beg) mod M of its head, M = 2^LM =
// min(L, 8): that lane alone loads the edge's alpha and source score, adds its term of
// c, and parks its dalpha and u; the head's lanes then add up their shares of c.  The
// partial dot products of a batch of 8 edges are reduce-scattered over aligned groups of
// M lanes, so lane q ends with the group's sums of its own 8 / M edges (7 exchanges for
// M = 8, 6 for M = 4, against a butterfly of log2 L levels for each edge), and L > 8
// adds the groups by a butterfly.  Bound by the gathers (128-byte lines) and the
// per-edge arrays.  Before, heads of fewer than 8 lanes ran the butterflies and parked in
// memory (64.3M edges, fp32, 8 heads of 16: 8.1 -> 7.1 ms) and heads of a ragged number
// of vectors or past one wavefront ran k_bwd_rows_any (2.5M edges, one head of 41 bf16:
// 0.61 -> 0.10 ms; 0.86M edges, 8 heads of 51: 1.23 -> 0.14 ms).
template <typename TX, int VEC, bool BUF, bool DOT, int LM, bool RAG, int PK = kParkSep>
__global__ __launch_bounds__(kBlock) void k_bwd_rows(BwdArgs a)
{
    constexpr int U = 8;
    constexpr int M = 1 << LM;
    constexpr int EPL = U / M;       // edges of a batch owned by a lane
    // 16-bit features stay packed: four dot2 instructions per 16-byte vector
    // instead of widening both operands to fp32 (half the registers).
    constexpr bool PACKED = sizeof(TX) == 2 && VEC == 8;
    const int log2S = a.log2S;
    const int S = 1 << log2S;
    const int lane = lane_id();
    const int lig = lane & (S - 1);
    const int gbase = lane & ~(S - 1);
    const int L = 1 << a.log2L;
    const int q = lig & (L - 1);
    const int hl = lig >> a.log2L;                      // head within the slab
    const int h = (int)blockIdx.y * a.HG + hl;
    const int H = a.H;
    const bool hact = hl < a.HG && h < H;
    const bool act = hact && q * VEC < a.D;
    const int over = (RAG && act && (q + 1) * VEC > a.D) ? (q + 1) * VEC - a.D : 0;   // masked front features
    const int64_t fe = act ? (int64_t)h * a.D + q * VEC - over : 0;
    const bool writer = hact && q < M;
    uint32_t keep[RAG ? 4 : 1];
    if constexpr (RAG) {
#pragma unroll
        for (int w = 0; w < 4; ++w)
            if constexpr (sizeof(TX) == 4) keep[w] = w >= over ? 0xffffffffu : 0u;
            else keep[w] = (2 * w >= over ? 0x0000ffffu : 0u) | (2 * w + 1 >= over ? 0xffff0000u : 0u);
    }
    const auto mask = [&](uint4 v) {
        if constexpr (RAG) return make_uint4(v.x & keep[0], v.y & keep[1], v.z & keep[2], v.w & keep[3]);
        else return v;
    };
    const UnitWalk walk = unit_walk(a.units != nullptr, a.u_lo, a.u_hi, a.lists, a.n_rows,
                                    kBlock >> log2S, threadIdx.x >> log2S);
    const int64_t stride = walk.step;
    const int64_t hi = walk.end;
    const RowGather<TX, VEC, BUF> X(a.X, a.x_bytes);
    const TX *__restrict__ P = static_cast<const TX *>(a.P);
    const int32_t *__restrict__ col = a.col;
    extern __shared__ float row_park[];
    float *const park_mine = row_park + (threadIdx.x >> log2S) * a.park_cap;

    int64_t u = walk.first;
    if (u >= hi) return;
    int4 d = fetch_bwd_unit(a, u, hi);
    int c_cur = 0;
    if (d.z > d.y) c_cur = col[d.y + lig < d.z - 1 ? d.y + lig : d.z - 1];
    for (;;) {
        const int64_t un = u + stride;
        const int4 dn = fetch_bwd_unit(a, un, hi);
        const int row = d.x, beg = d.y, end = d.z, part = d.w;
        // a whole row whose parked values fit this sub-group's LDS share parks them there
        // (pairs of heads on one lane, 8 edges of which a lane parks in a batch, in the records:
        // 8 heads of 8 bf16, 2.5M edges, 453 us through LDS, 415)
        constexpr bool PARK_LDS = !DOT && !(LM == 0 && PK != kParkSep);
        float *const lds =
            (PARK_LDS && part < 0 && (end - beg) * a.HG * (PK == kParkSep ? 1 : 2) <= a.park_cap) ? park_mine : nullptr;
        float p[PACKED ? 1 : VEC];
        uint4 pw = make_uint4(0u, 0u, 0u, 0u);
        if constexpr (VEC == 1) {
            p[0] = 0.f;
            if (act) load_vec<TX, 1>(P, (int64_t)row * a.W + fe, p);
        } else {
            if (act) {
                const u32x4_u v = *reinterpret_cast<const u32x4_u *>(P + (int64_t)row * a.W + fe);
                pw = mask(make_uint4(v.x, v.y, v.z, v.w));
            }
            if constexpr (!PACKED) RowGather<TX, VEC, BUF>::unpack16(pw.x, pw.y, pw.z, pw.w, p);
        }
        const float sd = (!DOT && hact) ? a.s_dst[(int64_t)row * H + h] : 0.f;
        // kParkStats: the row's softmax state for this lane's head
        const float rm = (PK == kParkStats && hact) ? a.row_stats[(int64_t)row * 2 * H + h] : 0.f;
        const float rrz = (PK == kParkStats && hact) ? a.row_stats[(int64_t)row * 2 * H + H + h] : 0.f;
        float c = 0.f;

        const int last = end - 1;
        for (int k0 = beg; k0 < end; k0 += S) {
            const int n = (end - k0 < S) ? end - k0 : S;
            const int c_nxt = col[k0 + S + lig < last ? k0 + S + lig : last];
            for (int j = 0; j < n; j += U) {
                uint4 xw[VEC > 1 ? U : 1];
                float x1[VEC > 1 ? 1 : U][1];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const bool ok = j + t < n;
                    const int cc = lane_bcast(c_cur, gbase + (ok ? j + t : j));
                    if constexpr (VEC == 1) X.load((int64_t)cc * a.W + fe, ok && act, x1[t]);
                    else xw[t] = X.load_raw16((int64_t)cc * a.W + fe, ok && act);
                }
                float pd[U];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    float s = 0.f;
                    if constexpr (VEC == 1) {
                        s = p[0] * x1[t][0];
                    } else {
                        const uint4 x = mask(xw[t]);
                        if constexpr (PACKED) {
                            s = dot2_acc<TX>(x.x, pw.x, s);
                            s = dot2_acc<TX>(x.y, pw.y, s);
                            s = dot2_acc<TX>(x.z, pw.z, s);
                            s = dot2_acc<TX>(x.w, pw.w, s);
                        } else {
                            float xv[VEC];
                            RowGather<TX, VEC, BUF>::unpack16(x.x, x.y, x.z, x.w, xv);
#pragma unroll
                            for (int e = 0; e < VEC; ++e) s = fmaf(p[e], xv[e], s);
                        }
                    }
                    pd[t] = s;
                }
                // this lane's edges of the batch: j + (q mod M) + M r
                float sum[EPL];
                reduce_scatter<LM>(pd, q & (M - 1), sum);
                if constexpr (M == 8)
                    for (int off = 8; off < L; off <<= 1) sum[0] += lane_xor(sum[0], off);
                // (a cross-lane read: every lane takes part; with several edges a lane their
                // scores and weights are requested together, without branches)
                float ss1[EPL], al1[EPL];
                if constexpr (!DOT) {
#pragma unroll
                    for (int r = 0; r < EPL; ++r) {
                        const int t = (q & (M - 1)) + M * r;
                        const int cme = lane_bcast(c_cur, gbase + j + t);
                        const bool own = j + t < n && writer;
                        if (EPL > 1 || own) {
                            ss1[r] = a.s_src[own ? (int64_t)cme * H + h : 0];
                            if constexpr (PK != kParkStats) al1[r] = a.alpha[own ? (int64_t)(k0 + j + t) * H + h : 0];
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < EPL; ++r) {
                    const int t = (q & (M - 1)) + M * r;
                    const int64_t k = k0 + j + t;
                    if (j + t < n && writer) {
                        if (DOT || PK == kParkSep || a.dalpha) a.dalpha[k * H + h] = sum[r];
                        if constexpr (!DOT) {
                            if constexpr (PK == kParkStats)
                                al1[r] = alpha_value(leaky_relu(sd + ss1[r], a.slope), rm, rrz);
                            c = fmaf(al1[r], sum[r], c);
                            park_edge<PK>(a, k * H + h, part >= 0, al1[r], sum[r],
                                          park_value(sd + ss1[r], a.slope, al1[r]), lds, (int)(k - beg) * a.HG + hl);
                        }
                    }
                }
            }
            c_cur = c_nxt;
        }
        const int c_first_next =
            (dn.z > dn.y) ? col[dn.y + lig < dn.z - 1 ? dn.y + lig : dn.z - 1] : 0;

        if constexpr (!DOT) {
            // the head's lanes hold shares of c (owners only, the others 0)
            c = group_sum(c, L);
            if (part >= 0) {
                if (hact && q == 0) a.gstats[(int64_t)part * a.sstride + h] = c;
            } else {
                // this lane's parked edges: offsets q, q + M, ... of the row
                constexpr int R = 4;
                float sdt = 0.f;
                if (writer) {
                    for (int o0 = q; o0 < end - beg; o0 += R * M) {
                        float al[R], da[R], uv[R];
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const int o = o0 + r * M;
                            const int oc = o < end - beg ? o : o0;
                            const int64_t i = ((int64_t)beg + oc) * H + h;
                            const int li = oc * a.HG + hl;
                            if constexpr (PK == kParkSep) {
                                // dalpha from its output; u from LDS (alpha from the input)
                                // or the record (alpha, u)
                                da[r] = a.dalpha[i];
                                const float2 p = lds ? make_float2(a.alpha[i], lds[li]) : a.rec[i];
                                al[r] = p.x;
                                uv[r] = p.y;
                            } else {
                                // the pair from LDS or the record: (dalpha, u) with alpha from
                                // the input, or (dalpha, v) holding alpha and u
                                const float2 p = lds ? make_float2(lds[2 * li], lds[2 * li + 1]) : a.rec[i];
                                da[r] = p.x;
                                if constexpr (PK == kParkStats) {
                                    const float2 q = unpark_stats(p.y, a.slope);
                                    al[r] = q.x;
                                    uv[r] = q.y;
                                } else {
                                    al[r] = a.alpha[i];
                                    uv[r] = p.y;
                                }
                            }
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const int o = o0 + r * M;
                            if (o < end - beg)
                                sdt = add_stored(sdt, finish_edge<PK>(a, ((int64_t)beg + o) * H + h, al[r], uv[r],
                                                                       da[r], c));
                        }
                    }
                }
                sdt = group_sum(sdt, L);
                if (hact && q == 0) a.ds_dst[(int64_t)row * H + h] = sdt;
            }
        }
        if (un >= hi) break;
        u = un;
        d = dn;
        c_cur = c_first_next;
    }
}

// Sum over the slots of one head in a wavefront laid out as (slot, head):
// lanes s * H + h, s < 64 / H.  The same fixed order in every lane of h.
__device__ __forceinline__ float slot_sum(float v, int H)
{
    if ((H & (H - 1)) == 0) {
        for (int off = H; off < kWave; off <<= 1) v += lane_xor(v, off);
        return v;
    }
    const int slots = kWave / H;
    const int h = lane_id() % H;
    float s = 0.f;
    for (int i = 0; i < slots; ++i) s += lane_bcast(v, i * H + h);
    return s;
}

// Pass 1 for any shape: a wavefront per unit, lanes as (edge slot, head),
// each lane forming whole dot products element by element.  Every edge is
// parked by the lane of its slot.
template <typename TX, typename TP, bool DOT, int PK = kParkSep>
__global__ __launch_bounds__(kBlock) void k_bwd_rows_any(BwdArgs a)
{
    const int lane = lane_id();
    const int H = a.H;
    const int eps = kWave / H;
    const int h = lane % H;
    const int slot = lane / H;
    const bool live = slot < eps;
    const UnitWalk walk = unit_walk(a.units != nullptr, a.u_lo, a.u_hi, a.lists, a.n_rows,
                                    kBlock / kWave, threadIdx.x / kWave);
    const int64_t hi = walk.end;
    const TX *__restrict__ X = static_cast<const TX *>(a.X);
    const TP *__restrict__ P = static_cast<const TP *>(a.P);
    for (int64_t u = walk.first; u < hi; u += walk.step) {
        const int4 d = fetch_bwd_unit(a, u, hi);
        const int row = d.x, beg = d.y, end = d.z, part = d.w;
        const float sd = DOT ? 0.f : a.s_dst[(int64_t)row * H + h];
        const float rm = PK == kParkStats ? a.row_stats[(int64_t)row * 2 * H + h] : 0.f;
        const float rrz = PK == kParkStats ? a.row_stats[(int64_t)row * 2 * H + H + h] : 0.f;
        float c = 0.f;
        if (live) {
            for (int k = beg + slot; k < end; k += eps) {
                const int j = a.col[k];
                float s = 0.f;
                for (int e = 0; e < a.D; ++e) {
                    float pv[1], xv[1];
                    load_vec<TP, 1>(P, (int64_t)row * a.W + (int64_t)h * a.D + e, pv);
                    load_vec<TX, 1>(X, (int64_t)j * a.W + (int64_t)h * a.D + e, xv);
                    s = fmaf(pv[0], xv[0], s);
                }
                if (DOT || PK == kParkSep || a.dalpha) a.dalpha[(int64_t)k * H + h] = s;
                if constexpr (!DOT) {
                    const float ss1 = a.s_src[(int64_t)j * H + h];
                    const float al = PK == kParkStats ? alpha_value(leaky_relu(sd + ss1, a.slope), rm, rrz)
                                                      : a.alpha[(int64_t)k * H + h];
                    c = fmaf(al, s, c);
                    park_edge<PK>(a, (int64_t)k * H + h, part >= 0, al, s, park_value(sd + ss1, a.slope, al),
                                  nullptr, 0);
                }
            }
        }
        if constexpr (DOT) continue;
        c = slot_sum(live ? c : 0.f, H);
        if (part >= 0) {
            if (slot == 0) a.gstats[(int64_t)part * a.sstride + h] = c;
            continue;
        }
        float sdt = 0.f;
        if (live) {
            for (int k = beg + slot; k < end; k += eps) {
                const int64_t i = (int64_t)k * H + h;
                const float2 r = a.rec[i];
                float g;
                if constexpr (PK == kParkSep) {
                    g = finish_edge<PK>(a, i, r.x, r.y, a.dalpha[i], c);           // (alpha, u)
                } else if constexpr (PK == kParkPair) {
                    g = finish_edge<PK>(a, i, a.alpha[i], r.y, r.x, c);            // (dalpha, u)
                } else {
                    const float2 q = unpark_stats(r.y, a.slope);                   // (dalpha, v)
                    g = finish_edge<PK>(a, i, q.x, q.y, r.x, c);
                }
                sdt = add_stored(sdt, g);
            }
        }
        sdt = slot_sum(live ? sdt : 0.f, H);
        if (slot == 0) a.ds_dst[(int64_t)row * H + h] = sdt;
    }
}

// Split rows, after pass 1: every neighbour group adds up the shares of c of
// all groups of its row, turns its parked edges into dscore and leaves its
// share of ds_dst.  One wavefront per group, lanes (slot, head); the shares
// are loaded by the slots side by side and summed over the slots in a fixed
// order (every group of a row forms the same c), and the next group's
// descriptors are fetched while this one is processed.
template <int PK>
__global__ __launch_bounds__(kBlock) void k_bwd_split_edges(BwdArgs a)
{
    const int lane = lane_id();
    const int H = a.H;
    const int eps = kWave / H;
    const int h = lane % H;
    const int slot = lane / H;
    const bool live = slot < eps;
    const int half = a.sstride >> 1;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    const int32_t np = *a.n_parts;
    int64_t p = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    if (p >= np) return;
    int4 d = a.part_units[p];
    int4 sr = a.split_rows[d.w];
    for (;;) {
        const int64_t pn = p + waves;
        const int4 dn = pn < np ? a.part_units[pn] : make_int4(0, 0, 0, 0);
        float cs = 0.f;
        if (live)
            for (int g = slot; g < sr.z; g += eps) cs += a.gstats[(int64_t)(sr.y + g) * a.sstride + h];
        const float c = slot_sum(live ? cs : 0.f, H);
        const int4 srn = pn < np ? a.split_rows[dn.w] : make_int4(0, 0, 0, 0);
        constexpr int R = 8;
        float sdt = 0.f;
        if (live) {
            for (int k0 = d.y + slot; k0 < d.z; k0 += R * eps) {
                float da[R], uv[R], al[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int k = k0 + r * eps;
                    const int64_t i = (int64_t)(k < d.z ? k : k0) * H + h;
                    if constexpr (PK == kParkSep) {         // dalpha and the u parked in dscore
                        da[r] = a.dalpha[i];
                        uv[r] = a.dscore[i];
                        al[r] = a.alpha[i];
                    } else if constexpr (PK == kParkPair) { // the parked pair (dalpha, u)
                        const float2 q = a.rec[i];
                        da[r] = q.x;
                        uv[r] = q.y;
                        al[r] = a.alpha[i];
                    } else {                                // (dalpha, v): alpha and u from v
                        const float2 q = a.rec[i];
                        const float2 w = unpark_stats(q.y, a.slope);
                        da[r] = q.x;
                        al[r] = w.x;
                        uv[r] = w.y;
                    }
                }
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int k = k0 + r * eps;
                    if (k < d.z) sdt = add_stored(sdt, finish_edge<PK>(a, (int64_t)k * H + h, al[r], uv[r], da[r], c));
                }
            }
        }
        sdt = slot_sum(live ? sdt : 0.f, H);
        if (slot == 0) a.gstats[p * a.sstride + half + h] = sdt;
        if (pn >= np) break;
        p = pn;
        d = dn;
        sr = srn;
    }
}

// ds[row, h] = sum of the groups' shares (slot order), one wavefront per split
// row; the shares sit at offset `base` of each partial slot's stats.
__global__ __launch_bounds__(kBlock) void k_split_head_sums(const int4 *__restrict__ split_rows,
                                                            const int32_t *__restrict__ n_split,
                                                            const float *__restrict__ gstats,
                                                            int sstride, int base, int H,
                                                            float *__restrict__ out)
{
    const int lane = lane_id();
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    const int32_t ns = *n_split;
    for (int64_t s = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; s < ns;
         s += waves) {
        const int4 d = split_rows[s];
        if (lane < H) {
            float v = 0.f;
            for (int g = 0; g < d.z; ++g) v += gstats[(int64_t)(d.y + g) * sstride + base + lane];
            out[(int64_t)d.x * H + lane] = v;
        }
    }
}

using BwdKernel = void (*)(BwdArgs);

template <typename TX, int VEC, bool BUF, bool RAG, bool DOT, int PK>
BwdKernel pick_rows_m(int lm)
{
    if (lm == 0) return k_bwd_rows<TX, VEC, BUF, DOT, 0, RAG, PK>;
    if (lm == 1) return k_bwd_rows<TX, VEC, BUF, DOT, 1, RAG, PK>;
    if (lm == 2) return k_bwd_rows<TX, VEC, BUF, DOT, 2, RAG, PK>;
    return k_bwd_rows<TX, VEC, BUF, DOT, 3, RAG, PK>;
}

// The 64-bit-address kernels (X past the buffer limit, or heads below a vector) mask
// whether or not the heads are ragged.
template <typename TX, bool DOT, int PK>
BwdKernel pick_rows_v(bool buf, int vec, bool rag, int lm)
{
    constexpr int V = (int)(16 / sizeof(TX));
    if (vec == 1) return pick_rows_m<TX, 1, false, false, DOT, PK>(lm);
    if (!buf) return pick_rows_m<TX, V, false, true, DOT, PK>(lm);
    return rag ? pick_rows_m<TX, V, true, true, DOT, PK>(lm) : pick_rows_m<TX, V, true, false, DOT, PK>(lm);
}

template <bool DOT, int PK>
BwdKernel pick_rows_t(int dt, bool buf, int vec, bool rag, int lm)
{
    if (dt == COGDL_F32) return pick_rows_v<float, DOT, PK>(buf, vec, rag, lm);
    if (dt == COGDL_BF16) return pick_rows_v<bf16_t, DOT, PK>(buf, vec, rag, lm);
    return pick_rows_v<f16_t, DOT, PK>(buf, vec, rag, lm);
}

// lm: log2 of the owner lanes per head; pk: the parking mode (the dot-product kernels
// have one)
template <bool DOT>
BwdKernel pick_rows(int dt, bool buf, int vec, bool rag, int lm, int pk)
{
    if constexpr (!DOT) {
        if (pk == kParkPair) return pick_rows_t<false, kParkPair>(dt, buf, vec, rag, lm);
        if (pk == kParkStats) return pick_rows_t<false, kParkStats>(dt, buf, vec, rag, lm);
    }
    return pick_rows_t<DOT, kParkSep>(dt, buf, vec, rag, lm);
}

template <typename TX, bool DOT, int PK>
BwdKernel pick_any_p(int pdt)
{
    if (pdt == COGDL_F32) return k_bwd_rows_any<TX, float, DOT, PK>;
    if (pdt == COGDL_BF16) return k_bwd_rows_any<TX, bf16_t, DOT, PK>;
    return k_bwd_rows_any<TX, f16_t, DOT, PK>;
}

template <bool DOT, int PK>
BwdKernel pick_any_t(int xdt, int pdt)
{
    if (xdt == COGDL_F32) return pick_any_p<float, DOT, PK>(pdt);
    if (xdt == COGDL_BF16) return pick_any_p<bf16_t, DOT, PK>(pdt);
    return pick_any_p<f16_t, DOT, PK>(pdt);
}

template <bool DOT>
BwdKernel pick_any(int xdt, int pdt, int pk)
{
    if constexpr (!DOT) {
        if (pk == kParkPair) return pick_any_t<false, kParkPair>(xdt, pdt);
        if (pk == kParkStats) return pick_any_t<false, kParkStats>(xdt, pdt);
    }
    return pick_any_t<DOT, kParkSep>(xdt, pdt);
}

unsigned wave_grid(int64_t work)
{
    int64_t b = (work + (kBlock / kWave) - 1) / (kBlock / kWave);
    if (b > 2048) b = 2048;
    if (b < 1) b = 1;
    return (unsigned)b;
}

// Pass 1 over the units of `plan` (or the rows in order): heads of up to 64 vectors with
// both operands of one format run the feature-parallel kernel, the rest the general one.
template <bool DOT>
cogdl_status rows_pass(BwdArgs a, const Plan *P, int xdt, int pdt, const char *name,
                       hipStream_t stream)
{
    const int64_t units = P ? P->cap_units : a.n_rows;
    const int v16 = 16 / dtype_bytes(xdt);
    const int pk = a.row_stats ? kParkStats : (a.dalpha && a.dscore) ? kParkSep : kParkPair;
    const int vec = a.D >= v16 ? v16 : 1;
    int L = next_pow2((a.D + vec - 1) / vec);
    // Dot products alone of up to 4 short ragged heads: the general kernel takes 64 / H edges
    // side by side, the feature-parallel one 8, and a lane sums up to 8 features faster than
    // a long row's chain of batches goes on (2 heads of 5 bf16, us, general / parallel:
    // without a plan 600k edges 98 / 469, 2.5M 378 / 1183, but 8M in rows of 16 238 / 124; with
    // one 15k 13 / 27, 600k 18 / 30, 2.5M 94 / 51; 8 heads of 6 without a plan 456 / 476).
    const bool short_heads = DOT && a.D <= 8 && a.H <= 4 && (a.D & (a.D - 1)) != 0 && (!P || P->nnz < 3 << 18);
    if (xdt == pdt && L <= kWave && !short_heads) {
        // sub-groups of at least 8 lanes, so that a chunk of column indices (one per lane)
        // fills a batch of 8 edges
        const int hp = next_pow2(a.H);
        while (L * hp < 8) L *= 2;
        a.HG = L * hp <= kWave ? a.H : kWave / L;
        const int S = L * next_pow2(a.HG);
        const int slabs = (a.H + a.HG - 1) / a.HG;
        a.log2S = log2i(S);
        a.log2L = log2i(L);
        BwdKernel k = pick_rows<DOT>(xdt, a.x_bytes <= kBufferMaxBytes, vec, a.D % vec != 0, L < 8 ? a.log2L : 3, pk);
        const int64_t upb = kBlock / S;
        a.park_cap = DOT ? 0 : kRowParkFloats / (int)upb;
        const size_t shm = DOT ? 0 : sizeof(float) * kRowParkFloats;
        int64_t blocks = (units + upb - 1) / upb;
        const int64_t res = resident_blocks(reinterpret_cast<const void *>(k), kBlock);
        if (blocks > res) blocks = res;
        blocks = list_grid(blocks, a.lists);
        COGDL_LAUNCH_SHM(name, k, dim3((unsigned)blocks, (unsigned)slabs), kBlock, shm, stream, a);
    } else {
        BwdKernel k = pick_any<DOT>(xdt, pdt, pk);
        a.park_cap = 0;
        int64_t blocks = (units + (kBlock / kWave) - 1) / (kBlock / kWave);
        const int64_t res = resident_blocks(reinterpret_cast<const void *>(k), kBlock);
        if (blocks > res) blocks = res;
        blocks = list_grid(blocks, a.lists);
        COGDL_LAUNCH(name, k, (unsigned)blocks, kBlock, stream, a);
    }
    return COGDL_OK;
}

cogdl_status check_heads(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *rowptr,
                         const int32_t *col, int32_t H, int32_t D)
{
    if (n_rows < 0 || n_cols < 0 || nnz < 0) return COGDL_ERR_INVALID;
    if (H < 1 || H > COGDL_MAX_HEADS || D < 1) return COGDL_ERR_INVALID;
    if (nnz > COGDL_MAX_NNZ || (int64_t)H * D > INT32_MAX) return COGDL_ERR_TOO_LARGE;
    if (n_rows > 0 && !rowptr) return COGDL_ERR_INVALID;
    if (nnz > 0 && (!col || n_rows == 0 || n_cols == 0)) return COGDL_ERR_INVALID;
    return COGDL_OK;
}

}  // namespace
}  // namespace cogdl

using namespace cogdl;

extern "C" {

cogdl_status cogdl_sddmm_dot(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *rowptr,
                             const int32_t *col, int32_t H, int32_t D, const void *P,
                             cogdl_dtype p_dtype, const void *Q, cogdl_dtype q_dtype, float *out,
                             const cogdl_plan *plan, hipStream_t stream)
{
    cogdl_status st = check_heads(n_rows, n_cols, nnz, rowptr, col, H, D);
    if (st != COGDL_OK) return st;
    if (!dtype_ok(p_dtype) || !dtype_ok(q_dtype)) return COGDL_ERR_DTYPE;
    if (nnz > 0 && (!P || !Q || !out)) return COGDL_ERR_INVALID;
    const Plan *Pl = plan_of(plan);
    if (Pl && (Pl->n_rows != n_rows || Pl->nnz != nnz)) return COGDL_ERR_PLAN;
    if (nnz == 0) return COGDL_OK;
    BwdArgs a{};
    a.units = Pl ? Pl->units : nullptr;
    if (Pl) set_units(a, all_units(*Pl));
    a.n_rows = n_rows;
    a.rowptr = rowptr;
    a.col = col;
    a.H = H;
    a.D = D;
    a.W = (int64_t)H * D;
    a.X = Q;
    a.x_bytes = (uint64_t)n_cols * (uint64_t)a.W * (uint64_t)dtype_bytes(q_dtype);
    a.P = P;
    a.dalpha = out;
    return rows_pass<true>(a, Pl, (int)q_dtype, (int)p_dtype, "sddmm_dot", stream);
}

}  // extern "C"

namespace cogdl {
namespace {

// The backward with the forward weights given (alpha) or rebuilt from the
// forward's row softmax states (row_stats): exactly one of them.
cogdl_status gat_backward_impl(int32_t n_rows, int32_t n_cols, int64_t nnz, const int32_t *rowptr,
                               const int32_t *col, const int32_t *colptr, const int32_t *row_t,
                               const int32_t *perm, int32_t H, int32_t D, const float *s_dst,
                               const float *s_src, float negative_slope, const float *alpha,
                               const float *row_stats, const void *X, cogdl_dtype x_dtype,
                               const void *dY, cogdl_dtype dy_dtype, void *dX, cogdl_dtype dx_dtype,
                               float *dalpha, float *dscore, float *ds_dst, float *ds_src,
                               float *edge_work, const cogdl_plan *plan, const cogdl_plan *plan_t,
                               hipStream_t stream)
{
    cogdl_status st = check_heads(n_rows, n_cols, nnz, rowptr, col, H, D);
    if (st != COGDL_OK) return st;
    if (!dtype_ok(x_dtype) || !dtype_ok(dy_dtype) || !dtype_ok(dx_dtype)) return COGDL_ERR_DTYPE;
    if (n_cols > 0 && (!colptr || !dX || !ds_src)) return COGDL_ERR_INVALID;
    if (n_rows > 0 && (!ds_dst || !s_dst || !dY)) return COGDL_ERR_INVALID;
    if (nnz > 0 && (!row_t || !perm || !s_src || (alpha == nullptr) == (row_stats == nullptr) || !X ||
                    !edge_work || (uintptr_t)edge_work % alignof(float2) != 0))
        return COGDL_ERR_INVALID;
    float2 *rec = reinterpret_cast<float2 *>(edge_work);
    const int64_t W = (int64_t)H * D;
    const Plan *Pr = plan_of(plan);
    const Plan *Pc = plan_of(plan_t);
    if (Pr && (Pr->n_rows != n_rows || Pr->nnz != nnz || Pr->max_heads < H)) return COGDL_ERR_PLAN;
    if (Pc && (Pc->n_rows != n_cols || Pc->nnz != nnz || Pc->max_feat < W || Pc->max_heads < H))
        return COGDL_ERR_PLAN;

    // pass 1 on the CSR: dalpha, dscore, ds_dst
    if (n_rows > 0) {
        BwdArgs a{};
        a.units = Pr ? Pr->units : nullptr;
        if (Pr) set_units(a, all_units(*Pr));
        a.n_rows = n_rows;
        a.rowptr = rowptr;
        a.col = col;
        a.H = H;
        a.D = D;
        a.W = W;
        a.s_dst = s_dst;
        a.s_src = s_src;
        a.slope = negative_slope;
        a.alpha = alpha;
        a.row_stats = row_stats;
        a.X = X;
        a.x_bytes = (uint64_t)n_cols * (uint64_t)W * (uint64_t)dtype_bytes(x_dtype);
        a.P = dY;
        a.dalpha = dalpha;
        a.dscore = dscore;
        a.rec = rec;
        a.ds_dst = ds_dst;
        a.gstats = Pr ? Pr->gstats : nullptr;
        a.sstride = Pr ? 2 * Pr->max_heads : 0;
        a.part_units = Pr ? Pr->part_units : nullptr;
        a.n_parts = Pr ? Pr->n_parts_dev() : nullptr;
        a.split_rows = Pr ? Pr->split_rows : nullptr;
        a.n_split = Pr ? Pr->n_split_dev() : nullptr;
        st = rows_pass<false>(a, Pr, (int)x_dtype, (int)dy_dtype, "gat_bwd_rows", stream);
        if (st != COGDL_OK) return st;
        if (Pr) {
            if (row_stats)
                COGDL_LAUNCH("gat_bwd_split_edges", k_bwd_split_edges<kParkStats>, wave_grid(Pr->cap_partials),
                             kBlock, stream, a);
            else if (dalpha && dscore)
                COGDL_LAUNCH("gat_bwd_split_edges", k_bwd_split_edges<kParkSep>, wave_grid(Pr->cap_partials),
                             kBlock, stream, a);
            else
                COGDL_LAUNCH("gat_bwd_split_edges", k_bwd_split_edges<kParkPair>, wave_grid(Pr->cap_partials),
                             kBlock, stream, a);
            COGDL_LAUNCH("gat_bwd_split_dst", k_split_head_sums, wave_grid(Pr->cap_split), kBlock,
                         stream, Pr->split_rows, Pr->n_split_dev(), Pr->gstats, a.sstride,
                         Pr->max_heads, H, ds_dst);
        }
    }
    if (n_cols == 0) return COGDL_OK;

    // pass 2 on the CSC: dX and ds_src
    const HeadMap m = head_map(H, D, dtype_bytes(dy_dtype), true);
    GatArgs g{};
    g.units = Pc ? Pc->units : nullptr;
    g.n_rows = n_cols;
    g.rowptr = colptr;
    g.col = row_t;
    g.H = H;
    g.D = D;
    g.W = W;
    g.alpha_in = alpha;
    g.X = dY;
    g.x_bytes = (uint64_t)n_rows * (uint64_t)W * (uint64_t)dtype_bytes(dy_dtype);
    g.Y = dX;
    g.partials = Pc ? Pc->partials : nullptr;
    g.pstride = Pc ? (Pc->max_feat + 7) / 8 * 8 : 0;
    g.gstats = Pc ? Pc->gstats : nullptr;
    g.sstride = Pc ? 2 * Pc->max_heads : 0;
    g.perm = perm;
    g.rec = rec;
    g.ds_out = ds_src;
    g.L = m.L;
    g.log2S = m.log2S;
    const bool buf = g.x_bytes <= kBufferMaxBytes;
    const int64_t units = Pc ? Pc->cap_units : n_cols;
    const bool tiny = Pc && m.tiny;
    if (Pc) set_units(g, tiny ? long_units(*Pc) : all_units(*Pc));
    {
        const int64_t upb = kBlock >> m.log2S;
        GatKernel k = gat_pick<true>((int)dy_dtype, (int)dx_dtype, m.vec, m.ch, buf, m.lm);
        int64_t blocks = (units + upb - 1) / upb;
        const int64_t res = resident_blocks(reinterpret_cast<const void *>(k), kBlock);
        if (blocks > res) blocks = res;
        blocks = list_grid(blocks, g.lists);
        COGDL_LAUNCH("gat_bwd_cols", k, dim3((unsigned)blocks, (unsigned)m.n_slabs), kBlock, stream, g);
    }
    if (tiny) {
        GatArgs b = g;
        set_units(b, tiny_units(*Pc));
        b.log2S = m.log2S - 2;
        const int64_t upb = kBlock >> b.log2S;
        GatKernel k = gat_pick<true>((int)dy_dtype, (int)dx_dtype, m.vec, 4, buf);
        int64_t blocks = (units + upb - 1) / upb;
        const int64_t res = resident_blocks(reinterpret_cast<const void *>(k), kBlock);
        if (blocks > res) blocks = res;
        blocks = list_grid(blocks, b.lists);
        COGDL_LAUNCH("gat_bwd_cols_tiny", k, dim3((unsigned)blocks, (unsigned)m.n_slabs), kBlock, stream, b);
    }
    if (!Pc) return COGDL_OK;
    st = sum_reduce_launch("gat_bwd_dx_reduce", *Pc, W, dX, (int)dx_dtype, false, nullptr,
                           COGDL_ACT_NONE, stream);
    if (st != COGDL_OK) return st;
    COGDL_LAUNCH("gat_bwd_split_src", k_split_head_sums, wave_grid(Pc->cap_split), kBlock, stream,
                 Pc->split_rows, Pc->n_split_dev(), Pc->gstats, g.sstride, 0, H, ds_src);
    return COGDL_OK;
}

}  // namespace
}  // namespace cogdl

extern "C" {

cogdl_status cogdl_gat_backward(int32_t n_rows, int32_t n_cols, int64_t nnz,
                                const int32_t *rowptr, const int32_t *col, const int32_t *colptr,
                                const int32_t *row_t, const int32_t *perm, int32_t H, int32_t D,
                                const float *s_dst, const float *s_src, float negative_slope,
                                const float *alpha, const void *X, cogdl_dtype x_dtype,
                                const void *dY, cogdl_dtype dy_dtype, void *dX,
                                cogdl_dtype dx_dtype, float *dalpha, float *dscore, float *ds_dst,
                                float *ds_src, float *edge_work, const cogdl_plan *plan,
                                const cogdl_plan *plan_t, hipStream_t stream)
{
    if (nnz > 0 && !alpha) return COGDL_ERR_INVALID;
    return gat_backward_impl(n_rows, n_cols, nnz, rowptr, col, colptr, row_t, perm, H, D, s_dst, s_src,
                             negative_slope, alpha, nullptr, X, x_dtype, dY, dy_dtype, dX, dx_dtype,
                             dalpha, dscore, ds_dst, ds_src, edge_work, plan, plan_t, stream);
}

cogdl_status cogdl_gat_backward_stats(int32_t n_rows, int32_t n_cols, int64_t nnz,
                                      const int32_t *rowptr, const int32_t *col,
                                      const int32_t *colptr, const int32_t *row_t,
                                      const int32_t *perm, int32_t H, int32_t D,
                                      const float *s_dst, const float *s_src,
                                      float negative_slope, const float *row_stats, const void *X,
                                      cogdl_dtype x_dtype, const void *dY, cogdl_dtype dy_dtype,
                                      void *dX, cogdl_dtype dx_dtype, float *dalpha,
                                      float *dscore, float *ds_dst, float *ds_src,
                                      float *edge_work, const cogdl_plan *plan,
                                      const cogdl_plan *plan_t, hipStream_t stream)
{
    if (nnz > 0 && !row_stats) return COGDL_ERR_INVALID;
    return gat_backward_impl(n_rows, n_cols, nnz, rowptr, col, colptr, row_t, perm, H, D, s_dst, s_src,
                             negative_slope, nullptr, row_stats, X, x_dtype, dY, dy_dtype, dX, dx_dtype,
                             dalpha, dscore, ds_dst, ds_src, edge_work, plan, plan_t, stream);
}

}  // extern "C"
