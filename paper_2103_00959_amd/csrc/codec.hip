// Activation compression: per-group b-bit quantization with stochastic
// rounding, the technique the paper extends to GNN training to shrink the
// activations kept for the backward pass (2, 3 and 4 bits in its evaluation).
//
// Format (n x F activations, groups of G consecutive features of a row, G a
// multiple of 64, the last group of a row possibly shorter):
//   stats[2g], stats[2g + 1] = (m, r): the group minimum and its step
//     r = (M - m) / (2^b - 1)  (0 for a constant group);
//   codes: per group, G / 64 blocks of b uint64 bit planes; plane p of a
//     block holds bit p of the codes of its 64 consecutive features.
// Encoding of x (flat index e = i * F + f), all in fp32:
//   q = clamp(floor(fma(x - m, s, u)), 0, 2^b - 1),  s = (2^b - 1) / (M - m),
// u the uniform of e from Philox4x32-10 (Salmon et al., SC 2011) at counter
// (e / 4, 0, 0) and key = seed, word e mod 4, top 24 bits times 2^-24.
// Decoding: x' = fma(q, r, m), an unbiased estimate of x within one step.
//
// Mapping on gfx950.  Groups of a power of two up to 4096 (rows of any width and alignment
// up to 512): 8 consecutive features per lane in 16-byte vectors, a group on G / 8
// adjacent lanes (several groups per wavefront), min/max by a butterfly within the group,
// each lane writing its byte of the planes of its 64-feature block; a kernel per code
// width, so that no plane past it is formed.  Other groups: a wavefront per group, one
// feature per lane, each block's b bit planes as b wavefront ballots.  Either way a
// group of bf16 features reads 2G bytes and writes G b / 8 + 8.
//
// Compression is bound by its vector instructions (Philox: 35 v_mad_u64_u32 and 36
// three-input xors for 8 features, then quantizing and packing), decompression by its
// stores.  2.4M x 256 bf16 at 2 bits: with planes handled for any width, planes assembled
// by lane exchanges, two-input xors and bf16 rounded by integer steps 0.66 and 0.44 ms;
// now 0.52 and 0.33 ms (1.4 GB each way).
#include "common.hpp"
#include "internal.hpp"

namespace cogdl {
namespace {

constexpr int kBlock = 256;

// a ^ b ^ c in one instruction (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// The four words of Philox4x32-10 at counter (c, 0, 0) (c = lo + 2^32 hi, the element
// index / 4) with key = seed.  Each 32 x 32 -> 64-bit product is one v_mad_u64_u32
// (separate high and low multiplies took 9% longer); the second and third counter words
// being zero leaves one product in the first round and, for a wave-uniform hi, one vector
// product in the second.
__device__ __forceinline__ uint4 philox4(uint64_t seed, uint32_t lo, uint32_t hi)
{
    uint32_t c0 = lo, c1 = hi, c2 = 0u, c3 = 0u;
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = round == 0 ? c1 ^ k0 : xor3(hi1, c1, k0);
        const uint32_t n2 = round == 0 ? hi0 ^ k1 : xor3(hi0, c3, k1);
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

__device__ __forceinline__ uint32_t philox_word(uint64_t seed, int64_t e)
{
    const uint4 r = philox4(seed, (uint32_t)(e >> 2), (uint32_t)(e >> 34));
    const int w = (int)(e & 3);
    return w == 0 ? r.x : w == 1 ? r.y : w == 2 ? r.z : r.w;
}

__device__ __forceinline__ float uniform24(uint32_t r) { return (float)(r >> 8) * (1.0f / 16777216.0f); }

__device__ __forceinline__ float wave_min(float v)
{
    return group_reduce(v, kWave, [](float a, float b) { return fminf(a, b); });
}

__device__ __forceinline__ float wave_max(float v)
{
    return group_reduce(v, kWave, [](float a, float b) { return fmaxf(a, b); });
}

struct CodecArgs {
    int64_t n;
    int32_t F;
    int32_t bits;
    int32_t G;
    int32_t ng;       // groups per row
    uint64_t seed;
    const void *A;
    uint64_t *codes;
    float *stats;
};

template <typename TA>
__global__ __launch_bounds__(kBlock) void k_compress(CodecArgs a)
{
    const int lane = lane_id();
    const int64_t groups = a.n * a.ng;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    const int nb = a.G / kWave;
    const float qmax = (float)((1 << a.bits) - 1);
    const TA *__restrict__ A = static_cast<const TA *>(a.A);
    for (int64_t g = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; g < groups;
         g += waves) {
        const int64_t i = g / a.ng;
        const int f0 = (int)(g % a.ng) * a.G;
        const int len = a.F - f0 < a.G ? a.F - f0 : a.G;
        const int64_t base = i * a.F + f0;
        float lo = INFINITY, hi = -INFINITY;
        for (int j = lane; j < len; j += kWave) {
            float x[1];
            load_vec<TA, 1>(A, base + j, x);
            lo = fminf(lo, x[0]);
            hi = fmaxf(hi, x[0]);
        }
        const float m = wave_min(lo), M = wave_max(hi);
        const float range = M - m;
        const float s = range > 0.f ? qmax / range : 0.f;
        const float r = range > 0.f ? range / qmax : 0.f;
        if (lane == 0) {
            a.stats[2 * g] = m;
            a.stats[2 * g + 1] = r;
        }
        uint64_t *__restrict__ w = a.codes + g * (int64_t)nb * a.bits;
        for (int t = 0; t < nb; ++t) {
            const int j = t * kWave + lane;
            uint32_t q = 0;
            if (j < len) {
                float x[1];
                load_vec<TA, 1>(A, base + j, x);
                const float u = uniform24(philox_word(a.seed, base + j));
                float v = floorf(fmaf(x[0] - m, s, u));
                v = v < 0.f ? 0.f : (v > qmax ? qmax : v);
                q = (uint32_t)v;
            }
            for (int p = 0; p < a.bits; ++p) {
                const uint64_t plane = __ballot((q >> p) & 1u);
                if (lane == p) w[(int64_t)t * a.bits + p] = plane;
            }
        }
    }
}

template <typename TO>
__global__ __launch_bounds__(kBlock) void k_decompress(int64_t n, int F, int bits, int G, int ng,
                                                       const uint64_t *__restrict__ codes,
                                                       const float *__restrict__ stats,
                                                       TO *__restrict__ out)
{
    const int lane = lane_id();
    const int64_t groups = n * ng;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    const int nb = G / kWave;
    for (int64_t g = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; g < groups;
         g += waves) {
        const int64_t i = g / ng;
        const int f0 = (int)(g % ng) * G;
        const int len = F - f0 < G ? F - f0 : G;
        const float m = stats[2 * g], r = stats[2 * g + 1];
        const uint64_t *__restrict__ w = codes + g * (int64_t)nb * bits;
        for (int t = 0; t < nb; ++t) {
            const int j = t * kWave + lane;
            uint32_t q = 0;
            for (int p = 0; p < bits; ++p)
                q |= (uint32_t)((w[(int64_t)t * bits + p] >> lane) & 1u) << p;
            if (j < len) {
                const float v[1] = {fmaf((float)q, r, m)};
                store_out<TO, 1>(out, i * F + f0 + j, v);
            }
        }
    }
}

cogdl_status check_codec(int64_t n, int32_t F, int32_t bits, int32_t group)
{
    if (n < 0 || F < 1 || bits < 1 || bits > 8 || group < kWave || group % kWave != 0)
        return COGDL_ERR_INVALID;
    return COGDL_OK;
}

unsigned codec_grid(int64_t groups)
{
    int64_t b = (groups + (kBlock / kWave) - 1) / (kBlock / kWave);
    if (b > 65536) b = 65536;
    if (b < 1) b = 1;
    return (unsigned)b;
}

// ------------------------------------------------ vectorized path
// Each lane holds 8 consecutive features, a group is LG = G / (8 NV) adjacent
// lanes (8 to 64) holding NV vectors each, so a wavefront reads and writes
// full 16-byte vectors and covers 64 / LG groups at a time.  A 64-feature
// block of codes is 8 lanes, each writing one byte per bit plane (its 8 codes).

template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> {
    __device__ static void load(const bf16_t *p, int64_t i, float (&o)[8]) { load_vec<bf16_t, 8>(p, i, o); }
    __device__ static void store(bf16_t *p, int64_t i, const float (&v)[8]) { store_vec<bf16_t, 8>(p, i, v); }
};
template <> struct Vec8<f16_t> {
    __device__ static void load(const f16_t *p, int64_t i, float (&o)[8]) { load_vec<f16_t, 8>(p, i, o); }
    __device__ static void store(f16_t *p, int64_t i, const float (&v)[8]) { store_vec<f16_t, 8>(p, i, v); }
};
template <> struct Vec8<float> {
    __device__ static void load(const float *p, int64_t i, float (&o)[8])
    {
        float lo[4], hi[4];
        load_vec<float, 4>(p, i, lo);
        load_vec<float, 4>(p, i + 4, hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) { o[e] = lo[e]; o[4 + e] = hi[e]; }
    }
    __device__ static void store(float *p, int64_t i, const float (&v)[8]) { store_vec<float, 8>(p, i, v); }
};

// Group g of the activations: the flat index of its first feature and its length.
struct RowSpan {
    int64_t base;
    int len;
};

template <bool RAG>
__device__ __forceinline__ RowSpan row_span(int64_t g, int G, int F, int ng)
{
    if constexpr (!RAG) return {g * G, G};
    int64_t i = g;
    int j = 0;
    if (ng > 1) {
        if (g <= INT32_MAX) i = (int64_t)((uint32_t)g / (uint32_t)ng);
        else i = g / ng;
        j = (int)(g - i * ng);
    }
    const int left = F - j * G;
    return {i * F + (int64_t)j * G, left < G ? left : G};
}

// How many of features [8 sl, 8 sl + 8) lie below len.
__device__ __forceinline__ int span_of(int len, int sl)
{
    const int m = len - 8 * sl;
    return m < 0 ? 0 : (m > 8 ? 8 : m);
}

// BITS: the code width, 0 for any (a.bits).  RAG (one vector a lane): any row width and
// alignment; the last group of a row may be shorter, a lane's features past it take its
// first one for the minimum and maximum and code 0, and the Philox words of 8 features
// off the 4-feature grid come from three blocks.
template <typename TA, int NV, int BITS, bool RAG>
__global__ __launch_bounds__(kBlock) void k_compress_v(CodecArgs a)
{
    const int bits = BITS > 0 ? BITS : a.bits;
    const int lane = lane_id();
    const int LG = a.G / (8 * NV);
    const int sl = lane & (LG - 1);
    const int per_wave = kWave / LG;
    const int64_t groups = a.n * a.ng;
    const int64_t wave = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const int64_t stride = (int64_t)gridDim.x * (kBlock / kWave) * per_wave;
    const float qmax = (float)((1 << bits) - 1);
    const int nb = a.G / kWave;
    const TA *__restrict__ A = static_cast<const TA *>(a.A);
    for (int64_t g = wave * per_wave + lane / LG; g - lane / LG < groups; g += stride) {
        const bool gok = g < groups;
        // the flat index of feature j of the group is base + j
        const RowSpan row = row_span<RAG>(g, a.G, a.F, a.ng);
        const int64_t base = row.base;
        const int mine = RAG ? (gok ? span_of(row.len, sl) : 0) : 8;   // features of this lane in the group
        float x[NV][8];
        float lo = INFINITY, hi = -INFINITY;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            if (RAG ? mine == 8 : gok) {
                Vec8<TA>::load(A, base + (int64_t)(v * LG + sl) * 8, x[v]);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float one[1] = {0.f};
                    if (RAG && mine > 0) load_vec<TA, 1>(A, base + sl * 8 + (e < mine ? e : 0), one);
                    x[v][e] = one[0];
                }
            }
            if (RAG && mine == 0) continue;
#pragma unroll
            for (int e = 0; e < 8; ++e) {         // (a group past the end writes nothing)
                lo = fminf(lo, x[v][e]);
                hi = fmaxf(hi, x[v][e]);
            }
        }
        lo = group_reduce(lo, LG, [](float u, float v) { return fminf(u, v); });
        hi = group_reduce(hi, LG, [](float u, float v) { return fmaxf(u, v); });
        const float range = hi - lo;
        const float s = range > 0.f ? qmax / range : 0.f;
        const float r = range > 0.f ? range / qmax : 0.f;
        if (gok && sl == 0) {
            a.stats[2 * g] = lo;
            a.stats[2 * g + 1] = r;
        }
        uint64_t *__restrict__ w = a.codes + g * (int64_t)nb * bits;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int64_t e0 = base + (int64_t)(v * LG + sl) * 8;
            uint32_t rw[8];                       // the 8 words of these features
            if constexpr (RAG) {
                const uint64_t c = (uint64_t)e0 >> 2;
                const uint4 r0 = philox4(a.seed, (uint32_t)c, (uint32_t)(c >> 32));
                const uint4 r1 = philox4(a.seed, (uint32_t)(c + 1), (uint32_t)((c + 1) >> 32));
                const int s = (int)(e0 & 3);
                uint4 r2 = make_uint4(0u, 0u, 0u, 0u);
                if (s != 0) r2 = philox4(a.seed, (uint32_t)(c + 2), (uint32_t)((c + 2) >> 32));
                const uint32_t w[11] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w, r2.x, r2.y, r2.z};
                // words s to s + 7 by masks: written as ?: the compiler indexes w in memory (48
                // bytes of scratch and 11 KB of LDS; at 2 bits 3000 x 1000 bf16 22 us a call, now 14,
                // 1M x 300 in groups of 512 1249 and 787)
                const uint32_t by1 = 0u - (uint32_t)(s & 1), by2 = 0u - (uint32_t)(s >> 1);
                uint32_t w1[10];
#pragma unroll
                for (int e = 0; e < 10; ++e) w1[e] = (w[e + 1] & by1) | (w[e] & ~by1);
#pragma unroll
                for (int e = 0; e < 8; ++e) rw[e] = (w1[e + 2] & by2) | (w1[e] & ~by2);
            } else {
                // e0 is a multiple of 8: two Philox blocks of 4.  A wavefront's features are
                // one aligned span of 512 NV (a power of two), so the high word of the
                // counter is the same in every lane.
                const uint32_t clo = (uint32_t)((uint64_t)e0 >> 2);
                const uint32_t chi = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint64_t)e0 >> 34));
                const uint4 r0 = philox4(a.seed, clo, chi);
                const uint4 r1 = philox4(a.seed, clo + 1, chi);
                const uint32_t w[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) rw[e] = w[e];
            }
            uint32_t q[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float u = uniform24(rw[e]);
                // the clamp to [0, qmax] as one median of three (t is finite); the conversion
                // truncates, which is the floor of a value that is not negative
                q[e] = (uint32_t)__builtin_amdgcn_fmed3f(fmaf(x[v][e] - lo, s, u), 0.f, qmax);
            }
            const int blk = (v * LG + sl) / 8;     // 64-feature block of these 8 features
            const int byte = sl & 7;               // their byte within the block's planes
            // each lane writes its own byte of every plane: the 8 lanes of a block fill a
            // word together
            uint8_t *__restrict__ w8 = reinterpret_cast<uint8_t *>(w + (int64_t)blk * bits) + byte;
#pragma unroll
            for (int p = 0; p < (BITS > 0 ? BITS : 8); ++p) {
                if (p >= bits) break;
                uint32_t frag = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) frag |= ((q[e] >> p) & 1u) << e;
                if constexpr (RAG) frag &= (1u << mine) - 1u;
                if (gok) w8[8 * p] = (uint8_t)frag;
            }
        }
    }
}

template <typename TO, int NV, int BITS, bool RAG>
__global__ __launch_bounds__(kBlock) void k_decompress_v(int64_t n, int F, int any_bits, int G, int ng,
                                                         const uint64_t *__restrict__ codes,
                                                         const float *__restrict__ stats,
                                                         TO *__restrict__ out)
{
    constexpr int PL = BITS > 0 ? BITS : 8;      // planes held (any_bits of them used)
    const int bits = BITS > 0 ? BITS : any_bits;
    const int lane = lane_id();
    const int LG = G / (8 * NV);
    const int sl = lane & (LG - 1);
    const int per_wave = kWave / LG;
    const int64_t groups = n * ng;
    const int64_t wave = (int64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave;
    const int64_t stride = (int64_t)gridDim.x * (kBlock / kWave) * per_wave;
    const int nb = G / kWave;
    const int byte = sl & 7;   // this lane's byte of each plane word of its block
    const uint32_t *__restrict__ c32 = reinterpret_cast<const uint32_t *>(codes);
    // a group's stats and, per vector and plane, the 32-bit half of the plane
    // word that holds this lane's byte; fetched one group ahead
    const auto fetch = [&](int64_t g, float &m, float &r, uint32_t (&h)[NV][PL]) {
        m = stats[2 * g];
        r = stats[2 * g + 1];
        const int64_t w0 = g * (int64_t)nb * bits;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int blk = (v * LG + sl) / 8;
#pragma unroll
            for (int p = 0; p < PL; ++p)
                h[v][p] = p < bits ? c32[2 * (w0 + (int64_t)blk * bits + p) + (byte >> 2)] : 0u;
        }
    };
    int64_t g = wave * per_wave + lane / LG;
    float mn = 0.f, rn = 0.f;
    uint32_t hn[NV][PL] = {};
    if (g < groups) fetch(g, mn, rn, hn);
    for (; g - lane / LG < groups; g += stride) {
        const bool gok = g < groups;
        const float m = mn, r = rn;
        uint32_t h[NV][PL];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int p = 0; p < PL; ++p) h[v][p] = hn[v][p];
        if (g + stride < groups) fetch(g + stride, mn, rn, hn);
        if (!gok) continue;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            uint32_t q[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
#pragma unroll
            for (int p = 0; p < PL; ++p) {
                const uint32_t b8 = (h[v][p] >> (8 * (byte & 3))) & 0xffu;
#pragma unroll
                for (int e = 0; e < 8; ++e) q[e] |= ((b8 >> e) & 1u) << p;
            }
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = fmaf((float)q[e], r, m);
            const RowSpan row = row_span<RAG>(g, G, F, ng);
            const int mine = RAG ? span_of(row.len, sl) : 8;
            const int64_t at = row.base + (int64_t)(v * LG + sl) * 8;
            if (mine == 8) {
                Vec8<TO>::store(out, at, y);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float one[1] = {y[e]};
                    if (e < mine) store_out<TO, 1>(out, at + e, one);
                }
            }
        }
    }
}

using CompressKernel = void (*)(CodecArgs);

// One vector a lane (groups up to 512; rag: of any row): a kernel per code width.  Larger
// groups of whole aligned rows: any width.
template <typename TA, bool RAG>
CompressKernel pick_compress_1(int bits)
{
    constexpr CompressKernel k[8] = {k_compress_v<TA, 1, 1, RAG>, k_compress_v<TA, 1, 2, RAG>,
                                     k_compress_v<TA, 1, 3, RAG>, k_compress_v<TA, 1, 4, RAG>,
                                     k_compress_v<TA, 1, 5, RAG>, k_compress_v<TA, 1, 6, RAG>,
                                     k_compress_v<TA, 1, 7, RAG>, k_compress_v<TA, 1, 8, RAG>};
    return k[bits - 1];
}

template <typename TA>
CompressKernel pick_compress_v(int nv, int bits, bool rag)
{
    if (rag) return pick_compress_1<TA, true>(bits);
    if (nv == 1) return pick_compress_1<TA, false>(bits);
    if (nv == 2) return k_compress_v<TA, 2, 0, false>;
    if (nv == 4) return k_compress_v<TA, 4, 0, false>;
    return k_compress_v<TA, 8, 0, false>;
}

template <typename TO>
using DecompressKernel = void (*)(int64_t, int, int, int, int, const uint64_t *, const float *, TO *);

template <typename TO, bool RAG>
DecompressKernel<TO> pick_decompress_1(int bits)
{
    constexpr DecompressKernel<TO> k[8] = {k_decompress_v<TO, 1, 1, RAG>, k_decompress_v<TO, 1, 2, RAG>,
                                           k_decompress_v<TO, 1, 3, RAG>, k_decompress_v<TO, 1, 4, RAG>,
                                           k_decompress_v<TO, 1, 5, RAG>, k_decompress_v<TO, 1, 6, RAG>,
                                           k_decompress_v<TO, 1, 7, RAG>, k_decompress_v<TO, 1, 8, RAG>};
    return k[bits - 1];
}

template <typename TO>
DecompressKernel<TO> pick_decompress_v(int nv, int bits, bool rag)
{
    if (rag) return pick_decompress_1<TO, true>(bits);
    if (nv == 1) return pick_decompress_1<TO, false>(bits);
    if (nv == 2) return k_decompress_v<TO, 2, 0, false>;
    if (nv == 4) return k_decompress_v<TO, 4, 0, false>;
    return k_decompress_v<TO, 8, 0, false>;
}

// Vectors per lane of the vectorized kernels (0: not applicable; a group's lanes are a
// power of two), and whether rows are ragged or unaligned.
struct VectorMap {
    int nv;
    bool rag;
};

VectorMap vector_map(int32_t F, int32_t group, const void *p)
{
    const bool rag = F % group != 0 || (uintptr_t)p % 16 != 0;
    if ((group & (group - 1)) != 0 || group > (rag ? 512 : 4096)) return {0, false};
    return {group > 512 ? group / 512 : 1, rag};
}

}  // namespace
}  // namespace cogdl

using namespace cogdl;

extern "C" {

cogdl_status cogdl_act_codec_size(int64_t n, int32_t F, int32_t bits, int32_t group,
                                  int64_t *code_words, int64_t *stat_floats)
{
    cogdl_status st = check_codec(n, F, bits, group);
    if (st != COGDL_OK) return st;
    if (!code_words || !stat_floats) return COGDL_ERR_INVALID;
    const int64_t ng = (F + group - 1) / group;
    *code_words = n * ng * (group / kWave) * bits;
    *stat_floats = n * ng * 2;
    return COGDL_OK;
}

cogdl_status cogdl_act_compress(int64_t n, int32_t F, const void *A, cogdl_dtype a_dtype,
                                int32_t bits, int32_t group, uint64_t seed, uint64_t *codes,
                                float *stats, hipStream_t stream)
{
    cogdl_status st = check_codec(n, F, bits, group);
    if (st != COGDL_OK) return st;
    if (!dtype_ok(a_dtype)) return COGDL_ERR_DTYPE;
    if (n > 0 && (!A || !codes || !stats)) return COGDL_ERR_INVALID;
    if (n == 0) return COGDL_OK;
    CodecArgs a{n, F, bits, group, (F + group - 1) / group, seed, A, codes, stats};
    const unsigned b = codec_grid(n * a.ng);
    const auto [nv, rag] = vector_map(F, group, A);
    if (nv > 0) {
        const int per_wave = kWave / (group / (8 * nv));
        CompressKernel k = a_dtype == COGDL_F32    ? pick_compress_v<float>(nv, bits, rag)
                           : a_dtype == COGDL_BF16 ? pick_compress_v<bf16_t>(nv, bits, rag)
                                                   : pick_compress_v<f16_t>(nv, bits, rag);
        // a grid past the resident size, no prefetch: a resident grid walking the
        // groups with the next one fetched ahead measured 10-15% slower here
        const unsigned bv = codec_grid((n * a.ng + per_wave - 1) / per_wave);
        COGDL_LAUNCH("act_compress", k, bv, kBlock, stream, a);
        return COGDL_OK;
    }
    if (a_dtype == COGDL_F32)
        COGDL_LAUNCH("act_compress", k_compress<float>, b, kBlock, stream, a);
    else if (a_dtype == COGDL_BF16)
        COGDL_LAUNCH("act_compress", k_compress<bf16_t>, b, kBlock, stream, a);
    else
        COGDL_LAUNCH("act_compress", k_compress<f16_t>, b, kBlock, stream, a);
    return COGDL_OK;
}

cogdl_status cogdl_act_decompress(int64_t n, int32_t F, int32_t bits, int32_t group,
                                  const uint64_t *codes, const float *stats, void *out,
                                  cogdl_dtype out_dtype, hipStream_t stream)
{
    cogdl_status st = check_codec(n, F, bits, group);
    if (st != COGDL_OK) return st;
    if (!dtype_ok(out_dtype)) return COGDL_ERR_DTYPE;
    if (n > 0 && (!out || !codes || !stats)) return COGDL_ERR_INVALID;
    if (n == 0) return COGDL_OK;
    const int ng = (F + group - 1) / group;
    const unsigned b = codec_grid(n * ng);
    const auto [nv, rag] = vector_map(F, group, out);
    if (nv > 0) {
        const int per_wave = kWave / (group / (8 * nv));
        const int64_t wv = (n * ng + per_wave - 1) / per_wave;
#define COGDL_DECOMP_V(TO)                                                                       \
    do {                                                                                         \
        const DecompressKernel<TO> k = pick_decompress_v<TO>(nv, bits, rag);                    \
        const unsigned bv = codec_grid(wv);    /* past the resident size: 2-4% faster */      \
        COGDL_LAUNCH("act_decompress", k, bv, kBlock, stream, n, F, bits, group, ng, codes, stats,  \
                     static_cast<TO *>(out));                                                    \
    } while (0)
        if (out_dtype == COGDL_F32) COGDL_DECOMP_V(float);
        else if (out_dtype == COGDL_BF16) COGDL_DECOMP_V(bf16_t);
        else COGDL_DECOMP_V(f16_t);
#undef COGDL_DECOMP_V
        return COGDL_OK;
    }
    if (out_dtype == COGDL_F32)
        COGDL_LAUNCH("act_decompress", k_decompress<float>, b, kBlock, stream, n, F, bits, group,
                     ng, codes, stats, static_cast<float *>(out));
    else if (out_dtype == COGDL_BF16)
        COGDL_LAUNCH("act_decompress", k_decompress<bf16_t>, b, kBlock, stream, n, F, bits, group,
                     ng, codes, stats, static_cast<bf16_t *>(out));
    else
        COGDL_LAUNCH("act_decompress", k_decompress<f16_t>, b, kBlock, stream, n, F, bits, group,
                     ng, codes, stats, static_cast<f16_t *>(out));
    return COGDL_OK;
}

}  // extern "C"
