// What the launches of product.hip and product_leaf.hip share: the error of a product against the score it stands for, the
// decoding of points into operands of v_mfma_f32_32x32x16_f16, selections by histogram and by counting.
#pragma once
#include "avq_internal.h"
#include "wave_topk.h"

namespace avq {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));


// entries (lanes with a kept point among 16) that a wave collects in LDS; 32 x 32 products add 64 at most
__host__ __device__ constexpr int product_pend(int steps) { return steps <= 14 ? 128 : 96; }
__host__ __device__ constexpr int product_qt(int steps) { return steps <= 7 ? 2 : 1; } // tiles of 32 queries in a stage
__host__ __device__ constexpr int product_ahead(int steps) { return steps <= 7 ? steps : steps == 10 ? 5 : steps == 14 ? 7 : 4; } // operands are read from LDS this many steps ahead; divides steps

constexpr int kProductMaxClasses = 32768;

inline int product_steps(int d) // steps of 16 dimensions, as a kernel has them
{
    const int s = (d + 15) / 16;
    return s <= 8 ? s : s + (s & 1);
}
inline int product_ct(int steps) { return steps <= 8 ? 4 : 2; }

struct ProductMeta { float xn, xe; int32_t exp; int32_t bad; }; // scaled: largest norm of a decoded point and of its conversion error
struct ProductQuery { float qn, qe; int32_t exp; int32_t bad; };
static_assert(sizeof(ProductMeta) <= kProductInfoBytes && sizeof(ProductQuery) <= kProductInfoBytes, "scratch");

// Norms from fp32 sums of squares: 2^-23 per term and the root's rounding are within the factor.
__device__ __forceinline__ float product_norm(float n2) { return 1.0002f * sqrtf(n2); }

// |p - s| in scaled units. Conversions: |<q, x> - <q', x'>| <= qn xe + qe (xn + xe). Sums of d products in fp32: the
// product's (from -T up: twice the magnitude) and the tables', 2^-23 a term. f16 subnormals, should they be flushed:
// 2^-14 a coordinate. fp32 results that underflow: 2^-126 a term in the unscaled scores. 8-bit tables: the integer sum is
// within half a unit a subspace (and the rounding of three fp32 operations on it) of the real one.
__device__ __forceinline__ float product_error(const ProductQuery &q, const ProductMeta &c, int d, int M, float unit)
{
    const float terms = (float)(d + M + 8), xn = c.xn, xe = c.xe;
    const float conv = q.qn * xe + q.qe * (xn + xe);
    const float acc = 3.0f * terms * 1.2e-7f * (q.qn + q.qe) * (xn + xe);
    const float flush = 6.2e-5f * sqrtf(terms) * (q.qn + q.qe + xn + xe);
    const float under = ldexpf(terms, q.exp + c.exp - 126);
    return 1.001f * (conv + acc + flush) + under + (unit > 0.0f ? 1.001f * ldexpf(unit, q.exp + c.exp) * (float)M * 0.5002f : 0.0f);
}

// This wave's points, CT x 32 of them, `apart` points from one 32 to the next, as operands. Their code bytes come to LDS first,
// as do 4-bit dictionaries (into `spare`, ROOM bytes of the workgroup's, or `pend`, BUF bytes of the wave's; left in memory where
// those are too small), so that a step waits for memory once, not at every byte and codeword. One body for all steps (as
// straight-line code for every kind of subspace they were 21,000 instructions), so that a step's registers are chosen by
// comparing its number. 10,000,000 x 128 points, 1,024 queries: 3.3 ms with the bytes and codewords read from memory, 2.7 this way.
// Called by the whole workgroup (a barrier in it).
template <int NS, int CT, int WAVES, int ROOM, int BUF>
__device__ __forceinline__ void product_decode(v8h (&a)[CT][NS], const ProductParams &p, int64_t first, int64_t apart, uint8_t *spare, uint4 *pend)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const int ds = p.d / p.M, kc = 1 << p.bits, nfull = p.NB / 4, tails = p.NB % 4;
    const uint32_t inv = ((1u << 20) + (uint32_t)ds - 1u) / (uint32_t)ds; // l / ds = l * inv >> 20 for l < 512
    const int own = CT * 32 * p.NB, all = WAVES * own;             // bytes of codes: a wave's, the workgroup's
    const int cb_bytes = kc * p.d * 2;
    const bool near = all <= ROOM;
    auto point = [&](int c, int i) -> int64_t { const int64_t at = first + c * apart + i; return at < p.n ? at : p.n - 1; }; // beyond the end: copies of the last one, not kept
    if (near) {
        uint8_t *const mine = spare + wave * own; // [CT][row of four planes: 8 slots of 16 bytes; plane: 8 of 4]
        for (int e = lane; e < CT * nfull * 8; e += 64) {
            const int c = e / (nfull * 8), r = e / 8 % nfull, g = e & 7;
            const int64_t i = first + c * apart + 4 * g; // whole blocks of 256 are there; the last one's points beyond n are zero
            const int64_t block = i >> 8 < (p.n + 255) >> 8 ? i >> 8 : 0;
            *(uint4 *)(mine + c * 32 * p.NB + r * 128 + g * 16) = *(const uint4 *)(p.codes + (size_t)block * 256 * p.NB + r * 1024 + ((i & 255) >> 2) * 16);
        }
        for (int e = lane; e < CT * tails * 8; e += 64) {
            const int c = e / (tails * 8), r = e / 8 % tails, g = e & 7;
            const int64_t i = first + c * apart + 4 * g;
            const int64_t block = i >> 8 < (p.n + 255) >> 8 ? i >> 8 : 0;
            *(uint32_t *)(mine + c * 32 * p.NB + nfull * 128 + r * 32 + g * 4) =
                *(const uint32_t *)(p.codes + (size_t)block * 256 * p.NB + nfull * 1024 + r * 256 + ((i & 255) >> 2) * 4);
        }
    }
    const _Float16 *cb16 = (const _Float16 *)p.cb16;
    if (cb_bytes <= 8192) { // 4-bit dictionaries (16-byte pieces: kc is 16)
        uint4 *to = nullptr;
        int from = 0, step = 0;
        if (near && all + cb_bytes <= ROOM) { to = (uint4 *)(spare + all); from = tid; step = WAVES * 64; }
        else if (cb_bytes <= BUF) { to = pend; from = lane; step = 64; }
        if (to != nullptr) {
            for (int e = from; e < cb_bytes / 16; e += step) to[e] = ((const uint4 *)p.cb16)[e];
            cb16 = (const _Float16 *)to;
        }
    }
    __syncthreads();
    const uint8_t *at[CT]; // the point's byte of plane 0
    int slot[CT];
    const int row = near ? 128 : 1024, plane = near ? 32 : 256; // bytes from one to the next
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int64_t i = point(c, j);
        slot[c] = near ? j >> 2 : (int)(i & 255) >> 2;
        at[c] = near ? spare + wave * own + c * 32 * p.NB + (j & 3) : p.codes + (size_t)(i >> 8) * 256 * p.NB + (i & 3);
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int k = 0; k < NS; ++k) a[c][k] = v8h{};
#pragma unroll 1
    for (int s = 0; s < NS; ++s) {
        const int l0 = 16 * s + 8 * h;
        auto word_of = [&](int c, int m) -> size_t { // of the dictionaries, for subspace m
            const int b = p.bits == 8 ? m : m >> 1;
            const int v = at[c][b < 4 * nfull ? (b >> 2) * row + slot[c] * 16 + (b & 3) * 4 : nfull * row + (b - 4 * nfull) * plane + slot[c] * 4];
            return (size_t)(m * kc + (p.bits == 8 ? v : (m & 1 ? v >> 4 : v & 15)));
        };
        v8h o[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) o[c] = v8h{};
        if (ds % 8 == 0) {
            const int m = (int)((uint32_t)l0 * inv >> 20);
            if (l0 < p.d)
#pragma unroll
                for (int c = 0; c < CT; ++c) o[c] = *(const v8h *)(cb16 + word_of(c, m) * ds + (l0 - m * ds));
        } else if (ds == 4) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (l0 + 4 * u >= p.d) continue;
                    const v4h w = *(const v4h *)(cb16 + word_of(c, l0 / 4 + u) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[c][4 * u + e] = w[e];
                }
        } else if (ds == 2) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (l0 + 2 * u >= p.d) continue;
                    const v2h w = *(const v2h *)(cb16 + word_of(c, l0 / 2 + u) * 2);
                    o[c][2 * u] = w[0];
                    o[c][2 * u + 1] = w[1];
                }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int l = l0 + u, m = (int)((uint32_t)l * inv >> 20);
                if (l >= p.d) continue;
#pragma unroll
                for (int c = 0; c < CT; ++c) o[c][u] = cb16[word_of(c, m) * ds + (l - m * ds)];
            }
        }
#pragma unroll
        for (int k = 0; k < NS; ++k)
            if (s == k)
#pragma unroll
                for (int c = 0; c < CT; ++c) a[c][k] = o[c];
    }
}

// What the refinement takes of a query: kept points, and of those the ones within 2 E of the R-th largest product. The
// rounding of 8-bit tables lets through several times R, that of f16 a few more than R.
template <bool U8> struct ProductRoom { static constexpr int kept = U8 ? 8192 : 4096, final = U8 ? 4096 : 2048; };

// Ranks by counting: out[rank] = key for the `want` largest of n distinct keys in LDS (keys[n] = 0 for n odd).
template <int PER>
__device__ __forceinline__ void rank_per(const u64 *keys, int n, int want, u64 *out, int tid)
{
    u64 mine[PER];
    int rank[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = tid + k * 256;
        mine[k] = i < n ? keys[i] : ~0ull;
        rank[k] = 0;
    }
    for (int t = 0; t < n; t += 2) {
        const ulonglong2 two = *(const ulonglong2 *)(keys + t);
#pragma unroll
        for (int k = 0; k < PER; ++k) rank[k] += (int)(two.x > mine[k]) + (int)(two.y > mine[k]);
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (tid + k * 256 < n && rank[k] < want) out[rank[k]] = mine[k];
}

template <int MOST>
__device__ __forceinline__ void rank_keys(const u64 *keys, int n, int want, u64 *out, int tid)
{
    if (n <= 256) rank_per<1>(keys, n, want, out, tid);
    else if (n <= 512) rank_per<2>(keys, n, want, out, tid);
    else if (n <= 1024) rank_per<4>(keys, n, want, out, tid);
    else rank_per<MOST / 256>(keys, n, want, out, tid);
}

// The smallest ordering value of the bin, of 256 between `from` and the largest value, that holds the R-th largest of `total`
// values at(i) that reach `from` (0: fewer than R do). hist: cleared. 256 threads; ends with a barrier.
struct BinScratch { uint32_t hist[256], wave_hi[4], wave_sum[4], found; };
template <class At>
__device__ __forceinline__ uint32_t rth_bin(BinScratch &b, uint32_t total, uint32_t from, uint32_t R, int tid, At at)
{
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t hi = 0u;
    for (uint32_t i = tid; i < total; i += 256u) { const uint32_t v = at(i); hi = v > hi ? v : hi; }
    for (int s = 32; s > 0; s >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)hi, s, 64);
        hi = o > hi ? o : hi;
    }
    if (lane == 0) b.wave_hi[wave] = hi;
    if (tid == 0) b.found = 0u;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) hi = b.wave_hi[w] > hi ? b.wave_hi[w] : hi;
    if (hi < from) return 0u; // of the whole workgroup
    const uint32_t range = hi - from;
    const int shift = range > 255u ? 24 - __clz((int)range) : 0; // range >> shift: at most 255
    for (uint32_t i = tid; i < total; i += 256u) {
        const uint32_t v = at(i);
        if (v >= from) atomicAdd(&b.hist[(v - from) >> shift], 1u);
    }
    __syncthreads();
    const uint32_t own = b.hist[tid];
    uint32_t suf = own; // of this bin and those above it
    for (int m = 1; m < 64; m <<= 1) {
        const uint32_t o = (uint32_t)__shfl_down((int)suf, m, 64);
        if (lane + m < 64) suf += o;
    }
    if (lane == 0) b.wave_sum[wave] = suf;
    __syncthreads();
    for (int w = wave + 1; w < 4; ++w) suf += b.wave_sum[w];
    if (suf >= R && suf - own < R) b.found = from + ((uint32_t)tid << shift);
    __syncthreads();
    return b.found;
}

} // namespace avq
