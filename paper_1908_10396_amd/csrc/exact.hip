// Exact inner-product search (paper Section 1: argmax over the database of <q, x_i>), by way of a bf16 matrix product.
//
// The results are those of an fp32 fma chain over the coordinates in order, for every point. Only the points that can
// be among a query's k best are scored that way: the matrix cores form all inner products from bf16 operands with fp32
// sums, and every value so computed is within E of the fp32 chain (exact_bound below, from the norms and the actual
// conversion errors of the 64 points at hand and of the query). Kept per query and 64 points is the largest value a.
// With theta the k-th largest of the a - E, k blocks hold a point at or above theta each, so no point of a block with
// a + E < theta can be among the k best, ties included; the other blocks (about k of them) are scored in fp32.
//
// Where the product decides little (copies of a few rows, rows that differ by less than the bf16 rounding of what they
// have in common, a query of zeros) a query's list of blocks is long; beyond exact_max_listed the plain kernel takes that
// query, as it does one whose norm is not finite or above 1e18. need[0] != 0: every query of the launch (a point with such
// a norm), need[1 + q]: query q.
//
// 1,183,514 x 100 points, 1,000 queries, k = 10: every point in fp32 took 20.8 ms (one 4-byte load and eight fmas a
// step, bound by the issue of the loads); this way 0.51 ms (product 0.33, which reads x once: 0.12 of matrix instructions,
// 0.09 to read x; selection and fp32 scores 0.20; the plain kernel's three launches, which leave at once, 0.014).
// bf16 rather than f16, whose range needs a scale first.
#include <algorithm>
#include <type_traits>
#include "avq_internal.h"
#include "wave_topk.h"

namespace avq {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kExactGroup = 8 * 64;   // points of a workgroup: a wave holds the operands of 64
constexpr float kExactMaxNorm = 1e18f; // products and sums of coordinates stay finite

// Norms from fp32 squares: what they lose to underflow is below 1e-18 a coordinate.
__device__ __forceinline__ float exact_norm(float n2, int terms) { return 1.0001f * sqrtf(n2) + 4e-18f * (float)terms; }

// |value of the product - fp32 chain| <= this: conversions qn ex + qe (xn + ex); fp32 sums of `terms` products in any
// order, twice (2^-24 each, 2^-23 taken); bf16 subnormals, should they be flushed.
__device__ __forceinline__ float exact_bound(float qn, float qe, float xn, float xe, int terms)
{
    const float conv = qn * xe + qe * (xn + xe);
    const float acc = 2.0f * (float)terms * 1.2e-7f * (qn + qe) * (xn + xe);
    return 1.001f * (conv + acc) + 1e-37f * (float)terms * (qn + xn + 1.0f);
}

// One workgroup per tile of 32 queries: operand order [step][lane][8], lane (row lane % 32, half lane / 32) holding
// coordinates 16 step + 8 half .. + 7; padding rows are zero. qnorm[q] = (norm, norm of the conversion error). Sets need.
__global__ void __launch_bounds__(256)
exact_pack_kernel(const float *__restrict__ queries, int nq, int d, int steps, v8bf *__restrict__ packed, float2 *__restrict__ qnorm,
                  uint32_t *__restrict__ need)
{
    const int tid = threadIdx.x, t = blockIdx.x;
    if (t == 0 && tid == 0) need[0] = 0u;
    const int r = tid >> 3, g = tid & 7, q = t * 32 + r;
    float n2 = 0.0f, e2 = 0.0f;
    if (q < nq)
        for (int l = g; l < d; l += 8) {
            const float v = queries[(size_t)q * d + l], e = v - (float)(__bf16)v;
            n2 += v * v;
            e2 += e * e;
        }
    for (int s = 4; s > 0; s >>= 1) { n2 += __shfl_xor(n2, s, 64); e2 += __shfl_xor(e2, s, 64); }
    if (g == 0 && q < nq) {
        const float qn = exact_norm(n2, d);
        qnorm[q] = make_float2(qn, exact_norm(e2, d));
        need[1 + q] = qn < kExactMaxNorm ? 0u : 1u;
    }
    for (int f = tid; f < steps * 64; f += 256) {
        const int lane = f & 63, s = f >> 6, qq = t * 32 + (lane & 31);
        v8bf o;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int l = 16 * s + 8 * (lane >> 5) + i;
            o[i] = (__bf16)(qq < nq && l < d ? queries[(size_t)qq * d + l] : 0.0f);
        }
        packed[(size_t)t * steps * 64 + f] = o;
    }
}

// Eight waves of 64 points, whose operands stay in registers (x is read once), against all queries, whose tiles of 32
// go through LDS up to two ahead (x: 473 MB, queries: 224 KB at the size above). The products of one accumulator are issued
// between the instructions that take the maximum of the other one (sched_barrier keeps the order): 0.46 -> 0.42 ms at the size
// above. 14 operands of two column tiles fit 128 registers but for a few outside the loop, so that two workgroups share a compute
// unit and one's row loads overlap the other's products: 0.33 (PAIR; fewer operands fit without being told). With one workgroup
// for a compute unit, or a few queries and hence nothing to overlap, those few registers are a loss (launch_exact has the line). More
// operands would spill in the loop (one column tile of 12: 14 loads from scratch every two tiles, each of which also waits for
// the staged ones; 1,183,514 x 160, 1,000 queries, exact search whole: 1,051 us with one workgroup and products and maxima one after
// the other, 1,090 with two, 971 with one). best[q][block of 64]: the workgroup's eight
// maxima of a query leave as 32 adjacent bytes. xnorm[block] = largest norm and conversion error of its points.
// PAIR: as many registers as let two share a compute unit.
template <int NS, int CT, bool PAIR>
__global__ void __launch_bounds__(512, PAIR ? 4 : 2)
exact_product_kernel(const float *__restrict__ x, int64_t n, int d, const v8bf *__restrict__ packed, int n_tiles, int nq,
                     float *__restrict__ best, int64_t best_stride, float2 *__restrict__ xnorm, uint32_t *__restrict__ need)
{
    __shared__ __align__(16) v8bf tile[3][NS * 64];
    __shared__ __align__(16) float mx[2][32][8];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const int64_t p0 = (int64_t)blockIdx.x * (8 * CT * 32) + wave * (CT * 32);
    const bool quad = (d & 3) == 0 && ((uintptr_t)x & 15) == 0;
    auto stage = [&](int t, int slot) {
        const v8bf *src = packed + (size_t)t * NS * 64;
        for (int s = wave; s < NS; s += 8)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + s * 64 + lane),
                                             (__attribute__((address_space(3))) void *)(tile[slot] + s * 64), 16, 0, 0);
    };
    stage(0, 0);
    if (n_tiles > 1) stage(1, 1);
    v8bf a[CT][NS];
    float xn = 0.0f, xe = 0.0f;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int64_t i = p0 + c * 32 + j;
        const bool live = i < n; // padding points are copies of the last one
        const float *row = x + (size_t)(live ? i : n - 1) * d;
        float n2 = 0.0f, e2 = 0.0f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int l0 = 16 * s + 8 * h;
            float v[8];
            if (quad && l0 + 8 <= d) {
                const float4 u = *(const float4 *)(row + l0), w = *(const float4 *)(row + l0 + 4);
                v[0] = u.x; v[1] = u.y; v[2] = u.z; v[3] = u.w;
                v[4] = w.x; v[5] = w.y; v[6] = w.z; v[7] = w.w;
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = l0 + u < d ? row[l0 + u] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const __bf16 b = (__bf16)v[u];
                const float e = v[u] - (float)b;
                n2 += v[u] * v[u];
                e2 += e * e;
                a[c][s][u] = b;
            }
        }
        n2 += __shfl_xor(n2, 32, 64);
        e2 += __shfl_xor(e2, 32, 64);
        const float cn = exact_norm(n2, d), ce = exact_norm(e2, d);
        if (live && !(cn < kExactMaxNorm)) atomicOr(need, 1u);
        xn = fmaxf(xn, cn);
        xe = fmaxf(xe, ce);
    }
    for (int s = 16; s > 0; s >>= 1) { xn = fmaxf(xn, __shfl_xor(xn, s, 64)); xe = fmaxf(xe, __shfl_xor(xe, s, 64)); }
    if (lane == 0) xnorm[(size_t)blockIdx.x * 8 + wave] = make_float2(xn, xe);
    const bool any = p0 < n;

    // wave t % 8 writes tile t's maxima: two lanes per query, 16 bytes each
    auto put = [&](int t) {
        if (wave != (t & 7)) return;
        const int q = t * 32 + (lane >> 1);
        if (q < nq)
            *(float4 *)(best + (size_t)q * best_stride + (size_t)blockIdx.x * 8 + 4 * (lane & 1)) = *(const float4 *)&mx[t & 1][lane >> 1][4 * (lane & 1)];
    };
    // the largest of an accumulator, two values an instruction (the maximum of IEEE 754-2019 quiets no operand first)
    float m = -INFINITY;
    auto take = [&](const v16f &v, int q) __attribute__((always_inline)) {
        m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, v[2 * q]), v[2 * q + 1]);
    };
    // column j of tile t is query j: this lane's 16 CT points of it, then the other half's
    auto finish = [&](int t) {
        const float o = __shfl_xor(m, 32, 64);
        if (h == 0) mx[t & 1][j][wave] = any ? fmaxf(m, o) : -INFINITY;
    };
    // the products of one accumulator (H) with a tile, while the values of the other one, formed before them, are taken
    v16f acc[2], zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) { zero[v] = 0.0f; acc[0][v] = acc[1][v] = -3e38f; }
    v8bf b[NS];
    auto half = [&](auto which, const v8bf *next) __attribute__((always_inline)) {
        constexpr int H = decltype(which)::value, O = 1 - H, ch = CT == 2 ? H : 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            acc[H] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ch][s], b[s], s == 0 ? zero : acc[H], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (q * NS / 8 == s) take(acc[O], q);
            asm volatile("" : "+v"(m)); // here, not past the products that hide it
            if (CT == 1 || H == 1) b[s] = next[s * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0): this wave's part of the first tiles is in LDS
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) b[s] = tile[0][s * 64 + lane];
    int slot = 0;
    auto after = [](int s) { return s == 2 ? 0 : s + 1; };
    // the tile after t is there, and the maxima written before; every wave has left the tile before t, whose place the one after
    // next takes
    auto turn = [&](int t) {
        __builtin_amdgcn_s_waitcnt(0x0f70);
        __syncthreads();
        if (t + 2 < n_tiles) stage(t + 2, after(after(slot)));
        slot = after(slot);
    };
    // (operands read beyond the last tile are not used)
    if constexpr (CT == 2) {
#pragma unroll 1
        for (int t = 0; t < n_tiles; ++t) {
            half(std::integral_constant<int, 0>{}, nullptr);
            if (t > 0) finish(t - 1);
            m = -INFINITY;
            turn(t);
            if (t > 0) put(t - 1); // read before the next barrier; the next maxima go to the other half of mx
            half(std::integral_constant<int, 1>{}, tile[slot]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) take(acc[1], q);
    } else { // the tiles take turns with the accumulators
        auto step = [&](auto which, int t) __attribute__((always_inline)) {
            turn(t);
            if (t > 1) put(t - 2);
            half(which, tile[slot]);
            if (t > 0) finish(t - 1);
            m = -INFINITY;
        };
#pragma unroll 1
        for (int t = 0; t < n_tiles; t += 2) {
            step(std::integral_constant<int, 0>{}, t);
            if (t + 1 < n_tiles) step(std::integral_constant<int, 1>{}, t + 1);
        }
        __syncthreads();
        if (n_tiles > 1) put(n_tiles - 2);
#pragma unroll
        for (int q = 0; q < 8; ++q) take((n_tiles & 1) ? acc[0] : acc[1], q);
    }
    finish(n_tiles - 1);
    __syncthreads();
    put(n_tiles - 1);
}

// One workgroup per query: theta by two histogram passes over the ordering values of a - E (its 22 high bits, rounded
// down: a lower theta only adds blocks), then the blocks that reach it as a list, a wave per block and a lane per point,
// fp32 chain, wave lists. There are at least 4 k blocks (exact_supported). More than max_listed (at most kExactBins)
// blocks: need[1 + q] is set and the plain kernel answers.
constexpr int kExactBins = 2048;
template <int kExactThreads>
__global__ void __launch_bounds__(kExactThreads)
exact_finish_kernel(const float *__restrict__ x, int64_t n, int d, const float *__restrict__ queries, const float *__restrict__ best,
                    int64_t n_blocks, int64_t best_stride, int block_points, const float2 *__restrict__ qnorm,
                    const float2 *__restrict__ xnorm, int ns, int k, uint32_t max_listed, uint32_t *__restrict__ need,
                    int32_t *__restrict__ ids_out, float *__restrict__ scores_out)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t hist[kExactBins], wave_sum[kExactThreads / 64], found[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = blockIdx.x;
    if ((need[0] | need[1 + q]) != 0u) return;
    constexpr int nw = kExactThreads / 64;
    const int C = 64 * ns;
    u64 *lists = (u64 *)smem, *mine = lists + (size_t)wave * C;
    u64 *pend = lists + (size_t)nw * C + wave * 64;
    float *qs = (float *)(lists + (size_t)nw * (C + 64));
    for (int l = tid; l < d; l += kExactThreads) qs[l] = queries[(size_t)q * d + l];
    wave_list_clear(mine, ns);
    const float *a = best + (size_t)q * best_stride;
    const float2 qe = qnorm[q];
    auto bound = [&](int64_t b) { const float2 e = xnorm[b]; return exact_bound(qe.x, qe.y, e.x, e.y, d); };
    // the bin of 11 bits that holds the left-th largest value with the given leading bits (all values: shift 21, prefix 0)
    uint32_t prefix = 0u, left = (uint32_t)k;
    for (int pass = 0; pass < 2; ++pass) {
        for (int b = tid; b < kExactBins; b += kExactThreads) hist[b] = 0u;
        __syncthreads();
        for (int64_t b = tid; b < n_blocks; b += kExactThreads) {
            const uint32_t o = ord_from_f32(a[b] - bound(b));
            if (pass == 0) atomicAdd(&hist[o >> 21], 1u);
            else if (o >> 21 == prefix) atomicAdd(&hist[(o >> 10) & 2047u], 1u);
        }
        __syncthreads();
        uint32_t h[kExactBins / kExactThreads], sum = 0u;
#pragma unroll
        for (int i = 0; i < kExactBins / kExactThreads; ++i) { h[i] = hist[tid * (kExactBins / kExactThreads) + i]; sum += h[i]; }
        uint32_t suf = sum; // of this lane and those above it
        for (int m = 1; m < 64; m <<= 1) {
            const uint32_t o = (uint32_t)__shfl_down((int)suf, m, 64);
            if (lane + m < 64) suf += o;
        }
        if (lane == 0) wave_sum[wave] = suf;
        __syncthreads();
        uint32_t above = suf - sum;
        for (int w = wave + 1; w < nw; ++w) above += wave_sum[w];
#pragma unroll
        for (int i = kExactBins / kExactThreads - 1; i >= 0; --i) {
            if (above < left && left <= above + h[i]) {
                found[0] = (uint32_t)(tid * (kExactBins / kExactThreads) + i);
                found[1] = above;
            }
            above += h[i];
        }
        __syncthreads();
        prefix = (prefix << 11) | found[0];
        left -= found[1];
        __syncthreads();
    }
    const float theta = f32_from_ord(prefix << 10); // the values of the bin are at or above it
    uint32_t *list = hist;
    if (tid == 0) found[0] = 0u;
    __syncthreads();
    for (int64_t b = tid; b < n_blocks; b += kExactThreads)
        if (a[b] + bound(b) >= theta) {
            const uint32_t at = atomicAdd(&found[0], 1u);
            if (at < kExactBins) list[at] = (uint32_t)b;
        }
    __syncthreads();
    const uint32_t n_list = found[0];
    if (n_list > max_listed) {
        if (tid == 0) need[1 + q] = 1u;
        return;
    }
    const bool quad = (d & 3) == 0 && ((uintptr_t)x & 15) == 0;
    u64 thr = 0ull;
    int cnt = 0;
    const uint32_t per = block_points == 32 ? 2 : 1; // blocks of a wave at a time
    for (uint32_t e = wave * per; e < n_list; e += nw * per) {
        const uint32_t mine_e = e + (per == 2 ? (uint32_t)lane >> 5 : 0u);
        const int64_t i = (int64_t)list[mine_e < n_list ? mine_e : e] * block_points + (lane & (block_points - 1));
        const bool valid = mine_e < n_list && i < n;
        const float *row = x + (size_t)(valid ? i : 0) * d;
        float s = 0.0f;
        int l = 0;
        if (quad)
#pragma unroll 8
            for (; l < d; l += 4) {
                const float4 v = *(const float4 *)(row + l);
                s = __fmaf_rn(qs[l], v.x, s);
                s = __fmaf_rn(qs[l + 1], v.y, s);
                s = __fmaf_rn(qs[l + 2], v.z, s);
                s = __fmaf_rn(qs[l + 3], v.w, s);
            }
        else
#pragma unroll 8
            for (; l < d; ++l) s = __fmaf_rn(qs[l], row[l], s);
        const u64 key = make_key(ord_from_f32(s), (int32_t)i);
        if (wave_push(mine, ns, pend, cnt, valid && key > thr, key)) thr = mine[k - 1];
    }
    if (cnt > 0) wave_list_flush(mine, ns, pend, cnt);
    for (int stride = 1; stride < nw; stride *= 2) {
        __syncthreads();
        if ((wave & (2 * stride - 1)) == 0) wave_list_merge_from(mine, ns, lists + (size_t)(wave + stride) * C);
    }
    if (wave == 0)
        for (int i = lane; i < k; i += 64) {
            const u64 key = mine[i];
            ids_out[(size_t)q * k + i] = key_id(key);
            scores_out[(size_t)q * k + i] = f32_from_ord(key_ord(key));
        }
}

static int exact_steps(int d)
{
    const int need = (d + 15) / 16;
    for (int s : {2, 3, 4, 7, 8, 12, 16})
        if (need <= s) return s;
    return 0;
}
// a few queries: sixteen waves share a query's blocks; many: eight, and twice the workgroups at once
static int exact_finish_threads(int nq) { return nq < 256 ? 1024 : 512; }
static size_t exact_finish_lds(int d, int k, int threads)
{
    return (size_t)(threads / 64) * (64 * ((k + 63) / 64) + 64) * sizeof(u64) + (size_t)d * sizeof(float);
}

namespace {
struct ExactWs {
    v8bf *packed;
    float2 *qnorm, *xnorm;
    float *best;
    uint32_t *need;
    int64_t stride;
};
size_t exact_ws_layout(int64_t n, int d, int nq, unsigned char *base, ExactWs *w)
{
    size_t off = 0;
    auto take = [&](size_t bytes) -> void * {
        const size_t at = off;
        off += (bytes + 255) & ~(size_t)255;
        return base ? (void *)(base + at) : nullptr;
    };
    const int64_t group = exact_steps(d) > 8 ? kExactGroup / 2 : kExactGroup;
    w->stride = (n + group - 1) / group * 8;
    w->need = (uint32_t *)take(sizeof(uint32_t) * (1 + (size_t)nq));
    w->packed = (v8bf *)take(sizeof(v8bf) * (size_t)((nq + 31) / 32) * exact_steps(d) * 64);
    w->qnorm = (float2 *)take(sizeof(float2) * (size_t)nq);
    w->xnorm = (float2 *)take(sizeof(float2) * (size_t)w->stride);
    w->best = (float *)take(sizeof(float) * (size_t)nq * w->stride);
    return off;
}
} // namespace

size_t exact_ws_bytes(int64_t n, int d, int nq)
{
    ExactWs w;
    return exact_ws_layout(n, d, nq, nullptr, &w);
}

// Queries of one launch, whose scratch takes at most `most` bytes: 32, a multiple of it, or all.
int exact_queries_per_launch(int64_t n, int d, int nq, size_t most)
{
    const size_t fixed = exact_ws_bytes(n, d, 32), per_32 = exact_ws_bytes(n, d, 64) - fixed + 1024; // (rounded up per array)
    const int64_t fit = most > fixed ? 32 + (int64_t)((most - fixed) / per_32) * 32 : 32;
    return (int)std::min<int64_t>(nq, fit);
}

// The plain kernel alone: d beyond the operands that registers hold, lists that do not fit LDS; and where too few blocks
// can be left out for what the selection costs, or a few queries' blocks keep a few compute units busy for long. Measured,
// plain / this: 2,000 x 100, 1,000 queries, k = 100: 0.15 / 0.36 ms; 20,000 x 100, one query: k = 10 74 / 44 us, k = 300 126 / 367;
// 200,000 x 100, one query, k = 300: 0.25 / 0.43 ms, 64 queries, k = 100: 0.58 / 0.20; 1,000,000 x 100, one query,
// k = 100: 0.57 / 0.30, 300: 0.74 / 0.60, 512: 1.12 / 0.91, x 32, k = 512: 0.99 / 0.49. Rounds of sixteen waves over about k
// blocks: one query, k = 48 / 64: 70,000 x 100: 104 / 104 and 104 / 114 us, 200,000 x 256: 159 / 161 and 158 / 195, four
// queries, k = 64: 123 / 125 and 178 / 192, eight: 202 / 209 (the latter); 500,000 x 100, one query, k = 64: 186 / 158.
// Two and three dimensions: as many points within the bf16 rounding of the best as to make a long list (k = 10, one query and
// 300: 300,000 x 2: 110 / 131 and 370 / 410 us, 20,000 x 2: 75 / 60 and 123 / 77; 1,000,000 x 3: 180 / 221 and 636 / 902,
// 300,000 x 3: 112 / 83 and 400 / 178; 1,000,000 x 4: 180 / 91 and 495 / 177).
bool exact_supported(int64_t n, int d, int nq, int k)
{
    if (nq < 1 || n < 256 * (int64_t)k || (k > 64 && nq < 16 && n < 1000000)) return false;
    if (d < 4 && n > (d == 2 ? 100000 : 500000)) return false;
    if (k > 48 && n < 400000 && ((nq == 1 && d > 64) || (nq < 8 && d > 200))) return false;
    return exact_steps(d) > 0 && exact_finish_lds(d, k, 1024) <= kMaxDynLds - 16 * 1024;
}

// The longest list of blocks that is scored here rather than by the plain kernel: 2 k (what a search takes anyway) and as
// much as half of that kernel's time pays for. Measured: a list costs 0.12 to 0.2 ns a point and coordinate while the
// queries have compute units to themselves, 0.55 ps x nq beyond some 364 queries (the caches' rate), the plain kernel
// about 75 us and n x d x (3.5 + 0.165 nq) ps. Every point a copy of one row, k = 10, the plain kernel alone / this way /
// the list whatever its length (us a call): 200,000 x 100 points, one query 103 / 142 / 2,530, 1,000 queries
// 2,830 / 3,025 / 10,940; 1,183,514 x 100, one query 465 / 646 / 24,640, 300 queries 5,790 / 6,330 / 29,500. At worst, lists
// just short of the line, a call takes 1.7 times the plain kernel's time (200,000 x 100 rows that share a component of
// ten times their norm, 16 queries: 178 / 294 / 314; with 300 queries 1,100 / 695).
static uint32_t exact_max_listed(int64_t n, int d, int nq, int k, int block_points)
{
    const double points = (190000.0 / d + (double)n * (0.009 + 0.0004 * nq)) / std::max(1.0, nq / 364.0);
    return (uint32_t)std::min<double>(kExactBins, 2.0 * k + points / block_points);
}

// nq as exact_queries_per_launch allows. *need_out: which queries the plain kernel has to answer (see the top).
int launch_exact(const float *x, int64_t n, int d, const float *queries, int nq, int k, void *ws, int32_t *ids_out,
                 float *scores_out, const uint32_t **need_out, hipStream_t st)
{
    ExactWs w;
    exact_ws_layout(n, d, nq, (unsigned char *)ws, &w);
    const int steps = exact_steps(d), tiles = (nq + 31) / 32, ns = (k + 63) / 64;
    const int block_points = steps > 8 ? 32 : 64;
    *need_out = w.need;
    hipLaunchKernelGGL(exact_pack_kernel, dim3((unsigned)tiles), dim3(256), 0, st, queries, nq, d, steps, w.packed, w.qnorm, w.need);
    // Two workgroups a compute unit: from 257 of them and three tiles of queries on, or 513 and two. 100 dimensions, one / two, us a
    // call: 77,000 points, 2 queries 42.8 / 45.1, 1,000 133.6 / 135.5; 200,000, 64 queries 65.4 / 66.3, 130 74.2 / 73.2, 1,000 182.6 / 170.7;
    // 400,000, 64 89.6 / 87.6; 1,183,514, 16 queries 191.9 / 197.4, 64 202.1 / 200.4, 130 226.4 / 212.6, 1,000 605 / 520.
    const int64_t groups = w.stride / 8;
    const bool pair = groups > 256 && tiles > (groups > 512 ? 1 : 2);
#define AVQ_EXACT(NS, CT, PAIR)                                                                                          \
    hipLaunchKernelGGL((exact_product_kernel<NS, CT, PAIR>), dim3((unsigned)(w.stride / 8)), dim3(512), 0, st, x, n, d, w.packed, \
                       tiles, nq, w.best, w.stride, w.xnorm, w.need)
    switch (steps) {
    case 2: AVQ_EXACT(2, 2, false); break;
    case 3: AVQ_EXACT(3, 2, false); break;
    case 4: AVQ_EXACT(4, 2, false); break;
    case 7:
        if (pair) AVQ_EXACT(7, 2, true);
        else AVQ_EXACT(7, 2, false);
        break;
    case 8: AVQ_EXACT(8, 2, false); break;
    case 12: AVQ_EXACT(12, 1, false); break;
    default: AVQ_EXACT(16, 1, false); break;
    }
#undef AVQ_EXACT
    static LdsLimitOnce once[2];
    AVQ_TRY(set_lds_limit((const void *)exact_finish_kernel<512>, kMaxDynLds - 16 * 1024, &once[0]));
    AVQ_TRY(set_lds_limit((const void *)exact_finish_kernel<1024>, kMaxDynLds - 16 * 1024, &once[1]));
    const int threads = exact_finish_threads(nq);
    hipLaunchKernelGGL(threads == 512 ? exact_finish_kernel<512> : exact_finish_kernel<1024>, dim3((unsigned)nq), dim3((unsigned)threads),
                       exact_finish_lds(d, k, threads), st, x, n, d, queries, w.best, (n + block_points - 1) / block_points, w.stride,
                       block_points, w.qnorm, w.xnorm, ns, k, exact_max_listed(n, d, nq, k, block_points), w.need, ids_out, scores_out);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

} // namespace avq
