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
// step, bound by the issue of the loads); this way 0.43 ms (product 0.27, which reads x once: 0.13 of matrix instructions,
// 0.08 to read x; selection and fp32 scores 0.15; the plain kernel's three launches, which leave at once, 0.014).
// bf16 rather than f16, whose range needs a scale first.
#include <algorithm>
#include <type_traits>
#include "avq_internal.h"
#include "lds_copy.h"
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
// coordinates 16 step + 4 half .. + 3 and 8 further on (the products may take them in any order, and a load of a point's row then
// covers 32 adjacent bytes); padding rows are zero. qnorm[q] = (norm, norm of the conversion error). Sets need.
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
            const int l = 16 * s + 4 * (lane >> 5) + (i & 3) + 2 * (i & 4);
            o[i] = (__bf16)(qq < nq && l < d ? queries[(size_t)qq * d + l] : 0.0f);
        }
        packed[(size_t)t * steps * 64 + f] = o;
    }
}

// Eight waves of 64 points, whose operands stay in registers (x is read once), against all queries, whose tiles of 32
// go through LDS up to two ahead (x: 473 MB, queries: 224 KB at the size above). The products of one accumulator are issued
// between the instructions that take the maximum of the other one (sched_barrier keeps the order). More operands of two
// column tiles than 8 steps would spill in the loop: one column tile. best[q][block of 64]: the workgroup's eight maxima of a
// query leave as 32 adjacent bytes. xnorm[block] = largest norm and conversion error of its points, xnorm8 of the workgroup's.
//
// A lane reads its points' coordinates itself, some steps ahead, four words a load whatever the row's alignment. PAIR (81 to 112
// dimensions): as many registers as let two workgroups share a compute unit, so that one's products go on while the other
// reads its rows (fewer dimensions need no more anyway). RUNS: those rows come through LDS besides, sixteen a wave at a time, as
// one run of memory, which reads each line once and whole; nt: past the caches, at 6 TB/s (1,183,514 x 100, one query: 211 us for
// the product with each lane its own rows and two workgroups, 129 with one, 111 this way).
// Bound by the reading of x, then the tiles (5.6 us each, 4.1 of matrix instructions at the 2.0 GHz that they leave). Product
// alone, 1,183,514 x 100, 1,024 queries: 310 us with a load waited for at a row's every step and the staged tile waited for
// before each tile's first operand, 270 now. Rows that are no whole quads word by word / four words a load, us a call, one query:
// 1,200,000 x 33 122 / 77, 400,000 x 97 139 / 89, 3,000,000 x 113 1,004 / 485, x 129 1,148 / 643. How many steps ahead makes
// little difference: 3,000,000 x 48, one query, 1 / 2 / 4 / 6 / all twelve: 172 / 177 / 166 / 165 / 166.
template <int NS, int CT, bool PAIR, bool RUNS>
__global__ void __launch_bounds__(512, PAIR ? 4 : 2)
exact_product_kernel(const float *__restrict__ x, int64_t n, int d, const v8bf *__restrict__ packed, int n_tiles, int nq,
                     float *__restrict__ best, int64_t best_stride, float2 *__restrict__ xnorm, uint32_t *__restrict__ need,
                     float2 *__restrict__ xnorm8, int nt)
{
    __shared__ __align__(16) v8bf tile[3][NS * 64];
    __shared__ __align__(16) float mx[2][32][8];
    __shared__ float2 norms[8];
    constexpr int kRows = 16; // (two workgroups of 7 steps share 160 KB)
    __shared__ __align__(16) uint4 rows_lds[8][RUNS ? kRows * NS * 4 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const int64_t p0 = (int64_t)blockIdx.x * (8 * CT * 32) + wave * (CT * 32);
    const bool quad = (d & 3) == 0 && ((uintptr_t)x & 15) == 0;
    auto stage = [&](int t, int slot) {
        const v8bf *src = packed + (size_t)t * NS * 64;
        for (int s = wave; s < NS; s += 8)
            lds_copy16(src + s * 64 + lane, tile[slot] + s * 64);
    };
    stage(0, 0);
    if (n_tiles > 1) stage(1, 1);
    v8bf a[CT][NS];
    float xn = 0.0f, xe = 0.0f, n2 = 0.0f, e2 = 0.0f;
    auto operand = [&](int c, int s, const float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const __bf16 b = (__bf16)v[u];
            const float e = v[u] - (float)b;
            n2 += v[u] * v[u];
            e2 += e * e;
            a[c][s][u] = b;
        }
    };
    auto end_of_points = [&](int c) __attribute__((always_inline)) {
        n2 += __shfl_xor(n2, 32, 64);
        e2 += __shfl_xor(e2, 32, 64);
        const float cn = exact_norm(n2, d), ce = exact_norm(e2, d);
        if (p0 + c * 32 + j < n && !(cn < kExactMaxNorm)) atomicOr(need, 1u);
        xn = fmaxf(xn, cn);
        xe = fmaxf(xe, ce);
        n2 = e2 = 0.0f;
    };
    if constexpr (RUNS) {
        // The rows come through LDS, kRows of them at a time, which are one run of memory: each line is read once, whole, and no
        // register holds what is on its way. Rows of an even number of quads are turned by their number (quad c of row r is at
        // place c + r of it), so that the lanes of a read are spread over the banks; others are by themselves.
        uint4 *const mine = rows_lds[wave];
        const int unit = quad ? d / 4 : d, total = kRows * unit, turn_by = quad && (unit & 1) == 0 ? 1 : 0; // 16 bytes, or 4
        const uint32_t inv = ((1u << 20) + (uint32_t)unit - 1u) / (uint32_t)unit; // e / unit = e inv >> 20 for e < 1024
        auto turned = [&](int r) { return turn_by * (r - unit * (int)((uint32_t)r * inv >> 20)); }; // r % unit
#pragma unroll
        for (int c = 0; c < CT; ++c) {
#pragma unroll
            for (int t = 0; t < 32 / kRows; ++t) {
                const int64_t r0 = p0 + c * 32 + t * kRows, start = r0 + kRows <= n ? r0 : n - kRows; // (n is 256 or more)
                const float *src = x + start * d;
                if (quad) {
                    for (int e0 = 0; e0 < total; e0 += 64) {
                        const int e = e0 + lane < total ? e0 + lane : 0; // (beyond the run: its start, not used)
                        const int r = (int)((uint32_t)e * inv >> 20);
                        int q = e - r * unit - turned(r);
                        q += q < 0 ? unit : 0;
                        if (nt) lds_copy16_once(src + (r * unit + q) * 4, mine + e0);
                        else lds_copy16(src + (r * unit + q) * 4, mine + e0);
                    }
                } else {
                    for (int e0 = 0; e0 < total; e0 += 64)
                        lds_copy4(src + (e0 + lane < total ? e0 + lane : 0), (float *)mine + e0);
                }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0)
                asm volatile("" ::: "memory");
                if ((j & ~(kRows - 1)) == t * kRows) {
                    const int64_t i = p0 + c * 32 + j;
                    const int r = (int)((i < n ? i : n - 1) - start); // padding points are copies of the last one
                    const int by = turned(r);
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        float v[8];
                        if (quad) {
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const int q = 4 * s + h + 2 * u;
                                int at = q + by;
                                at -= at >= unit ? unit : 0;
                                const float4 w = *(const float4 *)(mine + r * unit + (q < unit ? at : 0));
                                v[4 * u] = q < unit ? w.x : 0.0f; v[4 * u + 1] = q < unit ? w.y : 0.0f;
                                v[4 * u + 2] = q < unit ? w.z : 0.0f; v[4 * u + 3] = q < unit ? w.w : 0.0f;
                            }
                        } else {
#pragma unroll
                            for (int u = 0; u < 8; ++u) {
                                const int l = 16 * s + 4 * h + (u & 3) + 2 * (u & 4);
                                const float w = ((const float *)mine)[r * d + (l < d ? l : 0)];
                                v[u] = l < d ? w : 0.0f;
                            }
                        }
                        operand(c, s, v);
                        __builtin_amdgcn_sched_barrier(0); // (all reads first would spill)
                    }
                }
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0): the next rows take these ones' place
                asm volatile("" ::: "memory");
            }
            end_of_points(c);
        }
    } else if (NS == 7 && !PAIR && quad) {
        // as below, but a row's last words are left out by a choice rather than a branch (300,000 x 100, one query: 67.0 us a call,
        // 68.2 as below; other numbers of steps gain from the latter: 3,000,000 x 128, one query 402 / 386)
        const float *row[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int64_t i = p0 + c * 32 + j;
            row[c] = x + (size_t)(i < n ? i : n - 1) * d; // padding points are copies of the last one
        }
        float4 raw[NS][2];
        auto ask = [&](int e) __attribute__((always_inline)) {
            const int l = 16 * (e % NS) + 4 * h; // (beyond the row: its start, not used)
            raw[e % NS][0] = *(const float4 *)(row[e / NS] + (l < d ? l : 0));
            raw[e % NS][1] = *(const float4 *)(row[e / NS] + (l + 8 < d ? l + 8 : 0));
        };
#pragma unroll
        for (int e = 0; e < NS; ++e) ask(e);
#pragma unroll
        for (int e = 0; e < CT * NS; ++e) {
            const float4 u = raw[e % NS][0], w = raw[e % NS][1];
            const int l = 16 * (e % NS) + 4 * h;
            const bool in0 = l < d, in1 = l + 8 < d;
            const float v[8] = {in0 ? u.x : 0.0f, in0 ? u.y : 0.0f, in0 ? u.z : 0.0f, in0 ? u.w : 0.0f,
                                in1 ? w.x : 0.0f, in1 ? w.y : 0.0f, in1 ? w.z : 0.0f, in1 ? w.w : 0.0f};
            operand(e / NS, e % NS, v);
            if (e + NS < CT * NS) ask(e + NS);
            __builtin_amdgcn_sched_barrier(0);
            if (e % NS == NS - 1) end_of_points(e / NS);
        }
    } else if (d >= 4) {
        // A step's eight coordinates of a lane's point, those of kAsk steps asked for before they are used (without a branch
        // between them: one for the row's end had each wait for the one before). Four words are one load, at any word's
        // alignment; where a row's end lies within them, the row's last four are read and moved down.
        constexpr int kAsk = PAIR ? 2 : CT * NS < 6 ? CT * NS : 6; // (more spill in a pair)
        const float *row[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int64_t i = p0 + c * 32 + j;
            row[c] = x + (size_t)(i < n ? i : n - 1) * d; // padding points are copies of the last one
        }
        float raw[kAsk][2][4] = {};
        auto ask = [&](int e) __attribute__((always_inline)) {
            const int l = 16 * (e % NS) + 4 * h;
            // (Nothing of the row. A pair's rows end within the last step, but without the branch the compiler forms the addresses of
            // all steps first and spills 8 registers rather than none at six steps, 32 rather than 13 at seven: 700,000 x 96, one
            // query 102 us a call instead of 87.)
            if (PAIR && 16 * (e % NS) >= d) return;
            __builtin_memcpy(raw[e % kAsk][0], row[e / NS] + (l < d - 4 ? l : d - 4), 16);
            __builtin_memcpy(raw[e % kAsk][1], row[e / NS] + (l + 8 < d - 4 ? l + 8 : d - 4), 16);
        };
#pragma unroll
        for (int e = 0; e < kAsk; ++e) ask(e);
#pragma unroll
        for (int e = 0; e < CT * NS; ++e) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = raw[e % kAsk][u / 4][u % 4];
            if (16 * (e % NS) + 16 > d) { // the row's end
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    const int l = 16 * (e % NS) + 4 * h + 8 * g, by = l + 4 - d; // by: words beyond the end
                    const float w[4] = {v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                    if (!PAIR && (d & 3) == 0) { // four or none (a pair: more registers, spilled)
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[4 * g + u] = by <= 0 ? w[u] : 0.0f;
                    } else {
                        v[4 * g] = by <= 0 ? w[0] : by == 1 ? w[1] : by == 2 ? w[2] : by == 3 ? w[3] : 0.0f;
                        v[4 * g + 1] = by <= 0 ? w[1] : by == 1 ? w[2] : by == 2 ? w[3] : 0.0f;
                        v[4 * g + 2] = by <= 0 ? w[2] : by == 1 ? w[3] : 0.0f;
                        v[4 * g + 3] = by <= 0 ? w[3] : 0.0f;
                    }
                }
            }
            operand(e / NS, e % NS, v);
            if (e + kAsk < CT * NS) ask(e + kAsk);
            __builtin_amdgcn_sched_barrier(0);
            if (e % NS == NS - 1) end_of_points(e / NS);
        }
    } else { // two or three dimensions
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int64_t i = p0 + c * 32 + j;
            const float *row = x + (size_t)(i < n ? i : n - 1) * d;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                float v[8] = {};
                if (s == 0 && h == 0) {
                    v[0] = row[0];
                    v[1] = row[1];
                    v[2] = d == 3 ? row[2] : 0.0f;
                }
                operand(c, s, v);
            }
            end_of_points(c);
        }
    }
    for (int s = 16; s > 0; s >>= 1) { xn = fmaxf(xn, __shfl_xor(xn, s, 64)); xe = fmaxf(xe, __shfl_xor(xe, s, 64)); }
    if (lane == 0) norms[wave] = xnorm[(size_t)blockIdx.x * 8 + wave] = make_float2(xn, xe);
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
    if (tid == 0) {
        float2 most = norms[0];
        for (int w = 1; w < 8; ++w) most = make_float2(fmaxf(most.x, norms[w].x), fmaxf(most.y, norms[w].y));
        xnorm8[blockIdx.x] = most;
    }
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

// One workgroup per query. theta: the blocks are dealt to C classes, C a power of two from 8 k on, and theta is the k-th
// largest of the classes' a - E, each that of the class's largest a: a few of the k best may share a class, which only lowers
// theta a little, and a is read once, without the norms. Where that takes more than 256 classes, two histogram passes over the
// ordering values (22 high bits, rounded down) of each thread's two largest blocks; for more results than a quarter of the
// threads, of all blocks. Then the blocks that reach theta as a list - against the largest E of eight blocks first, so that few
// norms are read -, a wave per block and a lane per point, fp32 chain, wave lists. There are at least 4 k blocks
// (exact_supported). More than max_listed (at most kExactBins) blocks: need[1 + q] is set and the plain kernel answers.
// Bound by what it reads: some fifteen blocks of 25 KB a query at the size above, and a twice (150 KB); 0.13 to 0.15 ms for 1,000
// queries, 0.20 with the norms of all blocks read three times. One query on 3,000,000 x 32 points: 47 us with the threads of a
// class reading blocks C apart, 32 with adjacent threads at adjacent blocks and the classes' maxima exchanged. (Up to four threads a
// class read whole lines as they are, and the exchange would cost 1,000 queries at the size above 2 us.) Measured and dropped:
// the rows through LDS as one run of memory (0.13 at k = 10, but 427 us instead of 286 for the search of 300,000 x 64, 600
// queries, k = 100), sixteen loads of a lane at once (more registers: 1.31 ms instead of 1.15 at k = 100), registers for eight
// waves a SIMD (1,000 queries, k = 10 on 1,200,000 x 24: 169 us instead of 179, but k = 100 on x 100 1,218 instead of 1,009).
constexpr int kExactBins = 2048;
template <int kExactThreads>
__global__ void __launch_bounds__(kExactThreads)
exact_finish_kernel(const float *__restrict__ x, int64_t n, int d, const float *__restrict__ queries, const float *__restrict__ best,
                    int64_t n_blocks, int64_t best_stride, int block_points, const float2 *__restrict__ qnorm,
                    const float2 *__restrict__ xnorm, const float2 *__restrict__ xnorm8, int ns, int k, uint32_t max_listed,
                    uint32_t *__restrict__ need,
                    int32_t *__restrict__ ids_out, float *__restrict__ scores_out)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) uint32_t hist[kExactBins], wave_sum[kExactThreads / 64], found[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, q = blockIdx.x;
    if ((need[0] | need[1 + q]) != 0u) return;
    constexpr int nw = kExactThreads / 64;
    const int L = 64 * ns;
    u64 *lists = (u64 *)smem, *mine = lists + (size_t)wave * L;
    u64 *pend = lists + (size_t)nw * L + wave * 64;
    float *qs = (float *)(lists + (size_t)nw * (L + 64));
    for (int l = tid; l < d; l += kExactThreads) qs[l] = queries[(size_t)q * d + l];
    wave_list_clear(mine, ns);
    const float *a = best + (size_t)q * best_stride;
    const float2 qe = qnorm[q];
    auto bound = [&](int64_t b) { const float2 e = xnorm[b]; return exact_bound(qe.x, qe.y, e.x, e.y, d); };
    const bool classes = k <= kExactThreads / 4;
    int C = kExactThreads; // per = threads of a class, side by side
    while (C >= 16 * k && C > 64) C >>= 1;
    const int per_class = kExactThreads / C, cls = tid / per_class, sub = tid & (per_class - 1);
    const bool ranked = classes && C <= 256;
    const bool mixed = per_class > 4; // the threads of a class lie apart, and adjacent ones read adjacent blocks
    float low = -INFINITY, low2 = -INFINITY, theta; // of the class, or the largest two of this thread's blocks
    if (classes) {
        float top = -INFINITY, top2 = -INFINITY;
        uint32_t at = 0u, at2 = 0u;
        if (ranked) {
#pragma unroll 8
            for (uint32_t b = mixed ? tid : cls + C * sub; b < (uint32_t)n_blocks; b += kExactThreads) {
                const float v = a[b];
                at = v > top ? b : at;
                top = fmaxf(top, v);
            }
        } else {
#pragma unroll 4
            for (uint32_t b = tid; b < (uint32_t)n_blocks; b += kExactThreads) {
                const float v = a[b];
                at2 = v > top ? at : v > top2 ? b : at2;
                top2 = v > top ? top : fmaxf(v, top2);
                at = v > top ? b : at;
                top = fmaxf(top, v);
            }
            if (top2 > -INFINITY) low2 = top2 - bound(at2);
        }
        if (top > -INFINITY) low = top - bound(at);
    }
    if (ranked) { // the value that fewer than k exceed and k reach; a class's threads each count a part
        float *vals = (float *)hist, *spread = vals + kExactBins / 2;
        if (mixed) {
            spread[tid] = low; // block b is of class b % C, so this thread's blocks are of class tid % C
            __syncthreads();
            low = spread[cls + C * sub]; // the threads of a class side by side
        }
        for (int m = 1; m < per_class; m <<= 1) low = fmaxf(low, __shfl_xor(low, m, 64));
        if (sub == 0) vals[cls] = low;
        __syncthreads();
        uint32_t more = 0u, same = 0u;
        for (int e = sub * 4; e < C; e += per_class * 4) {
            const float4 v = *(const float4 *)(vals + e);
            more += (uint32_t)(v.x > low) + (uint32_t)(v.y > low) + (uint32_t)(v.z > low) + (uint32_t)(v.w > low);
            same += (uint32_t)(v.x == low) + (uint32_t)(v.y == low) + (uint32_t)(v.z == low) + (uint32_t)(v.w == low);
        }
        for (int m = 1; m < per_class; m <<= 1) { more += __shfl_xor((int)more, m, 64); same += __shfl_xor((int)same, m, 64); }
        if (more < (uint32_t)k && more + same >= (uint32_t)k) found[0] = __float_as_uint(low); // all that do have the same value
        __syncthreads();
        theta = __uint_as_float(found[0]);
    } else { // the bin of 11 bits that holds the left-th largest value with the given leading bits (all values: shift 21, prefix 0)
        uint32_t prefix = 0u, left = (uint32_t)k;
        for (int pass = 0; pass < 2; ++pass) {
            for (int b = tid; b < kExactBins; b += kExactThreads) hist[b] = 0u;
            __syncthreads();
            auto count = [&](float v) {
                const uint32_t o = ord_from_f32(v);
                if (pass == 0) atomicAdd(&hist[o >> 21], 1u);
                else if (o >> 21 == prefix) atomicAdd(&hist[(o >> 10) & 2047u], 1u);
            };
            if (!classes)
                for (int64_t b = tid; b < n_blocks; b += kExactThreads) count(a[b] - bound(b));
            else { count(low); count(low2); } // (-infinity: none; there are k others)
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
        theta = f32_from_ord(prefix << 10); // the values of the bin are at or above it
    }
    __syncthreads();
    uint32_t *list = hist;
    if (tid == 0) found[0] = 0u;
    __syncthreads();
#pragma unroll 4
    for (int64_t b = tid; b < n_blocks; b += kExactThreads) {
        const float v = a[b];
        const float2 e = xnorm8[b >> 3];
        if (v + exact_bound(qe.x, qe.y, e.x, e.y, d) >= theta && v + bound(b) >= theta) {
            const uint32_t to = atomicAdd(&found[0], 1u);
            if (to < kExactBins) list[to] = (uint32_t)b;
        }
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
        if ((wave & (2 * stride - 1)) == 0) wave_list_merge_from(mine, ns, lists + (size_t)(wave + stride) * L);
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
    for (int s : {2, 3, 4, 5, 6, 7, 8, 12, 16})
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
    float2 *qnorm, *xnorm, *xnorm8; // xnorm8: the largest of eight blocks
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
    w->xnorm8 = (float2 *)take(sizeof(float2) * (size_t)(w->stride / 8));
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
    // One workgroup a compute unit, two that read their rows themselves (pair), two whose rows come through LDS (runs). us a call,
    // k = 10. Seven steps, one / pair / runs: 140,000 x 100, 64 queries 62 / 66 / 67, 300 91 / 90 / 94; 600,000 x 100, 64 101 / 112 / 102,
    // 300 151 / 155 / 145, 1,000 285 / 273 / 262; 1,200,000 x 100, 1 184 / 212 / 150, 64 197 / 217 / 175, 300 276 / 275 / 236.
    // Six, pair / runs: 700,000 x 88, 1 84 / 94, 1,000 269 / 274; 1,000,000 x 88, 1 127 / 113, 64 138 / 139, 256 163 / 171, 640 274 / 276;
    // 1,400,000 x 96, 1 151 / 151, 30 169 / 160, 256 203 / 216, 400 252 / 260, 1,000 438 / 416; 2,000,000 x 88, 400 356 / 344.
    // Five, whose operands leave room for two workgroups anyway, one / runs: 700,000 x 72, 1 69 / 84, 1,000 214 / 220; 1,400,000 x 72, 1
    // 122 / 129, 1,000 375 / 368; 2,000,000 x 72, 400 288 / 297, 640 396 / 379, 1,000 512 / 478.
    // (65 to 96 dimensions by seven steps too: 400,000 x 72, 64 queries 77 us, by five 63; 400,000 x 96 83, by six 76.)
    // The caches hold on to x up to somewhat more than their size, for the rows that the selection reads: x 275 MB of 112 dimensions, past
    // the caches / not: one query 100 / 108, 64 125 / 117, 300 182 / 163; 400 MB 64 160 / 155, 300 224 / 213; 500 MB of 100, 64 191 / 192.
    const int64_t groups = w.stride / 8;
    const uint64_t mb = (sizeof(float) * (uint64_t)n * (uint64_t)d) >> 20;
    const bool beyond = mb > 256; // the Infinity Cache
    const int nt = beyond && (tiles == 1 || mb > 448);
    const bool pair = groups > 256 && mb <= 200 && tiles >= 8;
    const bool runs = steps == 5 ? mb > 448 && tiles > 16 : steps == 6 ? beyond && (tiles <= 2 || mb > (tiles > 16 ? 400 : 640))
                                                          : groups > 256 && (beyond || tiles >= 8);
#define AVQ_EXACT(NS, CT, PAIR, RUNS)                                                                                    \
    hipLaunchKernelGGL((exact_product_kernel<NS, CT, PAIR, RUNS>), dim3((unsigned)(w.stride / 8)), dim3(512), 0, st, x, n, d, w.packed, \
                       tiles, nq, w.best, w.stride, w.xnorm, w.need, w.xnorm8, nt)
    switch (steps) {
    case 2: AVQ_EXACT(2, 2, false, false); break;
    case 3: AVQ_EXACT(3, 2, false, false); break;
    case 4: AVQ_EXACT(4, 2, false, false); break;
    case 5:
        if (runs) AVQ_EXACT(5, 2, true, true);
        else AVQ_EXACT(5, 2, false, false);
        break;
    case 6:
        if (runs) AVQ_EXACT(6, 2, true, true);
        else AVQ_EXACT(6, 2, true, false);
        break;
    case 7:
        if (pair) AVQ_EXACT(7, 2, true, false);
        else if (runs) AVQ_EXACT(7, 2, true, true);
        else AVQ_EXACT(7, 2, false, false);
        break;
    case 8: AVQ_EXACT(8, 2, false, false); break;
    case 12: AVQ_EXACT(12, 1, false, false); break;
    default: AVQ_EXACT(16, 1, false, false); break;
    }
#undef AVQ_EXACT
    static LdsLimitOnce once[2];
    AVQ_TRY(set_lds_limit((const void *)exact_finish_kernel<512>, kMaxDynLds - 16 * 1024, &once[0]));
    AVQ_TRY(set_lds_limit((const void *)exact_finish_kernel<1024>, kMaxDynLds - 16 * 1024, &once[1]));
    const int threads = exact_finish_threads(nq);
    hipLaunchKernelGGL(threads == 512 ? exact_finish_kernel<512> : exact_finish_kernel<1024>, dim3((unsigned)nq), dim3((unsigned)threads),
                       exact_finish_lds(d, k, threads), st, x, n, d, queries, w.best, (n + block_points - 1) / block_points, w.stride,
                       block_points, w.qnorm, w.xnorm, w.xnorm8, ns, k, exact_max_listed(n, d, nq, k, block_points), w.need, ids_out, scores_out);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

} // namespace avq
