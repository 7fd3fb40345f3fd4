// Batches on a flat index: which points can be among a query's R best, by way of a matrix product.
//
// The ADC score of Section 4.1, sum_m <q^(m), c_{m, code}>, is the inner product of the query with the point its code
// stands for, so for many queries it is a matrix product with one row per point: 2 d operations a pair instead of a table
// look-up and an addition per subspace. The points are decoded from their codes into registers (f16, as operands of
// v_mfma_f32_32x32x16_f16) and meet all queries there; the codes are read once and no decoded point is ever stored.
//
// The results are still those of the table sums, in their stated order of additions: the product only decides which points
// are looked at. Every value p it forms is within E of the score s that ranks the point (product_error below). With p_(R)
// the R-th largest p, R points have s >= p_(R) - E, and a point with p < p_(R) - 2 E has s < p_(R) - E: the R best are
// among the points with p >= p_(R) - 2 E, ties included. Those are scored again with fp32 tables or with the 8-bit ones.
//
// p_(R) is guessed first: the sampling launch forms the products of every stride-th 32 points and keeps the largest of each
// class of them, and the r-th largest of a query's classes is the guess T. The full launch keeps what reaches T - 2 E. If R
// of the kept points reach T, so does p_(R), and nothing was missed; otherwise, or if more was kept than there is room for,
// the query is scanned plainly.
//
// f16 holds 11 bits of an operand: queries and dictionaries are scaled by powers of two to just below 2^14, and E is about
// a thousandth of |q| |x| (8-bit tables: the rounding of their entries, half a unit a subspace, is most of it). bf16, which
// needs no scale, would keep eight times as wide a margin, the i8 instruction at twice the rate thirty times.
//
// What bounds it: the matrix instructions, at the clock they leave. 1,183,514 points, 100 dimensions, 10,000 queries: 1.06 ms
// of them at 2.4 GHz, 1.4 at the 1.85 GHz that the counters show; the launch takes 1.98 when nothing is kept and 2.45 with
// its 320 kept points a query (a third of that for the entries in LDS, the rest for handing them over). A library's bf16
// product of the same size runs at the rate of 1.95 (1.2 PFLOP/s). The table look-ups on the matrix cores took 4.2 ms, 8-bit
// codes (1,999 queries) from byte tables 1.7 ms and 1.3 to score blocks, here 0.52 in all.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include "avq_internal.h"
#include "product_device.h"
#include "row_dot.h"

namespace avq {

constexpr int kProductWaves = 4;    // waves of a workgroup; two workgroups share a compute unit

__device__ __forceinline__ int scale_exp(float largest) // 2^result * largest is in [2^13, 2^14)
{
    if (!(largest > 0.0f)) return 0;
    int e;
    frexpf(largest, &e);
    return 14 - e;
}

// Workgroup 0: the dictionaries, scaled, as f16, and the norms that bound every decoded point. The others: 128 queries each,
// in operand order [tile of 32][step][lane][8], lane (row lane % 32, half lane / 32) holding coordinates 16 step + 8 half
// .. + 7, zero beyond d and nq (rows: [query][step][16] instead); their norms and scales; and what the launches after this one count in is cleared.
__global__ void __launch_bounds__(1024)
product_pack_kernel(const float *__restrict__ queries, int nq, int d, int steps, int n_tiles, const float *__restrict__ codebooks,
                    int M, int kc, _Float16 *__restrict__ cb16, ProductMeta *__restrict__ meta, v8h *__restrict__ packed,
                    ProductQuery *__restrict__ qinfo, uint32_t *__restrict__ kept_cnt, int cnt_stride, uint32_t *__restrict__ fail_clear,
                    int n_clear, int rows)
{
    __shared__ float wave_max[16];
    __shared__ uint32_t n2_max[256], e2_max[256];
    __shared__ int qexp[128], qbad[128];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.x == 0) {
        const int ds = d / M, total = M * kc * ds;
        float big = 0.0f;
        bool odd = false;
        for (int e = tid; e < total; e += 1024) {
            const float v = fabsf(codebooks[e]);
            big = fmaxf(big, v);
            odd = odd || !(v < INFINITY);
        }
        for (int s = 32; s > 0; s >>= 1) big = fmaxf(big, __shfl_xor(big, s, 64));
        if (__builtin_amdgcn_ballot_w64(odd) != 0ull) big = INFINITY;
        if (lane == 0) wave_max[wave] = big;
        if (tid < 256) { n2_max[tid] = 0u; e2_max[tid] = 0u; }
        if (tid < n_clear) fail_clear[tid] = 0u;
        __syncthreads();
        for (int w = 0; w < 16; ++w) big = fmaxf(big, wave_max[w]);
        const bool bad = !(big < INFINITY);
        const int ex = bad ? 0 : scale_exp(big);
        for (int w = tid; w < M * kc; w += 1024) {
            float n2 = 0.0f, e2 = 0.0f;
            for (int l = 0; l < ds; ++l) {
                const float v = bad ? 0.0f : ldexpf(codebooks[(size_t)w * ds + l], ex);
                const _Float16 h = (_Float16)v;
                const float e = v - (float)h;
                n2 += v * v;
                e2 += e * e;
                cb16[(size_t)w * ds + l] = h;
            }
            atomicMax(&n2_max[w / kc], __float_as_uint(n2)); // not negative: ordered like their bits
            atomicMax(&e2_max[w / kc], __float_as_uint(e2));
        }
        __syncthreads();
        if (wave == 0) {
            float n2 = 0.0f, e2 = 0.0f;
            for (int m = lane; m < M; m += 64) { n2 += __uint_as_float(n2_max[m]); e2 += __uint_as_float(e2_max[m]); }
            for (int s = 32; s > 0; s >>= 1) { n2 += __shfl_xor(n2, s, 64); e2 += __shfl_xor(e2, s, 64); }
            if (lane == 0) *meta = ProductMeta{product_norm(n2), product_norm(e2), ex, bad ? 1 : 0};
        }
        return;
    }
    const int q0 = ((int)blockIdx.x - 1) * 128;
    {
        const int r = tid >> 3, g = tid & 7, q = q0 + r;
        float big = 0.0f;
        bool odd = false;
        if (q < nq)
            for (int l = g; l < d; l += 8) {
                const float v = fabsf(queries[(size_t)q * d + l]);
                big = fmaxf(big, v);
                odd = odd || !(v < INFINITY);
            }
        int o = odd ? 1 : 0;
        for (int s = 4; s > 0; s >>= 1) { big = fmaxf(big, __shfl_xor(big, s, 64)); o |= __shfl_xor(o, s, 64); }
        const int ex = o ? 0 : scale_exp(big);
        float n2 = 0.0f, e2 = 0.0f;
        if (q < nq && !o)
            for (int l = g; l < d; l += 8) {
                const float v = ldexpf(queries[(size_t)q * d + l], ex), e = v - (float)(_Float16)v;
                n2 += v * v;
                e2 += e * e;
            }
        for (int s = 4; s > 0; s >>= 1) { n2 += __shfl_xor(n2, s, 64); e2 += __shfl_xor(e2, s, 64); }
        if (g == 0) {
            qexp[r] = ex;
            qbad[r] = o;
            if (q < nq) {
                qinfo[q] = ProductQuery{product_norm(n2), product_norm(e2), ex, o};
                kept_cnt[(size_t)q * cnt_stride] = 0u;
            }
        }
    }
    __syncthreads();
    for (int f = tid; f < 4 * steps * 64; f += 1024) {
        const int t = f / (steps * 64), s = f / 64 % steps, ln = f & 63, r = t * 32 + (ln & 31), q = q0 + r;
        const int tile = q0 / 32 + t;
        if (tile >= n_tiles) break;
        v8h o;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int l = 16 * s + 8 * (ln >> 5) + i;
            o[i] = (_Float16)(q < nq && l < d && !qbad[r] ? ldexpf(queries[(size_t)q * d + l], qexp[r]) : 0.0f);
        }
        packed[rows ? ((size_t)q * steps + s) * 2 + (ln >> 5) : ((size_t)tile * steps + s) * 64 + ln] = o;
    }
}

// Queries against points. A wave decodes the operands of CT x 32 points and keeps them; the queries' go through LDS, QT
// tiles of 32 at a time, in three buffers: while one is read, the next has arrived and the one after that is on its way. The products of a
// tile are formed in two halves of CT / 2 x 32 points, and while the matrix instructions of one half run, the vector unit
// looks at the other half's results: a step of 32 cycles has room for seven vector instructions of the same wave, and about
// three are needed. Two workgroups of four waves a compute unit, so that a barrier, or a wave busy with kept points, leaves
// the matrix unit to another wave.
// SAMPLE: every stride-th 32 points; a lane (query j, half h) leaves the largest product of each run of `run` (1, 4, 16,
// all) of its 16 CT accumulators in classes[q][class].
// Otherwise: what reaches thr[q] is kept: eight instructions find the largest of a lane's 16 products of 32 x 32. A lane that has one leaves its 16 accumulators in LDS, and 64 such entries at a time are gone through together:
// a lane per entry, one atomic addition and one store to kept[q] a point.
template <int NS, int CT, bool SAMPLE>
__global__ void __launch_bounds__(kProductWaves * 64, 2)
product_scan_kernel(const ProductParams p)
{
    constexpr int QT = product_qt(NS), PEND = product_pend(NS), HC = CT / 2;
    constexpr int W = product_ahead(NS);
    __shared__ __align__(16) v8h tile[3][QT * NS * 64];
    __shared__ __align__(16) float thr_s[3][64];
    __shared__ __align__(16) float4 pend_s[kProductWaves][PEND][4]; // a lane's accumulators
    __shared__ uint2 tags_s[kProductWaves][PEND]; // query of the chunk << 7 | point of the wave (accumulator 0's); the line
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const int64_t group = blockIdx.x % p.groups;
    const int chunk = blockIdx.x / p.groups;
    const int n_stages = p.n_tiles / QT; // n_tiles is a multiple of QT
    const int t0 = chunk * p.stages_per_chunk, t1 = t0 + p.stages_per_chunk < n_stages ? t0 + p.stages_per_chunk : n_stages;
    if (t0 >= t1) return;

    auto stage = [&](int t, int slot) {
        const v8h *src = (const v8h *)p.packed + (size_t)t * QT * NS * 64;
        v8h *dst = tile[slot];
        for (int s = wave; s < QT * NS; s += kProductWaves)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + s * 64 + lane),
                                             (__attribute__((address_space(3))) void *)(dst + s * 64), 16, 0, 0);
        if (!SAMPLE && wave == 0) // thr has room for 64 beyond the last tile
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(p.thr + (size_t)t * QT * 32 + lane),
                                             (__attribute__((address_space(3))) void *)thr_s[slot], 4, 0, 0);
    };
    stage(t0, 0);

    const int64_t apart = SAMPLE ? (int64_t)p.stride * 32 : 32; // points from one 32 to the next
    const int64_t first = (group * kProductWaves + wave) * CT * apart;
    float4(*const pend)[4] = pend_s[wave];
    uint2 *const tags = tags_s[wave];

    v8h a[CT][NS];
    product_decode<NS, CT, kProductWaves, 2 * QT * NS * 1024, PEND * 64>(a, p, first, apart, (uint8_t *)&tile[1][0], (uint4 *)&pend[0][0]);

    const int left = p.n - first < CT * 32 ? (int)(p.n - first) : CT * 32; // !SAMPLE: this wave's points
    int cnt = 0;                                                           // entries in its buffer
    auto hand_over = [&](int take) __attribute__((always_inline)) { // the first `take` (at most 64)
        wave_lds_fence();
        uint32_t hits = 0u;
        uint2 tag = make_uint2(0u, 0u);
        if (lane < take) {
            tag = tags[lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float4 w = pend[lane][r];
                const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (x[v] >= __uint_as_float(tag.y) && (int)(tag.x & 127u) + 8 * r + v < left) hits |= 1u << (4 * r + v);
            }
        }
        const uint32_t q = (tag.x >> 7) + (uint32_t)t0 * QT * 32;
        while (__builtin_amdgcn_ballot_w64(hits != 0u) != 0ull) {
            if (hits != 0u) {
                const int v = __builtin_ctz(hits);
                hits &= hits - 1u;
                const uint32_t id = (uint32_t)first + (tag.x & 127u) + 8 * (v >> 2) + (v & 3);
                const uint32_t pos = atomicAdd(p.kept_cnt + (size_t)q * p.cnt_stride, 1u);
                // beyond kept_cap the query is scanned plainly, and nothing more of it is wanted (a stale line keeps a few more)
                if (pos < (uint32_t)p.kept_cap) p.kept[(size_t)q * p.kept_cap + pos] = ((u64)ord_from_f32(((const float *)pend[lane])[v]) << 32) | id;
                else p.thr[q] = INFINITY;
            }
        }
        wave_lds_fence();
        cnt -= take;
        if (lane < cnt) { // the others move up
#pragma unroll
            for (int r = 0; r < 4; ++r) pend[lane][r] = pend[take + lane][r];
            tags[lane] = tags[take + lane];
        }
        wave_lds_fence();
    };

    v16f acc[CT], zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = -INFINITY;
    auto max2 = [](float x, float y) __attribute__((always_inline)) -> float { return __builtin_elementwise_maximum(x, y); };
    // The i-th of the eight instructions that find the largest of 16. (The IEEE 754-2019 maximum: no operand is quieted first,
    // and it takes three.)
    auto max_part = [&](float &m, const v16f &x, int i) __attribute__((always_inline)) {
        if (i == 0) m = max2(max2(x[0], x[1]), x[2]);
        else if (i < 7) m = max2(max2(m, x[2 * i + 1]), x[2 * i + 2]);
        else m = max2(m, x[15]);
    };
    // what reaches the line among tile tl of the chunk and half `which`
    auto keep_half = [&](auto which, int tl, float line, const float (&big)[HC]) __attribute__((always_inline)) {
        constexpr int H = decltype(which)::value;
#pragma unroll
        for (int cc = 0; cc < HC; ++cc) {
            const int c = H * HC + cc;
            const u64 mask = __builtin_amdgcn_ballot_w64(big[cc] >= line);
            if (__builtin_expect(mask == 0ull, 1)) continue;
            if (__builtin_expect(cnt > PEND - 64, 0)) hand_over(cnt < 64 ? cnt : 64);
            const int to = cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (big[cc] >= line) {
#pragma unroll
                for (int r = 0; r < 4; ++r) pend[to][r] = make_float4(acc[c][4 * r], acc[c][4 * r + 1], acc[c][4 * r + 2], acc[c][4 * r + 3]);
                tags[to] = make_uint2(((uint32_t)tl * 32u + (uint32_t)j) << 7 | (uint32_t)(4 * h + c * 32), __float_as_uint(line));
            }
            cnt += (int)__popcll(mask);
        }
    };
    float first_half = -INFINITY; // SAMPLE, one class a lane: its first half's largest
    auto sample_half = [&](auto which, int tl, const float (&big)[HC]) __attribute__((always_inline)) {
        constexpr int H = decltype(which)::value;
        const int q = (t0 * QT + tl) * 32 + j;
        const bool part = first + (CT - 1) * apart + 32 > p.n; // some of the points are not there
        if (part) {
            int64_t rest = p.n - first - 4 * h;
            asm volatile("" : "+v"(rest)); // the compares below stay in here
#pragma unroll
            for (int cc = 0; cc < HC; ++cc)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if ((H * HC + cc) * apart + 8 * (v / 4) + v % 4 >= rest) acc[H * HC + cc][v] = -INFINITY;
        }
        float m[HC];
#pragma unroll
        for (int cc = 0; cc < HC; ++cc) {
            m[cc] = big[cc];
            if (part)
#pragma unroll
                for (int i = 0; i < 8; ++i) max_part(m[cc], acc[H * HC + cc], i);
        }
        if (tl < 0 || q >= p.nq) return;
        const int per_lane = CT * 16 / p.run;
        float *dst = p.classes + (size_t)q * p.n_classes + ((size_t)(group * kProductWaves + wave) * 2 + h) * per_lane;
        if (p.run > 16) {
#pragma unroll
            for (int cc = 1; cc < HC; ++cc) m[0] = max2(m[0], m[cc]);
            if (H == 0) first_half = m[0];
            else dst[0] = max2(m[0], first_half);
        } else {
#pragma unroll
            for (int cc = 0; cc < HC; ++cc) {
                const int c = H * HC + cc;
                if (p.run == 16) {
                    dst[c] = m[cc];
                } else if (p.run == 4) {
                    *(float4 *)(dst + c * 4) = make_float4(max2(max2(acc[c][0], acc[c][1]), max2(acc[c][2], acc[c][3])),
                                                           max2(max2(acc[c][4], acc[c][5]), max2(acc[c][6], acc[c][7])),
                                                           max2(max2(acc[c][8], acc[c][9]), max2(acc[c][10], acc[c][11])),
                                                           max2(max2(acc[c][12], acc[c][13]), max2(acc[c][14], acc[c][15])));
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        *(float4 *)(dst + c * 16 + 4 * r) = make_float4(acc[c][4 * r], acc[c][4 * r + 1], acc[c][4 * r + 2], acc[c][4 * r + 3]);
                }
            }
        }
    };

    // the first stage, and its first operands
    __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0): this wave's part is in LDS
    __syncthreads();
    if (t0 + 1 < t1) stage(t0 + 1, 1);
    v8h b[W]; // operand of step s in b[s % W]
#pragma unroll
    for (int s = 0; s < W; ++s) b[s] = tile[0][s * 64 + lane];
    float line = SAMPLE ? 0.0f : thr_s[0][j], line_before = INFINITY; // of the tile at hand, and of the one before
    int slot = 0;
#pragma unroll 1
    for (int t = t0; t < t1; ++t) {
        const int slot1 = slot == 2 ? 0 : slot + 1, slot2 = slot1 == 2 ? 0 : slot1 + 1;
#pragma unroll 1
        for (int u = 0; u < QT; ++u) {
            const int tl = (t - t0) * QT + u;
            const bool last = u == QT - 1;
            const v8h *cur = tile[slot] + u * NS * 64, *nxt = tile[last ? slot1 : slot] + (last ? 0 : u + 1) * NS * 64;
            // One half's products; between its matrix instructions, the largest of the other half's and the reads of operands W
            // steps ahead. The barriers for the scheduler keep that order.
            float big[HC];
            auto half = [&](auto which, const v8h *next) __attribute__((always_inline)) {
                constexpr int H = decltype(which)::value, O = 1 - H;
#pragma unroll
                for (int s = 0; s < NS; ++s) {
#pragma unroll
                    for (int cc = 0; cc < HC; ++cc) {
                        acc[H * HC + cc] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[H * HC + cc][s], b[s % W], s == 0 ? zero : acc[H * HC + cc], 0, 0, 0);
#pragma unroll
                        for (int i = (s * HC + cc) * 8 / NS; i < (s * HC + cc + 1) * 8 / NS; ++i) max_part(big[i / 8], acc[O * HC + i / 8], i % 8);
                        if (cc < HC - 1) __builtin_amdgcn_sched_barrier(0);
                    }
                    if (W < NS || H == 1) // the first half's operands are still there
                        b[s % W] = s + W < NS ? cur[(s + W) * 64 + lane] : next[(s + W - NS) * 64 + lane];
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int cc = 0; cc < HC; ++cc) asm volatile("" : "+v"(big[cc])); // found here, not where a branch wants it
            };
            half(std::integral_constant<int, 0>{}, cur);
            if constexpr (SAMPLE) sample_half(std::integral_constant<int, 1>{}, tl - 1, big);
            else keep_half(std::integral_constant<int, 1>{}, tl - 1, line_before, big);
            if (last && t + 1 < t1) {
                // the next stage is there; every wave has left the one before this, whose buffer the one after next takes
                __builtin_amdgcn_s_waitcnt(0x0f70);
                __syncthreads();
                if (t + 2 < t1) stage(t + 2, slot2);
            }
            half(std::integral_constant<int, 1>{}, nxt); // operands beyond the last tile: not used
            line_before = line;
            if (!SAMPLE) line = thr_s[last ? slot1 : slot][last ? j : (u + 1) * 32 + j];
            if constexpr (SAMPLE) sample_half(std::integral_constant<int, 0>{}, tl, big);
            else keep_half(std::integral_constant<int, 0>{}, tl, line_before, big);
        }
        slot = slot1;
    }
    const int last_tl = (t1 - t0) * QT - 1;
    float big[HC];
#pragma unroll
    for (int cc = 0; cc < HC; ++cc)
#pragma unroll
        for (int i = 0; i < 8; ++i) max_part(big[cc], acc[HC + cc], i);
    if constexpr (SAMPLE) {
        sample_half(std::integral_constant<int, 1>{}, last_tl, big);
    } else {
        keep_half(std::integral_constant<int, 1>{}, last_tl, line_before, big);
        while (cnt > 0) hand_over(cnt < 64 ? cnt : 64);
    }
}

// Per query: T, the r-th largest of its S classes (found to a 2^-11th of its value or of the spread, from below), 2 E, and
// the line T - 2 E of the full launch; +infinity where the product decides nothing (values out of range, tables without
// one). One wave per query for S <= 2048 (THREADS 64, four queries a workgroup), otherwise a workgroup.
template <int THREADS, int PER>
__global__ void __launch_bounds__(THREADS == 64 ? 256 : THREADS)
product_bound_kernel(const float *__restrict__ classes, int S, int r, int nq, int nq_pad, int d, int M, const float *__restrict__ unit,
                     bool u8, const ProductQuery *__restrict__ qinfo, const ProductMeta *__restrict__ meta, float *__restrict__ thr,
                     float *__restrict__ margin, float *__restrict__ guess, const int32_t *__restrict__ leaf_ids,
                     const float *__restrict__ leaf_ip, int L)
{
    constexpr bool WIDE = THREADS > 64;
    constexpr int NW = THREADS / 64;
    __shared__ int wave_cnt[2][NW];
    __shared__ uint32_t wave_lo[NW], wave_hi[NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = WIDE ? (int)blockIdx.x : (int)blockIdx.x * 4 + wave;
    const int first = WIDE ? (int)threadIdx.x : lane;
    if (q >= nq) { // WIDE: the whole workgroup leaves
        if (q < nq_pad && first == 0) thr[q] = INFINITY;
        return;
    }
    uint32_t mine[PER], lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = first + k * THREADS;
        const float v = i < S ? classes[(size_t)q * S + i] : leaf_ip ? 0.0f : -INFINITY;
        mine[k] = leaf_ip ? __float_as_uint(v) : v > -INFINITY ? ord_from_f32(v) : 0u;
        if (mine[k] != 0u) { lo = mine[k] < lo ? mine[k] : lo; hi = mine[k] > hi ? mine[k] : hi; }
    }
    for (int s = 32; s > 0; s >>= 1) {
        const uint32_t a = (uint32_t)__shfl_xor((int)lo, s, 64), b = (uint32_t)__shfl_xor((int)hi, s, 64);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
    }
    if (WIDE) {
        if (lane == 0) { wave_lo[wave] = lo; wave_hi[wave] = hi; }
        __syncthreads();
        for (int w = 0; w < NW; ++w) { lo = wave_lo[w] < lo ? wave_lo[w] : lo; hi = wave_hi[w] > hi ? wave_hi[w] : hi; }
    }
    int parity = 0;
    auto count_ge = [&](uint32_t v) -> int {
        int cn = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) cn += (int)__popcll(__builtin_amdgcn_ballot_w64(mine[k] >= v));
        if (WIDE) {
            if (lane == 0) wave_cnt[parity][wave] = cn;
            __syncthreads();
            cn = 0;
            for (int w = 0; w < NW; ++w) cn += wave_cnt[parity][w];
            parity ^= 1;
        }
        return cn;
    };
    bool ok = hi != 0u && count_ge(lo) >= r;
    if (ok) {
        ++hi; // finite values stay below the largest word: count_ge(lo) >= r > count_ge(hi)
        while (hi - lo > 4096u) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            if (count_ge(mid) >= r) lo = mid; else hi = mid;
        }
    }
    // leaves: the largest |<q, center>|; infinite where one is not finite, which leaves no line to compare with
    float ip = 0.0f;
    if (leaf_ip) {
        for (int l = lane; l < L; l += 64) {
            if (leaf_ids[(size_t)q * L + l] < 0) continue; // no such leaf
            const float v = fabsf(leaf_ip[(size_t)q * L + l]);
            ip = v < INFINITY ? fmaxf(ip, v) : INFINITY;
        }
        for (int s = 32; s > 0; s >>= 1) ip = fmaxf(ip, __shfl_xor(ip, s, 64));
    }
    if (first != 0) return;
    const ProductQuery qi = qinfo[q];
    const ProductMeta me = *meta;
    const float un = u8 ? unit[q] : 0.0f;
    // with leaves the score is rounded twice more, as is the product with <q, center>
    const float ip_s = ldexpf(ip, qi.exp + me.exp);
    const float m2 = 2.0f * (product_error(qi, me, d, M, un) + 6e-7f * ip_s);
    // the unscaled scores and the sums on the way to them are finite
    const bool range = !qi.bad && !me.bad && ldexpf(qi.qn, -qi.exp) * ldexpf(me.xn, -me.exp) < 1e36f && (!u8 || un > 0.0f);
    const bool none = !ok && leaf_ip != nullptr; // everything in the probed leaves is kept
    ok = (ok || none) && range && m2 < 1e30f && ip_s < 1e30f && ip < 1e36f;
    margin[q] = ok ? m2 : -1.0f;
    guess[q] = none ? -INFINITY : f32_from_ord(lo);
    thr[q] = !ok ? INFINITY : none ? -INFINITY : f32_from_ord(lo) - m2;
}

// One workgroup per query: checks the guess, finds the R-th largest product among the kept points, scores what lies within
// 2 E of it as the plain scan would (fp32: the sum of the entries of a byte, bytes in order; 8-bit tables: the integer sum),
// ranks it, scores the R best against the points themselves where asked, and writes the answer. A chain of dependent
// steps per query, so what counts is their number: histograms instead of bisections, the bytes of a code loaded together. A
// query it cannot answer gets its tables laid out for the plain scan.
template <bool U8, int BITS>
__global__ void __launch_bounds__(256)
product_refine_kernel(const ProductRefineParams r)
{
    constexpr int FINAL = ProductRoom<U8>::final;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BinScratch bins;
    __shared__ int n_fin_s, slot_s;
    const int tid = threadIdx.x, q = blockIdx.x;
    u64 *keys = (u64 *)smem;                           // [FINAL]
    u64 *best = keys + FINAL;                          // [R + 1]; with 8-bit tables, first the finalists that stay
    float *qs = (float *)(best + r.R + (r.R & 1) + 2); // [d]
    float *tbl = qs + ((r.d + 3) & ~3);                // 4-bit codes: [2 NB][16], the fp32 tables or the 8-bit ones as numbers
    const int ds = r.d / r.M;
    const uint32_t total = r.kept_cnt[(size_t)q * r.cnt_stride];
    const float m2 = r.margin[q]; // 2 E
    bool ok = m2 >= 0.0f && total <= (uint32_t)r.kept_cap;
    int why = m2 >= 0.0f ? 1 : 3;
    if (r.force_fail_odd && (q & 1)) { ok = false; why = 3; }
    if (tid == 0) n_fin_s = 0;
    bins.hist[tid] = 0u;
    const u64 *kept = r.kept + (size_t)q * r.kept_cap;
    for (int l = tid; l < r.d; l += 256) qs[l] = r.queries[(size_t)q * r.d + l];
    if (ok) {
        const uint32_t bin = rth_bin(bins, total, ord_from_f32(r.guess[q]), (uint32_t)r.R, tid, [&](uint32_t i) { return (uint32_t)(kept[i] >> 32); });
        if (bin == 0u) { // fewer than R reach T
            ok = false;
            why = 2;
        } else {
            const uint32_t keep = ord_from_f32(f32_from_ord(bin) - m2);
            bins.hist[tid] = 0u;
            for (uint32_t i = tid; i < total; i += 256u) {
                const u64 e = kept[i];
                if ((uint32_t)(e >> 32) < keep) continue;
                const int slot = atomicAdd(&n_fin_s, 1);
                if (slot < FINAL) keys[slot] = (uint32_t)e;
            }
            if (BITS == 4) {
                const uint8_t *tab8 = U8 ? r.lut8 + (size_t)q * r.M * 16 : nullptr;
                for (int e = tid; e < 2 * r.NB * 16; e += 256) {
                    const int m = e >> 4;
                    float s = 0.0f;
                    if (m < r.M) {
                        if (U8) {
                            s = __uint_as_float(tab8[e]);
                        } else {
                            const float *c = r.codebooks + (size_t)e * ds;
                            for (int l = 0; l < ds; ++l) s = __fmaf_rn(qs[m * ds + l], c[l], s);
                        }
                    }
                    tbl[e] = s;
                }
            }
        }
    }
    __syncthreads();
    int n_fin = n_fin_s;
    ok = ok && n_fin <= FINAL;
    if (!ok) {
        if (tid == 0) {
            slot_s = (int)atomicAdd(r.fail_count, 1u);
            r.fail_list[slot_s] = q;
            atomicAdd(r.fail_total, 1u); // statistics of the call: 1 = too many kept points, 2 = bound guessed too high, 3 = other
            atomicAdd(r.fail_total + why, 1u);
        }
        __syncthreads();
        const int entries = r.M << BITS;
        const size_t row = (size_t)slot_s * entries;
        for (int e = tid; e < entries; e += 256) {
            if (U8) {
                ((uint8_t *)r.fail_lut)[row + e] = r.lut8[(size_t)q * entries + e];
            } else {
                const float *c = r.codebooks + (size_t)e * ds;
                float s = 0.0f;
                for (int l = 0; l < ds; ++l) s = __fmaf_rn(qs[(e >> BITS) * ds + l], c[l], s);
                ((float *)r.fail_lut)[row + e] = s;
            }
        }
        return;
    }
    const uint8_t *tab8 = U8 && BITS == 8 ? r.lut8 + (size_t)q * r.M * 256 : nullptr;
    for (int i = tid; i < n_fin; i += 256) {
        const int32_t id = (int32_t)(uint32_t)keys[i]; // replaced by the key below, by this thread
        // the row's bytes, 28 at a time: whole words from the one its first byte lies in (there is room behind the last row)
        const size_t at = (size_t)id * r.NB;
        const int shift = 8 * (int)(at & 3);
        const uint32_t *row = (const uint32_t *)(r.codes + (at & ~(size_t)3));
        uint32_t si = 0u;
        float sf = 0.0f;
        for (int b0 = 0; b0 < r.NB; b0 += 28) {
            uint32_t w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = b0 + 4 * u < r.NB + 3 ? row[b0 / 4 + u] : 0u;
#pragma unroll
            for (int u = 0; u < 7; ++u) {
                const uint32_t word = (uint32_t)((((u64)w[u + 1] << 32) | w[u]) >> shift);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int b = b0 + 4 * u + e;
                    if (b >= r.NB) continue;
                    const uint32_t byte = (word >> (8 * e)) & 255u;
                    if (BITS == 4) {
                        const float t0 = tbl[2 * b * 16 + (byte & 15u)], t1 = tbl[(2 * b + 1) * 16 + (byte >> 4)];
                        if (U8) si += __float_as_uint(t0) + __float_as_uint(t1);
                        else sf = __fadd_rn(sf, __fadd_rn(t0, t1));
                    } else if (U8) {
                        si += tab8[b * 256 + byte];
                    } else {
                        const float *c = r.codebooks + ((size_t)b * 256 + byte) * ds;
                        float v = 0.0f;
                        for (int l = 0; l < ds; ++l) v = __fmaf_rn(qs[b * ds + l], c[l], v);
                        sf = __fadd_rn(sf, v);
                    }
                }
            }
        }
        keys[i] = U8 ? make_key(si + 1u, id) : make_key(ord_from_f32(sf), id);
    }
    __syncthreads();
    const int want = r.reorder ? r.R : r.k; // k is R without reordering
    if (U8 && n_fin > 512) {
        // most of them are not among the R best: those below the bin of the R-th go before the ranking, which is quadratic
        const uint32_t bin = rth_bin(bins, (uint32_t)n_fin, 1u, (uint32_t)want, tid, [&](uint32_t i) { return key_ord(keys[i]); });
        if (tid == 0) n_fin_s = 0;
        u64 stay[FINAL / 256];
        int n_stay = 0;
#pragma unroll
        for (int u = 0; u < FINAL / 256; ++u) {
            const int i = tid + u * 256;
            stay[u] = i < n_fin && key_ord(keys[i]) >= bin ? keys[i] : 0ull;
            n_stay += stay[u] != 0ull;
        }
        __syncthreads();
        int to = n_stay > 0 ? atomicAdd(&n_fin_s, n_stay) : 0;
#pragma unroll
        for (int u = 0; u < FINAL / 256; ++u)
            if (stay[u] != 0ull) keys[to++] = stay[u];
        __syncthreads();
        n_fin = n_fin_s;
    }
    if (tid == 0 && (n_fin & 1)) keys[n_fin] = 0ull; // n_fin odd: below FINAL, which is even
    __syncthreads();
    rank_keys<FINAL>(keys, n_fin, want, best, tid); // at least R of them
    __syncthreads();
    int32_t *ids = r.ids_out + (size_t)q * r.k;
    float *scores = r.scores_out + (size_t)q * r.k;
    if (r.reorder) {
        for (int i = tid; i < r.R; i += 256) {
            const int32_t id = key_id(best[i]);
            keys[i] = make_key(ord_from_f32(row_dot_chain(qs, r.x + (size_t)id * r.d, r.d)), id);
        }
        if (tid == 0 && (r.R & 1)) keys[r.R] = 0ull;
        __syncthreads();
        rank_keys<512>(keys, r.R, r.k, best, tid); // all of best has been read
        __syncthreads();
    }
    for (int i = tid; i < r.k; i += 256) {
        const u64 key = best[i];
        float s;
        if (U8 && !r.reorder) s = __fmaf_rn((float)(int)(key_ord(key) - 1u), r.scale[q], r.bias[q]);
        else s = f32_from_ord(key_ord(key));
        ids[i] = key_id(key);
        scores[i] = s;
    }
}

// The answer of a query that was scanned plainly (workgroup b: fail_list[b]), from the scan's lists: merged, and scored against
// the points where asked.
__global__ void __launch_bounds__(1024)
product_fallback_kernel(const ProductRefineParams r, const u64 *__restrict__ partial, int max_chunks, int tile_queries, int ns, int u8)
{
    if (blockIdx.x >= *r.fail_count) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int n_chunks = scan_dynamic_chunks(((int)*r.fail_count + tile_queries - 1) / tile_queries, max_chunks);
    const int C = 64 * ns, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_waves = blockDim.x >> 6;
    const int q = r.fail_list[blockIdx.x];
    u64 *lists = (u64 *)smem;
    u64 *mine = lists + (size_t)wave * C;
    float *qs = (float *)(lists + (size_t)n_waves * C); // [d]
    for (int l = threadIdx.x; l < r.d; l += blockDim.x) qs[l] = r.queries[(size_t)q * r.d + l];
    wave_list_clear(mine, ns);
    for (int c = wave; c < n_chunks; c += n_waves) wave_list_merge_from(mine, ns, partial + ((size_t)blockIdx.x * n_chunks + c) * C);
    __syncthreads();
    if (wave > 0) return;
    for (int w = 1; w < n_waves; ++w) wave_list_merge_from(mine, ns, lists + (size_t)w * C);
    if (r.reorder) {
        u64 *again = lists + (size_t)(n_waves > 1 ? 1 : 0) * C; // another wave's list, merged by now
        u64 nk[8];
        const int slots = (r.R + 63) / 64; // at most 8
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int i = s * 64 + lane;
            nk[s] = 0ull;
            if (i < r.R && mine[i]) {
                const int32_t id = key_id(mine[i]);
                nk[s] = make_key(ord_from_f32(row_dot_chain(qs, r.x + (size_t)id * r.d, r.d)), id);
            }
        }
        wave_lds_fence();
        mine = again;
        wave_list_clear(mine, ns);
#pragma unroll
        for (int s = 0; s < 8; ++s)
            if (s < slots) wave_list_insert_sorted(mine, ns, wave_sort_desc(nk[s]));
    }
    for (int i = lane; i < r.k; i += 64) {
        const u64 key = mine[i]; // 0: none, the probed leaves of a partitioned index hold fewer points
        float s = -INFINITY;
        if (key) s = u8 && !r.reorder ? __fmaf_rn((float)(int)(key_ord(key) - 1u), r.scale[q], r.bias[q]) : f32_from_ord(key_ord(key));
        r.ids_out[(size_t)q * r.k + i] = key ? key_id(key) : -1;
        r.scores_out[(size_t)q * r.k + i] = s;
    }
}

// ---- host side -----------------------------------------------------------------

bool product_supported(int d, int M, int64_t n, int R) { return d <= 256 && M <= 256 && R < n && R <= AVQ_MAX_SELECT; }

// The launches for nq queries: grids, sample, classes.
ProductPlan product_plan(int nq, int64_t n, int d, int R, bool u8)
{
    ProductPlan pl{};
    pl.steps = product_steps(d);
    const int ct = product_ct(pl.steps), qt = product_qt(pl.steps);
    pl.n_tiles = ((nq + 31) / 32 + qt - 1) / qt * qt;
    const int64_t per = (int64_t)kProductWaves * ct * 32;
    pl.groups = (n + per - 1) / per;
    // 512 workgroups run side by side; the queries are cut into chunks until the last round is nearly full. Decoding costs a
    // workgroup about as much as four stages.
    auto cut = [&](int64_t groups, int32_t *per_chunk, int32_t *chunks) {
        const int stages = pl.n_tiles / qt;
        double best = 1e300;
        for (int c = 1; c <= stages && c <= 512; ++c) {
            const int spc = (stages + c - 1) / c, real = (stages + spc - 1) / spc;
            const double cost = std::ceil((double)groups * real / 512.0) * (4.0 + spc);
            if (cost < best * 0.999) { best = cost; *per_chunk = spc; *chunks = real; }
        }
    };
    cut(pl.groups, &pl.stages_per_chunk, &pl.chunks);
    // The sample: a 16th of the points (64th, ... of very many: classes for one workgroup's registers), more of a small index, all
    // of one below 25,000 points (or where R is not small against it), whose guess is then exact. mu of the R best fall into
    // the sample on average (Poisson); the r-th best of it is below the R-th best of all unless r or more do.
    int64_t stride = 16;
    while (stride > 1 && n / stride < std::max<int64_t>(12500, (int64_t)32 * R)) stride /= 2;
    while (n / stride / (ct * 16) > kProductMaxClasses / 4) stride *= 2;
    pl.stride = (int32_t)stride;
    const double mu = (double)R / (double)stride;
    pl.r = stride == 1 ? R : std::max(8, (int)std::ceil(mu + 5.0 * std::sqrt(mu) + 1.0));
    const int64_t subs = ((n + 31) / 32 + stride - 1) / stride;
    pl.sample_groups = (subs + kProductWaves * ct - 1) / (kProductWaves * ct);
    cut(pl.sample_groups, &pl.sample_stages_per_chunk, &pl.sample_chunks);
    // class size: as many products as leave eight classes per rank, and no more classes than the bound kernel holds
    pl.run = ct * 16;
    const int64_t lanes = pl.sample_groups * kProductWaves * 2;
    while (pl.run > 1 && lanes * (ct * 16 / pl.run) < (int64_t)8 * pl.r) pl.run = pl.run > 16 ? 16 : pl.run / 4;
    if (stride == 1)
        while (pl.run > 1 && lanes * (ct * 16 / pl.run) < n && lanes * (ct * 16 / pl.run) * 4 <= 8192) pl.run = pl.run > 16 ? 16 : pl.run / 4;
    pl.n_classes = (int32_t)(lanes * (ct * 16 / pl.run));
    pl.kept_cap = u8 ? ProductRoom<true>::kept : ProductRoom<false>::kept;
    pl.cnt_stride = spread_stride(nq);
    return pl;
}

template <int NS, int CT>
static int launch_product_ns(const ProductParams &p, bool sample, hipStream_t st)
{
    const int64_t grid = p.groups * p.chunks;
    if (grid > 0x7fffffff) { set_error("scan: grid too large"); return AVQ_EINVAL; }
    if (sample) hipLaunchKernelGGL((product_scan_kernel<NS, CT, true>), dim3((unsigned)grid), dim3(kProductWaves * 64), 0, st, p);
    else hipLaunchKernelGGL((product_scan_kernel<NS, CT, false>), dim3((unsigned)grid), dim3(kProductWaves * 64), 0, st, p);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_scan(const ProductParams &p, bool sample, hipStream_t st)
{
    switch (product_steps(p.d)) {
    case 1: return launch_product_ns<1, 4>(p, sample, st);
    case 2: return launch_product_ns<2, 4>(p, sample, st);
    case 3: return launch_product_ns<3, 4>(p, sample, st);
    case 4: return launch_product_ns<4, 4>(p, sample, st);
    case 5: return launch_product_ns<5, 4>(p, sample, st);
    case 6: return launch_product_ns<6, 4>(p, sample, st);
    case 7: return launch_product_ns<7, 4>(p, sample, st);
    case 8: return launch_product_ns<8, 4>(p, sample, st);
    case 10: return launch_product_ns<10, 2>(p, sample, st);
    case 12: return launch_product_ns<12, 2>(p, sample, st);
    case 14: return launch_product_ns<14, 2>(p, sample, st);
    case 16: return launch_product_ns<16, 2>(p, sample, st);
    default: set_error("scan: %d dimensions", p.d); return AVQ_EINVAL;
    }
}

int launch_product_pack(const ProductParams &p, const float *queries, const float *codebooks, uint32_t *fail_clear, int n_clear, bool rows,
                        hipStream_t st)
{
    hipLaunchKernelGGL(product_pack_kernel, dim3(1 + (p.n_tiles + 3) / 4), dim3(1024), 0, st, queries, p.nq, p.d, product_steps(p.d),
                       p.n_tiles, codebooks, p.M, 1 << p.bits, (_Float16 *)p.cb16, p.meta, (v8h *)p.packed, p.qinfo, p.kept_cnt,
                       p.cnt_stride, fail_clear, n_clear, rows ? 1 : 0);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_bound(const ProductParams &p, int r, const float *unit, float *margin, float *guess, const int32_t *leaf_ids,
                         const float *leaf_ip, int L, hipStream_t st)
{
    const int S = p.n_classes, nq_pad = p.n_tiles * 32;
    const bool u8 = unit != nullptr;
    auto go = [&](auto kern, int threads, int grid) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), 0, st, p.classes, S, r, p.nq, nq_pad, p.d, p.M, unit, u8, p.qinfo, p.meta, p.thr, margin, guess, leaf_ids,
                           leaf_ip, L);
    };
    if (S <= 512) go(product_bound_kernel<64, 8>, 256, (nq_pad + 3) / 4);
    else if (S <= 1280) go(product_bound_kernel<64, 20>, 256, (nq_pad + 3) / 4);
    else if (S <= 2048) go(product_bound_kernel<64, 32>, 256, (nq_pad + 3) / 4);
    else if (S <= 8192) go(product_bound_kernel<256, 32>, 256, nq_pad);
    else if (S <= kProductMaxClasses) go(product_bound_kernel<1024, 32>, 1024, nq_pad);
    else { set_error("scan: %d classes", S); return AVQ_EINVAL; }
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_refine(const ProductRefineParams &r, bool u8, int bits, hipStream_t st)
{
    const size_t lds = sizeof(u64) * ((u8 ? ProductRoom<true>::final : ProductRoom<false>::final) + (size_t)r.R + 4) +
                       sizeof(float) * (((size_t)r.d + 3) / 4 * 4) + (bits == 4 ? (size_t)2 * r.NB * 64 : 0);
    if (u8 && bits == 4) hipLaunchKernelGGL((product_refine_kernel<true, 4>), dim3(r.nq), dim3(256), lds, st, r);
    else if (u8) hipLaunchKernelGGL((product_refine_kernel<true, 8>), dim3(r.nq), dim3(256), lds, st, r);
    else if (bits == 4) hipLaunchKernelGGL((product_refine_kernel<false, 4>), dim3(r.nq), dim3(256), lds, st, r);
    else hipLaunchKernelGGL((product_refine_kernel<false, 8>), dim3(r.nq), dim3(256), lds, st, r);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_fallback(const ProductRefineParams &r, const u64 *partial, int max_chunks, int tile_queries, int ns, bool u8, hipStream_t st)
{
    int waves = 1;
    while (waves < 16 && waves * 4 <= max_chunks) waves *= 2;
    const size_t lds = sizeof(u64) * (size_t)waves * 64 * ns + sizeof(float) * (size_t)r.d;
    static LdsLimitOnce attr_done;
    AVQ_TRY(set_lds_limit((const void *)product_fallback_kernel, kMaxDynLds, &attr_done));
    hipLaunchKernelGGL(product_fallback_kernel, dim3(r.nq), dim3(waves * 64), lds, st, r, partial, max_chunks, tile_queries, ns, u8 ? 1 : 0);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

} // namespace avq
