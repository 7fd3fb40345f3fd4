// Batches on a partitioned index through a matrix product: the points of every probed leaf against the queries that probe it.
//
// As in product.hip the products decide which points are scored, with the same bound E on their error; a point's score here is
// its table sum plus <query, leaf center>. The (query, leaf) pairs are grouped by leaf. A first launch keeps the largest product
// of every class of 64 points (16, 4 where a query's leaves hold few points): R classes hold a point at or above the R-th
// largest of them, so that is a lower bound T of the R-th best product, and no guess: nothing has to be checked. A second launch
// keeps what reaches T - 2 E; those points are scored with the tables, ranked, and the R best scored exactly. A workgroup takes
// a block of 256 points and up to 512 queries, whose operands it gathers row by row.
//
// 10,000 queries, 100 of 2,000 leaves of 1,183,514 x 100 points: 2.8 to 3.0 ms with
// one-hot sums on the matrix cores against the R-th best of a query's first eight leaves (2,809 queries kept more than there was
// room for and were scanned again), 1.1 ms this way: 0.33 a launch, a third of it decoding.
#include <algorithm>
#include <type_traits>
#include "avq_internal.h"
#include "product_device.h"
#include "row_dot.h"
#include "wave_topk.h"

namespace avq {

constexpr int kLeafQueries = 512; // queries of a leaf that a workgroup takes

__global__ void __launch_bounds__(256)
product_clear_kernel(uint4 *__restrict__ a, int64_t na, uint4 *__restrict__ b, int64_t nb)
{
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < na + nb; i += step) {
        if (i < na) a[i] = make_uint4(0u, 0u, 0u, 0u);
        else b[i - na] = make_uint4(0u, 0u, 0u, 0u);
    }
}

// pair (query, slot) -> its place in the leaf's list, and <q, center>, scaled
__global__ void __launch_bounds__(256)
product_pairs_kernel(const int32_t *__restrict__ leaf_ids, const float *__restrict__ leaf_ip, const uint32_t *__restrict__ pos, int64_t n_pairs,
                     int L, const uint32_t *__restrict__ off, const ProductQuery *__restrict__ qinfo,
                     const ProductMeta *__restrict__ meta, uint32_t *__restrict__ qlist, float *__restrict__ pair_ip)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_pairs) return;
    const int32_t leaf = leaf_ids[i];
    if (leaf < 0) return;
    const uint32_t q = (uint32_t)(i / L), slot = (uint32_t)(i % L);
    const uint32_t to = off[leaf] + pos[i];
    qlist[to] = (q << 9) | slot;
    pair_ip[to] = ldexpf(leaf_ip[i], qinfo[q].exp + meta->exp);
}

// One workgroup: the items, (leaf, block and chunk of its queries).
__global__ void __launch_bounds__(1024)
product_items_kernel(const uint32_t *__restrict__ cnt, const int32_t *__restrict__ leaf_blk, int n_leaves, int most_items, uint2 *__restrict__ items,
                     uint32_t *__restrict__ n_items)
{
    __shared__ uint32_t part[1024];
    const int tid = threadIdx.x, per = (n_leaves + 1023) / 1024, lo = tid * per, hi = lo + per < n_leaves ? lo + per : n_leaves;
    auto chunks = [](uint32_t c) -> uint32_t { return (c + kLeafQueries - 1) / kLeafQueries; };
    uint32_t sum = 0u;
    for (int l = lo; l < hi; ++l) sum += (uint32_t)(leaf_blk[l + 1] - leaf_blk[l]) * chunks(cnt[l]);
    part[tid] = sum;
    __syncthreads();
    for (int d = 1; d < 1024; d *= 2) {
        const uint32_t x = tid >= d ? part[tid - d] : 0u;
        __syncthreads();
        part[tid] += x;
        __syncthreads();
    }
    if (tid == 1023) *n_items = part[tid]; // at most most_items
    uint32_t at = part[tid] - sum;
    for (int l = lo; l < hi; ++l) {
        const uint32_t b0 = (uint32_t)leaf_blk[l], b1 = (uint32_t)leaf_blk[l + 1], n_chunks = chunks(cnt[l]);
        for (uint32_t c = 0; c < n_chunks; ++c)
            for (uint32_t k = b0; k < b1; ++k, ++at)
                if (at < (uint32_t)most_items) items[at] = make_uint2((uint32_t)l, k << 8 | c);
    }
}

// pair_line[pair] = thr[query] - <q, center>: what a product has to reach
__global__ void __launch_bounds__(256)
product_lines_kernel(const uint32_t *__restrict__ qlist, const float *__restrict__ pair_ip, const float *__restrict__ thr, const uint32_t *__restrict__ off,
                     const uint32_t *__restrict__ cnt, int n_lists, int64_t n_pairs, float *__restrict__ pair_line)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_pairs || i >= (int64_t)off[n_lists - 1] + cnt[n_lists - 1]) return; // (fewer pairs than n_pairs where a query has fewer leaves)
    pair_line[i] = thr[qlist[i] >> 9] - pair_ip[i];
}

// The halves and their interleaving are those of product_scan_kernel; here a workgroup is 256 / (32 CT) waves, so four of them
// share a compute unit (two from 9 steps on), the operands of a tile's 32 queries are gathered, and a lane's line is its pair's.
template <int NS, int CT, bool SAMPLE>
__global__ void __launch_bounds__(64 * 8 / CT, 2)
product_leaf_kernel(const ProductLeafParams p)
{
    constexpr int WAVES = 8 / CT, PEND = product_pend(NS), HC = CT / 2, W = product_ahead(NS);
    __shared__ __align__(16) v8h tile[3][NS * 64];
    __shared__ __align__(16) float4 pend_s[WAVES][PEND][4]; // a lane's accumulators
    __shared__ uint2 tags_s[WAVES][PEND];                   // place in the chunk's list << 7 | point of the wave (accumulator 0's); the line
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    if (blockIdx.x >= *p.n_items) return;
    const uint2 it = p.items[blockIdx.x];
    const int leaf = (int)it.x;
    const int64_t blk = it.y >> 8;
    const uint32_t chunk = it.y & 255u;
    const uint32_t rest = p.leaf_cnt[leaf] - chunk * kLeafQueries, at_list = p.leaf_off[leaf] + chunk * kLeafQueries;
    const int n_q = (int)(rest < kLeafQueries ? rest : kLeafQueries);
    const uint32_t *const list = p.qlist + at_list;
    const float *const lines = (SAMPLE ? p.pair_ip : p.pair_line) + at_list;
    const int nt = (n_q + 31) / 32;

    auto entry_of = [&](int t) -> uint32_t { return t * 32 + j < n_q ? list[t * 32 + j] : 0xffffffffu; };
    auto line_of = [&](int t) -> float { return t * 32 + j < n_q ? lines[t * 32 + j] : INFINITY; };
    auto stage = [&](int slot, uint32_t e) {
        const v8h *row = (const v8h *)p.base.packed + (size_t)(e == 0xffffffffu ? 0u : e >> 9) * (2 * NS) + h;
        for (int s = wave; s < NS; s += WAVES)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(row + 2 * s),
                                             (__attribute__((address_space(3))) void *)(&tile[slot][0] + s * 64), 16, 0, 0);
    };
    uint32_t e_before = 0xffffffffu, e = entry_of(0), e1 = entry_of(1);
    float line_before = INFINITY, line = line_of(0), line1 = line_of(1);
    stage(0, e);
    float4(*const pend)[4] = pend_s[wave];
    uint2 *const tags = tags_s[wave];
    const int64_t first = blk * 256 + wave * (CT * 32);
    v8h a[CT][NS];
    product_decode<NS, CT, WAVES, 2 * NS * 1024, PEND * 64>(a, p.base, first, 32, (uint8_t *)&tile[1][0], (uint4 *)&pend[0][0]);
    int left = 0; // this wave's points: padding slots come last
#pragma unroll
    for (int c = 0; c < CT; ++c) left += (int)__popcll(__builtin_amdgcn_ballot_w64(h == 0 && p.perm[first + c * 32 + j] >= 0));
    left = __builtin_amdgcn_readfirstlane(left);
    const int leaf_blocks = p.leaf_blk[leaf + 1] - p.leaf_blk[leaf];
    const int per_lane = CT * 16 / p.run; // classes; a block has 256 / run
    const int first_class = ((int)(blk - p.leaf_blk[leaf]) * (256 / p.run)) % p.pair_classes + (wave * 2 + h) * per_lane;
    float first_half = -INFINITY;         // SAMPLE, one class a lane: its first half's largest

    int cnt = 0; // entries in the wave's buffer
    auto hand_over = [&](int take) __attribute__((always_inline)) { // the first `take` (at most 64)
        wave_lds_fence();
        uint32_t hits = 0u, en = 0u;
        uint2 tag = make_uint2(0u, 0u);
        float ip = 0.0f;
        if (lane < take) {
            tag = tags[lane];
            en = list[tag.x >> 7];
            ip = p.pair_ip[at_list + (tag.x >> 7)];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float4 w = pend[lane][r];
                const float x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (x[v] >= __uint_as_float(tag.y) && (int)(tag.x & 127u) + 8 * r + v < left) hits |= 1u << (4 * r + v);
            }
        }
        const uint32_t q = en >> 9;
        while (__builtin_amdgcn_ballot_w64(hits != 0u) != 0ull) {
            if (hits != 0u) {
                const int v = __builtin_ctz(hits);
                hits &= hits - 1u;
                const uint32_t at = (uint32_t)first + (tag.x & 127u) + 8 * (v >> 2) + (v & 3);
                const uint32_t pos = atomicAdd(p.base.kept_cnt + (size_t)q * p.base.cnt_stride, 1u);
                if (pos < (uint32_t)p.base.kept_cap) {
                    p.base.kept[(size_t)q * p.base.kept_cap + pos] = ((u64)ord_from_f32(((const float *)pend[lane])[v] + ip) << 32) | at;
                    p.kept_slot[(size_t)q * p.base.kept_cap + pos] = (uint16_t)(en & 511u);
                }
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
    auto max_part = [&](float &m, const v16f &x, int i) __attribute__((always_inline)) { // the i-th of eight instructions
        if (i == 0) m = max2(max2(x[0], x[1]), x[2]);
        else if (i < 7) m = max2(max2(m, x[2 * i + 1]), x[2 * i + 2]);
        else m = max2(m, x[15]);
    };
    auto keep_half = [&](auto which, int tl, float ln, const float (&big)[HC]) __attribute__((always_inline)) {
        constexpr int H = decltype(which)::value;
#pragma unroll
        for (int cc = 0; cc < HC; ++cc) {
            const int c = H * HC + cc;
            const u64 mask = __builtin_amdgcn_ballot_w64(big[cc] >= ln);
            if (__builtin_expect(mask == 0ull, 1)) continue;
            if (__builtin_expect(cnt > PEND - 64, 0)) hand_over(cnt < 64 ? cnt : 64);
            const int to = cnt + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (big[cc] >= ln) {
#pragma unroll
                for (int r = 0; r < 4; ++r) pend[to][r] = make_float4(acc[c][4 * r], acc[c][4 * r + 1], acc[c][4 * r + 2], acc[c][4 * r + 3]);
                tags[to] = make_uint2(((uint32_t)tl * 32u + (uint32_t)j) << 7 | (uint32_t)(4 * h + c * 32), __float_as_uint(ln));
            }
            cnt += (int)__popcll(mask);
        }
    };
    // a lane's classes: the largest of all its products, of the 16 of each 32 points, or of every four, plus <q, center>
    auto sample_half = [&](auto which, uint32_t en, float ip, const float (&big)[HC]) __attribute__((always_inline)) {
        constexpr int H = decltype(which)::value;
        const bool part = left < CT * 32;
        if (part) { // some of the points are not there
            int rest_points = left - 4 * h;
            asm volatile("" : "+v"(rest_points)); // the compares below stay in here
#pragma unroll
            for (int cc = 0; cc < HC; ++cc)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if ((H * HC + cc) * 32 + 8 * (v / 4) + v % 4 >= rest_points) acc[H * HC + cc][v] = -INFINITY;
        }
        float m[HC];
#pragma unroll
        for (int cc = 0; cc < HC; ++cc) {
            m[cc] = big[cc];
            if (part)
#pragma unroll
                for (int i = 0; i < 8; ++i) max_part(m[cc], acc[H * HC + cc], i);
        }
        float all = m[0];
#pragma unroll
        for (int cc = 1; cc < HC; ++cc) all = max2(all, m[cc]);
        if (H == 0) first_half = all;
        if (en == 0xffffffffu) return;
        uint32_t *dst = p.classes + ((size_t)(en >> 9) * p.L + (en & 511u)) * p.pair_classes + first_class;
        auto put = [&](int i, float x) __attribute__((always_inline)) {
            if (x == -INFINITY) return;
            const uint32_t o = ord_from_f32(x + ip);
            if (leaf_blocks * (256 / p.run) <= p.pair_classes) dst[i] = o;
            else atomicMax(dst + i, o); // the blocks of a large leaf share the classes
        };
        if (p.run == 4) {
#pragma unroll
            for (int cc = 0; cc < HC; ++cc) {
                const v16f &x = acc[H * HC + cc];
#pragma unroll
                for (int r = 0; r < 4; ++r) put((H * HC + cc) * 4 + r, max2(max2(x[4 * r], x[4 * r + 1]), max2(x[4 * r + 2], x[4 * r + 3])));
            }
        } else if (p.run == 16) {
#pragma unroll
            for (int cc = 0; cc < HC; ++cc) put(H * HC + cc, m[cc]);
        } else if (H == 1) {
            put(0, max2(all, first_half));
        }
    };

    __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0): this wave's part of the first tile is in LDS
    __syncthreads();
    if (nt > 1) stage(1, e1);
    uint32_t e2 = entry_of(2);
    v8h b[W]; // operand of step s in b[s % W]
#pragma unroll
    for (int s = 0; s < W; ++s) b[s] = tile[0][s * 64 + lane];
    int slot = 0;
#pragma unroll 1
    for (int t = 0; t < nt; ++t) {
        const int slot1 = slot == 2 ? 0 : slot + 1, slot2 = slot1 == 2 ? 0 : slot1 + 1;
        const v8h *cur = tile[slot], *nxt = tile[slot1];
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
        if (left > 0) {
            half(std::integral_constant<int, 0>{}, cur);
            if constexpr (SAMPLE) sample_half(std::integral_constant<int, 1>{}, e_before, line_before, big);
            else keep_half(std::integral_constant<int, 1>{}, t - 1, line_before, big);
        }
        if (t + 1 < nt) {
            // the next tile is there; every wave has left the one before this, whose buffer the one after next takes
            __builtin_amdgcn_s_waitcnt(0x0f70);
            __syncthreads();
            if (t + 2 < nt) stage(slot2, e2);
        }
        const uint32_t e3 = entry_of(t + 3);
        const float line2 = line_of(t + 2);
        if (left > 0) {
            half(std::integral_constant<int, 1>{}, nxt); // operands beyond the last tile: not used
            if constexpr (SAMPLE) sample_half(std::integral_constant<int, 0>{}, e, line, big);
            else keep_half(std::integral_constant<int, 0>{}, t, line, big);
        }
        e_before = e; e = e1; e1 = e2; e2 = e3;
        line_before = line; line = line1; line1 = line2;
        slot = slot1;
    }
    if (left > 0) {
        float big[HC];
#pragma unroll
        for (int cc = 0; cc < HC; ++cc)
#pragma unroll
            for (int i = 0; i < 8; ++i) max_part(big[cc], acc[HC + cc], i);
        if constexpr (SAMPLE) {
            sample_half(std::integral_constant<int, 1>{}, e_before, line_before, big);
        } else {
            keep_half(std::integral_constant<int, 1>{}, nt - 1, line_before, big);
            while (cnt > 0) hand_over(cnt < 64 ? cnt : 64);
        }
    }
}

// As product_refine_kernel, per query: the kept points' table sums plus <q, center>.
template <bool U8, int BITS>
__global__ void __launch_bounds__(256)
product_leaf_refine_kernel(const ProductLeafRefineParams r)
{
    constexpr int FINAL = ProductRoom<U8>::final;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ BinScratch bins;
    __shared__ int n_fin_s, slot_s;
    const ProductRefineParams &b = r.base;
    const int tid = threadIdx.x, q = blockIdx.x;
    u64 *keys = (u64 *)smem;                           // [FINAL]
    u64 *best = keys + FINAL;                          // [R + 1]
    float *ips = (float *)(best + b.R + (b.R & 1) + 2); // [FINAL] <q, center> of the finalists
    float *qs = ips + FINAL;                           // [d]
    float *tbl = qs + ((b.d + 3) & ~3);                // 4-bit codes: [2 NB][16], the fp32 tables or the 8-bit ones as numbers
    const int ds = b.d / b.M;
    const uint32_t total = b.kept_cnt[(size_t)q * b.cnt_stride];
    const float m2 = b.margin[q], guess = b.guess[q]; // 2 E, T (-infinity: none)
    bool ok = m2 >= 0.0f && total <= (uint32_t)b.kept_cap;
    int why = m2 >= 0.0f ? 1 : 3;
    if (b.force_fail_odd && (q & 1)) { ok = false; why = 3; }
    if (tid == 0) n_fin_s = 0;
    bins.hist[tid] = 0u;
    const u64 *kept = b.kept + (size_t)q * b.kept_cap;
    for (int l = tid; l < b.d; l += 256) qs[l] = b.queries[(size_t)q * b.d + l];
    const float scale = U8 ? b.scale[q] : 0.0f, bias = U8 ? b.bias[q] : 0.0f;
    if (ok) {
        uint32_t keep = 0u;
        if (total > (uint32_t)b.R || guess > -INFINITY) {
            const uint32_t bin = rth_bin(bins, total, guess > -INFINITY ? ord_from_f32(guess) : 1u, (uint32_t)b.R, tid, [&](uint32_t i) { return (uint32_t)(kept[i] >> 32); });
            if (bin == 0u) { // fewer than R reach T
                ok = false;
                why = 2;
            } else {
                keep = ord_from_f32(f32_from_ord(bin) - m2);
            }
            bins.hist[tid] = 0u;
        } else {
            __syncthreads(); // the same number of barriers is not needed: the whole workgroup is here
        }
        if (ok) {
            for (uint32_t i = tid; i < total; i += 256u) {
                const u64 e = kept[i];
                if ((uint32_t)(e >> 32) < keep) continue;
                const int slot = atomicAdd(&n_fin_s, 1);
                if (slot < FINAL) {
                    keys[slot] = (uint32_t)r.perm[(uint32_t)e];
                    ips[slot] = r.leaf_ip[(size_t)q * r.L + r.kept_slot[(size_t)q * b.kept_cap + i]];
                }
            }
            if (BITS == 4) {
                const uint8_t *tab8 = U8 ? b.lut8 + (size_t)q * b.M * 16 : nullptr;
                for (int e = tid; e < 2 * b.NB * 16; e += 256) {
                    const int m = e >> 4;
                    float s = 0.0f;
                    if (m < b.M) {
                        if (U8) {
                            s = __uint_as_float(tab8[e]);
                        } else {
                            const float *c = b.codebooks + (size_t)e * ds;
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
    if (!ok) { // its tables and leaves beside those of the other such queries, for the plain scan
        if (tid == 0) {
            slot_s = (int)atomicAdd(b.fail_count, 1u);
            b.fail_list[slot_s] = q;
            atomicAdd(b.fail_total, 1u); // statistics of the call: 1 = too many kept points, 2 = bound too high, 3 = other
            atomicAdd(b.fail_total + why, 1u);
            if (U8) { r.fail_scale[slot_s] = scale; r.fail_bias[slot_s] = bias; }
        }
        __syncthreads();
        const int entries = b.M << BITS;
        const size_t row = (size_t)slot_s * entries;
        for (int e = tid; e < entries; e += 256) {
            if (U8) {
                ((uint8_t *)b.fail_lut)[row + e] = b.lut8[(size_t)q * entries + e];
            } else {
                const float *c = b.codebooks + (size_t)e * ds;
                float s = 0.0f;
                for (int l = 0; l < ds; ++l) s = __fmaf_rn(qs[(e >> BITS) * ds + l], c[l], s);
                ((float *)b.fail_lut)[row + e] = s;
            }
        }
        for (int l = tid; l < r.L; l += 256) {
            r.fail_ip[(size_t)slot_s * r.L + l] = r.leaf_ip[(size_t)q * r.L + l];
            r.fail_ids[(size_t)slot_s * r.L + l] = r.leaf_ids[(size_t)q * r.L + l];
        }
        return;
    }
    const uint8_t *tab8 = U8 && BITS == 8 ? b.lut8 + (size_t)q * b.M * 256 : nullptr;
    for (int i = tid; i < n_fin; i += 256) {
        const int32_t id = (int32_t)(uint32_t)keys[i]; // replaced by the key below, by this thread
        // the row's bytes, 28 at a time: whole words from the one its first byte lies in (there is room behind the last row)
        const size_t at = (size_t)id * b.NB;
        const int shift = 8 * (int)(at & 3);
        const uint32_t *row = (const uint32_t *)(b.codes + (at & ~(size_t)3));
        uint32_t si = 0u;
        float sf = 0.0f;
        for (int b0 = 0; b0 < b.NB; b0 += 28) {
            uint32_t w[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) w[u] = b0 + 4 * u < b.NB + 3 ? row[b0 / 4 + u] : 0u;
#pragma unroll
            for (int u = 0; u < 7; ++u) {
                const uint32_t word = (uint32_t)((((u64)w[u + 1] << 32) | w[u]) >> shift);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = b0 + 4 * u + e;
                    if (k >= b.NB) continue;
                    const uint32_t byte = (word >> (8 * e)) & 255u;
                    if (BITS == 4) {
                        const float t0 = tbl[2 * k * 16 + (byte & 15u)], t1 = tbl[(2 * k + 1) * 16 + (byte >> 4)];
                        if (U8) si += __float_as_uint(t0) + __float_as_uint(t1);
                        else sf = __fadd_rn(sf, __fadd_rn(t0, t1));
                    } else if (U8) {
                        si += tab8[k * 256 + byte];
                    } else {
                        const float *c = b.codebooks + ((size_t)k * 256 + byte) * ds;
                        float v = 0.0f;
                        for (int l = 0; l < ds; ++l) v = __fmaf_rn(qs[k * ds + l], c[l], v);
                        sf = __fadd_rn(sf, v);
                    }
                }
            }
        }
        const float s = U8 ? __fmaf_rn((float)(int)si, scale, __fadd_rn(bias, ips[i])) : __fadd_rn(sf, ips[i]);
        keys[i] = make_key(ord_from_f32(s), id);
    }
    __syncthreads();
    const int want = b.reorder ? b.R : b.k; // k is R without reordering
    if (n_fin > 512) {
        // most of them are not among the R best: those below the bin of the R-th go before the ranking, which is quadratic
        const uint32_t bin = n_fin > want ? rth_bin(bins, (uint32_t)n_fin, 1u, (uint32_t)want, tid, [&](uint32_t i) { return key_ord(keys[i]); }) : 0u;
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
    rank_keys<FINAL>(keys, n_fin, want, best, tid);
    __syncthreads();
    const int found = n_fin < want ? n_fin : want; // fewer points than that in all probed leaves
    int n_out = found;
    if (b.reorder) {
        for (int i = tid; i < found; i += 256) {
            const int32_t id = key_id(best[i]);
            keys[i] = make_key(ord_from_f32(row_dot_chain(qs, b.x + (size_t)id * b.d, b.d)), id);
        }
        if (tid == 0 && (found & 1)) keys[found] = 0ull;
        __syncthreads();
        rank_keys<512>(keys, found, b.k, best, tid); // all of best has been read
        __syncthreads();
        n_out = found < b.k ? found : b.k;
    }
    for (int i = tid; i < b.k; i += 256) {
        b.ids_out[(size_t)q * b.k + i] = i < n_out ? key_id(best[i]) : -1;
        b.scores_out[(size_t)q * b.k + i] = i < n_out ? f32_from_ord(key_ord(best[i])) : -INFINITY;
    }
}

// ---- host side -----------------------------------------------------------------

bool product_leaf_supported(int d, int M, int n_leaves, int64_t n_blocks, int64_t max_leaf_blocks, int nq, int L, int R)
{
    return d <= 256 && M <= 256 && L >= 2 && L <= 512 && nq <= (1 << 16) && n_leaves <= (1 << 20) && n_blocks < (1 << 24) &&
           max_leaf_blocks <= 1024 && R <= AVQ_MAX_SELECT;
}

// Every leaf's blocks once, and again for every further kLeafQueries of its queries (a query probes a leaf once).
static int64_t product_leaf_items(int nq, int L, int64_t n_blocks, int64_t max_leaf_blocks)
{
    return n_blocks + std::min(max_leaf_blocks * ((int64_t)nq * L / kLeafQueries), n_blocks * (nq / kLeafQueries));
}

bool product_leaf_narrow(int L, int n_leaves, int R) { return (double)L < (R > 256 ? 0.06 : 0.03) * n_leaves; }

// Scratch for nq queries: words, slots and items of the launches.
ProductLeafPlan product_leaf_plan(int nq, int L, int n_leaves, int64_t n, int64_t n_blocks, int64_t max_leaf_blocks, int d, int R, bool u8)
{
    ProductLeafPlan pl{};
    pl.steps = product_steps(d);
    pl.n_tiles = (nq + 127) / 128 * 4;
    // Classes as large as leave three of them per result, at most all of a lane's products. Where a query probes a few leaves in
    // a hundred, its best points lie in a few of those, and large classes would leave a line far below them and more points than
    // there is room for: smaller ones, and with many results more blocks with classes of their own. (10,000,000 points, 3,000 queries, R =
    // 500, 20 of 2,000 leaves: 320 classes 18.8 ms, every query scanned plainly, 20,480 of them 3.5; 4,000,000, 40 of 4,000 leaves,
    // R = 100 1.41 / 1.16, R = 500 4.2 / 1.9. Classes of four points where 100 leaves are probed cost too much otherwise: 2.3 / 14 ms.)
    const double points = (double)L * (double)n / n_leaves;
    const int whole = product_ct(pl.steps) * 16;
    const bool narrow = product_leaf_narrow(L, n_leaves, R);
    pl.run = points >= 3.0 * whole * R && !narrow ? whole : points >= 48.0 * R && !(narrow && R > 256 && L <= 128) ? 16 : 4;
    // up to four blocks of a leaf have classes of their own
    const int64_t own_blocks = narrow && R > 256 ? 16 : 4;
    pl.pair_classes = (int)std::min<int64_t>(own_blocks, std::max<int64_t>(1, max_leaf_blocks)) * (256 / pl.run);
    while ((int64_t)L * pl.pair_classes > kProductMaxClasses && pl.pair_classes > 256 / pl.run) pl.pair_classes -= 256 / pl.run;
    while ((int64_t)L * pl.pair_classes > kProductMaxClasses && pl.run < 16) { pl.run = 16; pl.pair_classes = 16; }
    pl.n_classes = L * pl.pair_classes;
    pl.most_items = product_leaf_items(nq, L, n_blocks, max_leaf_blocks);
    pl.cnt_stride = spread_stride(nq);
    pl.kept_cap = u8 ? ProductRoom<true>::kept : ProductRoom<false>::kept;
    return pl;
}

// Queries of one part of a batch: as many as `most` bytes hold at `other` bytes a query beside the plan's, and no more than a
// launch of a workgroup per item allows (below 2^32 threads; fewer than kLeafQueries queries always do, as n_blocks is
// below 2^24).
int product_leaf_part(int nq, int L, int n_leaves, int64_t n, int64_t n_blocks, int64_t max_leaf_blocks, int d, int R, bool u8, size_t other, size_t most)
{
    const ProductLeafPlan pl = product_leaf_plan(nq, L, n_leaves, n, n_blocks, max_leaf_blocks, d, R, u8);
    const size_t row = (size_t)pl.n_classes * 4 + (size_t)pl.kept_cap * 10 + (size_t)pl.steps * 32 + (size_t)L * 24 + 256 + other;
    const int64_t threads = 64 * 8 / product_ct(pl.steps);
    int per = (int)std::min<int64_t>(nq, std::max<int64_t>(64, (int64_t)(most / row)));
    while (per >= kLeafQueries && product_leaf_items(per, L, n_blocks, max_leaf_blocks) * threads >= ((int64_t)1 << 32)) per -= per / 8;
    const int parts = (nq + per - 1) / per; // of about the same size
    return (nq + parts - 1) / parts;
}

int launch_product_clear(void *a, size_t a_bytes, void *b, size_t b_bytes, hipStream_t st)
{
    const int64_t na = (int64_t)(a_bytes / 16), nb = (int64_t)(b_bytes / 16), n = na + nb;
    hipLaunchKernelGGL(product_clear_kernel, dim3((unsigned)std::min<int64_t>(2048, (n + 255) / 256)), dim3(256), 0, st, (uint4 *)a, na, (uint4 *)b, nb);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_pairs(const ProductLeafParams &p, const int32_t *leaf_ids, const float *leaf_ip, const uint32_t *pos, int n_leaves,
                         uint2 *items, int64_t most_items, uint32_t *n_items, hipStream_t st)
{
    const int64_t n_pairs = (int64_t)p.base.nq * p.L;
    hipLaunchKernelGGL(product_pairs_kernel, dim3((unsigned)((n_pairs + 255) / 256)), dim3(256), 0, st, leaf_ids, leaf_ip, pos, n_pairs, p.L,
                       p.leaf_off, p.base.qinfo, p.base.meta, p.qlist, p.pair_ip);
    hipLaunchKernelGGL(product_items_kernel, dim3(1), dim3(1024), 0, st, p.leaf_cnt, p.leaf_blk, n_leaves, (int)most_items, items, n_items);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_lines(const ProductLeafParams &p, int n_leaves, hipStream_t st)
{
    const int64_t n_pairs = (int64_t)p.base.nq * p.L;
    hipLaunchKernelGGL(product_lines_kernel, dim3((unsigned)((n_pairs + 255) / 256)), dim3(256), 0, st, p.qlist, p.pair_ip, p.base.thr, p.leaf_off,
                       p.leaf_cnt, n_leaves, n_pairs, p.pair_line);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

template <int NS, int CT>
static int launch_product_leaf_ns(const ProductLeafParams &p, bool sample, int64_t most_items, hipStream_t st)
{
    const unsigned grid = (unsigned)most_items;
    if (sample) hipLaunchKernelGGL((product_leaf_kernel<NS, CT, true>), dim3(grid), dim3(64 * 8 / CT), 0, st, p);
    else hipLaunchKernelGGL((product_leaf_kernel<NS, CT, false>), dim3(grid), dim3(64 * 8 / CT), 0, st, p);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

int launch_product_leaf(const ProductLeafParams &p, bool sample, int64_t most_items, hipStream_t st)
{
    switch (product_steps(p.base.d)) {
    case 1: return launch_product_leaf_ns<1, 4>(p, sample, most_items, st);
    case 2: return launch_product_leaf_ns<2, 4>(p, sample, most_items, st);
    case 3: return launch_product_leaf_ns<3, 4>(p, sample, most_items, st);
    case 4: return launch_product_leaf_ns<4, 4>(p, sample, most_items, st);
    case 5: return launch_product_leaf_ns<5, 4>(p, sample, most_items, st);
    case 6: return launch_product_leaf_ns<6, 4>(p, sample, most_items, st);
    case 7: return launch_product_leaf_ns<7, 4>(p, sample, most_items, st);
    case 8: return launch_product_leaf_ns<8, 4>(p, sample, most_items, st);
    case 10: return launch_product_leaf_ns<10, 2>(p, sample, most_items, st);
    case 12: return launch_product_leaf_ns<12, 2>(p, sample, most_items, st);
    case 14: return launch_product_leaf_ns<14, 2>(p, sample, most_items, st);
    case 16: return launch_product_leaf_ns<16, 2>(p, sample, most_items, st);
    default: set_error("scan: %d dimensions", p.base.d); return AVQ_EINVAL;
    }
}

int launch_product_leaf_refine(const ProductLeafRefineParams &r, bool u8, int bits, hipStream_t st)
{
    const size_t fin = u8 ? ProductRoom<true>::final : ProductRoom<false>::final;
    const size_t lds = sizeof(u64) * (fin + (size_t)r.base.R + 4) + sizeof(float) * (fin + ((size_t)r.base.d + 3) / 4 * 4) +
                       (bits == 4 ? (size_t)2 * r.base.NB * 64 : 0);
    static LdsLimitOnce attr_done[4];
    auto go = [&](auto kern, LdsLimitOnce *once) -> int {
        AVQ_TRY(set_lds_limit((const void *)kern, 96 * 1024, once));
        hipLaunchKernelGGL(kern, dim3(r.base.nq), dim3(256), lds, st, r);
        AVQ_HIP(hipGetLastError());
        return AVQ_OK;
    };
    if (u8 && bits == 4) return go(product_leaf_refine_kernel<true, 4>, &attr_done[0]);
    if (u8) return go(product_leaf_refine_kernel<true, 8>, &attr_done[1]);
    if (bits == 4) return go(product_leaf_refine_kernel<false, 4>, &attr_done[2]);
    return go(product_leaf_refine_kernel<false, 8>, &attr_done[3]);
}

} // namespace avq
