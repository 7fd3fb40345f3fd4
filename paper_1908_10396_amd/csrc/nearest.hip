// Nearest centers, and Lloyd's algorithm for the leaf centers (paper Section 4; Section 5.3's tree).
//
// The nearest center of a point is the one with the largest s_j = <x, c_j> - ||c_j||^2 / 2, a matrix product of
// points and centers. It is formed on the matrix cores in f16, with fp32 sums, and only has to name the few
// centers that can be nearest: every s_j computed that way is within a bound E(x) of the real one (nearest_bound
// below), so a center whose value is more than 2 E under the largest is not the nearest. Per point the kernel
// keeps the two best centers and what bounds the third best value. Mostly the best one stands alone; a few points in a
// hundred are decided between two centers, and a few in a thousand against all of them, by fp64 squared distances, lowest
// index on ties: the assignment is that of an fp64 evaluation of every distance.
//
// 262,144 x 100 points, 2,000 centers: product and bookkeeping 0.139 ms (0.062 ms of matrix instructions at the 1.9 GHz it
// runs at, 0.036 ms for the points' operands and the lists; the vector instructions, 65 for every 32 x 32 values against
// seven matrix instructions, are the longer of the two that overlap), open points 0.05 ms; every distance in fp64 took 21 ms.
// 1,183,514 points: 0.58 + 0.08 ms (73 ms). With the products and the vector instructions of a tile one after the other, four
// of those for each value and a tile ahead, it was 0.20 and 1.05 ms.
#include <cmath>
#include <type_traits>
#include "avq_internal.h"

namespace avq {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

// Three further coordinates carry the term -||c||^2 / 2: the point holds kOne in each, the center a three-term f16
// split of the value. Coordinates are scaled by a power of two so that the largest center coordinate lies in
// [128, 256): far above the f16 subnormals, and no sum can reach the value of a padding center (-60000 kOne) as long
// as the point's coordinates stay below kMaxCoord; a point outside that is decided in fp64.
constexpr float kOne = 2048.0f, kMaxCoord = 1024.0f, kPadBias = -60000.0f;

// what the kernels share about the centers of one call (device memory)
struct NearMeta {
    float scale;           // the power of two
    uint32_t norm, err, bias; // float bits of the largest ||c||, ||c - c'||, ||c||^2 / 2 (scaled)
    uint32_t n_pairs, n_all;  // points to decide between two centers / against all
};

__global__ void __launch_bounds__(256)
near_absmax_kernel(const float *__restrict__ c, int64_t count, float *__restrict__ part, NearMeta *__restrict__ meta)
{
    __shared__ float red[256];
    float m = 0.0f;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) m = fmaxf(m, fabsf(c[i]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        meta->norm = 0u; meta->err = 0u; meta->bias = 0u; meta->n_pairs = 0u; meta->n_all = 0u;
    }
}
constexpr int kAbsmaxBlocks = 64;

// One workgroup per tile of 32 centers: the tile in operand order, [step][lane][8 halves], lane (row r = lane % 32,
// half lane / 32) holding coordinates 16 step + 8 (lane / 32) .. + 7 of center r. Clears the tile's pair counters.
__global__ void __launch_bounds__(256)
near_pack_kernel(const float *__restrict__ centers, int k, int d, int steps, const float *__restrict__ absmax,
                 v8h *__restrict__ packed, NearMeta *__restrict__ meta, uint32_t *__restrict__ cnt, int cnt_stride)
{
    __shared__ double part_n[256], part_e[256];
    __shared__ float bias[32][3];
    const int tid = threadIdx.x, t = blockIdx.x;
    float mx = 0.0f;
    for (int i = 0; i < kAbsmaxBlocks; ++i) mx = fmaxf(mx, absmax[i]);
    int e = 0;
    if (mx > 0.0f) { (void)frexpf(mx, &e); } // mx in [2^(e-1), 2^e)
    const float scale = mx > 0.0f ? ldexpf(1.0f, 8 - e < 120 ? 8 - e : 120) : 1.0f;
    if (t == 0 && tid == 0) meta->scale = scale;
    // norms and conversion errors: eight threads per center
    const int r = tid >> 3, g = tid & 7, j = t * 32 + r;
    double nn = 0.0, ee = 0.0;
    if (j < k) {
        for (int l = g; l < d; l += 8) {
            const float v = centers[(size_t)j * d + l] * scale;
            const double dv = (double)v, de = dv - (double)(float)(_Float16)v;
            nn += dv * dv;
            ee += de * de;
        }
    }
    part_n[tid] = nn;
    part_e[tid] = ee;
    __syncthreads();
    if (g == 0) {
        for (int u = 1; u < 8; ++u) { nn += part_n[tid + u]; ee += part_e[tid + u]; }
        double b = j < k ? -0.5 * nn / (double)kOne : (double)kPadBias;
        for (int u = 0; u < 3; ++u) {
            const float h = (float)(_Float16)(float)b;
            bias[r][u] = h;
            b -= (double)h;
        }
        if (j < k) {
            cnt[(size_t)j * cnt_stride] = 0u;
            atomicMax(&meta->norm, __float_as_uint((float)(sqrt(nn) * 1.0001)));
            atomicMax(&meta->err, __float_as_uint((float)(sqrt(ee) * 1.0001)));
            atomicMax(&meta->bias, __float_as_uint((float)(0.5 * nn * 1.0001)));
        }
    }
    __syncthreads();
    for (int f = tid; f < steps * 64; f += 256) {
        const int lane = f & 63, s = f >> 6, row = lane & 31, jj = t * 32 + row;
        v8h o;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int l = 16 * s + 8 * (lane >> 5) + i;
            float v = 0.0f;
            if (l < d) v = jj < k ? centers[(size_t)jj * d + l] * scale : 0.0f;
            else if (l < d + 3) v = bias[row][l - d];
            o[i] = (_Float16)v;
        }
        packed[(size_t)t * steps * 64 + f] = o;
    }
}

// |s computed - s| <= E. nx = ||x||, ex = ||x - x'|| of the point and the largest norm, error and bias of the centers:
// the conversions move <x, c> by at most ex ||c|| + ||x'|| ||c - c'||; fp32 accumulation of `terms` products by at most
// terms 2^-24 of the sum of magnitudes (2^-23 taken: the order and the rounding inside the instruction are its own);
// the position packed into the four lowest bits by 2^-19 of the value; f16 subnormals, should they be flushed, by 2^-14
// per coordinate.
__device__ __forceinline__ float nearest_bound(float nx, float ex, int terms, const NearMeta &m)
{
    const float cn = __uint_as_float(m.norm), ce = __uint_as_float(m.err), cb = __uint_as_float(m.bias);
    const float mag = nx * cn + cb;
    return 1.001f * (ex * cn + (nx + ex) * ce + ((float)terms * 1.2e-7f + 1.91e-6f) * mag + 6.2e-5f * sqrtf((float)terms) * (nx + cn + kOne));
}

// 64 points per wave as two column tiles of 32 (their operands stay in registers; one column tile above 141 coordinates), all
// centers as row tiles through LDS, up to two tiles ahead. A lane sees 16 centers of a tile for its point (lanes j and j + 32
// share point j % 32). The products of one accumulator are issued between the vector instructions that look through the other
// one, so that both units work (sched_barrier keeps the order). A group of
// four values gives its largest to the three best and its second to a bound on what was passed over, 11.5 instructions instead
// of 16 (0.175 -> 0.160 ms); a single tile to a stage leaves room for three waves per SIMD (0.160 -> 0.150). FEW: one column tile, and
// every value goes to the three best: among few centers the second is often in the best one's group, whose point would then
// be decided against all.
// assign[i] = nearest center; points that need fp64 go to pairs (point, center, center, -) and all_list (point).
// cnt / pos (optional): as in launch_nearest.
template <int NS, int CT, bool FEW>
__global__ void __launch_bounds__(256, 2)
nearest_mfma_kernel(const float *__restrict__ x, int64_t n, int d, const v8h *__restrict__ packed, int n_tiles, int k,
                    NearMeta *__restrict__ meta, int32_t *__restrict__ assign, int4 *__restrict__ pairs,
                    int32_t *__restrict__ all_list, uint32_t *__restrict__ cnt, int cnt_stride, uint32_t *__restrict__ pos)
{
    constexpr int G = CT == 2 || (FEW && NS <= 9) ? 4 : 2, Q = 4 * G; // the rows come in parts of G steps: Q quads of coordinates
    constexpr int kStage = NS * 64, kRows = 4 * 32 * Q;
    __shared__ __align__(16) v8h tile[2 * kStage + (kStage > kRows ? kStage : kRows)]; // three tiles; the third's place holds rows first
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), j = lane & 31, h = lane >> 5;
    const float scale = meta->scale;
    auto to_lds16 = [](const void *src, v8h *dst) __attribute__((always_inline)) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    };
    auto to_lds4 = [](const void *src, v8h *dst) __attribute__((always_inline)) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)dst, 4, 0, 0);
    };
    auto stage = [&](int t, int slot) { // a tile is NS KB in operand order: each wave copies a quarter of it
        for (int s = wave; s < NS; s += 4) to_lds16(packed + (size_t)t * kStage + s * 64 + lane, tile + slot * kStage + s * 64);
    };

    // The operands of the points. A wave's rows go through LDS, a part of 16 G coordinates of 32 rows at a time, in pieces that
    // are contiguous in memory (the code for rows read directly, by aligned quads or by single values, took 200 registers and
    // more, or spilled them). Quad q of row r lies at place q ^ turn(r), so that
    // lanes of different rows read different banks.
    v8h b[CT][NS];
    float nx[CT], ex[CT];
    bool far_out[CT];
    const int64_t p0 = (int64_t)blockIdx.x * (4 * CT * 32) + wave * (CT * 32);
    const bool quad = (d & 3) == 0 && ((uintptr_t)x & 15) == 0;
    v8h *rows = tile + 2 * kStage + wave * (32 * Q);
    auto turned = [](int r) { return Q == 16 ? r & 15 : (r >> 1) & 7; };
    auto fetch = [&](int c, int s0) __attribute__((always_inline)) {
        auto from = [&](int r, int l) { // coordinate l of row r; past the last ones: some in range, not used
            const int64_t i = p0 + c * 32 + r;
            return x + (size_t)(i < n ? i : n - 1) * d + l;
        };
        if (quad) {
#pragma unroll 4
            for (int e = lane; e < 32 * Q; e += 64) {
                const int r = e / Q, l = 16 * s0 + 4 * ((e % Q) ^ turned(r));
                to_lds16(from(r, l < d ? l : d - 4), rows + (e - lane));
            }
        } else {
#pragma unroll 4
            for (int e = lane; e < 32 * Q * 4; e += 64) {
                const int r = e / (4 * Q), l = 16 * s0 + 4 * ((e % (4 * Q) / 4) ^ turned(r)) + (e & 3);
                to_lds4(from(r, l < d ? l : d - 1), rows + (e - lane) / 4);
            }
        }
    };
    fetch(0, 0);
    stage(0, 0);
    if (n_tiles > 1) stage(1, 1);
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        float n2 = 0.0f, e2 = 0.0f, mx = 0.0f;
        int own = d - 8 * h; // coordinate 16 s + u of this lane's half is one of the row's below this
        asm volatile("" : "+v"(own)); // (compared anew for each column tile: kept, the results are a hundred registers)
#pragma unroll
        for (int s0 = 0; s0 < NS; s0 += G) {
            // a part goes to registers, the next one is asked for, then it is converted
            __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
            float4 part[2 * G];
#pragma unroll
            for (int u = 0; u < 2 * G; ++u) part[u] = *(const float4 *)(rows + j * Q + ((4 * (u / 2) + 2 * h + u % 2) ^ turned(j)));
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xc07f); // lgkmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
            if (s0 + G < NS) fetch(c, s0 + G);
            else if (c + 1 < CT) fetch(c + 1, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int g = 0; g < G && s0 + g < NS; ++g) {
                const int s = s0 + g;
                const float v[8] = {part[2 * g].x, part[2 * g].y, part[2 * g].z, part[2 * g].w,
                                    part[2 * g + 1].x, part[2 * g + 1].y, part[2 * g + 1].z, part[2 * g + 1].w};
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const float sv = 16 * s + u < own ? v[u] * scale : 0.0f;
                    const _Float16 hv = (_Float16)fminf(fmaxf(sv, -kMaxCoord), kMaxCoord);
                    const float de = sv - (float)hv;
                    mx = fmaxf(mx, fabsf(sv));
                    n2 += sv * sv;
                    e2 += de * de;
                    b[c][s][u] = 16 * s + u >= own && 16 * s + u < own + 3 ? (_Float16)kOne : hv;
                }
            }
        }
        n2 += __shfl_xor(n2, 32, 64);
        e2 += __shfl_xor(e2, 32, 64);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        nx[c] = sqrtf(n2) * 1.0001f;
        ex[c] = sqrtf(e2) * 1.0001f;
        far_out[c] = !(mx <= kMaxCoord);
    }
    float best[CT], second[CT], third[CT], passed[CT];
    int t_best[CT], t_second[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) { best[c] = second[c] = third[c] = passed[c] = -INFINITY; t_best[c] = t_second[c] = 0; }

    // four of a tile's 16 values: their positions in the lowest bits, their largest into the three best, their second into what
    // stands for a third best that was passed over (the maximum of IEEE 754-2019 quiets no operand first)
    auto take = [&](int c, const v16f &value, int v) __attribute__((always_inline)) {
        float a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = __uint_as_float((__float_as_uint(value[v + u]) & 0xfffffff0u) | (uint32_t)(v + u));
        if constexpr (FEW) { // every value into the three best
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                third[c] = __builtin_amdgcn_fmed3f(second[c], third[c], a[u]);
                second[c] = __builtin_amdgcn_fmed3f(best[c], second[c], a[u]);
                best[c] = __builtin_elementwise_maximum(best[c], a[u]);
            }
            return;
        }
        const float m3 = __builtin_elementwise_maximum(__builtin_elementwise_maximum(a[0], a[1]), a[2]);
        const float s3 = __builtin_amdgcn_fmed3f(a[0], a[1], a[2]);
        const float m4 = __builtin_elementwise_maximum(m3, a[3]), s4 = __builtin_amdgcn_fmed3f(m3, s3, a[3]);
        passed[c] = __builtin_elementwise_maximum(passed[c], s4);
        third[c] = __builtin_amdgcn_fmed3f(second[c], third[c], m4);
        second[c] = __builtin_amdgcn_fmed3f(best[c], second[c], m4);
        best[c] = __builtin_elementwise_maximum(best[c], m4);
    };
    // (the first values taken are below every real one; an infinity with position bits would be no number)
    // one tile's products for one column tile (H), while the values before them (of column tile O and its tile t_old) are taken
    v16f acc[2], zero;
#pragma unroll
    for (int v = 0; v < 16; ++v) { zero[v] = 0.0f; acc[0][v] = acc[1][v] = -3e38f; }
    v8h a[NS];
    auto half = [&](auto which, const v8h *next, int t_old) __attribute__((always_inline)) {
        constexpr int H = decltype(which)::value, O = 1 - H, ch = CT == 2 ? H : 0, co = CT == 2 ? O : 0;
        const float b_old = best[co], s_old = second[co];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            acc[H] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[s], b[ch][s], s == 0 ? zero : acc[H], 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (q * NS / 4 == s) take(co, acc[O], 4 * q);
            asm volatile("" : "+v"(third[co]), "+v"(passed[co])); // here, not past the products that hide it
            if (CT == 1 || H == 1) a[s] = next[s * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
        }
        int t_s = second[co] == b_old ? t_best[co] : t_old;
        asm volatile("" : "+v"(t_s)); // selects, no branches
        t_second[co] = second[co] == s_old ? t_second[co] : t_s;
        t_best[co] = best[co] == b_old ? t_best[co] : t_old;
    };
    __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0): this wave's part of the first stages is in LDS
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) a[s] = tile[s * 64 + lane];
    int slot = 0;
    auto after = [](int s) { return s == 2 ? 0 : s + 1; };
    // the tile after t is there; every wave has left the one before t, whose place the one after next takes
    auto turn = [&](int t) {
        if (t + 1 < n_tiles) {
            __builtin_amdgcn_s_waitcnt(0x0f70);
            __syncthreads();
            if (t + 2 < n_tiles) stage(t + 2, after(after(slot)));
        }
        slot = after(slot);
    };
    // (operands read beyond the last tile are not used)
    if constexpr (CT == 2) {
#pragma unroll 1
        for (int t = 0; t < n_tiles; ++t) {
            half(std::integral_constant<int, 0>{}, tile, t - 1);
            turn(t);
            half(std::integral_constant<int, 1>{}, tile + slot * kStage, t);
        }
    } else { // the tiles take turns with the accumulators
#pragma unroll 1
        for (int t = 0; t < n_tiles; t += 2) {
            turn(t);
            half(std::integral_constant<int, 0>{}, tile + slot * kStage, t - 1);
            if (t + 1 < n_tiles) {
                turn(t + 1);
                half(std::integral_constant<int, 1>{}, tile + slot * kStage, t);
            }
        }
    }
    // the last values
    {
        const bool odd = CT == 1 && (n_tiles & 1);
        constexpr int c = CT - 1;
        const float b_old = best[c], s_old = second[c];
        const int t = n_tiles - 1;
#pragma unroll
        for (int v = 0; v < 16; v += 4) take(c, odd ? acc[0] : acc[1], v);
        t_second[c] = second[c] == s_old ? t_second[c] : (second[c] == b_old ? t_best[c] : t);
        t_best[c] = best[c] == b_old ? t_best[c] : t;
    }
    const NearMeta m = *meta;
    // the two lists' places are asked for once per workgroup (once per wave and column tile, the additions to one line took
    // 0.015 ms of 0.175)
    uint32_t *room = (uint32_t *)tile; // [0] pairs, [1] all of this workgroup, [2], [3] their places
    __syncthreads();
    if (tid < 2) room[tid] = 0u;
    __syncthreads();
    int kind[CT], own_b[CT], own_s[CT];
    uint32_t at[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        // center of accumulator v of half h: row 8 (v / 4) + 4 h + v % 4 of its tile
        auto id_of = [&](float v, int t) -> int {
            const int w = (int)(__float_as_uint(v) & 15u);
            return t * 32 + 8 * (w >> 2) + 4 * h + (w & 3);
        };
        float b1 = best[c], s1 = second[c], r1 = third[c];
        int ib = id_of(b1, t_best[c]), is = id_of(s1, t_second[c]);
        const float b2 = __shfl_xor(b1, 32, 64), s2 = __shfl_xor(s1, 32, 64), r2 = __shfl_xor(r1, 32, 64);
        const int ib2 = __shfl_xor(ib, 32, 64), is2 = __shfl_xor(is, 32, 64);
        // the three best of the two halves' three best
        if (b2 > b1) { // second best: b1 or s2
            r1 = b1 > s2 ? fmaxf(s1, s2) : fmaxf(b1, r2);
            const bool own = b1 > s2;
            is = own ? ib : is2;
            s1 = own ? b1 : s2;
            b1 = b2;
            ib = ib2;
        } else {
            r1 = s1 > b2 ? fmaxf(r1, b2) : fmaxf(s1, s2);
            const bool own = s1 > b2;
            is = own ? is : ib2;
            s1 = own ? s1 : b2;
        }
        const int64_t i = p0 + c * 32 + j;
        r1 = fmaxf(r1, fmaxf(passed[c], __shfl_xor(passed[c], 32, 64)));
        kind[c] = 0;
        own_b[c] = ib;
        own_s[c] = is;
        if (h != 0 || i >= n) continue;
        const float e2 = 2.0f * nearest_bound(nx[c], ex[c], NS * 16, m);
        // (equal best values: one of the two positions may be that of the other, both came from accumulators)
        if (far_out[c] || !(b1 - r1 > e2) || ib >= k || (!(b1 - s1 > e2) && (is >= k || b1 == s1))) {
            kind[c] = 2;
            at[c] = atomicAdd(&room[1], 1u);
        } else if (!(b1 - s1 > e2)) {
            kind[c] = 1;
            at[c] = atomicAdd(&room[0], 1u);
        } else {
            assign[i] = ib;
            if (cnt) pos[i] = atomicAdd(&cnt[(size_t)ib * cnt_stride], 1u);
        }
    }
    __syncthreads();
    if (tid < 2) room[2 + tid] = room[tid] ? atomicAdd(tid ? &meta->n_all : &meta->n_pairs, room[tid]) : 0u;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int i = (int)(p0 + c * 32 + j);
        if (kind[c] == 1) pairs[room[2] + at[c]] = make_int4(i, own_b[c], own_s[c], 0);
        else if (kind[c] == 2) all_list[room[3] + at[c]] = i;
    }
}

// The points the product leaves open, by fp64 squared distances. Pairs: half a wave per center. All: a workgroup per
// point, a thread per center in turn, over the centers by coordinate ([d][k]), eight of their values in flight (one
// at a time, the loads' latency made this kernel the longest of an iteration: 0.74 ms against 0.2 for the product).
constexpr int kNearMaxDim = 17 * 16 - 3;
__global__ void __launch_bounds__(256)
nearest_decide_kernel(const float *__restrict__ x, int d, const float *__restrict__ centers, const float *__restrict__ centers_t,
                      int k, const NearMeta *__restrict__ meta, const int4 *__restrict__ pairs, const int32_t *__restrict__ all_list,
                      int32_t *__restrict__ assign, uint32_t *__restrict__ cnt, int cnt_stride, uint32_t *__restrict__ pos)
{
    __shared__ double xs[kNearMaxDim];
    __shared__ double red_d[4];
    __shared__ int red_j[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t n_pairs = meta->n_pairs, n_all = meta->n_all;
    for (uint32_t e = blockIdx.x; e < n_all; e += gridDim.x) {
        const int i = all_list[e];
        for (int l = tid; l < d; l += 256) xs[l] = (double)x[(size_t)i * d + l];
        __syncthreads();
        double bestd = INFINITY;
        int best = k;
        for (int j = tid; j < k; j += 256) {
            double dd = 0.0;
            const float *col = centers_t + j;
            int l = 0;
            for (; l + 8 <= d; l += 8) {
                float c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) c[u] = col[(size_t)(l + u) * k];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const double t = xs[l + u] - (double)c[u];
                    dd += t * t;
                }
            }
            for (; l < d; ++l) {
                const double t = xs[l] - (double)col[(size_t)l * k];
                dd += t * t;
            }
            if (dd < bestd) { bestd = dd; best = j; }
        }
        for (int s = 32; s > 0; s >>= 1) {
            const double od = __shfl_xor(bestd, s, 64);
            const int oj = __shfl_xor(best, s, 64);
            if (od < bestd || (od == bestd && oj < best)) { bestd = od; best = oj; }
        }
        if (lane == 0) { red_d[wave] = bestd; red_j[wave] = best; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < 4; ++w)
                if (red_d[w] < bestd || (red_d[w] == bestd && red_j[w] < best)) { bestd = red_d[w]; best = red_j[w]; }
            if (best >= k) best = 0; // no finite distance
            assign[i] = best;
            if (cnt) pos[i] = atomicAdd(&cnt[(size_t)best * cnt_stride], 1u);
        }
        __syncthreads();
    }
    for (uint32_t e = blockIdx.x * 4 + wave; e < n_pairs; e += gridDim.x * 4) {
        const int4 p = pairs[e];
        const int j = lane < 32 ? p.y : p.z;
        const float *row = x + (size_t)p.x * d, *c = centers + (size_t)j * d;
        double dd = 0.0;
        for (int l = lane & 31; l < d; l += 32) {
            const double t = (double)row[l] - (double)c[l];
            dd += t * t;
        }
        for (int s = 16; s > 0; s >>= 1) dd += __shfl_xor(dd, s, 64);
        const double od = __shfl_xor(dd, 32, 64);
        if (lane == 0) {
            const int best = dd < od || (dd == od && p.y < p.z) ? p.y : p.z;
            assign[p.x] = best;
            if (cnt) pos[p.x] = atomicAdd(&cnt[(size_t)best * cnt_stride], 1u);
        }
    }
}

static int near_steps(int d) // matrix instructions per tile: 16 coordinates each, three of them for the bias
{
    const int need = (d + 3 + 15) / 16;
    for (int s : {2, 3, 5, 7, 9, 13, 17})
        if (need <= s) return s;
    return 0;
}

bool nearest_supported(int d, int k) { return near_steps(d) > 0 && k >= 1; }

namespace {
struct NearWs {
    v8h *packed;
    float *absmax;
    NearMeta *meta;
    int4 *pairs;
    int32_t *all_list;
};
size_t near_ws_layout(int64_t n, int d, int k, unsigned char *base, NearWs *w)
{
    size_t off = 0;
    auto take = [&](size_t bytes) -> void * {
        const size_t at = off;
        off += (bytes + 255) & ~(size_t)255;
        return base ? (void *)(base + at) : nullptr;
    };
    const int tiles = (k + 31) / 32;
    w->packed = (v8h *)take(sizeof(v8h) * (size_t)tiles * near_steps(d) * 64);
    w->absmax = (float *)take(sizeof(float) * kAbsmaxBlocks);
    w->meta = (NearMeta *)take(sizeof(NearMeta));
    w->pairs = (int4 *)take(sizeof(int4) * (size_t)n);
    w->all_list = (int32_t *)take(sizeof(int32_t) * (size_t)n);
    return off;
}
} // namespace

size_t nearest_ws_bytes(int64_t n, int d, int k, int cnt_stride)
{
    NearWs w;
    return near_ws_layout(n, d, k, nullptr, &w) + sizeof(uint32_t) * (size_t)k * cnt_stride;
}

// assign[i] = nearest center of row i (n < 2^31). cnt / pos (both or neither): cnt[j * cnt_stride] = rows of center j,
// pos[i] = place of row i among those of its center (any order); without them the last part of ws serves as cnt.
int launch_nearest(const float *x, int64_t n, int d, const float *centers, const float *centers_t, int k, void *ws,
                   int32_t *assign, uint32_t *cnt, int cnt_stride, uint32_t *pos, hipStream_t st)
{
    NearWs w;
    const int steps = near_steps(d);
    if (steps == 0 || n < 1 || n > 0x7fffffff) { set_error("nearest: dimension %d or n out of range", d); return AVQ_EINVAL; }
    const size_t at = near_ws_layout(n, d, k, (unsigned char *)ws, &w);
    uint32_t *cnt_any = cnt ? cnt : (uint32_t *)((unsigned char *)ws + at);
    const int tiles = (k + 31) / 32;
    hipLaunchKernelGGL(near_absmax_kernel, dim3(kAbsmaxBlocks), dim3(256), 0, st, centers, (int64_t)k * d, w.absmax, w.meta);
    hipLaunchKernelGGL(near_pack_kernel, dim3((unsigned)tiles), dim3(256), 0, st, centers, k, d, steps, w.absmax, w.packed, w.meta,
                       cnt_any, cnt ? cnt_stride : 1);
    // Few points or centers: the kernel's way in and out and the points left to nearest_decide_kernel count, not the products. Leaf
    // training (10 iterations) whole, us, all in turns / as FEW: 4,000 x 100 points, 64 centers 522 / 451 (466 with the kernel before that),
    // 50,000, 64 744 / 694, 256 841 / 828, 120,000, 64 757 / 733, 512 1,184 / 1,270; x 36 points: 4,000, 64 400 / 370 (362), 50,000, 128
    // 568 / 551, 256 571 / 587, 250,000, 20 562 / 547, 64 594 / 604.
    const bool few = n * tiles <= (int64_t)1 << 18;
    auto go = [&](auto kern, int points) {
        hipLaunchKernelGGL(kern, dim3((unsigned)((n + points - 1) / points)), dim3(256), 0, st, x, n, d, w.packed, tiles, k, w.meta, assign,
                           w.pairs, w.all_list, cnt, cnt_stride, pos);
    };
#define AVQ_NEAR(NS, CT)                                                    \
    do {                                                                    \
        if (few) go(nearest_mfma_kernel<NS, 1, true>, 4 * 32);              \
        else go(nearest_mfma_kernel<NS, CT, false>, 4 * CT * 32);           \
    } while (0)
    switch (steps) {
    case 2: AVQ_NEAR(2, 2); break;
    case 3: AVQ_NEAR(3, 2); break;
    case 5: AVQ_NEAR(5, 2); break;
    case 7: AVQ_NEAR(7, 2); break;
    case 9: AVQ_NEAR(9, 2); break;
    case 13: AVQ_NEAR(13, 1); break;
    default: AVQ_NEAR(17, 1); break;
    }
#undef AVQ_NEAR
    hipLaunchKernelGGL(nearest_decide_kernel, dim3(2048), dim3(256), 0, st, x, d, centers, centers_t, k, w.meta, w.pairs, w.all_list,
                       assign, cnt, cnt_stride, pos);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// ---- Lloyd's algorithm for the leaf centers ----------------------------------------------

// One workgroup: exclusive sums of the counts (cnt[j * stride]).
__global__ void __launch_bounds__(1024)
near_offsets_kernel(const uint32_t *__restrict__ cnt, int cnt_stride, int k, uint32_t *__restrict__ off)
{
    __shared__ uint32_t part[1024];
    const int tid = threadIdx.x;
    const int per = (k + 1023) / 1024, lo = tid * per, hi = lo + per < k ? lo + per : k;
    uint32_t s = 0u;
    for (int j = lo; j < hi; ++j) s += cnt[(size_t)j * cnt_stride];
    part[tid] = s;
    __syncthreads();
    for (int st = 1; st < 1024; st *= 2) {
        const uint32_t a = tid >= st ? part[tid - st] : 0u;
        __syncthreads();
        part[tid] += a;
        __syncthreads();
    }
    uint32_t o = part[tid] - s;
    for (int j = lo; j < hi; ++j) { off[j] = o; o += cnt[(size_t)j * cnt_stride]; }
    if (tid == 1023) off[k] = part[1023];
}

__global__ void __launch_bounds__(256)
near_scatter_kernel(const int32_t *__restrict__ assign, const uint32_t *__restrict__ pos, const uint32_t *__restrict__ off,
                    int64_t n, int32_t *__restrict__ order)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) order[off[assign[i]] + pos[i]] = (int32_t)i;
}

// One workgroup per center: the mean of its rows (fp64 sums: eight waves take the rows in turn, a lane two coordinates
// at a time), rounded to fp32; a center without rows stays. Also writes the center by coordinate.
__global__ void __launch_bounds__(512)
near_means_kernel(const float *__restrict__ x, int d, const int32_t *__restrict__ order, const uint32_t *__restrict__ off, int k,
                  float *__restrict__ centers, float *__restrict__ centers_t)
{
    __shared__ double red[8][128];
    const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t lo = off[j], hi = off[j + 1];
    if (hi == lo) return;
    for (int d0 = 0; d0 < d; d0 += 128) {
        const int a = d0 + lane, b = a + 64;
        double sa = 0.0, sb = 0.0;
        for (uint32_t r = lo + wave; r < hi; r += 32) { // four rows in flight
            float va[4], vb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = r + 8 * u < hi;
                const float *row = x + (size_t)order[in ? r + 8 * u : r] * d;
                va[u] = in && a < d ? row[a] : 0.0f;
                vb[u] = in && b < d ? row[b] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) { sa += (double)va[u]; sb += (double)vb[u]; }
        }
        red[wave][lane] = sa;
        red[wave][lane + 64] = sb;
        __syncthreads();
        if (tid < 128 && d0 + tid < d) {
            double s = 0.0;
            for (int w = 0; w < 8; ++w) s += red[w][tid];
            const float v = (float)(s / (double)(hi - lo));
            centers[(size_t)j * d + d0 + tid] = v;
            centers_t[(size_t)(d0 + tid) * k + j] = v;
        }
        __syncthreads();
    }
}

// the first centers: rows drawn by init_row, one per center
__global__ void __launch_bounds__(64)
near_init_kernel(const float *__restrict__ x, int64_t n, int d, int k, uint64_t seed, float *__restrict__ centers,
                 float *__restrict__ centers_t)
{
    const int j = blockIdx.x;
    const float *row = x + (size_t)init_row(seed, 0u, (uint64_t)j, (uint64_t)k, (uint64_t)n) * d;
    for (int l = threadIdx.x; l < d; l += 64) {
        const float v = row[l];
        centers[(size_t)j * d + l] = v;
        centers_t[(size_t)l * k + j] = v;
    }
}

int kmeans_leaves_device(const float *x, int64_t n, int d, int k, int iters, uint64_t seed, float *centers, float *centers_t,
                         DevBuf *ws, hipStream_t st)
{
    if (n < k) { set_error("k-means: %lld points for %d centers", (long long)n, k); return AVQ_EINVAL; }
    const int stride = spread_stride(k);
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b_near = up(nearest_ws_bytes(n, d, k, stride)), b_n = up(sizeof(int32_t) * (size_t)n),
                 b_cnt = up(sizeof(uint32_t) * (size_t)k * stride), b_off = up(sizeof(uint32_t) * ((size_t)k + 1));
    AVQ_TRY(ws->reserve(b_near + 3 * b_n + b_cnt + b_off));
    unsigned char *p = ws->as<unsigned char>();
    void *near = p;
    int32_t *assign = (int32_t *)(p += b_near);
    uint32_t *pos = (uint32_t *)(p += b_n);
    int32_t *order = (int32_t *)(p += b_n);
    uint32_t *cnt = (uint32_t *)(p += b_n);
    uint32_t *off = (uint32_t *)(p += b_cnt);
    hipLaunchKernelGGL(near_init_kernel, dim3((unsigned)k), dim3(64), 0, st, x, n, d, k, seed, centers, centers_t);
    for (int it = 0; it < iters; ++it) {
        AVQ_TRY(launch_nearest(x, n, d, centers, centers_t, k, near, assign, cnt, stride, pos, st));
        hipLaunchKernelGGL(near_offsets_kernel, dim3(1), dim3(1024), 0, st, cnt, stride, k, off);
        hipLaunchKernelGGL(near_scatter_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, assign, pos, off, n, order);
        hipLaunchKernelGGL(near_means_kernel, dim3((unsigned)k), dim3(512), 0, st, x, d, order, off, k, centers, centers_t);
    }
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

} // namespace avq
