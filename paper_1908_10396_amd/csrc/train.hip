// Dictionary learning and encoding.
//
// Dictionaries: Lloyd's algorithm under the l2 loss, per subspace (paper
// Section 4: the k-means objective; Section 5.1 learns the dictionary this way
// and then assigns codes under the anisotropic loss; Section 4.1 names it as the
// initialisation). Encoding: the partition-assignment step of Section 4.1 under
// the loss eta*||r_par||^2 + ||r_perp||^2 of Section 3.2.
//
// The results are arg-mins, and they have to agree with a plain reference
// evaluation in fp64 except at exact ties: everything is decided in fp64, but for
// the encode search, which takes what fp32 decides beyond its error bound.
#include "avq_internal.h"
#include "wave_topk.h"

namespace avq {

// ---- eta (Section 3.2, Theorem 3.4) --------------------------------------------

__host__ __device__ inline double clamp_ratio_sq(double T, double norm)
{
    const double r = T / norm;
    const double u = r * r;
    return u > 0.999 ? 0.999 : u;
}

// int_0^alpha sin^d by composite Simpson (smooth integrand, fixed fine grid).
__host__ __device__ inline double sin_power_integral(int d, double alpha)
{
    const int N = 8192;
    const double h = alpha / N;
    double s = (d == 0 ? 2.0 : pow(sin(alpha), (double)d));
    for (int i = 1; i < N; ++i) {
        const double f = d == 0 ? 1.0 : pow(sin(i * h), (double)d);
        s += (i & 1) ? 4.0 * f : 2.0 * f;
    }
    return s * h / 3.0;
}

__host__ __device__ inline double eta_of_norm(int d, double T, double norm, int mode, double eta_explicit)
{
    if (mode == AVQ_ETA_EXPLICIT) return eta_explicit;
    if (!(norm > 0.0) || d < 2) return 1.0;
    const double u = clamp_ratio_sq(T, norm);
    if (mode == AVQ_ETA_EXACT) {
        // eta = h_par / h_perp = (d-1) (I_{d-2} / I_d - 1), I_d = int_0^alpha sin^d,
        // alpha = arccos(T / ||x||)
        const double alpha = acos(sqrt(u));
        return (double)(d - 1) * (sin_power_integral(d - 2, alpha) / sin_power_integral(d, alpha) - 1.0);
    }
    // the limit of Theorem 3.4 as a proxy, floored at 1 (Theorem 3.3: h_par >= h_perp)
    const double eta = (double)(d - 1) * u / (1.0 - u);
    return eta < 1.0 ? 1.0 : eta;
}

double eta_host(int d, double T, double norm, int mode) { return eta_of_norm(d, T, norm, mode, 1.0); }

// ---- k-means ----------------------------------------------------------------------

// ---- the dictionaries of all subspaces at once --------------------------------------
//
// Lloyd's algorithm for every subspace in the same launches: an iteration is one pass of all (point, subspace)
// pairs (pq_lloyd_kernel) and one small kernel that turns the sums into codewords. The points are laid out by
// coordinate first ([d][n], residuals formed once, in fp64, where there are leaf centers), so that a wave reads
// 64 values of a coordinate side by side; from row-major points each lane would touch a line of its own.
// The kernel is bound by vector instructions. For the usual subspace sizes it takes the largest <x, c> - ||c||^2 / 2 in
// fp32, ds + 3 instructions for a codeword, where it leads the second by more than both can be off by; the others, one
// pair in tens of thousands, and all pairs of other sizes are decided by fp64 distances, 3 ds + 3 instructions each (the same
// rate, one by one). 262,144 points x 50 subspaces x 16 codewords of 2 dimensions: 46 us an iteration (67 all in fp64) and
// 5 us for the codewords; with a launch sequence per subspace, row-major points and one copy of the sums 51 + 5 + 9 us per
// subspace and iteration. Where fp32 decides little (equal codewords, points close together but far from the origin), a pair
// takes both searches (109 us): a wave that sees so leaves the fp32 search out, and marks the subspace for the iterations
// after this one. Training whole, unit vectors / copies of a row, us: 262,144 x 100, 50 subspaces of 16 codewords 1,360 / 1,350
// all in fp64, 1,000 / 2,040 without that mark, 990 / 1,350 with it; 25 of 256 codewords 14,450 / 14,430, 8,000 / 22,700, 7,990 / 14,540.

// x [n][d] -> xt [cols][n], columns col0 .. col0 + cols - 1; XT double: the residual to centers[assign[i]]
template <typename XT>
__global__ void __launch_bounds__(256)
points_by_coordinate_kernel(const float *__restrict__ x, int64_t n, int d, int col0, int cols,
                            const float *__restrict__ centers, const int32_t *__restrict__ assign, XT *__restrict__ xt)
{
    __shared__ XT tile[32][65]; // [coordinate][point]
    const int64_t i0 = (int64_t)blockIdx.x * 64;
    const int c0 = blockIdx.y * 32;
    for (int e = threadIdx.x; e < 64 * 32; e += 256) {
        const int p = e >> 5, c = e & 31;
        if (i0 + p < n && c0 + c < cols) {
            const size_t at = (size_t)(col0 + c0 + c);
            XT v = (XT)x[(size_t)(i0 + p) * d + at];
            if (centers) v -= (XT)centers[(size_t)assign[i0 + p] * d + at];
            tile[c][p] = v;
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 64 * 32; e += 256) {
        const int c = e >> 6, p = e & 63;
        if (i0 + p < n && c0 + c < cols) xt[(size_t)(c0 + c) * n + i0 + p] = tile[c][p];
    }
}

// the first codewords: the row drawn by init_row, for codeword j = blockIdx.x * 256 + threadIdx.x of subspace m0 + blockIdx.y
template <typename XT>
__global__ void __launch_bounds__(256)
pq_init_kernel(const XT *__restrict__ xt, int64_t n, int ds, int k, int m0, uint64_t seed, float *__restrict__ cb,
               double *__restrict__ cb64, uint32_t *__restrict__ hard)
{
    const int j = blockIdx.x * 256 + threadIdx.x, m = blockIdx.y;
    if (j == 0) hard[m] = 0u;
    if (j >= k) return;
    const uint64_t i = init_row(seed, (uint32_t)(1 + m0 + m), (uint64_t)j, (uint64_t)k, (uint64_t)n);
    for (int l = 0; l < ds; ++l) {
        const float v = (float)xt[(size_t)(m * ds + l) * n + i];
        cb[((size_t)m * k + j) * ds + l] = v;
        cb64[((size_t)m * k + j) * ds + l] = (double)v;
    }
}

constexpr int kLloydFp32Points = 512; // of a workgroup (two steps), from which on the fp32 search pays

// nearest codeword by fp64 distances, the lowest index on ties
template <int DS, int KC>
__device__ __forceinline__ int lloyd_nearest(const double (&xv)[DS], const double *cb, int k_rt)
{
    const int k = KC ? KC : k_rt;
    int best = 0;
    double bestd = INFINITY;
#pragma unroll 16
    for (int j = 0; j < k; ++j) {
        double t = xv[0] - cb[j * DS];
        double dd = t * t;
#pragma unroll
        for (int l = 1; l < DS; ++l) {
            t = xv[l] - cb[j * DS + l];
            dd += t * t;
        }
        best = dd < bestd ? j : best;
        bestd = fmin(dd, bestd);
    }
    return best;
}

// One subspace (blockIdx.y) and per_block points per workgroup: the nearest codeword of every point (by fp64
// squared distances, lowest index on ties), the point added to that codeword's sums in LDS, the workgroup's sums to
// part_sum[m][entry][blk] and part_cnt[m][codeword][blk]. `copies` of the sums side by side in LDS keep the lanes
// of a wave, which share a few codewords, from adding to the same word: 32 of them put a wave's additions into
// separate banks. copies = 0: the sums do not fit LDS and go to part_* (n_slots = 1, cleared before) directly.
// DS = dimensions per subspace, KC = codewords (0: known at run time only). FAST: with the fp32 search. hard[m]: set where it
// decided little.
template <int DS, int KC, bool FAST, typename XT>
__global__ void __launch_bounds__(256, FAST && KC == 16 && DS < 4 ? 8 : 1) // (eight waves a SIMD: one round of workgroups)
pq_lloyd_kernel(const XT *__restrict__ xt, int64_t n, int ds_rt, int k_rt, int per_block, const float *__restrict__ cb32,
                const double *__restrict__ cb64, uint32_t *hard, int copies, int n_slots, double *__restrict__ part_sum,
                uint32_t *__restrict__ part_cnt)
{
    extern __shared__ __align__(16) double lloyd_lds[]; // [k * ds][copies], then uint32 [k][copies] and float [260]
    const int ds = DS ? DS : ds_rt, k = KC ? KC : k_rt;
    const int m = blockIdx.y, tid = threadIdx.x;
    double *lsum = lloyd_lds;
    uint32_t *lcnt = (uint32_t *)(lloyd_lds + (size_t)k * ds * copies);
    for (int e = tid; e < k * ds * copies; e += 256) lsum[e] = 0.0;
    for (int e = tid; e < k * copies; e += 256) lcnt[e] = 0u;
    float *bias = (float *)(lcnt + k * copies), *c_max = bias + 256;
    const bool search = FAST && per_block >= kLloydFp32Points;
    if (search) { // -||c||^2 / 2 of the codewords (at most 256) and their largest norm
        double n2 = 0.0;
        if (tid < k)
            for (int l = 0; l < ds; ++l) { const double c = cb64[((size_t)m * k + tid) * ds + l]; n2 += c * c; }
        bias[tid] = (float)(-0.5 * n2);
        float cm = (float)sqrt(n2) * 1.0001f;
        for (int w = 1; w < 64; w <<= 1) cm = fmaxf(cm, __shfl_xor(cm, w, 64));
        if ((tid & 63) == 0) c_max[tid >> 6] = cm;
    }
    __syncthreads();
    const double *cb = cb64 + (size_t)m * k * ds;
    const XT *xm = xt + (size_t)m * ds * n;
    const int64_t first = (int64_t)blockIdx.x * per_block;
    const int64_t end = first + per_block < n ? first + per_block : n;
    double *gsum = part_sum + (size_t)m * k * ds * n_slots;
    uint32_t *gcnt = part_cnt + (size_t)m * k * n_slots;
    const int copy = copies > 0 ? (tid & (copies - 1)) : 0;
    const float *cf = cb32 + (size_t)m * k * ds;
    if constexpr (DS != 0) {
        auto load = [&](int64_t i, double (&xv)[DS]) __attribute__((always_inline)) {
#pragma unroll
            for (int l = 0; l < DS; ++l) xv[l] = (double)xm[(size_t)l * n + i];
        };
        auto add = [&](int best, const double (&xv)[DS]) __attribute__((always_inline)) {
            if (copies > 0) {
#pragma unroll
                for (int l = 0; l < DS; ++l)
                    __hip_atomic_fetch_add(&lsum[(best * DS + l) * copies + copy], xv[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(&lcnt[best * copies + copy], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                for (int l = 0; l < DS; ++l) unsafeAtomicAdd(&gsum[(size_t)best * DS + l], xv[l]);
                atomicAdd(&gcnt[best], 1u);
            }
        };
        if constexpr (!FAST) {
            for (int64_t i = first + tid; i < end; i += 256) {
                double xv[DS];
                load(i, xv);
                add(lloyd_nearest<DS, KC>(xv, cb, k), xv);
            }
        } else {
            bool direct = !search || hard[m] != 0u; // this wave: fp64 distances for every point
            const float cn = search ? fmaxf(fmaxf(c_max[0], c_max[1]), fmaxf(c_max[2], c_max[3])) : 0.0f;
            const float cb_half = 0.5f * cn * cn;
            float bias16[16];
            if (KC == 16 && search) {
#pragma unroll
                for (int u = 0; u < 16; ++u) bias16[u] = bias[u];
            }
            int debt = 0; // of this wave: steps with points that take fp64 distances (many: two), less those without
            for (int64_t i = first + tid; i < end; i += 256) {
                int best = 0;
                double xv[DS];
                load(i, xv);
                float xf[DS], xn = 0.0f; // xn: at least the norm
#pragma unroll
                for (int l = 0; l < DS; ++l) {
                    xf[l] = (float)xv[l];
                    xn += fabsf(xf[l]);
                }
                bool open = true; // whether it takes the fp64 distances
                if (!direct) {
                    // the two largest <x, c> - ||c||^2 / 2 in fp32, the codeword's place among 16 in the lowest bits
                    float top = -INFINITY, second = -INFINITY;
                    int block = 0;
                    for (int j0 = 0; j0 < k; j0 += 16) {
                        const float old = top;
#pragma unroll
                        for (int u = 0; u < 16; ++u) {
                            float v = KC == 16 ? bias16[u] : bias[j0 + u];
#pragma unroll
                            for (int l = 0; l < DS; ++l) v = __fmaf_rn(xf[l], cf[(j0 + u) * DS + l], v);
                            v = __uint_as_float((__float_as_uint(v) & 0xfffffff0u) | (uint32_t)u);
                            second = __builtin_amdgcn_fmed3f(top, second, v);
                            top = __builtin_elementwise_maximum(top, v);
                        }
                        block = top == old ? block : j0;
                    }
                    best = block + (int)(__float_as_uint(top) & 15u);
                    // what a value can be off by: x rounded to fp32, the bias and DS sums rounded, the place (2^-19 of it); the last
                    // two terms: products under the smallest normal number, and the rounding of the fp64 distances
                    const float mag = xn * cn + cb_half;
                    const float e = ((float)(DS + 4) * 6.0e-8f + 1.91e-6f) * 1.01f * mag + 1e-36f + 1e-14f * (xn + cn) * (xn + cn);
                    open = !(top - second > 2.0f * e); // not by more than both can be off by
                    // a wave that often has such points does the work twice: it, and the launches after this one, leave the fp32 search out
                    const int n_open = (int)__popcll(__builtin_amdgcn_ballot_w64(open));
                    debt += n_open >= 16 ? 2 : n_open > 0 ? 1 : debt > 0 ? -1 : 0;
                    if (__builtin_expect(debt >= 4, 0)) {
                        direct = true;
                        hard[m] = 1u;
                    }
                }
                if (open) best = lloyd_nearest<DS, KC>(xv, cb, k);
                add(best, xv);
            }
        }
    } else {
        for (int64_t i = first + tid; i < end; i += 256) {
            int best = 0;
            double bestd = INFINITY;
            for (int j0 = 0; j0 < k; j0 += 8) { // k is a multiple of 16
                double dd[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) dd[u] = 0.0;
                for (int l = 0; l < ds; ++l) {
                    const double v = (double)xm[(size_t)l * n + i];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double t = v - cb[(size_t)(j0 + u) * ds + l];
                        dd[u] += t * t;
                    }
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    best = dd[u] < bestd ? j0 + u : best;
                    bestd = fmin(dd[u], bestd);
                }
            }
            if (copies > 0) {
                for (int l = 0; l < ds; ++l)
                    __hip_atomic_fetch_add(&lsum[(size_t)(best * ds + l) * copies + copy], (double)xm[(size_t)l * n + i],
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(&lcnt[best * copies + copy], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                for (int l = 0; l < ds; ++l) unsafeAtomicAdd(&gsum[(size_t)best * ds + l], (double)xm[(size_t)l * n + i]);
                atomicAdd(&gcnt[best], 1u);
            }
        }
    }
    if (copies == 0) return;
    __syncthreads();
    for (int e = tid; e < k * ds; e += 256) {
        double s = 0.0;
        for (int c = 0; c < copies; ++c) s += lsum[(size_t)e * copies + ((c + e) & (copies - 1))];
        gsum[(size_t)e * n_slots + blockIdx.x] = s;
    }
    for (int j = tid; j < k; j += 256) {
        uint32_t s = 0u;
        for (int c = 0; c < copies; ++c) s += lcnt[j * copies + ((c + j) & (copies - 1))];
        gcnt[(size_t)j * n_slots + blockIdx.x] = s;
    }
}

// One wave per codeword: the workgroups' sums added up, the mean rounded to fp32 (an empty cluster keeps its codeword).
__global__ void __launch_bounds__(64)
pq_codewords_kernel(const double *__restrict__ part_sum, const uint32_t *__restrict__ part_cnt, int n_slots, int ds, int k,
                    float *__restrict__ cb, double *__restrict__ cb64)
{
    const size_t mj = (size_t)blockIdx.y * k + blockIdx.x;
    const int lane = threadIdx.x;
    uint32_t cnt = 0u;
    for (int b = lane; b < n_slots; b += 64) cnt += part_cnt[mj * n_slots + b];
    for (int s = 32; s > 0; s >>= 1) cnt += (uint32_t)__shfl_xor((int)cnt, s, 64);
    if (cnt == 0u) return;
    for (int l = 0; l < ds; ++l) {
        double sum = 0.0;
        for (int b = lane; b < n_slots; b += 64) sum += part_sum[(mj * ds + l) * n_slots + b];
        for (int s = 32; s > 0; s >>= 1) sum += __shfl_xor(sum, s, 64);
        if (lane == 0) {
            const float v = (float)(sum / (double)cnt);
            cb[mj * ds + l] = v;
            cb64[mj * ds + l] = (double)v;
        }
    }
}

template <typename XT>
static int pq_kmeans_group(const float *x, int64_t n, int d, int m0, int Mg, int ds, int k, int iters, uint64_t seed,
                           const float *centers, const int32_t *assign, float *codebooks, DevBuf *ws, hipStream_t st)
{
    // one round of workgroups (eight of 256 threads per compute unit are resident: two more would be a second round of
    // them), each with at least one step of work
    const int n_blk = (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 2048 / Mg));
    const int per_block = (int)(((n + n_blk - 1) / n_blk + 255) / 256 * 256);
    const size_t copy_bytes = (size_t)k * (ds * sizeof(double) + sizeof(uint32_t));
    int copies = 32;
    while (copies > 1 && copies * copy_bytes > 32 * 1024) copies /= 2;
    if (copy_bytes > 120 * 1024) copies = 0;
    const int n_slots = copies ? n_blk : 1;
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b_xt = up(sizeof(XT) * (size_t)n * Mg * ds), b_cb = up(sizeof(double) * (size_t)Mg * k * ds),
                 b_sum = up(sizeof(double) * (size_t)Mg * k * ds * n_slots), b_cnt = up(sizeof(uint32_t) * (size_t)Mg * k * n_slots);
    AVQ_TRY(ws->reserve(b_xt + b_cb + b_sum + b_cnt + up(sizeof(uint32_t) * (size_t)Mg)));
    XT *xt = ws->as<XT>();
    double *cb64 = (double *)(ws->as<unsigned char>() + b_xt);
    double *part_sum = (double *)((unsigned char *)cb64 + b_cb);
    uint32_t *part_cnt = (uint32_t *)((unsigned char *)part_sum + b_sum);
    uint32_t *hard = (uint32_t *)((unsigned char *)part_cnt + b_cnt); // subspaces whose points mostly take fp64 distances
    hipLaunchKernelGGL(points_by_coordinate_kernel<XT>, dim3((unsigned)((n + 63) / 64), (unsigned)((Mg * ds + 31) / 32)), dim3(256), 0,
                       st, x, n, d, m0 * ds, Mg * ds, centers, assign, xt);
    hipLaunchKernelGGL(pq_init_kernel<XT>, dim3((unsigned)((k + 255) / 256), (unsigned)Mg), dim3(256), 0, st, xt, n, ds, k, m0, seed,
                       codebooks, cb64, hard);
    const dim3 grid((unsigned)n_blk, (unsigned)Mg);
    // The fp32 search from two steps of a workgroup on (training, us, without / with it: 4,000 x 100, 50 subspaces of 16 codewords
    // 203 / 207, 10,000 254 / 260, 20,000 298 / 282; 25 of 256 codewords 5,000 870 / 1,506, 20,000 1,630 / 2,020, 40,000 2,760 /
    // 2,460). Eight dimensions: the kernel that has both is the faster one for fp64 distances too (5,000 x 256 2,070 / 1,590).
    const bool fast = per_block >= kLloydFp32Points || ds == 8;
    const size_t lds = copies * copy_bytes + (fast ? 260 * sizeof(float) : 0);
    for (int it = 0; it < iters; ++it) {
        if (copies == 0) AVQ_HIP(hipMemsetAsync(part_sum, 0, b_sum + b_cnt, st));
        auto go = [&](auto kern, LdsLimitOnce *once) -> int {
            AVQ_TRY(set_lds_limit((const void *)kern, kMaxDynLds, once));
            hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, xt, n, ds, k, per_block, codebooks, cb64, hard, copies, n_slots, part_sum,
                               part_cnt);
            return AVQ_OK;
        };
#define AVQ_LLOYD(DS, KC)                                                                                          \
    do {                                                                                                           \
        static LdsLimitOnce once[2];                                                                               \
        if (fast && DS != 0) AVQ_TRY(go(pq_lloyd_kernel<DS, KC, DS != 0, XT>, &once[1]));                          \
        else AVQ_TRY(go(pq_lloyd_kernel<DS, KC, false, XT>, &once[0]));                                            \
    } while (0)
        if (k == 16) {
            switch (ds) {
            case 1: AVQ_LLOYD(1, 16); break;
            case 2: AVQ_LLOYD(2, 16); break;
            case 3: AVQ_LLOYD(3, 16); break;
            case 4: AVQ_LLOYD(4, 16); break;
            default: AVQ_LLOYD(0, 0); break;
            }
        } else {
            switch (ds) {
            case 2: AVQ_LLOYD(2, 0); break;
            case 4: AVQ_LLOYD(4, 0); break;
            case 8: AVQ_LLOYD(8, 0); break;
            default: AVQ_LLOYD(0, 0); break;
            }
        }
#undef AVQ_LLOYD
        hipLaunchKernelGGL(pq_codewords_kernel, dim3((unsigned)k, (unsigned)Mg), dim3(64), 0, st, part_sum, part_cnt, n_slots, ds, k,
                           codebooks, cb64);
    }
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// The M dictionaries of [k][d / M] codewords (16 or 256), drawn with stream ids 1 + m.
// Groups of subspaces whose points by coordinate stay under a gigabyte of scratch.
int pq_kmeans_device(const float *x, int64_t n, int d, int M, int k, int iters, uint64_t seed, const float *resid_centers,
                     const int32_t *resid_assign, float *codebooks, DevBuf *ws, hipStream_t st)
{
    if (n < k) { set_error("k-means: %lld points for %d centers", (long long)n, k); return AVQ_EINVAL; }
    const int ds = d / M;
    const size_t per_m = (size_t)n * ds * (resid_centers ? sizeof(double) : sizeof(float));
    int group = (int)std::max<size_t>(1, std::min<size_t>((size_t)M, ((size_t)1 << 30) / per_m));
    for (int m0 = 0; m0 < M;) {
        const int Mg = std::min(group, M - m0);
        float *cb = codebooks + (size_t)m0 * k * ds;
        const int rc = resid_centers ? pq_kmeans_group<double>(x, n, d, m0, Mg, ds, k, iters, seed, resid_centers, resid_assign, cb, ws, st)
                                     : pq_kmeans_group<float>(x, n, d, m0, Mg, ds, k, iters, seed, nullptr, nullptr, cb, ws, st);
        if (rc == AVQ_ENOMEM && Mg > 1) { // nothing was launched yet: fewer subspaces at a time
            group = (Mg + 1) / 2;
            continue;
        }
        AVQ_TRY(rc);
        m0 += Mg;
    }
    return AVQ_OK;
}

// ---- nearest centers of rows beyond the matrix-core kernels (nearest.hip) ----------------
//
// One thread per point: nearest center in fp64 squared l2 (lowest index on ties); the point's values are staged in
// LDS, transposed, so the inner loop reads them conflict-free; every lane reads the same center value. ACCUM: add
// the point into sums/counts; else write the assignment. For dimensions that nearest_supported() refuses.
template <bool ACCUM>
__global__ void __launch_bounds__(256)
nearest_kernel(const float *__restrict__ x, int64_t n, int d, int k, const float *__restrict__ centers, double *__restrict__ sums,
               unsigned long long *__restrict__ counts, int32_t *__restrict__ assign)
{
    extern __shared__ float staged[]; // [d][blockDim.x]
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int bs = blockDim.x;
    if (i >= n) return; // no barriers below: a thread reads its own column only
    for (int l = 0; l < d; ++l) staged[l * bs + threadIdx.x] = x[(size_t)i * d + l];
    int best = 0;
    double bestd = INFINITY;
    for (int j = 0; j < k; ++j) {
        const float *c = centers + (size_t)j * d;
        double dd = 0.0;
        for (int l = 0; l < d; ++l) {
            const double t = (double)staged[l * bs + threadIdx.x] - (double)c[l];
            dd += t * t;
        }
        if (dd < bestd) { bestd = dd; best = j; }
    }
    if (ACCUM) {
        for (int l = 0; l < d; ++l) atomicAdd(&sums[(size_t)best * d + l], (double)staged[l * bs + threadIdx.x]);
        atomicAdd(&counts[best], 1ull);
    } else {
        assign[i] = best;
    }
}

__global__ void init_centers_kernel(const float *__restrict__ x, int64_t n, int d, int k, uint64_t seed, float *__restrict__ centers)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)k * d) return;
    centers[t] = x[(size_t)init_row(seed, 0u, (uint64_t)(t / d), (uint64_t)k, (uint64_t)n) * d + t % d];
}

__global__ void update_centers_kernel(const double *__restrict__ sums, const unsigned long long *__restrict__ counts, int k, int d,
                                      float *__restrict__ centers)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)k * d) return;
    const unsigned long long c = counts[t / d];
    if (c > 0) centers[t] = (float)(sums[t] / (double)c); // an empty cluster keeps its center
}

// workgroups of at most 64 KB of staged values where that leaves 64 threads, so that several share a compute unit
static int nearest_block_size(int d)
{
    int bs = 256;
    while (bs > 64 && (size_t)bs * d * sizeof(float) > 64 * 1024) bs /= 2;
    return bs;
}

static int nearest_stage_bytes(int d, size_t *bytes)
{
    *bytes = (size_t)nearest_block_size(d) * d * sizeof(float);
    if (*bytes > 150 * 1024) { set_error("nearest center: dimension %d too large", d); return AVQ_EINVAL; }
    return AVQ_OK;
}

int kmeans_device(const float *x, int64_t n, int d, int k, int iters, uint64_t seed, float *centers, hipStream_t st)
{
    if (n < k) { set_error("k-means: %lld points for %d centers", (long long)n, k); return AVQ_EINVAL; }
    size_t lds = 0;
    AVQ_TRY(nearest_stage_bytes(d, &lds));
    const int bs = nearest_block_size(d);
    const size_t b_sums = sizeof(double) * (size_t)k * d, b_counts = sizeof(unsigned long long) * (size_t)k;
    DevBuf ws;
    AVQ_TRY(ws.reserve(b_sums + b_counts));
    double *sums = ws.as<double>();
    unsigned long long *counts = (unsigned long long *)(ws.as<unsigned char>() + b_sums);
    const unsigned eg = (unsigned)(((int64_t)k * d + 255) / 256);
    auto body = [&]() -> int {
        static LdsLimitOnce attr_done;
        AVQ_TRY(set_lds_limit((const void *)nearest_kernel<true>, kMaxDynLds, &attr_done));
        hipLaunchKernelGGL(init_centers_kernel, dim3(eg), dim3(256), 0, st, x, n, d, k, seed, centers);
        for (int it = 0; it < iters; ++it) {
            AVQ_HIP(hipMemsetAsync(ws.p, 0, b_sums + b_counts, st));
            hipLaunchKernelGGL(nearest_kernel<true>, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), lds, st, x, n, d, k, centers, sums,
                               counts, (int32_t *)nullptr);
            hipLaunchKernelGGL(update_centers_kernel, dim3(eg), dim3(256), 0, st, sums, counts, k, d, centers);
        }
        AVQ_HIP(hipGetLastError());
        AVQ_HIP(hipStreamSynchronize(st));
        return AVQ_OK;
    };
    const int rc = body();
    ws.release();
    return rc;
}

int launch_assign_nearest(const float *x, int64_t n, int d, const float *centers, int k, int32_t *assign, hipStream_t st)
{
    size_t lds = 0;
    AVQ_TRY(nearest_stage_bytes(d, &lds));
    const int bs = nearest_block_size(d);
    static LdsLimitOnce attr_done;
    AVQ_TRY(set_lds_limit((const void *)nearest_kernel<false>, kMaxDynLds, &attr_done));
    hipLaunchKernelGGL(nearest_kernel<false>, dim3((unsigned)((n + bs - 1) / bs)), dim3(bs), lds, st, x, n, d, k, centers,
                       (double *)nullptr, (unsigned long long *)nullptr, assign);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// Definition 4.1's assignment step with the leaf centers as codewords: every point to the center of smallest
// anisotropic loss. With r = x - c: ||r||^2 = ||x||^2 - 2<c,x> + ||c||^2 and <r,x> = ||x||^2 - <c,x>, so the
// loss ||r||^2 + (eta - 1) <r,x>^2 / ||x||^2 (Section 3.2) needs <c,x> and ||c||^2 only; fp64. A workgroup
// holds 64 points in LDS; thread (point p, group g of 4) takes the centers j = g, g + 4, ...; lowest index
// on equal loss.
__global__ void __launch_bounds__(256)
assign_aniso_kernel(const float *__restrict__ x, int64_t n, int d, const float *__restrict__ centers, int k,
                    int eta_mode, double T, double eta_explicit, int32_t *__restrict__ assign)
{
    extern __shared__ double xs[]; // [64][d + 1], then best loss [4][64] and best index [4][64]
    const int ld = d + 1;
    double *best_loss = xs + (size_t)64 * ld;
    int *best_idx = (int *)(best_loss + 256);
    const int tid = threadIdx.x, p = tid & 63, g = tid >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * 64;
    for (int e = tid; e < 64 * d; e += 256) {
        const int pp = e / d, l = e - pp * d;
        xs[(size_t)pp * ld + l] = i0 + pp < n ? (double)x[(size_t)(i0 + pp) * d + l] : 0.0;
    }
    __syncthreads();
    const double *xp = xs + (size_t)p * ld;
    double nx2 = 0.0;
    for (int l = 0; l < d; ++l) nx2 += xp[l] * xp[l];
    const double eta = eta_of_norm(d, T, sqrt(nx2), eta_mode, eta_explicit);
    const double w = nx2 > 0.0 ? (eta - 1.0) / nx2 : 0.0;
    double bl = 0.0;
    int bi = -1;
    for (int j = g; j < k; j += 4) {
        const float *c = centers + (size_t)j * d;
        double cx = 0.0, cc = 0.0;
        for (int l = 0; l < d; ++l) {
            const double cv = (double)c[l];
            cx += cv * xp[l];
            cc += cv * cv;
        }
        const double rx = nx2 - cx;
        const double loss = (nx2 - 2.0 * cx + cc) + w * rx * rx;
        if (bi < 0 || loss < bl) { bl = loss; bi = j; }
    }
    best_loss[g * 64 + p] = bl;
    best_idx[g * 64 + p] = bi;
    __syncthreads();
    if (g == 0 && i0 + p < n) {
        for (int gg = 1; gg < 4; ++gg) {
            const double l2 = best_loss[gg * 64 + p];
            const int j2 = best_idx[gg * 64 + p];
            if (j2 >= 0 && (bi < 0 || l2 < bl || (l2 == bl && j2 < bi))) { bl = l2; bi = j2; }
        }
        assign[i0 + p] = bi;
    }
}

static size_t assign_aniso_lds(int d) { return sizeof(double) * ((size_t)64 * (d + 1) + 256) + sizeof(int) * 256; }

int check_assign(int d, int k, bool aniso)
{
    size_t lds = 0;
    if (aniso ? assign_aniso_lds(d) <= kMaxDynLds : nearest_supported(d, k)) return AVQ_OK;
    if (!aniso) return nearest_stage_bytes(d, &lds);
    set_error("assign: dimension %d too large", d);
    return AVQ_EINVAL;
}

int launch_assign_aniso(const float *x, int64_t n, int d, const float *centers, int k, int eta_mode, double T,
                        double eta_explicit, int32_t *assign, hipStream_t st)
{
    const size_t lds = assign_aniso_lds(d);
    AVQ_TRY(check_assign(d, k, true));
    static LdsLimitOnce attr_done;
    AVQ_TRY(set_lds_limit((const void *)assign_aniso_kernel, kMaxDynLds, &attr_done));
    hipLaunchKernelGGL(assign_aniso_kernel, dim3((unsigned)((n + 63) / 64)), dim3(256), lds, st, x, n, d, centers, k,
                       eta_mode, T, eta_explicit, assign);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// ---- encoding under the anisotropic loss ------------------------------------------

// With r = x - x~, p = <r, x>, e = ||r||^2: ||r_par||^2 = p^2/||x||^2 and ||r_perp||^2 = e - p^2/||x||^2, so the loss
// is e + w p^2, w = (eta - 1) / ||x||^2. p and e are sums over the subspaces; with the other subspaces' part P of p
// fixed, codeword j of subspace m gives e_m(j) + w (P + p_m(j))^2 up to a constant.
//
// encode_aniso_kernel (16 codewords of 1 to 4 dimensions): a lane per point. What decides a codeword is, with
// t = <c, x>, u = <c, x - center>, q = P + <x - center, x>,
//     f(j) = ||c||^2 - 2 u + w t^2 - 2 w q t,
// formed in fp32: ds + 2 operations (ds + ds + 3 with leaf centers) and two and a half to keep the best (its index in its
// low bits) and the second best. f is within eps F of its real value, F a bound of the terms' magnitudes, so a codeword that
// leads by more than 2 eps F is the arg-min; else the lane evaluates those that do not trail by as much in fp64 as above (one
// (point, subspace) in some thousands). q = p + <codeword in use, x> is kept and updated in fp64. The codes are therefore
// those of an fp64 evaluation.
//
// The points of a wave need different numbers of passes: a lane whose point is done takes the wave's next point at the
// end of the sweep over the subspaces, so that no lane waits for the slowest of 64 (4.4 sweeps on average at the Glove
// shape, eight at most). A lane asks for its point's coordinates four subspaces ahead, 32 bytes at 2 dimensions; the
// dictionaries are in LDS. On a partitioned index the points are taken leaf by leaf, and the lanes' leaf centers mostly
// are one and the same.
//
// Bound by vector operations: some 180 a step, idle lanes counted, 0.26 a clock and SIMD at 2.1 GHz by the counters; more waves a
// compute unit than twelve change nothing. avq_encode of
// 1,183,514 x 100 points, 50 subspaces, 2.18 ms with the rows of a wave's points in LDS, which left room for five waves a
// compute unit, 1.43 this way (2,000 leaves: 3.96 / 2.83); 10^6 x 128, 64 subspaces 2.97 / 1.69; 500,000 x 192, 96 of them
// 5.25 / 1.86; 200,000 x 384, 192: 12.6 / 2.5; a thread per point with every codeword in fp64: 9.3 (11.8) ms at the first.
// Windows of points handed out by a counter instead of split evenly: 2.63 -> 2.34 ms, as one SIMD of four held two waves.
struct EncodeParams {
    const float *x;
    int64_t n, n_slots;
    const int32_t *order; // slot -> point (-1: none), NULL: slot i is point i
    int32_t d, M, NB, passes;
    const float *codebooks;   // [M][codewords][dimensions]
    const float *leaf_centers;
    const int32_t *leaf_assign;
    int32_t eta_mode;
    double T, eta_explicit;
    const double *w_in;       // NULL: w from eta_mode here
    uint8_t *packed;
    uint32_t *distinct;       // 16 codewords: per dictionary a bit for each that equals none before it
    uint32_t *next_window;    // windows of slots, one a lane, are handed out: waves that share a SIMD get fewer
    int32_t top_up;           // leaves, and more windows than waves: lanes without a point take the next window's while others are at work
    int32_t code_stride;      // bytes (odd dwords)
};

__global__ void __launch_bounds__(64)
encode_tables_kernel(const float *__restrict__ codebooks, int ds, float *__restrict__ tab, float2 *__restrict__ lim,
                     uint32_t *__restrict__ distinct, uint32_t *__restrict__ next_window)
{
    const int m = blockIdx.x, lane = threadIdx.x;
    if (m == 0 && lane == 0) *next_window = 0u;
    float cm = 0.0f, ccm = 0.0f;
    uint32_t alike = lane < 16 ? (1u << lane) - 1u : ~0u; // of the codewords before this lane's, those that equal it
    if (lane < 16) {
        const float *c = codebooks + ((size_t)m * 16 + lane) * ds;
        float *o = tab + ((size_t)m * 16 + lane) * (ds + 1);
        double cc = 0.0;
        for (int l = 0; l < ds; ++l) {
            o[l] = c[l];
            uint32_t same = 0u;
            for (int j = 0; j < 16; ++j) same |= (c[l] == __shfl(c[l], j, 64) ? 1u : 0u) << j;
            alike &= same;
            cc += (double)c[l] * (double)c[l];
            cm = fmaxf(cm, fabsf(c[l]));
        }
        o[ds] = (float)cc;
        ccm = (float)cc;
    }
    const uint64_t first = __builtin_amdgcn_ballot_w64(alike == 0u);
    for (int s = 32; s > 0; s >>= 1) { cm = fmaxf(cm, __shfl_xor(cm, s, 64)); ccm = fmaxf(ccm, __shfl_xor(ccm, s, 64)); }
    if (lane == 0) {
        lim[m] = make_float2(cm * 1.0001f, ccm * 1.0001f);
        distinct[m] = (uint32_t)first;
    }
}

// The same for 256 codewords (encode_wide_kernel): operands [m][(32 codewords g, two dimensions s) / 4][64][4], the lane's
// word of (g, s) being coordinate 2 s + lane / 32 of codeword 32 g + lane % 32; cc [m][256].
__global__ void __launch_bounds__(256)
encode_operands_kernel(const float *__restrict__ codebooks, int ds, float *__restrict__ operands, float *__restrict__ cc_out,
                       float2 *__restrict__ lim, uint32_t *__restrict__ next_window)
{
    __shared__ float wave_cm[4], wave_ccm[4];
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    if (m == 0 && tid == 0) *next_window = 0u;
    const float *c = codebooks + ((size_t)m * 256 + tid) * ds;
    float cm = 0.0f;
    double cc = 0.0;
    for (int l = 0; l < ds; ++l) {
        const float v = c[l];
        const int at = (tid >> 5) * (ds / 2) + (l >> 1);
        operands[((size_t)m * ds + at / 4) * 256 + ((l & 1) * 32 + (tid & 31)) * 4 + at % 4] = v;
        cc += (double)v * (double)v;
        cm = fmaxf(cm, fabsf(v));
    }
    cc_out[m * 256 + tid] = (float)cc;
    float ccm = (float)cc;
    for (int s = 32; s > 0; s >>= 1) { cm = fmaxf(cm, __shfl_xor(cm, s, 64)); ccm = fmaxf(ccm, __shfl_xor(ccm, s, 64)); }
    if (lane == 0) { wave_cm[tid >> 6] = cm; wave_ccm[tid >> 6] = ccm; }
    __syncthreads();
    if (tid == 0) {
        for (int v = 1; v < 4; ++v) { cm = fmaxf(cm, wave_cm[v]); ccm = fmaxf(ccm, wave_ccm[v]); }
        lim[m] = make_float2(cm * 1.0001f, ccm * 1.0001f);
    }
}

// (eta - 1) / ||x||^2 of every point, for the mode whose eta is an integral per point
__global__ void __launch_bounds__(256)
encode_weights_kernel(const float *__restrict__ x, int64_t n, int d, int eta_mode, double T, double eta_explicit, double *__restrict__ w)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float *xi = x + (size_t)i * d;
    double nx2 = 0.0;
    for (int l = 0; l < d; ++l) nx2 += (double)xi[l] * (double)xi[l];
    const double eta = eta_of_norm(d, T, sqrt(nx2), eta_mode, eta_explicit);
    w[i] = nx2 > 0.0 ? (eta - 1.0) / nx2 : 0.0;
}

// (eta - 1) / ||x||^2 of a point
__device__ __forceinline__ double encode_weight(const EncodeParams &p, int id, double nx2)
{
    if (p.w_in) return p.w_in[id];
    double eta = p.eta_explicit;
    if (p.eta_mode != AVQ_ETA_EXPLICIT) { // the limit of Theorem 3.4, floored at 1 (see eta_of_norm)
        eta = 1.0;
        if (nx2 > 0.0) {
            const double u = clamp_ratio_sq(p.T, sqrt(nx2));
            eta = fmax((double)(p.d - 1) * u / (1.0 - u), 1.0);
        }
    }
    return nx2 > 0.0 ? (eta - 1.0) / nx2 : 0.0;
}

// floats at a float's alignment; one load of several words takes that on this machine
template <int N>
__device__ __forceinline__ void load_floats(const float *__restrict__ at, float (&v)[N])
{
    __builtin_memcpy(v, at, sizeof(v));
}

template <int DS, bool RES>
__global__ void __launch_bounds__(512, 4)
encode_aniso_kernel(const EncodeParams p, const float *__restrict__ tables, const float2 *__restrict__ limits)
{
    constexpr int KC = 16, kAhead = RES && DS > 2 ? 2 : 4; // subspaces whose coordinates are asked for while the ones before are at work
    extern __shared__ __align__(16) float enc_lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = p.M, d = p.d;
    float *tab_lds = enc_lds; // [M][KC][DS + 1]
    float2 *lim_lds = (float2 *)(enc_lds + M * KC * (DS + 1)); // [M]
    uint8_t *codes = (uint8_t *)(enc_lds + M * (KC * (DS + 1) + 2)) + (size_t)wave * 64 * p.code_stride;
    uint8_t *my_codes = codes + (size_t)lane * p.code_stride;
    for (int e = threadIdx.x; e < M * KC * (DS + 1); e += blockDim.x) tab_lds[e] = tables[e];
    for (int e = threadIdx.x; e < M; e += blockDim.x) lim_lds[e] = limits[e];
    __syncthreads();
    for (int e = 0; e < p.code_stride; e += 4) *(uint32_t *)(my_codes + e) = 0u;

    int win_id = -1, win_left = 0;  // the window's points not yet taken: those of lanes 0 .. win_left - 1
    bool first = true, drained = false; // drained: no windows left
    int id = -1, stage = 0;         // this lane's point (-1: none) and pass (-1: nearest codewords first)
    double P = 0.0, w = 0.0; // P = <x - center - codewords, x>, the codewords chosen so far
    const float *xi = p.x, *ce_row = RES ? p.leaf_centers : nullptr;
    bool changed = false;
    constexpr float kEps = (1.9074e-6f + (2 * DS + 8 + (RES ? 4 : 0)) * 6.0e-8f) * 1.05f;

    auto lanes_below = [](u64 mask) -> int { return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u)); };
    for (;;) {
        // lanes without a point take the wave's next ones
        u64 need = __builtin_amdgcn_ballot_w64(id < 0);
        bool taken = false;
        while (need != 0ull) {
            if (win_left == 0) {
                if (drained || (RES && !p.top_up && __builtin_amdgcn_ballot_w64(id >= 0) != 0ull)) break;
                uint32_t w64 = blockIdx.x * (blockDim.x >> 6) + wave; // the first window; the others by the counter
                if (!first) {
                    if (lane == 0) w64 = gridDim.x * (blockDim.x >> 6) + atomicAdd(p.next_window, 1u);
                    w64 = __builtin_amdgcn_readfirstlane(w64);
                }
                first = false;
                const int64_t s0 = (int64_t)w64 * 64, s = s0 + lane;
                if (s0 >= p.n_slots) { drained = true; break; }
                const int slot = s < p.n_slots ? (p.order ? p.order[s] : (int)s) : -1;
                const u64 there = __builtin_amdgcn_ballot_w64(slot >= 0);
                win_left = (int)__popcll(there);
                // the points move to lanes 0 .. win_left - 1
                const int to = slot >= 0 ? lanes_below(there) : win_left + lanes_below(~there);
                win_id = __builtin_amdgcn_ds_permute(to << 2, slot);
                continue;
            }
            const int rank = lanes_below(need), n_need = (int)__popcll(need);
            const int who = __builtin_amdgcn_ds_bpermute((win_left - 1 - rank) << 2, win_id);
            if (id < 0 && rank < win_left) { id = who; taken = true; }
            win_left = win_left > n_need ? win_left - n_need : 0;
            need = __builtin_amdgcn_ballot_w64(id < 0);
        }
        if (__builtin_amdgcn_ballot_w64(id >= 0) == 0ull) break;
        if (taken) {
            stage = -1;
            xi = p.x + (size_t)id * d;
            if constexpr (RES) ce_row = p.leaf_centers + (size_t)p.leaf_assign[id] * d;
            double nx2 = 0.0, cx = 0.0;
            auto term = [&](float xl, float cl) {
                const double v = (double)xl;
                nx2 += v * v;
                if constexpr (RES) cx = fma((double)cl, v, cx);
            };
            int l = 0;
            constexpr int kSome = RES ? 16 : 32;
            for (; l + kSome <= d; l += kSome) {
                float v[kSome], c[RES ? kSome : 1];
                load_floats(xi + l, v);
                if constexpr (RES) load_floats(ce_row + l, c);
#pragma unroll
                for (int e = 0; e < kSome; ++e) term(v[e], c[RES ? e : 0]);
            }
            for (; l + 4 <= d; l += 4) {
                float v[4], c[RES ? 4 : 1];
                load_floats(xi + l, v);
                if constexpr (RES) load_floats(ce_row + l, c);
#pragma unroll
                for (int e = 0; e < 4; ++e) term(v[e], c[RES ? e : 0]);
            }
            for (; l < d; ++l) term(xi[l], RES ? ce_row[l] : 0.0f);
            P = nx2 - cx;
            w = encode_weight(p, id, nx2);
        }
        const bool active = id >= 0;
        const bool init = stage < 0;
        const double wl = init ? 0.0 : w, w2 = 2.0 * wl;
        const float wf = (float)wl;
        changed = false;

        auto load_codeword = [&](int m, int j, float (&c)[DS]) {
            typedef const __attribute__((address_space(3))) float lds_float;
            lds_float *src = (lds_float *)(tab_lds + (m * KC + j) * (DS + 1));
#pragma unroll
            for (int l = 0; l < DS; ++l) c[l] = src[l];
        };
        // this point's (and its center's) coordinates of subspaces m .. m + kAhead - 1; nothing beyond the row
        auto load_rows = [&](int m, float (&xs)[kAhead * DS], float (&ces)[RES ? kAhead * DS : 1]) {
            const int l0 = m * DS;
            if (l0 + kAhead * DS <= d) {
                load_floats(xi + l0, xs);
                if constexpr (RES) load_floats(ce_row + l0, ces);
            } else {
#pragma unroll
                for (int l = 0; l < kAhead * DS; ++l) {
                    xs[l] = l0 + l < d ? xi[l0 + l] : 0.0f;
                    if constexpr (RES) ces[l] = l0 + l < d ? ce_row[l0 + l] : 0.0f;
                }
            }
        };
        // One subspace: xv, ce its coordinates, cur the codeword in use, `code` its index.
        auto step = [&](int m, const float (&xv)[DS], const float (&ce)[RES ? DS : 1], const float (&cur)[DS], int code) {
            // q = (p of the other subspaces) + <x - center, x> of this one = P + <codeword in use, x>
            double t_cur = 0.0;
            float sx = 0.0f, sr = 0.0f, xrf[RES ? DS : 1];
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                t_cur = fma((double)cur[l], (double)xv[l], t_cur);
                sx += fabsf(xv[l]);
                if constexpr (RES) { xrf[l] = (float)((double)xv[l] - (double)ce[l]); sr += fabsf(xrf[l]); }
            }
            if (init) t_cur = 0.0;
            const double q = P + t_cur;
            const float Bf = (float)fma(w2, q, RES ? 0.0 : 2.0);
            const float2 lim = lim_lds[m];
            const float T = lim.x * sx;
            float F = fmaf(T, fmaf(wf, T, fabsf(Bf)), lim.y);
            if constexpr (RES) F = fmaf(2.0f * lim.x, sr, F);
            const float lead = fmaf(F, 2.0f * kEps, 2.0e-37f);

            // a half of the codewords at a time: more need more than the 128 registers of four waves a SIMD (as it is, 30 and, with
            // leaf centers, 40 are spilled at 4 dimensions, 7 and 4 with leaf centers at 3 and 2)
            constexpr int kPart = 8, kPart4 = kPart * (DS + 1) / 4;
            typedef float four_floats __attribute__((ext_vector_type(4)));
            typedef const __attribute__((address_space(3))) four_floats lds_float4;
            four_floats part[kPart4];
            auto load_part = [&](int j0) { // of the codewords j0 .. j0 + kPart - 1
                lds_float4 *src = (lds_float4 *)(tab_lds + (m * KC + j0) * (DS + 1));
                asm volatile("" : "+v"(src));
#pragma unroll
                for (int e = 0; e < kPart4; ++e) part[e] = src[e];
            };
            float best = INFINITY, second = INFINITY;
            auto entry = [&](int j, int l) -> float { // coordinate l of codeword j of the part (a constant), l = DS: ||c||^2
                const int at = (j % kPart) * (DS + 1) + l;
                return part[at / 4][at % 4];
            };
            auto value = [&](int v) -> float { // f of codeword v of the part, its index in the low bits
                auto c = [&](int l) -> float { return entry(v, l); };
                float t = xv[0] * c(0);
#pragma unroll
                for (int l = 1; l < DS; ++l) t = fmaf(xv[l], c(l), t);
                float f = c(DS);
                if constexpr (RES) {
                    float u = xrf[0] * c(0);
#pragma unroll
                    for (int l = 1; l < DS; ++l) u = fmaf(xrf[l], c(l), u);
                    f = fmaf(-2.0f, u, f);
                }
                f = fmaf(t, fmaf(wf, t, -Bf), f);
                return __uint_as_float((__float_as_uint(f) & 0xfffffff0u) | (uint32_t)v);
            };
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                if (v % kPart == 0) load_part(v);
                const float f0 = value(v), f1 = value(v + 1);
                // Two at a time: the second smallest of (best, f0, f1) is their median. (Instructions by name: as fminf,
                // each would be preceded by one that quiets its operands; a NaN is dropped either way.)
                const float mid = __builtin_amdgcn_fmed3f(best, f0, f1);
                asm("v_min_f32 %0, %1, %2" : "=v"(second) : "v"(second), "v"(mid));
                asm("v_min3_f32 %0, %1, %2, %3" : "=v"(best) : "v"(best), "v"(f0), "v"(f1));
            }
            int pick = (int)(__float_as_uint(best) & 15u);
            const bool open = active && !(second - best > lead);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(open) != 0ull, 0)) {
                if (open) {
                    // Equal codewords leave this open at every step: those that f does not rule out are found once more, without
                    // those that equal an earlier one, and up to four taken one by one. (200,000 x 100 points, 50 dictionaries, three
                    // passes: 253 us; of 8 pairs of equal codewords 474 with both of a pair evaluated and 443 with one, five
                    // alike 792 and 423, all sixteen alike 440 and 255.)
                    double bestv = INFINITY, xr[DS], xx = 0.0;
                    uint32_t left = 0u;
#pragma unroll
                    for (int v = 0; v < KC; ++v) {
                        if (v % kPart == 0) load_part(v);
                        left |= value(v) - best > lead ? 0u : 1u << v;
                    }
                    left &= p.distinct[m];
                    pick = 0;
#pragma unroll
                    for (int l = 0; l < DS; ++l) {
                        xr[l] = (double)xv[l] - (RES ? (double)ce[RES ? l : 0] : 0.0);
                        xx = fma(xr[l], (double)xv[l], xx);
                    }
                    auto try_codeword = [&](int j, auto coordinate) {
                        double pm = 0.0, em = 0.0;
#pragma unroll
                        for (int l = 0; l < DS; ++l) {
                            const double r = xr[l] - (double)coordinate(l);
                            pm = fma(r, (double)xv[l], pm);
                            em = fma(r, r, em);
                        }
                        const double pp = init ? 0.0 : (q - xx) + pm;
                        const double v = em + wl * pp * pp;
                        if (v < bestv) { bestv = v; pick = j; }
                    };
                    if (__builtin_amdgcn_ballot_w64(__popc(left) > 4) != 0ull) {
#pragma unroll
                        for (int j = 0; j < KC; ++j) {
                            if (j % kPart == 0) load_part(j);
                            try_codeword(j, [&](int l) { return entry(j, l); });
                        }
                    } else {
                        while (left != 0u) {
                            const int j = __builtin_ctz(left);
                            left &= left - 1u;
                            float c[DS];
                            load_codeword(m, j, c);
                            try_codeword(j, [&](int l) { return c[l]; });
                        }
                    }
                }
            }
            const bool other = active && (init || pick != code);
            if (__builtin_amdgcn_ballot_w64(other) != 0ull) {
                if (other) {
                    float c[DS];
                    load_codeword(m, pick, c);
                    double t_new = 0.0;
#pragma unroll
                    for (int l = 0; l < DS; ++l) t_new = fma((double)c[l], (double)xv[l], t_new);
                    my_codes[m] = (uint8_t)pick;
                    P = q - t_new;
                    changed = true;
                }
            }
        };
        // One sweep over the subspaces.
        float xs[kAhead * DS], ces[RES ? kAhead * DS : 1];
        load_rows(0, xs, ces);
#pragma unroll 1
        for (int m = 0; m < M; m += kAhead) {
            float xn[kAhead * DS], cen[RES ? kAhead * DS : 1], cur[kAhead][DS];
            const uint32_t four = *(const uint32_t *)(my_codes + (m & ~3)); // codes of a row start at a word, and end in one
            int code[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                code[u] = (int)(four >> (8 * ((m + u) & 3))) & 255;
                if (m + u < M) load_codeword(m + u, code[u], cur[u]);
            }
            load_rows(m + kAhead < M ? m + kAhead : 0, xn, cen);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (m + u >= M) break;
                float xv[DS], ce[RES ? DS : 1];
#pragma unroll
                for (int l = 0; l < DS; ++l) {
                    xv[l] = xs[u * DS + l];
                    if constexpr (RES) ce[l] = ces[u * DS + l];
                }
                step(m + u, xv, ce, cur[u], code[u]);
            }
#pragma unroll
            for (int l = 0; l < kAhead * DS; ++l) {
                xs[l] = xn[l];
                if constexpr (RES) ces[l] = cen[l];
            }
        }
        const bool done = active && (init ? p.passes == 0 : !changed || stage + 1 >= p.passes);
        stage = init ? 0 : stage + 1;
        if (done) {
            uint8_t *out = p.packed + (size_t)id * p.NB;
            for (int e = 0; e < p.code_stride && e / 2 < p.NB; e += 4) {
                const uint32_t v = *(const uint32_t *)(my_codes + e);
                out[e / 2] = (uint8_t)((v & 15u) | ((v >> 4) & 0xf0u));
                if (e / 2 + 1 < p.NB) out[e / 2 + 1] = (uint8_t)(((v >> 16) & 15u) | ((v >> 20) & 0xf0u));
            }
            id = -1;
        }
    }
}

// 256 codewords of 2, 4 or 8 dimensions, as above: a wave takes 32 points, lanes j and j + 32 the same one. <c, x> for 32
// codewords at a time comes from the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: two dimensions of 32 codewords against
// 32 points), which leaves a lane 16 of them; with leaf centers a second product has the terms linear in c, <c, y>, y = 2 (x -
// center) + 2 w q x. The operands are asked for a subspace ahead, in the order the instruction takes them; ||c||^2 is in LDS
// where it fits. Bound by the vector operations on the products (72 for 16 of a lane's) beside the matrix instruction.
// A lane per point with the codewords as scalar operands waited for each sixteen of them, as the scalar cache does not hold
// the dictionaries, and left a small call's few waves alone with 1,800 operations a step. avq_encode, that way / this way:
// 100,000 x 100, 25 subspaces 4.25 / 1.28 ms; 21,382 of them 2.73 / 0.60; 40,000 x 256, 32 subspaces 2.56 / 0.83, with 200
// leaves 4.44 / 1.70; 300,000 x 36, 9 subspaces 1.35 / 0.62; 2,000 of them 0.53 / 0.13.
typedef float v16f __attribute__((ext_vector_type(16)));
template <int DS, bool RES, bool CC_LDS>
__global__ void __launch_bounds__(512, 2)
encode_wide_kernel(const EncodeParams p, const float *__restrict__ operands, const float *__restrict__ cc_all,
                   const float2 *__restrict__ limits)
{
    constexpr int KC = 256, G = 8, S = DS / 2; // groups of 32 codewords, steps of two dimensions
    extern __shared__ __align__(16) float enc_lds[];
    const int lane = threadIdx.x & 63, j = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = p.M, d = p.d;
    typedef float four_floats __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(3))) four_floats lds_float4;
    float *cc_lds = enc_lds; // [M][256]
    uint8_t *my_codes = (uint8_t *)(enc_lds + (CC_LDS ? M * KC : 0)) + (size_t)(wave * 32 + j) * p.code_stride;
    if (CC_LDS) {
        for (int e = threadIdx.x; e < M * KC; e += blockDim.x) cc_lds[e] = cc_all[e];
        __syncthreads();
    }
    if (h == 0)
        for (int e = 0; e < p.code_stride; e += 4) *(uint32_t *)(my_codes + e) = 0u;

    int win_id = -1, win_left = 0;  // the window's points not yet taken: those of lanes 0 .. win_left - 1 of either half
    bool first = true, drained = false; // drained: no windows left
    int id = -1, stage = 0;
    double P = 0.0, w = 0.0;
    const float *xi = p.x, *ce_row = RES ? p.leaf_centers : nullptr;
    // the error of f, in units of F: that of the instructions, and of the index in the low bits
    constexpr float kEps = (1.9074e-6f + (2 * DS + 8 + (RES ? 6 : 0)) * 6.0e-8f) * 1.05f;
    auto below = [&](uint32_t mask) -> int { return (int)__popc(mask & ((1u << j) - 1u)); };

    for (;;) {
        // points for those who have none (both halves alike)
        uint32_t need = (uint32_t)__builtin_amdgcn_ballot_w64(id < 0);
        bool taken = false;
        while (need != 0u) {
            if (win_left == 0) {
                if (drained || (RES && !p.top_up && __builtin_amdgcn_ballot_w64(id >= 0) != 0ull)) break;
                uint32_t w32 = blockIdx.x * (blockDim.x >> 6) + wave; // the first window; the others by the counter
                if (!first) {
                    if (lane == 0) w32 = gridDim.x * (blockDim.x >> 6) + atomicAdd(p.next_window, 1u);
                    w32 = __builtin_amdgcn_readfirstlane(w32);
                }
                first = false;
                const int64_t s0 = (int64_t)w32 * 32, s = s0 + j;
                if (s0 >= p.n_slots) { drained = true; break; }
                const int slot = s < p.n_slots ? (p.order ? p.order[s] : (int)s) : -1;
                const uint32_t there = (uint32_t)__builtin_amdgcn_ballot_w64(slot >= 0);
                win_left = (int)__popc(there);
                const int to = slot >= 0 ? below(there) : win_left + below(~there); // the points move to the front
                win_id = __builtin_amdgcn_ds_permute((to + 32 * h) << 2, slot);
                continue;
            }
            const int rank = below(need), n_need = (int)__popc(need);
            const int who = __builtin_amdgcn_ds_bpermute(((win_left - 1 - rank) & 31) << 2, win_id);
            if (id < 0 && rank < win_left) { id = who; taken = true; }
            win_left = win_left > n_need ? win_left - n_need : 0;
            need = (uint32_t)__builtin_amdgcn_ballot_w64(id < 0);
        }
        if (__builtin_amdgcn_ballot_w64(id >= 0) == 0ull) break;
        if (taken) {
            stage = -1;
            xi = p.x + (size_t)id * d;
            if constexpr (RES) ce_row = p.leaf_centers + (size_t)p.leaf_assign[id] * d;
            double nx2 = 0.0, cx = 0.0;
            auto term = [&](float xl, float cl) {
                const double v = (double)xl;
                nx2 += v * v;
                if constexpr (RES) cx = fma((double)cl, v, cx);
            };
            constexpr int kSome = 16;
            int l = 0;
            for (; l + kSome <= d; l += kSome) {
                float v[kSome], c[RES ? kSome : 1];
                load_floats(xi + l, v);
                if constexpr (RES) load_floats(ce_row + l, c);
#pragma unroll
                for (int e = 0; e < kSome; ++e) term(v[e], c[RES ? e : 0]);
            }
            for (; l < d; ++l) term(xi[l], RES ? ce_row[l] : 0.0f);
            P = nx2 - cx;
            w = encode_weight(p, id, nx2);
        }
        const bool active = id >= 0;
        const bool init = stage < 0;
        const double wl = init ? 0.0 : w, w2 = 2.0 * wl;
        const float wf = (float)wl;
        bool changed = false;

        struct Step { // what a step needs and does not depend on the steps before it
            float xv[DS], ce[RES ? DS : 1], cur[DS];
            float a[G * S];
            float2 lim;
            int code;
        };
        auto load_step = [&](int m, Step &s) {
            s.code = my_codes[m];
            load_floats(xi + m * DS, s.xv);
            if constexpr (RES) load_floats(ce_row + m * DS, s.ce);
            s.lim = limits[m];
            // [m][G * S / 4][64][4]
#pragma unroll
            for (int e = 0; e < G * S / 4; ++e) {
                const four_floats v = *(const four_floats *)(operands + (((size_t)m * (G * S / 4) + e) * 64 + lane) * 4);
#pragma unroll
                for (int i = 0; i < 4; ++i) s.a[e * 4 + i] = v[i];
            }
            load_floats(p.codebooks + ((size_t)m * KC + s.code) * DS, s.cur);
        };
        Step now;
        load_step(0, now);
#pragma unroll 1
        for (int m = 0; m < M; ++m) {
            Step next;
            load_step(m + 1 < M ? m + 1 : 0, next);
            // q = (p of the other subspaces) + <x - center, x> of this one = P + <codeword in use, x>
            double t_cur = 0.0;
            float sx = 0.0f, sr = 0.0f, xrf[RES ? DS : 1];
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                t_cur = fma((double)now.cur[l], (double)now.xv[l], t_cur);
                sx += fabsf(now.xv[l]);
                if constexpr (RES) { xrf[l] = (float)((double)now.xv[l] - (double)now.ce[l]); sr += fabsf(xrf[l]); }
            }
            if (init) t_cur = 0.0;
            const double q = P + t_cur;
            const float Bf = (float)fma(w2, q, RES ? 0.0 : 2.0);
            const float T = now.lim.x * sx;
            float F = fmaf(T, fmaf(wf, T, fabsf(Bf)), now.lim.y);
            if constexpr (RES) F = fmaf(2.0f * now.lim.x, sr, F);
            // (the instruction may drop products below 2^-126)
            const float lead = fmaf(F, 2.0f * kEps, fmaf(2.0f * DS * 2.4e-38f, fmaf(wf, T, fabsf(Bf)), 2.0e-37f));

            float b[S], y[RES ? S : 1];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                b[s] = h ? now.xv[2 * s + 1] : now.xv[2 * s];
                if constexpr (RES) y[s] = fmaf(Bf, b[s], 2.0f * (h ? xrf[2 * s + 1] : xrf[2 * s]));
            }
            float best = INFINITY, second = INFINITY;
            int group = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                v16f t, u, zero;
#pragma unroll
                for (int v = 0; v < 16; ++v) zero[v] = 0.0f;
                t = __builtin_amdgcn_mfma_f32_32x32x2f32(now.a[g * S], b[0], zero, 0, 0, 0);
#pragma unroll
                for (int s = 1; s < S; ++s) t = __builtin_amdgcn_mfma_f32_32x32x2f32(now.a[g * S + s], b[s], t, 0, 0, 0);
                if constexpr (RES) {
                    u = __builtin_amdgcn_mfma_f32_32x32x2f32(now.a[g * S], y[0], zero, 0, 0, 0);
#pragma unroll
                    for (int s = 1; s < S; ++s) u = __builtin_amdgcn_mfma_f32_32x32x2f32(now.a[g * S + s], y[s], u, 0, 0, 0);
                }
                const float old = best;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    four_floats cc;
                    if constexpr (CC_LDS) cc = *(lds_float4 *)(cc_lds + m * KC + g * 32 + 8 * r + 4 * h);
                    else cc = *(const four_floats *)(cc_all + (size_t)m * KC + g * 32 + 8 * r + 4 * h);
                    float f[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float tv = t[4 * r + e];
                        if constexpr (RES) f[e] = fmaf(wf * tv, tv, cc[e]) - u[4 * r + e];
                        else f[e] = fmaf(tv, fmaf(wf, tv, -Bf), cc[e]);
                        f[e] = __uint_as_float((__float_as_uint(f[e]) & 0xfffffff0u) | (uint32_t)(4 * r + e));
                    }
#pragma unroll
                    for (int e = 0; e < 4; e += 2) { // as in encode_aniso_kernel
                        const float mid = __builtin_amdgcn_fmed3f(best, f[e], f[e + 1]);
                        asm("v_min_f32 %0, %1, %2" : "=v"(second) : "v"(second), "v"(mid));
                        asm("v_min3_f32 %0, %1, %2, %3" : "=v"(best) : "v"(best), "v"(f[e]), "v"(f[e + 1]));
                    }
                }
                group = best == old ? group : g;
            }
            const int v = (int)(__float_as_uint(best) & 15u);
            int pick = group * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
            { // the other half's codewords
                const float ob = __shfl_xor(best, 32, 64), os = __shfl_xor(second, 32, 64);
                const int op = __shfl_xor(pick, 32, 64);
                second = fminf(fmaxf(best, ob), fminf(second, os));
                pick = ob < best ? op : pick;
                best = fminf(best, ob);
            }
            const bool open = active && !(second - best > lead);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(open) != 0ull, 0)) {
                if (open) { // in fp64, each half of the codewords by one of the point's lanes
                    double bestv = INFINITY, xr[DS], xx = 0.0;
                    pick = 128 * h;
#pragma unroll
                    for (int l = 0; l < DS; ++l) {
                        xr[l] = (double)now.xv[l] - (RES ? (double)now.ce[RES ? l : 0] : 0.0);
                        xx = fma(xr[l], (double)now.xv[l], xx);
                    }
                    const float *cb = p.codebooks + ((size_t)m * KC + 128 * h) * DS;
#pragma unroll 4
                    for (int c = 0; c < 128; ++c) {
                        float cv[DS];
                        load_floats(cb + c * DS, cv);
                        double pm = 0.0, em = 0.0;
#pragma unroll
                        for (int l = 0; l < DS; ++l) {
                            const double r = xr[l] - (double)cv[l];
                            pm = fma(r, (double)now.xv[l], pm);
                            em = fma(r, r, em);
                        }
                        const double pp = init ? 0.0 : (q - xx) + pm;
                        const double val = em + wl * pp * pp;
                        if (val < bestv) { bestv = val; pick = 128 * h + c; }
                    }
                    const double ov = __shfl_xor(bestv, 32, 64);
                    const int op = __shfl_xor(pick, 32, 64);
                    if (ov < bestv || (ov == bestv && op < pick)) pick = op;
                }
            }
            const bool other = active && (init || pick != now.code);
            if (__builtin_amdgcn_ballot_w64(other) != 0ull) {
                if (other) {
                    float c[DS];
                    load_floats(p.codebooks + ((size_t)m * KC + pick) * DS, c);
                    double t_new = 0.0;
#pragma unroll
                    for (int l = 0; l < DS; ++l) t_new = fma((double)c[l], (double)now.xv[l], t_new);
                    if (h == 0) my_codes[m] = (uint8_t)pick;
                    P = q - t_new;
                    changed = true;
                }
            }
            now = next;
        }
        const bool done = active && (init ? p.passes == 0 : !changed || stage + 1 >= p.passes);
        stage = init ? 0 : stage + 1;
        if (done) {
            if (h == 0) {
                uint8_t *out = p.packed + (size_t)id * p.NB;
                for (int e = 0; e < p.NB; ++e) out[e] = my_codes[e];
            }
            id = -1;
        }
    }
}

// Every other shape (16 codewords of 8 dimensions; other numbers of dimensions per subspace; few subspaces, see
// encode_few_steps): a thread per point, all in fp64, the terms of the current codewords kept per subspace. DS = dimensions per
// subspace known at compile time (0: any): the point's sub-vector then stays in registers while its codewords (wave-
// uniform, read through the scalar cache) pass by, instead of being read again for every codeword from a row that no
// neighbouring lane shares. 200,000 points, 4-bit codes, DS known against any: 128 = 16 x 8 dimensions 0.72 against 5.98 ms a
// call, 512 = 128 x 4 6.1 against 35.7, 512 = 256 x 2 21.0 against 77.8.
constexpr int kMaxM = 256;
template <int DS>
__global__ void __launch_bounds__(128)
encode_kernel(const float *__restrict__ x, int64_t n, int d, int M, int kc, int bits,
              const float *__restrict__ codebooks, const float *__restrict__ leaf_centers,
              const int32_t *__restrict__ leaf_assign, int eta_mode, double T, double eta_explicit,
              int passes, uint8_t *__restrict__ packed)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int ds = DS ? DS : d / M;
    const float *xi = x + (size_t)i * d;
    const float *ce = leaf_centers ? leaf_centers + (size_t)leaf_assign[i] * d : nullptr;
    constexpr int kReg = DS ? DS : 1;
    double xv_m[kReg], xr_m[kReg]; // DS != 0: x^(m) and x^(m) - center^(m) of the subspace entered last
    uint8_t code[kMaxM];
    double pm_cur[kMaxM], em_cur[kMaxM]; // terms of the current codeword of every subspace
    double pm_after[kMaxM], em_after[kMaxM]; // their sums over the subspaces after m, as of the start of a pass

    double nx2 = 0.0;
    for (int l = 0; l < d; ++l) nx2 += (double)xi[l] * (double)xi[l];
    const double eta = eta_of_norm(d, T, sqrt(nx2), eta_mode, eta_explicit);
    const double w = nx2 > 0.0 ? (eta - 1.0) / nx2 : 0.0;

    auto enter = [&](int m) {
        if constexpr (DS != 0) {
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                xv_m[l] = (double)xi[m * DS + l];
                xr_m[l] = xv_m[l] - (ce ? (double)ce[m * DS + l] : 0.0);
            }
        }
    };
    // terms of subspace m for codeword j: pm = <r^(m), x^(m)>, em = ||r^(m)||^2
    auto terms = [&](int m, int j, double &pm, double &em) {
        const float *c = codebooks + ((size_t)m * kc + j) * ds;
        pm = 0.0;
        em = 0.0;
        if constexpr (DS != 0) {
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                const double r = xr_m[l] - (double)c[l];
                pm = fma(r, xv_m[l], pm);
                em = fma(r, r, em);
            }
        } else {
            for (int l = 0; l < ds; ++l) {
                const double xv = (double)xi[m * ds + l];
                const double r = (xv - (ce ? (double)ce[m * ds + l] : 0.0)) - (double)c[l];
                pm = fma(r, xv, pm);
                em = fma(r, r, em);
            }
        }
    };

    // start: l2-nearest codeword of the (residual) sub-vector in every subspace
    for (int m = 0; m < M; ++m) {
        int best = 0;
        double bestd = INFINITY, bestp = 0.0;
        enter(m);
        for (int j = 0; j < kc; ++j) {
            double pm, em;
            terms(m, j, pm, em);
            if (em < bestd) { bestd = em; bestp = pm; best = j; }
        }
        code[m] = (uint8_t)best;
        pm_cur[m] = bestp;
        em_cur[m] = bestd;
    }
    for (int pass = 0; pass < passes; ++pass) {
        bool changed = false;
        // p and e of the other subspaces = the subspaces before m (running sums of this pass) + those after
        // it (sums formed here, from the last subspace down): M additions per pass instead of M per subspace
        double after_p = 0.0, after_e = 0.0;
        for (int m = M - 1; m >= 0; --m) {
            pm_after[m] = after_p;
            em_after[m] = after_e;
            after_p += pm_cur[m];
            after_e += em_cur[m];
        }
        double before_p = 0.0, before_e = 0.0;
        for (int m = 0; m < M; ++m) {
            const double Pr = before_p + pm_after[m], Er = before_e + em_after[m];
            int best = 0;
            double bestv = INFINITY, bestp = 0.0, beste = 0.0;
            enter(m);
            for (int j = 0; j < kc; ++j) {
                double pm, em;
                terms(m, j, pm, em);
                const double p = Pr + pm, e = Er + em;
                const double v = e + w * p * p;
                if (v < bestv) { bestv = v; best = j; bestp = pm; beste = em; }
            }
            if (best != code[m]) {
                code[m] = (uint8_t)best;
                pm_cur[m] = bestp;
                em_cur[m] = beste;
                changed = true;
            }
            before_p += pm_cur[m];
            before_e += em_cur[m];
        }
        if (!changed) break;
    }
    const int NB = (M * bits + 7) / 8;
    uint8_t *out = packed + (size_t)i * NB;
    if (bits == 8) {
        for (int m = 0; m < M; ++m) out[m] = code[m];
    } else {
        for (int b = 0; b < NB; ++b) {
            uint8_t v = code[2 * b] & 15;
            if (2 * b + 1 < M) v |= (uint8_t)((code[2 * b + 1] & 15) << 4);
            out[b] = v;
        }
    }
}

template <int DS>
static int launch_encode_one(EncodeParams p, const float *tab, const float2 *lim, hipStream_t st)
{
    // waves per workgroup: as many resident per compute unit as the 160 KB of LDS and the registers allow; few points are
    // spread over the compute units first
    const int most = DS <= 2 && p.leaf_centers == nullptr ? 20 : 16;
    const size_t shared = (size_t)p.M * (16 * (DS + 1) + 2) * 4, per_wave = (size_t)64 * p.code_stride;
    // windows that hold points: in order of the leaves, whose slots are whole blocks of 256, a leaf's last one may be short
    const int64_t groups = p.order ? std::min<int64_t>((p.n_slots + 63) / 64, p.n / 64 + p.n_slots / 256) : (p.n_slots + 63) / 64;
    const int wanted = (int)std::min<int64_t>(8, std::max<int64_t>(1, (groups + 255) / 256));
    int waves = 0, resident = 0;
    for (int w = 1; w <= wanted; ++w) {
        const size_t need = shared + w * per_wave;
        if (need > kMaxDynLds) break;
        const int r = std::min<int>(most, (int)(kMaxDynLds / need) * w);
        if (r > resident) { resident = r; waves = w; }
    }
    if (waves == 0) return 1; // does not fit: the caller takes the plain kernel
    // a resident set of waves, one for each window with points, and one a compute unit for windows without
    const int64_t total = std::max(std::min<int64_t>(groups, (int64_t)256 * resident), std::min<int64_t>((p.n_slots + 63) / 64, 256));
    const dim3 grid((unsigned)((total + waves - 1) / waves));
    const size_t lds = shared + waves * per_wave;
    // As many waves as windows: a wave whose window has few points (a leaf's last ones) leaves the next window to another wave, rather
    // than filling its lanes from it and having the rest of it wait for them. us a call, filling / leaving, 60 leaves: 9,000 x 192, 96
    // subspaces 607 / 397; 30,000 x 100, 50 396 / 296.
    p.top_up = groups > (int64_t)grid.x * waves;
    static LdsLimitOnce flat_done, res_done;
    AVQ_TRY(set_lds_limit((const void *)encode_aniso_kernel<DS, false>, kMaxDynLds, &flat_done));
    AVQ_TRY(set_lds_limit((const void *)encode_aniso_kernel<DS, true>, kMaxDynLds, &res_done));
    if (p.leaf_centers) hipLaunchKernelGGL((encode_aniso_kernel<DS, true>), grid, dim3(64 * waves), lds, st, p, tab, lim);
    else hipLaunchKernelGGL((encode_aniso_kernel<DS, false>), grid, dim3(64 * waves), lds, st, p, tab, lim);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

template <int DS>
static int launch_encode_wide(EncodeParams p, const float *operands, const float *cc, const float2 *lim, hipStream_t st)
{
    const size_t shared = (size_t)p.M * 1024, per_wave = (size_t)32 * p.code_stride;
    const bool cc_lds = shared + 4 * per_wave <= kMaxDynLds;
    const size_t fixed = cc_lds ? shared : 0;
    const int64_t groups = p.order ? std::min<int64_t>((p.n_slots + 31) / 32, p.n / 32 + p.n_slots / 256) : (p.n_slots + 31) / 32;
    // waves per workgroup: few points are spread over the compute units first
    const int wanted = (int)std::min<int64_t>(8, std::max<int64_t>(1, (groups + 255) / 256));
    int waves = 0, resident = 0;
    for (int w = 1; w <= wanted; ++w) {
        const size_t need = fixed + w * per_wave;
        if (need > kMaxDynLds) break;
        const int r = std::min<int>(8, (int)(kMaxDynLds / need) * w);
        if (r >= resident) { resident = r; waves = w; }
    }
    if (waves == 0) return 1;
    const int64_t total = std::max(std::min<int64_t>(groups, (int64_t)256 * resident), std::min<int64_t>((p.n_slots + 31) / 32, 256));
    const dim3 grid((unsigned)((total + waves - 1) / waves)), block(64 * waves);
    p.top_up = groups > (int64_t)grid.x * waves;
    const size_t lds = fixed + waves * per_wave;
    static LdsLimitOnce done[4];
#define AVQ_WIDE(RES, CC, I)                                                                                          \
    do {                                                                                                              \
        AVQ_TRY(set_lds_limit((const void *)encode_wide_kernel<DS, RES, CC>, kMaxDynLds, &done[I]));                  \
        hipLaunchKernelGGL((encode_wide_kernel<DS, RES, CC>), grid, block, lds, st, p, operands, cc, lim);            \
    } while (0)
    if (p.leaf_centers) {
        if (cc_lds) AVQ_WIDE(true, true, 0);
        else AVQ_WIDE(true, false, 1);
    } else {
        if (cc_lds) AVQ_WIDE(false, true, 2);
        else AVQ_WIDE(false, false, 3);
    }
#undef AVQ_WIDE
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// Few subspaces: a thread per point in fp64 is done before the fp32 search's waves, which share the windows by one counter and set up
// their tables each. The lines lie where the two are level. One avq_encode, fp64 / fp32 search (us): 16 codewords of 1 dimension,
// three passes: 4,000 points, 2 subspaces 32 / 27; 100,000, 3 43 / 46, 4 51 / 46; 1,000,000, 3 165 / 209, 4 237 / 210; no pass: 4,000,
// 3 28 / 28, 4 31 / 28; 1,000,000, 7 171 / 215, 8 294 / 215; of 2: 4,000, 2 28 / 28, 3 36 / 30; 100,000, 5 48 / 49, 6 54 / 51; no pass:
// 16,000, 6 31 / 32; 100,000, 12 54 / 53; of 3: 4,000, 1 31 / 28; 300,000, 2 77 / 81, 3 127 / 88; no pass: 3 71 / 82, 4 94 / 81; of 4:
// 16,000, 2 31 / 31, 3 35 / 34; 100,000, 4 49 / 51, 5 56 / 56; no pass: 16,000, 4 30 / 31, 5 33 / 33; 300,000, 7 92 / 101, 8 107 / 95.
// 256 of 2: 40,000, 1 76 / 63, 300,000, 1 132 / 148, 2 235 / 164, no pass: 2 123 / 146, 3 168 / 152; of 4: 100,000, 1 94 / 86, no pass:
// 58 / 72, 2 97 / 81; of 8: 100,000, 1 124 / 102, no pass: 73 / 80. At 40,000 points the lines are those of fewer points.
static bool encode_few_steps(int64_t n, int ds, int kc, int M, int passes)
{
    const bool many = n >= 65536; // points: measured at 40,000 and 100,000
    if (kc == 16) {
        const int most[2][2][5] = {{{0, 3, 6, 1, 4}, {0, 0, 2, 0, 2}}, {{0, 7, 12, 3, 7}, {0, 3, 5, 2, 4}}}; // by many, passes, ds
        return M <= most[many][passes > 0][ds];
    }
    return many && M <= (ds == 2) + (passes == 0);
}

int launch_encode(const float *x, int64_t n, int d, int M, int kc, int bits, const float *codebooks, const float *leaf_centers,
                  const int32_t *leaf_assign, const int32_t *order, int64_t n_slots, int eta_mode, double T, double eta_explicit,
                  int passes, uint8_t *packed, DevBuf *ws, hipStream_t st)
{
    if (M > kMaxM) { set_error("encode: M = %d exceeds %d", M, kMaxM); return AVQ_EINVAL; }
    if (M < 1 || d % M != 0) { set_error("encode: d = %d is not a multiple of M = %d", d, M); return AVQ_EINVAL; }
    const int ds = d / M;
    int rc = AVQ_ENOMEM; // AVQ_ENOMEM or 1: the kernel below, which needs no scratch, takes the points
    const size_t b_tab = (sizeof(float) * (size_t)M * kc * (ds + 1) + 255) & ~(size_t)255, b_lim = sizeof(float2) * (size_t)kMaxM + 256 + 4 * (size_t)kMaxM;
    const bool weights = eta_mode == AVQ_ETA_EXACT;
    if ((kc == 16 ? ds >= 1 && ds <= 4 : ds == 2 || ds == 4 || ds == 8) && !encode_few_steps(n, ds, kc, M, passes))
        rc = ws->reserve(b_tab + b_lim + (weights ? sizeof(double) * (size_t)n : 0));
    if (rc == AVQ_OK) {
        EncodeParams p;
        p.x = x; p.order = order; p.n = n; p.n_slots = order ? n_slots : n;
        p.d = d; p.M = M; p.NB = (M * bits + 7) / 8; p.passes = passes;
        p.codebooks = codebooks;
        float *tab = ws->as<float>();                                // [M][kc][ds + 1]: codeword, ||c||^2
        float2 *lim = (float2 *)(ws->as<unsigned char>() + b_tab); // [M]: largest |coordinate|, largest ||c||^2
        p.leaf_centers = leaf_centers; p.leaf_assign = leaf_assign;
        p.eta_mode = eta_mode; p.T = T; p.eta_explicit = eta_explicit;
        p.w_in = weights ? (const double *)(ws->as<unsigned char>() + b_tab + b_lim) : nullptr;
        p.packed = packed;
        p.next_window = (uint32_t *)(lim + kMaxM);
        p.distinct = p.next_window + 64;
        p.code_stride = 4 * (((M + 3) / 4) | 1);
        float *cc = tab + (size_t)M * kc * ds; // 256 codewords: after their operands
        if (kc == 16)
            hipLaunchKernelGGL(encode_tables_kernel, dim3((unsigned)M), dim3(64), 0, st, codebooks, ds, tab, lim, p.distinct, p.next_window);
        else
            hipLaunchKernelGGL(encode_operands_kernel, dim3((unsigned)M), dim3(256), 0, st, codebooks, ds, tab, cc, lim, p.next_window);
        if (weights)
            hipLaunchKernelGGL(encode_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, n, d, eta_mode, T,
                               eta_explicit, (double *)p.w_in);
        if (kc == 16) {
            switch (ds) {
            case 1: rc = launch_encode_one<1>(p, tab, lim, st); break;
            case 2: rc = launch_encode_one<2>(p, tab, lim, st); break;
            case 3: rc = launch_encode_one<3>(p, tab, lim, st); break;
            default: rc = launch_encode_one<4>(p, tab, lim, st); break;
            }
        } else {
            switch (ds) {
            case 2: rc = launch_encode_wide<2>(p, tab, cc, lim, st); break;
            case 4: rc = launch_encode_wide<4>(p, tab, cc, lim, st); break;
            default: rc = launch_encode_wide<8>(p, tab, cc, lim, st); break;
            }
        }
    }
    if (rc != 1 && rc != AVQ_ENOMEM) return rc;
#define AVQ_ENCODE(DS)                                                                                                              \
    hipLaunchKernelGGL(encode_kernel<DS>, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, st, x, n, d, M, kc, bits, codebooks,      \
                       leaf_centers, leaf_assign, eta_mode, T, eta_explicit, passes, packed)
    switch (ds) {
    case 2: AVQ_ENCODE(2); break;
    case 4: AVQ_ENCODE(4); break;
    case 8: AVQ_ENCODE(8); break;
    default: AVQ_ENCODE(0); break;
    }
#undef AVQ_ENCODE
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// ---- joint dictionary update under the anisotropic loss ---------------------------------
//
// Section 4.2 alternates assignment and codeword update; with the codes fixed the loss is a
// convex quadratic in the stacked dictionaries c (D = M*kc*ds unknowns) and Appendix 7.5
// gives its normal equations
//     (sum_i B_i^T A_i B_i) c = sum_i h_par,i B_i^T x_i,
//     A_i = h_perp,i I + (h_par,i - h_perp,i) x_i x_i^T / ||x_i||^2,
// where B_i picks codeword code_i[m] of every dictionary m (x~_i = B_i c). With h_perp = 1,
// h_par = eta_i and s_i = B_i^T x_i (x_i's coordinates scattered to its codewords' slots):
//     A = diag(counts) + sum_i w_i s_i s_i^T,  w_i = (eta_i - 1)/||x_i||^2,  b = sum_i eta_i s_i.
// A is never formed: conjugate gradients need only v -> A v, one pass over the points with
// a gather of d values of v, a dot product and a scatter-add. Codewords no point uses keep
// their value (unit diagonal, right-hand side = old value). All in fp64.

// bits 32: one int32 per subspace (the leaf assignment seen as the code of a one-dictionary quantizer)
__device__ __forceinline__ int code_at(const uint8_t *row, int m, int bits)
{
    if (bits == 32) return ((const int32_t *)row)[m];
    return bits == 8 ? (int)row[m] : (int)((row[m >> 1] >> (4 * (m & 1))) & 15);
}

// One wave per point (grid-stride): w_i, counts, right-hand side and the rank-one part of A's diagonal.
__global__ void __launch_bounds__(256)
pq_update_setup_kernel(const float *__restrict__ x, int64_t n, int d, int M, int kc, int bits, int NB,
                       const uint8_t *__restrict__ codes, const float *__restrict__ centers,
                       const int32_t *__restrict__ assign, int eta_mode, double T, double eta_explicit,
                       double *__restrict__ w_out, double *__restrict__ eta_out, double *__restrict__ b,
                       double *__restrict__ dA, unsigned int *__restrict__ cnt)
{
    const int lane = threadIdx.x & 63;
    const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int ds = d / M;
    for (int64_t i = wave0; i < n; i += n_waves) {
        const float *xi = x + (size_t)i * d;
        const uint8_t *ci = codes + (size_t)i * NB;
        // with leaf centers g: x~ = g + B c, the loss still against x; the right-hand side is B^T A (x - g),
        // A v = v + w x (x^T v); without, A x = eta x
        const float *gi = centers ? centers + (size_t)assign[i] * d : nullptr;
        double part = 0.0, xr = 0.0;
        for (int a = lane; a < d; a += 64) {
            part += (double)xi[a] * (double)xi[a];
            if (gi) xr += (double)xi[a] * ((double)xi[a] - (double)gi[a]);
        }
        for (int m = 32; m > 0; m >>= 1) { part += __shfl_xor(part, m, 64); xr += __shfl_xor(xr, m, 64); }
        const double nx2 = part;
        const double eta = eta_of_norm(d, T, sqrt(nx2), eta_mode, eta_explicit);
        const double wi = nx2 > 0.0 ? (eta - 1.0) / nx2 : 0.0;
        if (lane == 0) {
            w_out[i] = wi;
            eta_out[i] = eta;
        }
        for (int a = lane; a < d; a += 64) {
            const int m = a / ds;
            const int slot = m * kc + code_at(ci, m, bits);
            const double rhs = gi ? ((double)xi[a] - (double)gi[a]) + wi * xr * (double)xi[a] : eta * (double)xi[a];
            unsafeAtomicAdd(&b[(size_t)slot * ds + (a - m * ds)], rhs);
            if (wi != 0.0) unsafeAtomicAdd(&dA[(size_t)slot * ds + (a - m * ds)], wi * (double)xi[a] * (double)xi[a]);
            if (a == m * ds) atomicAdd(&cnt[slot], 1u);
        }
    }
}

// y += sum_i w_i s_i (s_i^T v). One wave per point. With use_lds the sum is accumulated per
// workgroup in LDS (D doubles) and added to y once per workgroup; otherwise (D too large for
// LDS) every term goes to y directly.
__global__ void __launch_bounds__(256)
pq_update_matvec_kernel(const float *__restrict__ x, int64_t n, int d, int M, int kc, int bits, int NB,
                        const uint8_t *__restrict__ codes, const double *__restrict__ w,
                        const double *__restrict__ v, double *__restrict__ y, int D, int use_lds)
{
    extern __shared__ double acc_lds[]; // [D] when use_lds
    double *acc = use_lds ? acc_lds : y;
    if (use_lds) {
        for (int r = threadIdx.x; r < D; r += blockDim.x) acc_lds[r] = 0.0;
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
    const int ds = d / M;
    for (int64_t i = wave0; i < n; i += n_waves) {
        const float *xi = x + (size_t)i * d;
        const uint8_t *ci = codes + (size_t)i * NB;
        double t = 0.0;
        for (int a = lane; a < d; a += 64) {
            const int m = a / ds;
            const int r = (m * kc + code_at(ci, m, bits)) * ds + (a - m * ds);
            t += (double)xi[a] * v[r];
        }
        for (int m = 32; m > 0; m >>= 1) t += __shfl_xor(t, m, 64);
        const double wt = w[i] * t;
        if (wt != 0.0) {
            for (int a = lane; a < d; a += 64) {
                const int m = a / ds;
                const int r = (m * kc + code_at(ci, m, bits)) * ds + (a - m * ds);
                if (use_lds) atomicAdd(&acc_lds[r], wt * (double)xi[a]);
                else unsafeAtomicAdd(&acc[r], wt * (double)xi[a]);
            }
        }
    }
    if (!use_lds) return;
    __syncthreads();
    for (int r = threadIdx.x; r < D; r += blockDim.x)
        if (acc_lds[r] != 0.0) unsafeAtomicAdd(&y[r], acc_lds[r]);
}

// Conjugate gradients with the diagonal of A as preconditioner (exact in one step when every
// eta_i = 1, where A is diagonal). state[0] = r.z, state[1] = b.b, state[2] = iterations done,
// state[3] = r.r. One workgroup.
// mode 0 (start, after y = A c0 is complete): r = b - y, z = r/dA, p = z, y = diag(count) * p.
// mode 1 (step, after y = A p is complete): the usual update, then y = diag(count) * p for the next product.
__global__ void __launch_bounds__(1024)
pq_update_cg_kernel(int mode, int D, int ds, const unsigned int *__restrict__ cnt, const double *__restrict__ b,
                    const double *__restrict__ dA, double *__restrict__ c, double *__restrict__ r,
                    double *__restrict__ p, double *__restrict__ y, double *__restrict__ state, double tol2)
{
    __shared__ double red[1024];
    const int tid = threadIdx.x, nt = blockDim.x;
    auto reduce = [&](double v) -> double {
        red[tid] = v;
        __syncthreads();
        for (int s = nt >> 1; s > 0; s >>= 1) {
            if (tid < s) red[tid] += red[tid + s];
            __syncthreads();
        }
        const double out = red[0];
        __syncthreads();
        return out;
    };
    auto diag = [&](int e) -> double { const unsigned int k = cnt[e / ds]; return k ? (double)k : 1.0; };
    if (mode == 0) {
        double rz = 0.0, rr = 0.0, bb = 0.0;
        for (int e = tid; e < D; e += nt) {
            const double re = b[e] - y[e];
            const double ze = re / dA[e];
            r[e] = re;
            p[e] = ze;
            rz += re * ze;
            rr += re * re;
            bb += b[e] * b[e];
        }
        rz = reduce(rz);
        rr = reduce(rr);
        bb = reduce(bb);
        for (int e = tid; e < D; e += nt) y[e] = diag(e) * p[e];
        if (tid == 0) { state[0] = rz; state[1] = bb; state[2] = 0.0; state[3] = rr; }
        return;
    }
    const double rz = state[0];
    if (rz == 0.0 || state[3] <= tol2 * state[1]) return; // converged: later steps of a burst do nothing
    double pap = 0.0;
    for (int e = tid; e < D; e += nt) pap += p[e] * y[e];
    pap = reduce(pap);
    const double alpha = rz / pap;
    double rz2 = 0.0, rr2 = 0.0;
    for (int e = tid; e < D; e += nt) {
        c[e] += alpha * p[e];
        const double re = r[e] - alpha * y[e];
        r[e] = re;
        rz2 += re * re / dA[e];
        rr2 += re * re;
    }
    rz2 = reduce(rz2);
    rr2 = reduce(rr2);
    const double beta = rz2 / rz;
    for (int e = tid; e < D; e += nt) {
        const double pe = r[e] / dA[e] + beta * p[e];
        p[e] = pe;
        y[e] = diag(e) * pe;
    }
    if (tid == 0) { state[0] = rz2; state[2] += 1.0; state[3] = rr2; }
}

// c0 (the current dictionaries, as doubles), the right-hand side of unused codewords,
// y = diag(count) * c0, and the counts added to A's diagonal
__global__ void pq_update_init_kernel(int D, int ds, const unsigned int *__restrict__ cnt,
                                      const float *__restrict__ codebooks, double *__restrict__ c,
                                      double *__restrict__ b, double *__restrict__ y, double *__restrict__ dA)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= D) return;
    const double c0 = (double)codebooks[e];
    c[e] = c0;
    const unsigned int k = cnt[e / ds];
    if (k == 0u) b[e] = c0;
    y[e] = (k ? (double)k : 1.0) * c0;
    dA[e] += k ? (double)k : 1.0;
}

__global__ void pq_update_store_kernel(int D, const double *__restrict__ c, float *__restrict__ codebooks)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < D) codebooks[e] = (float)c[e];
}

// scratch: doubles w[n], eta[n], then b, c, r, p, y, dA of D each, state[4]; then cnt[M*kc] unsigned
size_t pq_update_scratch_bytes(int64_t n, int D, int slots)
{
    return sizeof(double) * ((size_t)2 * n + (size_t)6 * D + 4) + sizeof(unsigned int) * (size_t)slots;
}

int pq_joint_update_device(const float *x, int64_t n, int d, int M, int kc, int bits, const uint8_t *codes,
                           const float *centers, const int32_t *assign,
                           int eta_mode, double T, double eta_explicit, float *codebooks, void *scratch,
                           int max_iters, double tol, int *iters_out, double *rel_residual_out, hipStream_t st)
{
    const int ds = d / M, D = M * kc * ds, slots = M * kc, NB = (M * bits + 7) / 8;
    const int use_lds = (size_t)D * sizeof(double) <= 64 * 1024;
    double *w = (double *)scratch, *eta = w + n, *b = eta + n, *c = b + D, *r = c + D, *p = r + D, *y = p + D, *dA = y + D;
    double *state = dA + D;
    unsigned int *cnt = (unsigned int *)(state + 4);
    AVQ_HIP(hipMemsetAsync(b, 0, sizeof(double) * ((size_t)6 * D + 4) + sizeof(unsigned int) * (size_t)slots, st));
    const int grid = (int)std::min<int64_t>(1024, (n + 3) / 4);
    hipLaunchKernelGGL(pq_update_setup_kernel, dim3(grid), dim3(256), 0, st, x, n, d, M, kc, bits, NB, codes,
                       centers, assign, eta_mode, T, eta_explicit, w, eta, b, dA, cnt);
    AVQ_HIP(hipGetLastError());
    const int vgrid = (D + 255) / 256;
    hipLaunchKernelGGL(pq_update_init_kernel, dim3(vgrid), dim3(256), 0, st, D, ds, cnt, codebooks, c, b, y, dA);
    AVQ_HIP(hipGetLastError());
    const size_t lds = use_lds ? sizeof(double) * (size_t)D : 0;
    static LdsLimitOnce attr_done;
    AVQ_TRY(set_lds_limit((const void *)pq_update_matvec_kernel, 64 * 1024, &attr_done));
    // y = A c0
    hipLaunchKernelGGL(pq_update_matvec_kernel, dim3(grid), dim3(256), lds, st, x, n, d, M, kc, bits, NB, codes, w, c, y, D, use_lds);
    AVQ_HIP(hipGetLastError());
    hipLaunchKernelGGL(pq_update_cg_kernel, dim3(1), dim3(1024), 0, st, 0, D, ds, cnt, b, dA, c, r, p, y, state, tol * tol);
    AVQ_HIP(hipGetLastError());
    double host_state[4] = {0, 0, 0, 0};
    int done = 0;
    const int check_every = 16;
    while (done < max_iters) {
        const int burst = std::min(check_every, max_iters - done);
        for (int it = 0; it < burst; ++it) {
            hipLaunchKernelGGL(pq_update_matvec_kernel, dim3(grid), dim3(256), lds, st, x, n, d, M, kc, bits, NB, codes, w, p, y, D, use_lds);
            hipLaunchKernelGGL(pq_update_cg_kernel, dim3(1), dim3(1024), 0, st, 1, D, ds, cnt, b, dA, c, r, p, y, state, tol * tol);
        }
        AVQ_HIP(hipGetLastError());
        done += burst;
        AVQ_HIP(hipMemcpyAsync(host_state, state, sizeof(host_state), hipMemcpyDeviceToHost, st));
        AVQ_HIP(hipStreamSynchronize(st));
        if (host_state[1] == 0.0 || host_state[3] <= tol * tol * host_state[1]) break;
    }
    hipLaunchKernelGGL(pq_update_store_kernel, dim3(vgrid), dim3(256), 0, st, D, c, codebooks);
    AVQ_HIP(hipGetLastError());
    if (iters_out) *iters_out = (int)host_state[2];
    if (rel_residual_out) *rel_residual_out = host_state[1] > 0.0 ? sqrt(host_state[3] / host_state[1]) : 0.0;
    return AVQ_OK;
}

} // namespace avq
