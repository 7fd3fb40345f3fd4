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
// encode_aniso_kernel (16 codewords of 1 to 4 dimensions, 256 of 2, 4 or 8): a lane per point. What decides a codeword is, with
// t = <c, x>, u = <c, x - center>, q = P + <x - center, x>,
//     f(j) = ||c||^2 - 2 u + w t^2 - 2 w q t,
// formed in fp32 with the codewords as scalar operands: ds + 2 operations (ds + ds + 3 with leaf centers) and three
// to keep the best (its index in its low bits) and the second best. f is within eps F of its real value, F a bound of
// the terms' magnitudes, so a codeword that leads by more than 2 eps F is the arg-min; else the lane evaluates every
// codeword in fp64 as above (one (point, subspace) in some thousands). q = p + <codeword in use, x> is kept and
// updated in fp64. The codes are therefore those of an fp64 evaluation.
//
// The points of a wave need different numbers of passes: a lane whose point is done takes the wave's next point at the
// end of the sweep over the subspaces, so that no lane waits for the slowest of 64. (x of the points in LDS, row by
// row, for 16 codewords; with 256 the rows are read from memory again, 32 bytes for 1,800 operations.) The rows of 64
// points leave room for fewer waves a compute unit as d grows: five at 100 dimensions, two at 192, one from 240 on, where
// this kernel still wins (200,000 x 384 points, 192 subspaces: 10.1 ms a call, 14.7 all in fp64), but not if many codewords
// of a dictionary are equal (all in pairs: 12.7 against 8.6); beyond about 420 dimensions no wave fits. On a
// partitioned index the points are taken leaf by leaf, and the lanes' leaf centers mostly are one and the same.
// Bound by vector operations and by the chain from one subspace's choice to the next one's q: 1,183,514 x 100 points,
// 50 subspaces of 16 codewords: 2.34 ms (1.5 ms of vector operations at five waves per compute unit; 2.91 ms with leaf
// centers), against 9.3 (11.8) ms for a thread per point with every codeword in fp64 and its state in scratch memory.
// Windows of points handed out by a counter instead of split evenly: 2.63 -> 2.34 ms, as one SIMD of four holds two waves.
struct EncodeParams {
    const float *x;
    int64_t n_slots;
    const int32_t *order; // slot -> point (-1: none), NULL: slot i is point i
    int32_t d, M, NB, passes;
    const float *codebooks;   // [M][KC][DS]
    const float *leaf_centers;
    const int32_t *leaf_assign;
    int32_t eta_mode;
    double T, eta_explicit;
    const double *w_in;       // NULL: w from eta_mode here
    uint8_t *packed;
    uint32_t *next_window;    // windows of 64 slots are handed out: waves that share a SIMD get fewer
    int32_t row_stride, code_stride; // row_stride: floats per staged row (odd); code_stride: bytes (odd dwords)
};

__global__ void __launch_bounds__(64)
encode_tables_kernel(const float *__restrict__ codebooks, int kc, int ds, float *__restrict__ tab, float2 *__restrict__ lim,
                     uint32_t *__restrict__ next_window)
{
    const int m = blockIdx.x, lane = threadIdx.x;
    if (m == 0 && lane == 0) *next_window = 0u;
    float cm = 0.0f, ccm = 0.0f;
    for (int j = lane; j < kc; j += 64) {
        const float *c = codebooks + ((size_t)m * kc + j) * ds;
        float *o = tab + ((size_t)m * kc + j) * (ds + 1);
        double cc = 0.0;
        for (int l = 0; l < ds; ++l) {
            o[l] = c[l];
            cc += (double)c[l] * (double)c[l];
            cm = fmaxf(cm, fabsf(c[l]));
        }
        o[ds] = (float)cc;
        ccm = fmaxf(ccm, (float)cc);
    }
    for (int s = 32; s > 0; s >>= 1) { cm = fmaxf(cm, __shfl_xor(cm, s, 64)); ccm = fmaxf(ccm, __shfl_xor(ccm, s, 64)); }
    if (lane == 0) lim[m] = make_float2(cm * 1.0001f, ccm * 1.0001f);
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

template <int DS, int KC, bool RES>
__global__ void __launch_bounds__(512)
encode_aniso_kernel(const EncodeParams p, const float *__restrict__ tables, const float2 *__restrict__ limits)
{
    constexpr bool kStage = KC == 16; // rows of x and the dictionaries in LDS
    extern __shared__ __align__(16) float enc_lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n_waves = blockDim.x >> 6;
    const int M = p.M, d = p.d;
    constexpr int kTab4 = 4 * (DS + 1); // float4s of a subspace's table of 16 codewords
    float *tab_lds = enc_lds; // kStage: [M][KC][DS + 1]
    float2 *lim_lds = (float2 *)(enc_lds + M * KC * (DS + 1)); // kStage: [M]
    float *rows = enc_lds + (kStage ? M * (KC * (DS + 1) + 2) + wave * 64 * p.row_stride : 0);
    uint8_t *codes = (uint8_t *)(enc_lds + (kStage ? M * (KC * (DS + 1) + 2) + n_waves * 64 * p.row_stride : 0)) +
                     (size_t)wave * 64 * p.code_stride;
    uint8_t *my_codes = codes + (size_t)lane * p.code_stride;
    const float *my_row = rows + (size_t)lane * p.row_stride; // kStage
    if (kStage) {
        for (int e = threadIdx.x; e < M * KC * (DS + 1); e += blockDim.x) tab_lds[e] = tables[e];
        for (int e = threadIdx.x; e < M; e += blockDim.x) lim_lds[e] = limits[e];
        __syncthreads();
    }
    for (int e = 0; e < p.code_stride; e += 4) *(uint32_t *)(my_codes + e) = 0u;

    int win_id = -1;                // this lane's slot of the window: its point
    u64 win = 0ull;                 // slots of the window not yet taken
    bool drained = false;           // no windows left
    int id = -1, stage = 0;         // this lane's point (-1: none) and pass (-1: nearest codewords first)
    double P = 0.0, w = 0.0; // P = <x - center - codewords, x>, the codewords chosen so far
    const float *xi = p.x, *ce_row = nullptr;
    bool changed = false;
    constexpr float kEps = (1.9074e-6f + (2 * DS + 8 + (RES ? 4 : 0)) * 6.0e-8f) * 1.05f;

    for (;;) {
        // lanes without a point take the wave's next ones
        u64 need = __builtin_amdgcn_ballot_w64(id < 0), taken = 0ull;
        while (need != 0ull) {
            if (win == 0ull) {
                if (drained) break;
                uint32_t w64 = 0u;
                if (lane == 0) w64 = atomicAdd(p.next_window, 1u);
                const int64_t s0 = (int64_t)__builtin_amdgcn_readfirstlane(w64) * 64, s = s0 + lane;
                if (s0 >= p.n_slots) { drained = true; break; }
                win_id = s < p.n_slots ? (p.order ? p.order[s] : (int)s) : -1;
                win = __builtin_amdgcn_ballot_w64(win_id >= 0);
                continue;
            }
            const int t = __builtin_ctzll(need), from = __builtin_ctzll(win);
            const int who = __builtin_amdgcn_readlane(win_id, from);
            need &= need - 1;
            win &= win - 1;
            taken |= 1ull << t;
            if (lane == t) id = who;
            if constexpr (kStage) {
                const float *src = p.x + (size_t)who * d;
                for (int c = 0; c < d; c += 64)
                    if (c + lane < d)
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(src + c + lane),
                                                         (__attribute__((address_space(3))) void *)(rows + t * p.row_stride + c), 4, 0, 0);
            }
        }
        if (__builtin_amdgcn_ballot_w64(id >= 0) == 0ull) break;
        if (taken != 0ull) {
            __builtin_amdgcn_s_waitcnt(0x0f70); // vmcnt(0): the rows are in LDS
            wave_lds_fence();
            if ((taken >> lane) & 1) {
                stage = -1;
                if constexpr (!kStage) xi = p.x + (size_t)id * d;
                if constexpr (RES) ce_row = p.leaf_centers + (size_t)p.leaf_assign[id] * d;
                double nx2 = 0.0, cx = 0.0;
#pragma unroll 4
                for (int l = 0; l < d; ++l) {
                    const double v = (double)(kStage ? my_row[l] : xi[l]);
                    nx2 += v * v;
                    if constexpr (RES) cx = fma((double)ce_row[l], v, cx);
                }
                P = nx2 - cx;
                if (p.w_in) {
                    w = p.w_in[id];
                } else {
                    double eta = p.eta_explicit;
                    if (p.eta_mode != AVQ_ETA_EXPLICIT) { // the limit of Theorem 3.4, floored at 1 (see eta_of_norm)
                        eta = 1.0;
                        if (nx2 > 0.0) {
                            const double u = clamp_ratio_sq(p.T, sqrt(nx2));
                            eta = fmax((double)(d - 1) * u / (1.0 - u), 1.0);
                        }
                    }
                    w = nx2 > 0.0 ? (eta - 1.0) / nx2 : 0.0;
                }
            }
        }
        const bool active = id >= 0;
        const bool init = stage < 0;
        const double wl = init ? 0.0 : w, w2 = 2.0 * wl;
        const float wf = (float)wl;
        changed = false;

        // One sweep over the subspaces. What a step needs is asked for during the step before it (two sets of registers
        // that take turns): a compute unit holds five waves at 100 dimensions, too few to hide a load by another wave.
        struct Step {
            float xv[DS], ce[RES ? DS : 1], cur[DS];
            float4 tab[kStage ? kTab4 : 1]; // kStage: the subspace's codewords and ||c||^2
            float2 lim;
            int code;
        };
        auto read_lds = [](const float *at, float (&v)[DS]) {
            typedef const __attribute__((address_space(3))) float lds_float;
            lds_float *src = (lds_float *)at;
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                if (l == 2) asm volatile("" : "+v"(src)); // three words are not read as one (see build.py)
                v[l] = src[l];
            }
        };
        auto load_codeword = [&](int m, int j, float (&c)[DS]) {
            if constexpr (kStage) read_lds(tab_lds + (m * KC + j) * (DS + 1), c);
            else {
                const float *src = p.codebooks + ((size_t)m * KC + j) * DS;
#pragma unroll
                for (int l = 0; l < DS; ++l) c[l] = src[l];
            }
        };
        auto load_step = [&](int m, Step &s) { // all but the codeword in use, which waits for its index
            if constexpr (kStage) read_lds(my_row + m * DS, s.xv);
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                if constexpr (!kStage) s.xv[l] = xi[m * DS + l];
                if constexpr (RES) s.ce[l] = active ? ce_row[m * DS + l] : 0.0f;
            }
            s.code = my_codes[m];
            if constexpr (kStage) {
                const float4 *t = (const float4 *)(tab_lds + m * KC * (DS + 1));
#pragma unroll
                for (int e = 0; e < kTab4; ++e) s.tab[e] = t[e];
                s.lim = lim_lds[m]; // (a scalar load here would make the wave wait for every LDS read in flight)
            }
        };
        auto step = [&](int m, const Step &s, Step &nx) {
            const int mn = m + 1 < M ? m + 1 : 0;
            load_step(mn, nx);
            // q = (p of the other subspaces) + <x - center, x> of this one = P + <codeword in use, x>
            double t_cur = 0.0;
            float sx = 0.0f, sr = 0.0f, xrf[RES ? DS : 1];
#pragma unroll
            for (int l = 0; l < DS; ++l) {
                t_cur = fma((double)s.cur[l], (double)s.xv[l], t_cur);
                sx += fabsf(s.xv[l]);
                if constexpr (RES) { xrf[l] = (float)((double)s.xv[l] - (double)s.ce[l]); sr += fabsf(xrf[l]); }
            }
            if (init) t_cur = 0.0;
            const double q = P + t_cur;
            const float Bf = (float)fma(w2, q, RES ? 0.0 : 2.0);
            const float2 lim = kStage ? s.lim : limits[m];
            const float T = lim.x * sx;
            float F = fmaf(T, fmaf(wf, T, fabsf(Bf)), lim.y);
            if constexpr (RES) F = fmaf(2.0f * lim.x, sr, F);
            const float lead = fmaf(F, 2.0f * kEps, 2.0e-37f);

            float best = INFINITY, second = INFINITY;
            int group = 0;
            const float *tab = tables + (size_t)m * KC * (DS + 1); // wave-uniform: scalar loads and operands
            constexpr int kGroups = KC / 16;
            auto entry = [&](int j, int l) -> float { // coordinate l of codeword j (kStage: j a constant), l = DS: ||c||^2
                if constexpr (kStage) {
                    const float4 e = s.tab[(j * (DS + 1) + l) / 4];
                    const int r = (j * (DS + 1) + l) % 4;
                    return r == 0 ? e.x : r == 1 ? e.y : r == 2 ? e.z : e.w;
                } else {
                    return tab[j * (DS + 1) + l];
                }
            };
#pragma unroll 1
            for (int g = 0; g < kGroups; ++g) {
                const float old = best;
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    auto c = [&](int l) -> float { return entry(g * 16 + v, l); };
                    float t = s.xv[0] * c(0);
#pragma unroll
                    for (int l = 1; l < DS; ++l) t = fmaf(s.xv[l], c(l), t);
                    float f = c(DS);
                    if constexpr (RES) {
                        float u = xrf[0] * c(0);
#pragma unroll
                        for (int l = 1; l < DS; ++l) u = fmaf(xrf[l], c(l), u);
                        f = fmaf(-2.0f, u, f);
                    }
                    f = fmaf(t, fmaf(wf, t, -Bf), f);
                    f = __uint_as_float((__float_as_uint(f) & 0xfffffff0u) | (uint32_t)v);
                    second = __builtin_amdgcn_fmed3f(best, second, f);
                    // the smaller; the compiler makes it the minimum that drops a NaN (a true median would return -infinity)
                    best = __builtin_amdgcn_fmed3f(-INFINITY, best, f);
                }
                if (kGroups > 1) group = best == old ? group : g;
            }
            int pick = group * 16 + (int)(__float_as_uint(best) & 15u);
            load_codeword(mn, nx.code, nx.cur);
            const bool open = active && !(second - best > lead);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(open) != 0ull, 0)) {
                if (open) {
                    // Equal codewords leave this open at every step. The codewords come from registers, or several at a time
                    // (one at a time by scalar loads, each waited for: 1.50 ms where 200,000 x 100 points meet 50 dictionaries
                    // of 8 pairs of equal codewords, 0.95 this way; 0.56 without the pairs).
                    double bestv = INFINITY, xr[DS], xx = 0.0;
                    pick = 0;
#pragma unroll
                    for (int l = 0; l < DS; ++l) {
                        xr[l] = (double)s.xv[l] - (RES ? (double)s.ce[RES ? l : 0] : 0.0);
                        xx = fma(xr[l], (double)s.xv[l], xx);
                    }
                    auto try_codeword = [&](int j) {
                        double pm = 0.0, em = 0.0;
#pragma unroll
                        for (int l = 0; l < DS; ++l) {
                            const double r = xr[l] - (double)entry(j, l);
                            pm = fma(r, (double)s.xv[l], pm);
                            em = fma(r, r, em);
                        }
                        const double pp = init ? 0.0 : (q - xx) + pm;
                        const double v = em + wl * pp * pp;
                        if (v < bestv) { bestv = v; pick = j; }
                    };
                    if constexpr (kStage) {
#pragma unroll
                        for (int j = 0; j < KC; ++j) try_codeword(j);
                    } else {
                        constexpr int kAtOnce = DS == 8 ? 2 : 8; // eight of 8 dimensions take 218 registers instead of 110
#pragma unroll kAtOnce
                        for (int j = 0; j < KC; ++j) try_codeword(j);
                    }
                }
            }
            const bool other = active && (init || pick != s.code);
            if (__builtin_amdgcn_ballot_w64(other) != 0ull) {
                if (other) {
                    float c[DS];
                    load_codeword(m, pick, c);
                    double t_new = 0.0;
#pragma unroll
                    for (int l = 0; l < DS; ++l) t_new = fma((double)c[l], (double)s.xv[l], t_new);
                    my_codes[m] = (uint8_t)pick;
                    P = q - t_new;
                    changed = true;
                }
            }
        };
        Step even, odd;
        load_step(0, even);
        load_codeword(0, even.code, even.cur);
        int m = 0;
        for (; m + 1 < M; m += 2) {
            step(m, even, odd);
            step(m + 1, odd, even);
        }
        if (m < M) step(m, even, odd);
        const bool done = active && (init ? p.passes == 0 : !changed || stage + 1 >= p.passes);
        stage = init ? 0 : stage + 1;
        if (done) {
            uint8_t *out = p.packed + (size_t)id * p.NB;
            for (int e = 0; e < p.code_stride && (KC == 16 ? e / 2 : e) < p.NB; e += 4) {
                const uint32_t v = *(const uint32_t *)(my_codes + e);
                if constexpr (KC == 16) {
                    out[e / 2] = (uint8_t)((v & 15u) | ((v >> 4) & 0xf0u));
                    if (e / 2 + 1 < p.NB) out[e / 2 + 1] = (uint8_t)(((v >> 16) & 15u) | ((v >> 20) & 0xf0u));
                } else {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
                        if (e + b < p.NB) out[e + b] = (uint8_t)(v >> (8 * b));
                }
            }
            id = -1;
        }
    }
}

// Every other shape (16 codewords of 8 dimensions; rows of which LDS does not hold 64; other numbers of dimensions per
// subspace; few subspaces, see encode_few_steps): a thread per point, all in fp64, the terms of the current codewords kept per subspace. DS = dimensions per
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

template <int DS, int KC>
static int launch_encode_one(EncodeParams p, const float *tab, const float2 *lim, hipStream_t st)
{
    // waves per workgroup: as many resident per compute unit as the 160 KB of LDS allow, at most 16
    const size_t shared = KC == 16 ? (size_t)p.M * (KC * (DS + 1) + 2) * 4 : 0;
    const size_t per_wave = (KC == 16 ? (size_t)64 * p.row_stride * 4 : 0) + (size_t)64 * p.code_stride;
    int waves = 0, resident = 0;
    for (int w = 1; w <= 8; ++w) {
        const size_t need = shared + w * per_wave;
        if (need > kMaxDynLds) break;
        const int r = std::min<int>(16, (int)(kMaxDynLds / need) * w);
        if (r > resident) { resident = r; waves = w; }
    }
    if (waves == 0) return 1; // does not fit: the caller takes the plain kernel
    const int64_t groups = (p.n_slots + 63) / 64;
    const int64_t total = std::min<int64_t>(groups, (int64_t)256 * resident); // a resident set of waves
    const dim3 grid((unsigned)((total + waves - 1) / waves));
    const size_t lds = shared + waves * per_wave;
    static LdsLimitOnce flat_done, res_done;
    AVQ_TRY(set_lds_limit((const void *)encode_aniso_kernel<DS, KC, false>, kMaxDynLds, &flat_done));
    AVQ_TRY(set_lds_limit((const void *)encode_aniso_kernel<DS, KC, true>, kMaxDynLds, &res_done));
    if (p.leaf_centers) hipLaunchKernelGGL((encode_aniso_kernel<DS, KC, true>), grid, dim3(64 * waves), lds, st, p, tab, lim);
    else hipLaunchKernelGGL((encode_aniso_kernel<DS, KC, false>), grid, dim3(64 * waves), lds, st, p, tab, lim);
    AVQ_HIP(hipGetLastError());
    return AVQ_OK;
}

// Few subspaces: a thread per point in fp64 is done before the fp32 search's waves have handed out their points one by one
// and staged their rows. One avq_encode of 300,000 points, fp64 / fp32 search (us): 16 codewords of 2 dimensions, ten
// passes: 4 subspaces 75 / 127, 8 126 / 138, 10 153 / 142; no pass: 8 73 / 130, 16 139 / 139; of 1 dimension, ten passes: 4
// 96 / 126, 6 135 / 134; of 3: 2 82 / 125, 3 133 / 126; of 4: 4 91 / 129, 6 131 / 137; 256 of 2, no pass, 16,000 points: 2
// 64 / 81, 4 105 / 112, 6 145 / 145. (1,000,000 points, 2 subspaces of 2 dimensions, ten passes: 92 / 251.) At 500 to 16,000
// points the lines lie one or two subspaces lower.
static bool encode_few_steps(int ds, int kc, int M, int passes)
{
    if (kc == 16) {
        const int most[5] = {0, 4, 7, 2, 5}, most_no_pass[5] = {0, 10, 14, 4, 8}; // by ds
        return M <= (passes > 0 ? most : most_no_pass)[ds];
    }
    return M <= (ds == 2 ? (passes > 0 ? 2 : 4) : ds == 4 && passes == 0 ? 2 : 0);
}

int launch_encode(const float *x, int64_t n, int d, int M, int kc, int bits, const float *codebooks, const float *leaf_centers,
                  const int32_t *leaf_assign, const int32_t *order, int64_t n_slots, int eta_mode, double T, double eta_explicit,
                  int passes, uint8_t *packed, DevBuf *ws, hipStream_t st)
{
    if (M > kMaxM) { set_error("encode: M = %d exceeds %d", M, kMaxM); return AVQ_EINVAL; }
    if (M < 1 || d % M != 0) { set_error("encode: d = %d is not a multiple of M = %d", d, M); return AVQ_EINVAL; }
    const int ds = d / M;
    int rc = AVQ_ENOMEM; // AVQ_ENOMEM or 1: the kernel below, which needs no scratch, takes the points
    const size_t b_tab = (sizeof(float) * (size_t)M * kc * (ds + 1) + 255) & ~(size_t)255, b_lim = sizeof(float2) * (size_t)kMaxM + 256;
    const bool weights = eta_mode == AVQ_ETA_EXACT;
    if ((kc == 16 ? ds >= 1 && ds <= 4 : ds == 2 || ds == 4 || ds == 8) && !encode_few_steps(ds, kc, M, passes))
        rc = ws->reserve(b_tab + b_lim + (weights ? sizeof(double) * (size_t)n : 0));
    if (rc == AVQ_OK) {
        EncodeParams p;
        p.x = x; p.order = order; p.n_slots = order ? n_slots : n;
        p.d = d; p.M = M; p.NB = (M * bits + 7) / 8; p.passes = passes;
        p.codebooks = codebooks;
        float *tab = ws->as<float>();                                // [M][kc][ds + 1]: codeword, ||c||^2
        float2 *lim = (float2 *)(ws->as<unsigned char>() + b_tab); // [M]: largest |coordinate|, largest ||c||^2
        p.leaf_centers = leaf_centers; p.leaf_assign = leaf_assign;
        p.eta_mode = eta_mode; p.T = T; p.eta_explicit = eta_explicit;
        p.w_in = weights ? (const double *)(ws->as<unsigned char>() + b_tab + b_lim) : nullptr;
        p.packed = packed;
        p.next_window = (uint32_t *)(lim + kMaxM);
        p.row_stride = d | 1;
        p.code_stride = 4 * (((M + 3) / 4) | 1);
        hipLaunchKernelGGL(encode_tables_kernel, dim3((unsigned)M), dim3(64), 0, st, codebooks, kc, ds, tab, lim,
                           p.next_window);
        if (weights)
            hipLaunchKernelGGL(encode_weights_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, x, n, d, eta_mode, T,
                               eta_explicit, (double *)p.w_in);
        if (kc == 16) {
            switch (ds) {
            case 1: rc = launch_encode_one<1, 16>(p, tab, lim, st); break;
            case 2: rc = launch_encode_one<2, 16>(p, tab, lim, st); break;
            case 3: rc = launch_encode_one<3, 16>(p, tab, lim, st); break;
            default: rc = launch_encode_one<4, 16>(p, tab, lim, st); break;
            }
        } else {
            switch (ds) {
            case 2: rc = launch_encode_one<2, 256>(p, tab, lim, st); break;
            case 4: rc = launch_encode_one<4, 256>(p, tab, lim, st); break;
            default: rc = launch_encode_one<8, 256>(p, tab, lim, st); break;
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
