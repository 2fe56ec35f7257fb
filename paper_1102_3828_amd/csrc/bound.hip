// Lists that cannot hold anything within a query's bound (gfx950).
//
// No estimate of a (query, list) pair is below the sum of the smallest entries of its look-up table's rows (Eq. (5)),
//     L = sum_j min_k || r^j - p_jk ||^2 ,  r = x - c_l ,
// so once the sample has given a bound tau on the k'-th smallest estimate, a pair with L > tau needs neither a table nor a
// pass over its list: the short-list is the same without it.  Where the data is clustered most of the w lists are such
// (w is chosen for the queries that need many).
//
// L comes from the matrix cores without writing a table: ||r^j||^2 + min_k (||p_jk||^2 - 2 r^j . p_jk), the dot products in
// fp16 with the reproduction values as the rows of the product, so that a lane holds sixteen values of one pair's row and
// the minimum is taken in registers.  The margin covers every rounding of this against the fp32 table sums: fp16 rounding of
// both operands changes the products of a pair by at most 2^-10 sum_j 2 ||r^j|| max_k ||p_jk||, values below the smallest normal
// by 2^-14 each, and tables and fp32 sums are accurate to a few 2^-22 of sum_j (||r^j|| + max_k ||p_jk||)^2.
//
// Bound: vector instructions (24 per 16 values) and the staging of the codebook, once per workgroup.  64000 pairs at d = 128:
// 27 us; the tables of as many pairs take 164.  Measured (calls of 1000 queries x 64 lists, us before and now): 1024 lists of 10^5
// entries, four in a cluster, 2053 -> 1050 (7 % of the estimates are left to compute); 8192 lists of 3.7 10^3, k' = 10000,
// 1783 -> 1464; mixtures whose lists overlap more, 10^8 vectors and k' = 10000 2824 -> 2685, 10^9 and k' = 1000 4156 -> 3259.
#include "ivfr_internal.h"

#include <algorithm>
#include <type_traits>

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

#define PB_T 512

template <int M, int DS>
__global__ __launch_bounds__(PB_T) void pair_bound_kernel(const float* __restrict__ queries, const int32_t* __restrict__ probe,
                                                          int P, int w, const float* __restrict__ coarse,
                                                          const float* __restrict__ pq, const float* __restrict__ pq_norm,
                                                          const float* __restrict__ pq_maxnorm, const float* __restrict__ tau,
                                                          uint32_t* __restrict__ state) {
    constexpr int D = M * DS;
    constexpr int K = DS == 8 ? 8 : 16;          // dimensions per matrix instruction
    constexpr int V = K / 2;                     // of them in one lane
    constexpr int STEPS = DS / K;                // per sub-quantizer
    typedef typename std::conditional<K == 8, half4, half8>::type op_t;
    extern __shared__ char s_raw[];
    char* const s_cent = s_raw;                                                  // fp16 [M][256][DS], scaled
    float* const s_norm = reinterpret_cast<float*>(s_raw + IVFR_KS * D * 2);     // [M][256]
    const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, h = lane >> 5;
    float pmax[M], cmax = 0.f, nmax = 0.f;
#pragma unroll
    for (int j = 0; j < M; ++j) { pmax[j] = pq_maxnorm[j]; cmax = fmaxf(cmax, pmax[j]); nmax = fmaf(pmax[j], pmax[j], nmax); }
    int ce = 0;
    if (cmax > 0.f) (void)frexpf(cmax, &ce);
    const float s_c = cmax > 0.f ? ldexpf(1.f, 7 - ce) : 1.f;   // a power of two: the largest component is below 128
    for (int i = tid; i < IVFR_KS * D / 8; i += PB_T) {
        const float4 v0 = *reinterpret_cast<const float4*>(pq + (int64_t)i * 8);
        const float4 v1 = *reinterpret_cast<const float4*>(pq + (int64_t)i * 8 + 4);
        half8 hv;
        hv[0] = (_Float16)(v0.x * s_c); hv[1] = (_Float16)(v0.y * s_c); hv[2] = (_Float16)(v0.z * s_c); hv[3] = (_Float16)(v0.w * s_c);
        hv[4] = (_Float16)(v1.x * s_c); hv[5] = (_Float16)(v1.y * s_c); hv[6] = (_Float16)(v1.z * s_c); hv[7] = (_Float16)(v1.w * s_c);
        reinterpret_cast<half8*>(s_cent)[i] = hv;
    }
    for (int i = tid; i < M * IVFR_KS; i += PB_T) s_norm[i] = pq_norm[i];
    __syncthreads();
    // a wavefront takes 32 consecutive pairs: lanes row and row + 32 hold the halves of every step of pair row
    for (int64_t p0 = ((int64_t)blockIdx.x * (PB_T / 64) + (tid >> 6)) * 32; p0 < P; p0 += (int64_t)gridDim.x * (PB_T / 64) * 32) {
        const int64_t p = p0 + row < P ? p0 + row : P - 1;
        const float* x = queries + (p / w) * D + V * h;
        const float* c = coarse + (int64_t)probe[p] * D + V * h;
        float rn[M], amax = 0.f, rr = 0.f, ub = 0.f;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            float s2 = 0.f;
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
#pragma unroll
                for (int e = 0; e < V; e += 4) {
                    const int o = (j * STEPS + s) * K + e;
                    const float4 a = *reinterpret_cast<const float4*>(x + o), b = *reinterpret_cast<const float4*>(c + o);
                    const float v[4] = {a.x - b.x, a.y - b.y, a.z - b.z, a.w - b.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) { s2 = fmaf(v[i], v[i], s2); amax = fmaxf(amax, fabsf(v[i])); }
                }
            s2 += __shfl_xor(s2, 32, 64);
            rn[j] = s2;
            rr += s2;
            const float a = sqrtf(s2) + pmax[j];
            ub = fmaf(a, a, ub);
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
        int ae = 0;
        if (amax > 0.f) (void)frexpf(2.f * amax, &ae);
        const float s_a = amax > 0.f ? ldexpf(1.f, 9 - ae) : 1.f;   // largest |2 r s_a| in [256, 512)
        const float inv_s = 1.f / (s_a * s_c);
        op_t b[M * STEPS];
#pragma unroll
        for (int s = 0; s < M * STEPS; ++s)
#pragma unroll
            for (int e = 0; e < V; e += 4) {
                const float4 u = *reinterpret_cast<const float4*>(x + s * K + e), v = *reinterpret_cast<const float4*>(c + s * K + e);
                const float f = -2.f * s_a;
                b[s][e] = (_Float16)((u.x - v.x) * f); b[s][e + 1] = (_Float16)((u.y - v.y) * f);
                b[s][e + 2] = (_Float16)((u.z - v.z) * f); b[s][e + 3] = (_Float16)((u.w - v.w) * f);
            }
        float low = 0.f;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            float mn = INFINITY;
#pragma unroll 2
            for (int t = 0; t < 8; ++t) {   // 32 reproduction values
                floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    const op_t a = *reinterpret_cast<const op_t*>(s_cent + ((j * IVFR_KS + 32 * t + row) * DS + s * K + V * h) * 2);
                    if constexpr (K == 8) acc = __builtin_amdgcn_mfma_f32_32x32x8f16(a, b[j * STEPS + s], acc, 0, 0, 0);
                    else acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b[j * STEPS + s], acc, 0, 0, 0);
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 n = *reinterpret_cast<const float4*>(s_norm + j * IVFR_KS + 32 * t + 8 * g + 4 * h);
                    mn = fminf(mn, fminf(fmaf(acc[4 * g], inv_s, n.x), fmaf(acc[4 * g + 1], inv_s, n.y)));
                    mn = fminf(mn, fminf(fmaf(acc[4 * g + 2], inv_s, n.z), fmaf(acc[4 * g + 3], inv_s, n.w)));
                }
            }
            mn = fminf(mn, __shfl_xor(mn, 32, 64));
            low += fmaxf(0.f, rn[j] + mn);
        }
        const float margin = 1.05f * 9.765625e-4f * fmaxf(ub - rr - nmax, 0.f) + 7.62939453125e-6f * ub + D * 0.0390625f * inv_s;
        // (a comparison with something that is no number keeps the pair)
        const bool none = low - margin > tau[p / w];
        if (h == 0 && p0 + row < P) state[p] = (state[p] & ~IVFR_PAIR_KEPT) | (none ? 0u : IVFR_PAIR_KEPT);
    }
}

template <int M, int DS>
static size_t pair_bound_lds() { return (size_t)IVFR_KS * M * DS * 2 + (size_t)M * IVFR_KS * sizeof(float); }

#define IVFR_PB_ALL(F) F(4, 8) F(4, 16) F(4, 32) F(8, 8) F(8, 16) F(8, 32) F(16, 8) F(16, 16)

bool ivfr_pair_bound_supported(const ivfr_index* ix) {
#define IVFR_PB(MM, DD) if (ix->p.m == MM && ix->dsub == DD) return true;
    IVFR_PB_ALL(IVFR_PB)
#undef IVFR_PB
    return false;
}

int ivfr_launch_pair_bound(const ivfr_index* ix, const float* queries, const int32_t* probe, int nq, int w, const float* tau,
                           uint32_t* state, hipStream_t st) {
    const int P = nq * w;
    if (P <= 0) return IVFR_OK;
    const int grid = std::min(ix->n_cu, (P + PB_T / 2 - 1) / (PB_T / 2));   // 32 pairs per wavefront
#define IVFR_PB(MM, DD)                                                                                                        \
    if (ix->p.m == MM && ix->dsub == DD) {                                                                                     \
        hipLaunchKernelGGL((pair_bound_kernel<MM, DD>), dim3(grid), dim3(PB_T), (pair_bound_lds<MM, DD>()), st, queries, probe, P, \
                           w, ix->coarse, ix->pq, ix->pq_norm, ix->pq_maxnorm, tau, state);                                    \
        IVFR_HIP(hipGetLastError());                                                                                           \
        return IVFR_OK;                                                                                                        \
    }
    IVFR_PB_ALL(IVFR_PB)
#undef IVFR_PB
    ivfr_set_error("internal: no pair bound for m = %d and %d-dimensional sub-vectors", ix->p.m, ix->dsub);
    return IVFR_ERR_STATE;
}

// Dynamic LDS beyond 48 KB has to be allowed per kernel and device.
int ivfr_pair_bound_init() {
#define IVFR_PB(MM, DD)                                                                                                       \
    IVFR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(pair_bound_kernel<MM, DD>),                                    \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)pair_bound_lds<MM, DD>()));
    IVFR_PB_ALL(IVFR_PB)
#undef IVFR_PB
    return IVFR_OK;
}
