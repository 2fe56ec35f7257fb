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
// Bound: the reads of the codebook (from L2, once per workgroup) and the chain of a wavefront's products.  d = 128: 8 us for
// 8000 pairs, 11 for 16000, 23 for 64000 (33 with 32 pairs per workgroup); the tables of as many take 23, 44 and 145.  Listing and
// counting the kept pairs takes 27 instead of 22 at 64000: one returning addition a workgroup to one word, a thousand that queue up.  It
// replaces the kernel that counted them (8), while the grouping's two kernels behind it start with colder counts (17 -> 26 and 9 -> 13).
// Measured
// (calls of 1000 queries x 64 lists, us without and with): 1024 lists of 10^5
// entries, four in a cluster, 2053 -> 1050 (7 % of the estimates are left to compute); 8192 lists of 3.7 10^3, k' = 10000,
// 1783 -> 1464; mixtures whose lists overlap more, 10^8 vectors and k' = 10000 2824 -> 2685, 10^9 and k' = 1000 4156 -> 3259.  Where
// the lists overlap wholly nothing is left out, and the bounds are a loss (see BoundTries for its size and what follows from it).
#include "ivfr_internal.h"

#include <algorithm>
#include <type_traits>

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

#define PB_T 512
#define PB_WAVES (PB_T / 64)

// A workgroup takes 32 NP consecutive pairs; a wavefront a sub-quantizer (two at M = 16, half of one at M = 4): few pairs are spread
// over many compute units, and a wavefront has no more than sixteen products for each 32 of them.  Lanes row and row + 32 hold the
// halves of a step of pair row.  out: the lower bounds themselves (less the margin), else the pairs' state bits against tau.
template <int M, int DS, int NP>
__global__ __launch_bounds__(PB_T) void pair_bound_kernel(const float* __restrict__ queries, const int32_t* __restrict__ probe,
                                                          int P, int w, const float* __restrict__ coarse,
                                                          const float* __restrict__ pq, const float* __restrict__ pq_norm,
                                                          const float* __restrict__ pq_maxnorm, const float* __restrict__ tau,
                                                          uint32_t* __restrict__ state, float* __restrict__ out,
                                                          KeptPairs kept) {
    constexpr int D = M * DS;
    constexpr int K = DS == 8 ? 8 : 16;          // dimensions per matrix instruction
    constexpr int V = K / 2;                     // of them in one lane
    constexpr int STEPS = DS / K;                // per sub-quantizer
    constexpr int SPLIT = M < PB_WAVES ? PB_WAVES / M : 1;   // wavefronts per sub-quantizer
    constexpr int TILES = 8 / SPLIT;             // of 32 reproduction values, per wavefront
    typedef typename std::conditional<K == 8, half4, half8>::type op_t;
    __shared__ __align__(16) float s_norm[M * IVFR_KS];
    __shared__ float s_min[SPLIT][M][32 * NP], s_r2[M][32 * NP], s_flush[M][NP];
    const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, h = lane >> 5, wave = tid >> 6;
    const int64_t p0 = (int64_t)blockIdx.x * (32 * NP);
    for (int i = tid; i < M * IVFR_KS; i += PB_T) s_norm[i] = pq_norm[i];
    __syncthreads();
    const float* x[NP];
    const float* c[NP];
#pragma unroll
    for (int n = 0; n < NP; ++n) {
        const int64_t p = p0 + 32 * n + row < P ? p0 + 32 * n + row : P - 1;
        x[n] = queries + (p / w) * D + V * h;
        c[n] = coarse + (int64_t)probe[p] * D + V * h;
    }
    for (int j = wave / SPLIT; j < M; j += PB_WAVES / SPLIT) {
        // powers of two that bring the larger components of both operands to 2^6 .. 2^7 and 2^8 .. 2^9; 2^60 at the most, so that they,
        // their product and its inverse stay inside fp32 (components below 2^-52 lose bits then: s_flush counts in the same units)
        int ce = 0;
        const float pmax = pq_maxnorm[j];
        if (pmax > 0.f) (void)frexpf(pmax, &ce);
        const float s_c = pmax > 0.f ? ldexpf(1.f, min(7 - ce, 60)) : 1.f;
        op_t b[NP][STEPS];
        float inv_s[NP], mn[NP], r2[NP];
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            float v[STEPS * V];
            float s2 = 0.f, amax = 0.f;
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
#pragma unroll
                for (int e = 0; e < V; e += 4) {
                    const int o = j * DS + s * K + e;
                    const float4 a = *reinterpret_cast<const float4*>(x[n] + o), d = *reinterpret_cast<const float4*>(c[n] + o);
                    v[s * V + e] = a.x - d.x; v[s * V + e + 1] = a.y - d.y; v[s * V + e + 2] = a.z - d.z; v[s * V + e + 3] = a.w - d.w;
                }
#pragma unroll
            for (int i = 0; i < STEPS * V; ++i) { s2 = fmaf(v[i], v[i], s2); amax = fmaxf(amax, fabsf(v[i])); }
            r2[n] = s2 + __shfl_xor(s2, 32, 64);
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
            int ae = 0;
            if (amax > 0.f) (void)frexpf(2.f * amax, &ae);
            const float s_a = amax > 0.f ? ldexpf(1.f, min(9 - ae, 60)) : 1.f;
            inv_s[n] = 1.f / (s_a * s_c);
            mn[n] = INFINITY;
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
#pragma unroll
                for (int e = 0; e < V; ++e) b[n][s][e] = (_Float16)(v[s * V + e] * (-2.f * s_a));
        }
        const int t0 = (wave % SPLIT) * TILES;
#pragma unroll 4
        for (int t = t0; t < t0 + TILES; ++t) {   // 32 reproduction values
            op_t a[STEPS];
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const float* src = pq + ((int64_t)j * IVFR_KS + 32 * t + row) * DS + s * K + V * h;
#pragma unroll
                for (int e = 0; e < V; e += 4) {
                    const float4 f = *reinterpret_cast<const float4*>(src + e);
                    a[s][e] = (_Float16)(f.x * s_c); a[s][e + 1] = (_Float16)(f.y * s_c);
                    a[s][e + 2] = (_Float16)(f.z * s_c); a[s][e + 3] = (_Float16)(f.w * s_c);
                }
            }
#pragma unroll
            for (int n = 0; n < NP; ++n) {
                floatx16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    if constexpr (K == 8) acc = __builtin_amdgcn_mfma_f32_32x32x8f16(a[s], b[n][s], acc, 0, 0, 0);
                    else acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[s], b[n][s], acc, 0, 0, 0);
                }
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 nn = *reinterpret_cast<const float4*>(s_norm + j * IVFR_KS + 32 * t + 8 * g + 4 * h);
                    mn[n] = fminf(mn[n], fminf(fmaf(acc[4 * g], inv_s[n], nn.x), fmaf(acc[4 * g + 1], inv_s[n], nn.y)));
                    mn[n] = fminf(mn[n], fminf(fmaf(acc[4 * g + 2], inv_s[n], nn.z), fmaf(acc[4 * g + 3], inv_s[n], nn.w)));
                }
            }
        }
#pragma unroll
        for (int n = 0; n < NP; ++n) {
            const float m2 = fminf(mn[n], __shfl_xor(mn[n], 32, 64));
            if (h == 0) {
                s_min[wave % SPLIT][j][32 * n + row] = m2;
                if (wave % SPLIT == 0) s_r2[j][32 * n + row] = r2[n];
            }
            if (lane == 0 && wave % SPLIT == 0) s_flush[j][n] = DS * 0.0390625f * inv_s[n];   // (2^9 + 2^7) 2^-14 per dimension
        }
    }
    __syncthreads();
    if (tid >= 32 * NP || p0 + tid >= P) return;
    float low = 0.f, rr = 0.f, ub = 0.f, nmax = 0.f, flush = 0.f;
    for (int j = 0; j < M; ++j) {
        const float r2 = s_r2[j][tid], pm = pq_maxnorm[j];
        float mn = s_min[0][j][tid];
#pragma unroll
        for (int x2 = 1; x2 < SPLIT; ++x2) mn = fminf(mn, s_min[x2][j][tid]);
        low += fmaxf(0.f, r2 + mn);
        rr += r2;
        nmax = fmaf(pm, pm, nmax);
        const float a = sqrtf(r2) + pm;
        ub = fmaf(a, a, ub);
        flush += s_flush[j][tid >> 5];
    }
    low -= 1.05f * 9.765625e-4f * fmaxf(ub - rr - nmax, 0.f) + 7.62939453125e-6f * ub + flush;
    if (!(low < INFINITY)) low = -INFINITY;   // infinite or no number: nothing is known of the pair
    if (out) { out[p0 + tid] = low; return; }
    const bool none = low > tau[(p0 + tid) / w];
    state[p0 + tid] = (state[p0 + tid] & ~IVFR_PAIR_KEPT) | (none ? 0u : IVFR_PAIR_KEPT);
    // the kept pairs' list, in any order of the workgroups (one wavefront is left of each)
    static_assert(32 * NP <= 64, "the pairs of a workgroup are those of its first wavefront");
    const uint64_t mine = __ballot(!none);
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(kept.n, (uint32_t)__popcll(mine));
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (!none) {
        const int64_t p = p0 + tid;
        kept.pairs[at + (uint32_t)__popcll(mine & ((1ull << lane) - 1ull))] = (uint32_t)p;
        atomicAdd(&kept.list_np[2 * probe[p] + (kept.use8 && !kept.exact_only[p / w] ? 0 : 1)], 1u);
    }
}

#define IVFR_PB_ALL(F) F(4, 8) F(4, 16) F(4, 32) F(8, 8) F(8, 16) F(8, 32) F(16, 8) F(16, 16)

bool ivfr_pair_bound_supported(const ivfr_index* ix) {
#define IVFR_PB(MM, DD) if (ix->p.m == MM && ix->dsub == DD) return true;
    IVFR_PB_ALL(IVFR_PB)
#undef IVFR_PB
    return false;
}

int ivfr_launch_pair_bound(const ivfr_index* ix, const float* queries, const int32_t* probe, int nq, int w, const float* tau,
                           uint32_t* state, float* out, const KeptPairs& kept, hipStream_t st) {
    const int P = nq * w;
    if (P <= 0) return IVFR_OK;
#define IVFR_PB(MM, DD)                                                                                                        \
    if (ix->p.m == MM && ix->dsub == DD) {                                                                                     \
        /* two times 32 pairs share the codebook where every compute unit still has a workgroup */                             \
        if (P > 64 * ix->n_cu)                                                                                                 \
            hipLaunchKernelGGL((pair_bound_kernel<MM, DD, 2>), dim3((unsigned)((P + 63) / 64)), dim3(PB_T), 0, st, queries, probe, \
                               P, w, ix->coarse, ix->pq, ix->pq_norm, ix->pq_maxnorm, tau, state, out, kept);                        \
        else                                                                                                                   \
            hipLaunchKernelGGL((pair_bound_kernel<MM, DD, 1>), dim3((unsigned)((P + 31) / 32)), dim3(PB_T), 0, st, queries, probe, \
                               P, w, ix->coarse, ix->pq, ix->pq_norm, ix->pq_maxnorm, tau, state, out, kept);                        \
        IVFR_HIP(hipGetLastError());                                                                                           \
        return IVFR_OK;                                                                                                        \
    }
    IVFR_PB_ALL(IVFR_PB)
#undef IVFR_PB
    ivfr_set_error("internal: no pair bound for m = %d and %d-dimensional sub-vectors", ix->p.m, ix->dsub);
    return IVFR_ERR_STATE;
}
