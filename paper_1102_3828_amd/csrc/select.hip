// Segmented exact top-K selection by 64-bit key, one workgroup per segment (gfx950).
//
// Serves the three selections of the query stage: the w nearest coarse centroids
// (section 3.3), the k' smallest ADC estimates that form the short-list (step 1 of section
// 3.2) and the k smallest refined distances (step 3).  A key is (distance bits << 32) | index:
// non-negative IEEE floats order like their bit patterns, and the index in the low half makes
// every key distinct, so "the K smallest keys" is the K smallest distances with ties broken
// towards the lowest index, exactly.
//
// The selection itself (the K-th smallest key of a segment) is in select_core.h.
#include "select_core.h"

#include <algorithm>
#include <type_traits>

#define SORT_MAX 16384
#define BIN_SORT_MAX 8192   // results sorted through bins: their keys, bins and order fit the LDS

__device__ __forceinline__ int64_t seg_count(const uint32_t* counts, uint32_t cap, int seg, bool* over) {
    *over = false;
    uint32_t c = counts[seg];
    if (c > cap) { *over = true; return cap; }
    return c;
}

// ---- bound from a uniform sample --------------------------------------------------------------
// The sample holds n of the query's sq visited entries, so about mu = k' n / sq of the true k'
// best are in it (Poisson-like).  Taking the r-th smallest sampled estimate with r = mu + 5
// sqrt(mu) + 6 makes it all but certain (beyond five standard deviations) that at least k'
// visited entries lie at or below it; the filtered scan verifies that by counting.
// WALK: few workgroups walk over the segments (for batches in which hardly any query has a sample: launching a
// workgroup per query only to find its skip flag set costs more than the whole selection); otherwise one
// workgroup per segment.
template <bool WALK>
__global__ __launch_bounds__(SEL_T) void select_tau_kernel(const uint2* recs, const int32_t* ids, uint32_t id_stride,
                                                           CandLayout lay, const uint32_t* counts,
                                                           const unsigned long long* sq, int kprime,
                                                           int fixed_rank, const uint8_t* skip, float* tau,
                                                           uint32_t* tau_id, int values_only, int nseg) {
    __shared__ SelShared sh;
    // seg is uniform over the workgroup, so every barrier is reached by all its threads
    for (int seg = blockIdx.x; seg < nseg; seg += WALK ? (int)gridDim.x : nseg) {
        if (skip && skip[seg]) continue;
        bool over;
        int64_t n = seg_count(counts, values_only ? 0xFFFFFFFFu : lay.cap(seg), seg, &over);
        const double mu = (double)kprime * (double)n / (double)(sq[seg] ? sq[seg] : 1ull);
        // fixed_rank > 0: the records are a subset of the visited entries and their fixed_rank-th smallest is wanted
        const int64_t r = fixed_rank > 0 ? (int64_t)fixed_rank : (int64_t)ceil(mu + 5.0 * sqrt(mu) + 6.0);
        if (n < r || n == 0) {
            if (threadIdx.x == 0) {
                tau[seg] = INFINITY;
                if (tau_id) tau_id[seg] = 0xFFFFFFFFu;
            }
            continue;
        }
        // values only: the segment holds n bare estimates (4 bytes each) at the start of its record buffer.  The selection
        // ends with a barrier: its LDS state is free for the next segment
        const uint2* r0 = recs + lay.base(seg);
        const uint64_t pivot = values_only ? kth_key(sh, ValsSrc{reinterpret_cast<const uint32_t*>(r0), n}, (uint32_t)r)
                                           : kth_key(sh, MemRecsSrc{r0, n, ids, id_stride}, (uint32_t)r);
        if (threadIdx.x == 0) {
            tau[seg] = __uint_as_float((uint32_t)(pivot >> 32));
            if (tau_id) tau_id[seg] = (uint32_t)pivot;
        }
    }
}

int ivfr_launch_select_tau(const SelectArgs& a, const unsigned long long* sq, int kprime, int fixed_rank,
                           const uint8_t* skip, float* tau, uint32_t* tau_id, hipStream_t st, bool values_only,
                           bool mostly_skipped) {
    if (a.nseg <= 0) return IVFR_OK;
    if (mostly_skipped)
        hipLaunchKernelGGL(select_tau_kernel<true>, dim3(std::min(a.nseg, 256)), dim3(SEL_T), 0, st, a.recs, a.ids,
                           a.id_stride, a.lay, a.counts, sq, kprime, fixed_rank, skip, tau, tau_id, values_only ? 1 : 0, a.nseg);
    else
        hipLaunchKernelGGL(select_tau_kernel<false>, dim3(a.nseg), dim3(SEL_T), 0, st, a.recs, a.ids, a.id_stride,
                           a.lay, a.counts, sq, kprime, fixed_rank, skip, tau, tau_id, values_only ? 1 : 0, a.nseg);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// ---- unordered compaction of the K smallest records -----------------------------------------
__global__ __launch_bounds__(SEL_T, 4) void select_records_kernel(const uint2* recs, const int32_t* ids,
                                                               uint32_t id_stride,
                                                               CandLayout lay, const uint32_t* counts, int K,
                                                               int out_base,
                                                               const unsigned long long* sq, uint32_t* out_pos,
                                                               float* out_est, int32_t* out_n, int32_t* overflow,
                                                               int32_t* overflow_total) {
    __shared__ SelShared sh;
    __shared__ uint32_t s_slot;
    const int seg = blockIdx.x;
    const int q = out_base + seg;
    bool over;
    int64_t n = seg_count(counts, lay.cap(seg), seg, &over);
    // the filter was too tight if it kept fewer than k' although more entries were visited
    if (sq && n < K && (unsigned long long)n < sq[seg]) over = true;
    if (threadIdx.x == 0) {
        s_slot = 0;
        if (overflow) overflow[q] = over ? 1 : 0;
        if (over && overflow_total) atomicAdd(overflow_total, 1);
    }
    __syncthreads();
    if (over) {
        if (threadIdx.x == 0) out_n[q] = 0;
        return;
    }
    const MemRecsSrc s{recs + lay.base(seg), n, ids, id_stride};
    uint32_t* op = out_pos + (int64_t)q * K;
    float* oe = out_est + (int64_t)q * K;
    if (n <= K) {
        for (int64_t i = threadIdx.x; i < n; i += SEL_T) {
            const uint2 r = s.v[i];
            op[i] = r.y;
            oe[i] = __uint_as_float(r.x);
        }
        if (threadIdx.x == 0) out_n[q] = (int32_t)n;
        return;
    }
    auto take = [&](const auto& src) {
        const uint64_t pivot = kth_key(sh, src, (uint32_t)K);
        src.sweep([&](uint32_t est, uint32_t pos) {
            if (within(est, pivot, [&]() { return src.lo(pos); })) {
                const uint32_t slot = atomicAdd(&s_slot, 1u);
                if (slot < (uint32_t)K) { op[slot] = pos; oe[slot] = __uint_as_float(est); }
            }
        });
    };
    if (n <= 8 * SEL_T) { RegRecsSrc<8> regs; regs.n = n; regs.ids = ids; regs.id_stride = id_stride; regs.load(s.v); take(regs); }
    else if (n <= 26 * SEL_T) { RegRecsSrc<26> regs; regs.n = n; regs.ids = ids; regs.id_stride = id_stride; regs.load(s.v); take(regs); }
    else take(s);
    if (threadIdx.x == 0) out_n[q] = K;
}

int ivfr_launch_select_records(const SelectArgs& a, int out_base, const unsigned long long* sq, uint32_t* out_pos,
                               float* out_est, int32_t* out_n, int32_t* overflow, int32_t* overflow_total,
                               hipStream_t st) {
    if (a.nseg <= 0) return IVFR_OK;
    hipLaunchKernelGGL(select_records_kernel, dim3(a.nseg), dim3(SEL_T), 0, st, a.recs, a.ids, a.id_stride, a.lay, a.counts, a.K,
                       out_base, sq, out_pos, out_est, out_n, overflow, overflow_total);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// ---- sorted K smallest keys -----------------------------------------------------------------
// A segment's elements are 64-bit keys, or (VALS) bare distance words whose index in the segment is the low half of the
// key.  counts (optional) gives each segment's element count (int32, e.g. the short-list length).
// NR: elements per thread that are held in registers, at most NR SEL_T a segment; 0: any number, read from memory each time.  A kernel
// each: one for all sizes took 75 registers, three workgroups a compute unit instead of four (1000 queries, the probe of 8 of 51
// lists 11.0 us, so 5.2).
template <bool VALS, int NR>
__global__ __launch_bounds__(SEL_T, NR <= 4 ? 8 : 1) void select_sorted_kernel(const void* data, int64_t seg_stride,
                                                              int64_t fixed_count, const int32_t* counts, int K,
                                                              int n2, int out_base, int32_t* out_lo, float* out_hi) {
    extern __shared__ uint64_t sk[];   // n2 keys
    __shared__ SelShared sh;
    __shared__ uint32_t s_slot;
    const int seg = blockIdx.x;
    const int q = out_base + seg;
    int64_t n = counts ? (int64_t)counts[q] : fixed_count;
    if (threadIdx.x == 0) s_slot = 0;
    for (int i = threadIdx.x; i < n2; i += SEL_T) sk[i] = ~0ull;
    __syncthreads();
    typedef typename std::conditional<VALS, ValsSrc, KeysSrc>::type Src;
    typedef typename std::conditional<VALS, uint32_t, uint64_t>::type Elem;
    const Src s{static_cast<const Elem*>(data) + (int64_t)seg * seg_stride, n};
    int m_out;
    if (n <= K) {
        for (int64_t i = threadIdx.x; i < n; i += SEL_T) sk[i] = VALS ? ((uint64_t)s.v[i] << 32) | (uint32_t)i : (uint64_t)s.v[i];
        m_out = (int)n;
    } else {
        auto take = [&](const auto& src) {
            const uint64_t pivot = kth_key(sh, src, (uint32_t)K);
            src.sweep([&](uint32_t h, uint32_t l) {
                const uint64_t k = ((uint64_t)h << 32) | l;
                if (k <= pivot) {
                    const uint32_t slot = atomicAdd(&s_slot, 1u);
                    if (slot < (uint32_t)n2) sk[slot] = k;
                }
            });
        };
        if constexpr (NR == 0) take(s);
        else if constexpr (NR == 4) { if constexpr (VALS) take(RegValsSrc<4, Src>(s)); else take(RegKeysSrc<4>(s)); }
        else if (n <= 4 * SEL_T) { if constexpr (VALS) take(RegValsSrc<4, Src>(s)); else take(RegKeysSrc<4>(s)); }
        else { if constexpr (VALS) take(RegValsSrc<NR, Src>(s)); else take(RegKeysSrc<NR>(s)); }
        m_out = K;
    }
    __syncthreads();
    if (n2 <= SEL_RANK_SORT) {
        // few results: no sort
        const int m_have = n <= K ? m_out : (int)(s_slot < (uint32_t)n2 ? s_slot : (uint32_t)n2);
        write_ranked(sk, m_have, m_out, K, out_lo + (int64_t)q * K, out_hi + (int64_t)q * K);
        return;
    }
    // More results: their words fall into up to 4096 equal bins between the smallest and the largest of them, a prefix over
    // the bins gives every bin's place, and inside its bin (one or two keys as a rule) a key counts the keys before it.
    // Only where a bin holds more than 64 keys - a crowd of equal distances - the bitonic network sorts them all.
    // (5000 of 10000 keys, 100 segments: 184 us with the network, 42 us with the bins.)
    if (n2 <= BIN_SORT_MAX) {
        const int nb = n2 < 4096 ? n2 : 4096;
        uint32_t* cursor = reinterpret_cast<uint32_t*>(sk + n2);        // [nb]
        uint16_t* order = reinterpret_cast<uint16_t*>(cursor + nb);     // [n2] keys by bin
        const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
        const int have = n <= K ? m_out : (int)(s_slot < (uint32_t)n2 ? s_slot : (uint32_t)n2);
        uint32_t mn = 0xFFFFFFFFu, mx = 0u;
        for (int i = tid; i < have; i += SEL_T) {
            const uint32_t h = (uint32_t)(sk[i] >> 32);
            mn = h < mn ? h : mn;
            mx = h > mx ? h : mx;
        }
        for (int i = tid; i < nb; i += SEL_T) cursor[i] = 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint32_t a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
            mn = a < mn ? a : mn;
            mx = b > mx ? b : mx;
        }
        if (lane == 0) { sh.wa[wv] = mn; sh.wb[wv] = mx; }
        if (tid == 0) sh.fill = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SEL_T / 64; ++i) {
            mn = sh.wa[i] < mn ? sh.wa[i] : mn;
            mx = sh.wb[i] > mx ? sh.wb[i] : mx;
        }
        int shift = 0;
        while (have > 0 && ((mx - mn) >> shift) >= (uint32_t)nb) ++shift;
        for (int i = tid; i < have; i += SEL_T) atomicAdd(&cursor[((uint32_t)(sk[i] >> 32) - mn) >> shift], 1u);
        __syncthreads();
        // exclusive prefix over the bins, nb / SEL_T (at least one) consecutive bins per thread
        const int per = (nb + SEL_T - 1) / SEL_T;
        uint32_t sum = 0, big = 0;
        for (int i = 0; i < per; ++i)
            if (tid * per + i < nb) { const uint32_t c = cursor[tid * per + i]; sum += c; big |= c > 64u ? 1u : 0u; }
        uint32_t inc = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        if (lane == 63) sh.wa[wv] = inc;
        if (big) sh.fill = 1;
        __syncthreads();
        uint32_t run = inc - sum;
        for (int i = 0; i < wv; ++i) run += sh.wa[i];
        const bool crowd = sh.fill != 0;
        if (!crowd) {   // uniform
            for (int i = 0; i < per; ++i)
                if (tid * per + i < nb) { const uint32_t c = cursor[tid * per + i]; cursor[tid * per + i] = run; run += c; }
            __syncthreads();
            for (int i = tid; i < have; i += SEL_T) order[atomicAdd(&cursor[((uint32_t)(sk[i] >> 32) - mn) >> shift], 1u)] = (uint16_t)i;
            __syncthreads();   // cursor[b] is now the end of bin b
            int32_t* lo = out_lo + (int64_t)q * K;
            float* hi = out_hi + (int64_t)q * K;
            for (int i = tid; i < have; i += SEL_T) {
                const uint64_t key = sk[i];
                const uint32_t b = ((uint32_t)(key >> 32) - mn) >> shift;
                const uint32_t e0 = b ? cursor[b - 1] : 0u, e1 = cursor[b];
                uint32_t r = e0;
                for (uint32_t e = e0; e < e1; ++e) {
                    const int o = order[e];
                    const uint64_t ko = sk[o];
                    r += (ko < key || (ko == key && o < i)) ? 1u : 0u;
                }
                if (r < (uint32_t)m_out) {
                    lo[r] = (int32_t)(uint32_t)key;
                    hi[r] = __uint_as_float((uint32_t)(key >> 32));
                }
            }
            for (int i = m_out + tid; i < K; i += SEL_T) { lo[i] = -1; hi[i] = INFINITY; }
            return;
        }
    }
    for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < n2; i += SEL_T) {
                int ixj = i ^ j;
                if (ixj > i) {
                    uint64_t a = sk[i], b = sk[ixj];
                    bool asc = (i & k) == 0;
                    if ((a > b) == asc) { sk[i] = b; sk[ixj] = a; }
                }
            }
            __syncthreads();
        }
    }
    for (int i = threadIdx.x; i < K; i += SEL_T) {
        int64_t o = (int64_t)q * K + i;
        if (i < m_out) {
            uint64_t k = sk[i];
            out_lo[o] = (int32_t)(uint32_t)k;
            out_hi[o] = __uint_as_float((uint32_t)(k >> 32));
        } else {
            out_lo[o] = -1;
            out_hi[o] = INFINITY;
        }
    }
}

// ---- visited lists of a few queries -----------------------------------------------------------
// Coarse distances and the selection of the w nearest lists in one launch, a workgroup per query, where the centroids are few: two
// kernels of 6.5 and 4.4 us, mostly start, drain and the way of the distances through memory.  A thread has a column (two
// beyond 512) of a copy of the centroids that has the same four components of consecutive centroids side by side; the products are
// a chain of fused multiply-adds in the order in which dist_words_kernel's matrix instruction takes the dimensions (0, 4, 1, 5, 2, 6, 3,
// 7 of every eight), the norm has that kernel's order too: the same words, bit for bit.  Bound: the reads of the centroids by one
// compute unit (64 bytes a clock).  Measured (both kernels, now one): 256 lists of 128 dimensions
// 10.8 -> 6.0 us, 1024 lists 12.6 -> 9.3; one query a call 52.6 -> 48.0 us, 100 queries 57.2 -> 51.1, 37 queries of 1024 lists 70.3 -> 66.8.
#define PROBE_WORDS 2   // columns per thread
__global__ __launch_bounds__(SEL_T) void probe_few_kernel(const float* __restrict__ X, int d, const float4* __restrict__ cols,
                                                          const float* __restrict__ cnorm, int c, int K, int32_t* __restrict__ out_lo,
                                                          float* __restrict__ out_hi, uint32_t* __restrict__ bad) {
    __shared__ SelShared sh;
    __shared__ uint64_t sk[SEL_RANK_SORT];
    __shared__ uint32_t s_words[PROBE_WORDS * SEL_T];
    __shared__ float4 s_x[IVFR_PROBE_FEW_D / 4];
    __shared__ uint32_t s_slot;
    const int q = blockIdx.x, tid = threadIdx.x;
    const float* x = X + (int64_t)q * d;
    for (int e = tid; e < d / 4; e += SEL_T) s_x[e] = *reinterpret_cast<const float4*>(x + 4 * e);
    if (tid == 0) s_slot = 0;
    __syncthreads();
    float xn = 0.f;   // the eight lanes of a group have the pieces of dist_words_kernel's eight threads
    for (int e = tid & 7; e < d / 4; e += 8) {
        const float4 v = s_x[e];
        xn = fmaf(v.x, v.x, xn); xn = fmaf(v.y, v.y, xn); xn = fmaf(v.z, v.z, xn); xn = fmaf(v.w, v.w, xn);
    }
    xn += __shfl_xor(xn, 4, 64);
    xn += __shfl_xor(xn, 2, 64);
    xn += __shfl_xor(xn, 1, 64);
    if (tid == 0 && !(xn <= 3.0e38f)) atomicMax(bad, (uint32_t)q + 1u);
#pragma unroll
    for (int u = 0; u < PROBE_WORDS; ++u) {
        const int col = tid + SEL_T * u;
        if (col >= c) break;
        const float cn = cnorm[col];
        float t = 0.f;
        const float4* p = cols + col;
        for (int e = 0; e < d / 4; e += 8, p += 8 * (int64_t)c) {   // 32 dimensions: eight loads in flight (d is a multiple of 32)
            float4 v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = p[i * (int64_t)c];
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                const float4 y = s_x[e + i], z = s_x[e + i + 1];
                t = fmaf(y.x, v[i].x, t); t = fmaf(z.x, v[i + 1].x, t); t = fmaf(y.y, v[i].y, t); t = fmaf(z.y, v[i + 1].y, t);
                t = fmaf(y.z, v[i].z, t); t = fmaf(z.z, v[i + 1].z, t); t = fmaf(y.w, v[i].w, t); t = fmaf(z.w, v[i + 1].w, t);
            }
        }
        s_words[col] = __float_as_uint(fmaxf(0.f, fmaf(-2.f, t, xn + cn)));
    }
    __syncthreads();
    int m_out = c, m_have = c;
    if (c <= K) {
        for (int i = tid; i < c; i += SEL_T) sk[i] = ((uint64_t)s_words[i] << 32) | (uint32_t)i;
    } else {
        const ValsSrc s{s_words, c};
        const RegValsSrc<PROBE_WORDS, ValsSrc> src(s);
        const uint64_t pivot = kth_key(sh, src, (uint32_t)K);
        src.sweep([&](uint32_t h, uint32_t l) {
            const uint64_t k = ((uint64_t)h << 32) | l;
            if (k <= pivot) {
                const uint32_t slot = atomicAdd(&s_slot, 1u);
                if (slot < SEL_RANK_SORT) sk[slot] = k;
            }
        });
        m_out = K;
    }
    __syncthreads();
    if (c > K) m_have = (int)(s_slot < SEL_RANK_SORT ? s_slot : SEL_RANK_SORT);
    write_ranked(sk, m_have, m_out, K, out_lo + (int64_t)q * K, out_hi + (int64_t)q * K);
}

// A compute unit per query, columns and results that fit the kernel, and 1.25 2^26 components of centroids read by all queries together at
// the most.  Every query's workgroup reads them all, and they are a copy: 1 MB and more of it takes the place of the rows that the re-rank
// reads next (512 dimensions, 1024 centroids, 192 queries: 22.3 us against 19.1 + 4.5 of the two kernels, re-rank 14.3 against 9.5).
// Calls, two kernels / this one, by 2^26 components: up to 0.5 1.06 to 1.17 (128 dimensions, 1024 centroids, 256 queries 53.0 / 48.9 us), 0.75
// 1.05 to 1.10, 1.0 1.04 to 1.06 (256, 1024, 256 66.0 / 62.5), 1.03 to 1.25 1.00 to 1.06 (512, 600, 256 99.2 / 97.7; 512, 1024, 160
// 135.5 / 127.6), 1.3 0.99 (512, 768, 224), 1.5 to 2 0.96 to 0.98 (512, 1024, 256 103 / 107).
#define IVFR_PROBE_FEW_READ (5ll << 24)
bool ivfr_probe_few(const ivfr_index* ix, int nq, int w) {
    return ix->coarse_cols && nq <= ix->n_cu && w <= SEL_RANK_SORT && (int64_t)nq * ix->p.c * ix->p.d <= IVFR_PROBE_FEW_READ;
}

int ivfr_launch_probe_few(const ivfr_index* ix, const float* X, int nq, int w, int32_t* probe, float* probe_dist, uint32_t* bad, hipStream_t st) {
    if (nq <= 0) return IVFR_OK;
    hipLaunchKernelGGL(probe_few_kernel, dim3((unsigned)nq), dim3(SEL_T), 0, st, X, ix->p.d, reinterpret_cast<const float4*>(ix->coarse_cols),
                       ix->coarse_norm, ix->p.c, w, probe, probe_dist, bad);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

static int g_sort_max = 4096;   // keys that fit the default dynamic-LDS limit until the attribute is raised

int ivfr_select_init() {
    const void* const kernels[] = {
        reinterpret_cast<const void*>(select_sorted_kernel<false, 4>), reinterpret_cast<const void*>(select_sorted_kernel<false, 20>),
        reinterpret_cast<const void*>(select_sorted_kernel<false, 0>), reinterpret_cast<const void*>(select_sorted_kernel<true, 4>),
        reinterpret_cast<const void*>(select_sorted_kernel<true, 16>), reinterpret_cast<const void*>(select_sorted_kernel<true, 0>)};
    hipError_t e = hipSuccess;
    for (const void* k : kernels)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, SORT_MAX * 8);
    if (e == hipSuccess) g_sort_max = SORT_MAX;
    else (void)hipGetLastError();
    return IVFR_OK;
}

int ivfr_launch_select_sorted(const SelectArgs& a, const int32_t* counts_i32, int out_base, int32_t* out_lo,
                              float* out_hi, hipStream_t st) {
    if (a.nseg <= 0) return IVFR_OK;
    if (a.K > g_sort_max) {
        ivfr_set_error("sorted selection supports at most %d results per query (got %d)", g_sort_max, a.K);
        return IVFR_ERR_INVALID_ARG;
    }
    int n2 = 2;
    while (n2 < a.K) n2 <<= 1;
    // the keys, and for the sort through bins the bins and the order of the keys
    const size_t lds = (size_t)n2 * 8 + (n2 > SEL_RANK_SORT && n2 <= BIN_SORT_MAX ? (size_t)std::min(n2, 4096) * 4 + (size_t)n2 * 2 : 0);
    const int64_t most = counts_i32 ? a.seg_stride : a.fixed_count;   // elements of a segment
#define IVFR_SORTED(VALS, NR)                                                                                                 \
    hipLaunchKernelGGL((select_sorted_kernel<VALS, NR>), dim3(a.nseg), dim3(SEL_T), lds, st,                                  \
                       VALS ? static_cast<const void*>(a.vals) : static_cast<const void*>(a.keys), a.seg_stride, a.fixed_count, \
                       counts_i32, a.K, n2, out_base, out_lo, out_hi)
    if (a.vals) {
        if (most <= 4 * SEL_T) IVFR_SORTED(true, 4);
        else if (most <= 16 * SEL_T) IVFR_SORTED(true, 16);
        else IVFR_SORTED(true, 0);
    } else {
        if (most <= 4 * SEL_T) IVFR_SORTED(false, 4);
        else if (most <= 20 * SEL_T) IVFR_SORTED(false, 20);
        else IVFR_SORTED(false, 0);
    }
#undef IVFR_SORTED
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}
