// Steps a3 and a4 of a query in one workgroup: ADC scan of its visited lists (Eq. (5)) and the exact k' smallest estimates
// (gfx950).
//
// For visits of some 10^4 entries the general way - plan, sample, bound, scan, selection - is a chain of eight kernels that
// spend more time starting and draining than working, and writes every estimate to memory to read it back three times.
// Here a workgroup walks over its query's lists, one table in LDS at a time (the next one on its way in registers), and
// keeps what it finds in LDS:
//  - a visit that fits (twice CAP entries) keeps the bare estimates, entry e of the r-th list at its place in visit order;
//  - a longer one keeps records (estimate, position).  When fewer than a pass's worth of places are left, the k' smallest
//    so far are selected, the rest is dropped and the k'-th smallest becomes the bound for what follows.  Any k' entries at
//    or below a bound make it valid, so nothing can be missed, whatever the order of the entries; with entries in
//    no particular order k' ln(visit / CAP) of them pass the first bound.
// The selection is the one of select_core.h, on LDS.  Estimates are the sums of adc_sum in the scan kernels, the short-list
// is the one the general way finds.
#include "select_core.h"

#include <algorithm>

#define PASS (2 * SEL_T)   // entries per pass: two per thread

// bare estimates in visit order; an element's id is found through its list's place in the visit
struct PlacedSrc {
    const uint32_t* v;
    int64_t n;
    const uint32_t* pre;     // [w + 1] entries before each list
    const uint32_t* start;   // [w] position of each list
    int w;
    const int32_t* ids;
    uint32_t id_stride;
    __device__ __forceinline__ uint32_t position(uint32_t i) const {
        int lo = 0, hi = w;   // last list with pre[list] <= i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= i) lo = mid; else hi = mid;
        }
        return start[lo] + (i - pre[lo]);
    }
    __device__ __forceinline__ uint32_t lo(uint32_t i) const { return (uint32_t)ids[(size_t)position(i) * id_stride]; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep4(n, [&](int64_t i) { return v[i]; }, [](uint32_t x, int64_t i, B& f) { f(x, (uint32_t)i); }, body);
    }
};

template <int M>
__device__ __forceinline__ float table_sum(const float* lut, const uint32_t* wds) {   // the order of adc_sum
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int t = 0; t < M / 4; ++t) {
        const uint32_t v = wds[t];
        const float* L = lut + t * 4 * IVFR_KS;
        s0 += L[v & 0xff];
        s1 += L[IVFR_KS + ((v >> 8) & 0xff)];
        s0 += L[2 * IVFR_KS + ((v >> 16) & 0xff)];
        s1 += L[3 * IVFR_KS + (v >> 24)];
    }
    return s0 + s1;
}

template <int M, int CAP>
__global__ __launch_bounds__(SEL_T, M <= 16 ? 6 : 4) void scan_select_kernel(const uint8_t* __restrict__ codes, ScanSelectArgs a,
                                                            const uint32_t* __restrict__ list_start,
                                                            const uint32_t* __restrict__ list_len,
                                                            const int32_t* __restrict__ ids, uint32_t id_stride) {
    constexpr int T4 = M * IVFR_KS / 4;                      // 16-byte pieces of a table
    constexpr int TR = (T4 + SEL_T - 1) / SEL_T;             // per thread
    extern __shared__ float s_dyn[];
    float* const s_lut = s_dyn;                              // [M * 256]
    uint2* const s_rec = reinterpret_cast<uint2*>(s_lut + M * IVFR_KS);   // [CAP]
    uint32_t* const s_val = reinterpret_cast<uint32_t*>(s_rec);          // [2 CAP]
    uint32_t* const s_start = s_val + 2 * CAP;               // [w]
    uint32_t* const s_pre = s_start + a.w;                   // [w + 1]
    __shared__ SelShared sh;
    __shared__ uint32_t s_cnt[2][SEL_T / 64];
    __shared__ uint32_t s_fill;
    const int q = blockIdx.x, w = a.w;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the visited lists, and the entries before each
    for (int r = tid; r < w; r += SEL_T) {
        const int l = a.probe[(int64_t)q * w + r];
        s_start[r] = list_start[l];
        s_pre[r + 1] = list_len[l];
    }
    if (tid == 0) { s_pre[0] = 0; s_fill = 0; }
    __syncthreads();
    if (wave == 0) {
        uint32_t carry = 0;
        for (int r0 = 0; r0 < w; r0 += 64) {
            uint32_t v = r0 + lane < w ? s_pre[r0 + lane + 1] : 0u;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t o = __shfl_up(v, off, 64);
                if (lane >= off) v += o;
            }
            if (r0 + lane < w) s_pre[r0 + lane + 1] = carry + v;
            carry += __shfl(v, 63, 64);
        }
    }
    __syncthreads();
    const uint32_t total = s_pre[w];   // below 2^32: the launcher bounds w times the longest list
    const bool placed = total <= 2u * CAP;
    const uint32_t K = (uint32_t)a.kprime;
    uint32_t n = 0, parity = 0;        // records kept so far (uniform)
    float tau = INFINITY;
    float4 next[TR];
    auto fetch = [&](int r) {
        const PairTable pt = a.ts.pair((int64_t)q * w + r);
#pragma unroll
        for (int i = 0; i < TR; ++i)
            if (T4 % SEL_T == 0 || tid + SEL_T * i < T4) next[i] = pt.get4(4 * (tid + SEL_T * i));
    };
    auto next_list = [&](int r) { while (r < w && s_pre[r + 1] == s_pre[r]) ++r; return r; };   // skips empty lists
    int r = next_list(0);
    if (r < w) fetch(r);
    while (r < w) {
        __syncthreads();   // the previous table is no longer read
#pragma unroll
        for (int i = 0; i < TR; ++i)
            if (T4 % SEL_T == 0 || tid + SEL_T * i < T4) reinterpret_cast<float4*>(s_lut)[tid + SEL_T * i] = next[i];
        __syncthreads();
        const uint32_t start = s_start[r], pre = s_pre[r], len = s_pre[r + 1] - pre;
        const int rn = next_list(r + 1);
        if (rn < w) fetch(rn);
        for (uint32_t base = 0; base < len; base += PASS) {
            const uint32_t e = base + 2u * tid;
            const bool in0 = e < len, in1 = e + 1 < len;
            uint32_t wds[2][M / 4];
            if (in0) {   // lists start at multiples of 32 entries and end in padding: both codes are there to read
                const uint32_t* src = reinterpret_cast<const uint32_t*>(codes + ((uint64_t)start + e) * M);
#pragma unroll
                for (int t = 0; t < M / 4; ++t) { wds[0][t] = src[t]; wds[1][t] = src[M / 4 + t]; }
            } else {
#pragma unroll
                for (int t = 0; t < M / 4; ++t) wds[0][t] = wds[1][t] = 0;
            }
            const float e0 = table_sum<M>(s_lut, wds[0]), e1 = table_sum<M>(s_lut, wds[1]);
            if (placed) {
                if (in0) s_val[pre + e] = __float_as_uint(e0);
                if (in1) s_val[pre + e + 1] = __float_as_uint(e1);
                continue;
            }
            const bool k0 = in0 && e0 <= tau, k1 = in1 && e1 <= tau;
            const uint64_t m0 = __ballot(k0), m1 = __ballot(k1);
            const uint32_t n0 = __popcll(m0), n1 = __popcll(m1);
            if (lane == 0) s_cnt[parity][wave] = n0 + n1;
            __syncthreads();   // (a thread that is still reading the counts of the pass before last has not come here)
            uint32_t at = n, sum = 0;
#pragma unroll
            for (int i = 0; i < SEL_T / 64; ++i) {
                const uint32_t ci = s_cnt[parity][i];
                at += i < wave ? ci : 0u;
                sum += ci;
            }
            parity ^= 1u;
            const uint64_t below = (1ull << lane) - 1ull;
            if (k0) s_rec[at + __popcll(m0 & below)] = make_uint2(__float_as_uint(e0), start + e);
            if (k1) s_rec[at + n0 + __popcll(m1 & below)] = make_uint2(__float_as_uint(e1), start + e + 1);
            n += sum;
            if (n > CAP - PASS) {   // uniform; CAP - PASS >= k', so the k' smallest are among the n records
                __syncthreads();
                const uint64_t pivot = kth_key(sh, RecsSrc{s_rec, n, ids, id_stride}, K);
                const uint32_t p_hi = (uint32_t)(pivot >> 32), p_lo = (uint32_t)pivot;
                uint2 rec[CAP / SEL_T];
#pragma unroll
                for (int i = 0; i < CAP / SEL_T; ++i) rec[i] = (uint32_t)(tid + SEL_T * i) < n ? s_rec[tid + SEL_T * i] : make_uint2(0xFFFFFFFFu, 0u);
                if (tid == 0) s_fill = 0;
                __syncthreads();   // everything is in registers
#pragma unroll
                for (int i = 0; i < CAP / SEL_T; ++i) {
                    const bool keep = (uint32_t)(tid + SEL_T * i) < n &&
                                      (rec[i].x < p_hi || (rec[i].x == p_hi && (uint32_t)ids[(size_t)rec[i].y * id_stride] <= p_lo));
                    const uint64_t mk = __ballot(keep);
                    uint32_t first = 0;
                    if (lane == 0 && mk) first = atomicAdd(&s_fill, (uint32_t)__popcll(mk));
                    first = __builtin_amdgcn_readfirstlane(first);
                    const uint32_t slot = first + __popcll(mk & below);
                    if (keep && slot < K) s_rec[slot] = rec[i];
                }
                tau = __uint_as_float(p_hi);
                n = K;
                __syncthreads();
            }
        }
        r = rn;
    }
    __syncthreads();
    uint32_t* const op = a.out_pos + (int64_t)q * K;
    float* const oe = a.out_est ? a.out_est + (int64_t)q * K : nullptr;
    if (placed) n = total;
    if (tid == 0) {
        a.out_n[q] = (int32_t)(n < K ? n : K);
        atomicAdd(a.total, (unsigned long long)total);
        s_fill = 0;
    }
    uint64_t pivot = ~0ull;
    // (both selections end with a barrier; without one every element is taken and the barrier follows)
    if (placed) {
        const PlacedSrc s{s_val, n, s_pre, s_start, w, ids, id_stride};
        if (n > K) pivot = kth_key(sh, s, K);
        else __syncthreads();
        const uint32_t p_hi = (uint32_t)(pivot >> 32), p_lo = (uint32_t)pivot;
        const bool all = n <= K;
        for (uint32_t i0 = 0; i0 < n; i0 += SEL_T) {
            const uint32_t i = i0 + tid;
            const uint32_t est = i < n ? s_val[i] : 0u;
            const bool take = i < n && (all || est < p_hi || (est == p_hi && s.lo(i) <= p_lo));
            const uint64_t mk = __ballot(take);
            uint32_t first = 0;
            if (lane == 0 && mk) first = atomicAdd(&s_fill, (uint32_t)__popcll(mk));
            first = __builtin_amdgcn_readfirstlane(first);
            const uint32_t slot = first + __popcll(mk & ((1ull << lane) - 1ull));
            if (take && slot < K) { op[slot] = s.position(i); if (oe) oe[slot] = __uint_as_float(est); }
        }
    } else {
        const RecsSrc s{s_rec, n, ids, id_stride};
        if (n > K) pivot = kth_key(sh, s, K);
        else __syncthreads();
        const uint32_t p_hi = (uint32_t)(pivot >> 32), p_lo = (uint32_t)pivot;
        const bool all = n <= K;
        for (uint32_t i0 = 0; i0 < n; i0 += SEL_T) {
            const uint32_t i = i0 + tid;
            const uint2 rec = i < n ? s_rec[i] : make_uint2(0u, 0u);
            const bool take = i < n && (all || rec.x < p_hi || (rec.x == p_hi && s.lo(rec.y) <= p_lo));
            const uint64_t mk = __ballot(take);
            uint32_t first = 0;
            if (lane == 0 && mk) first = atomicAdd(&s_fill, (uint32_t)__popcll(mk));
            first = __builtin_amdgcn_readfirstlane(first);
            const uint32_t slot = first + __popcll(mk & ((1ull << lane) - 1ull));
            if (take && slot < K) { op[slot] = rec.y; if (oe) oe[slot] = __uint_as_float(rec.x); }
        }
    }
}

// Places for records: a pass and the short-list must fit; small ones leave room for more workgroups per compute unit.
static int record_places(int kprime) { return kprime <= 512 ? 2048 : (kprime <= 2048 ? 4096 : 8192); }

static size_t scan_select_lds(int m, int cap, int w) {
    return (size_t)m * IVFR_KS * sizeof(float) + (size_t)cap * sizeof(uint2) + (2 * (size_t)w + 1) * sizeof(uint32_t);
}

bool ivfr_scan_select_supported(const ivfr_index* ix, int w, int kprime) {
    return kprime <= 8192 - 2 * PASS && w <= 512 && (uint64_t)w * ix->max_len < 0xFFFFFFF0ull;
}

#define IVFR_SS_ALL(F) F(4, 2048) F(4, 4096) F(4, 8192) F(8, 2048) F(8, 4096) F(8, 8192) F(16, 2048) F(16, 4096) F(16, 8192) \
    F(32, 2048) F(32, 4096) F(32, 8192) F(64, 2048) F(64, 4096) F(64, 8192)

int ivfr_launch_scan_select(const ivfr_index* ix, const ScanSelectArgs& a, hipStream_t st) {
    if (a.nq <= 0) return IVFR_OK;
    const int m = ix->p.m, cap = record_places(a.kprime);
    const size_t lds = scan_select_lds(m, cap, a.w);
#define IVFR_SS(MM, CC)                                                                                                    \
    if (m == MM && cap == CC)                                                                                              \
        hipLaunchKernelGGL((scan_select_kernel<MM, CC>), dim3((unsigned)a.nq), dim3(SEL_T), lds, st, ix->codes, a, ix->list_start, \
                           ix->list_len, reinterpret_cast<const int32_t*>(ix->rec), (uint32_t)(ix->rec_stride / 4));
    IVFR_SS_ALL(IVFR_SS)
#undef IVFR_SS
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Dynamic LDS beyond 48 KB has to be allowed per kernel and device.
int ivfr_scan_select_init() {
#define IVFR_SS(MM, CC)                                                                                                 \
    IVFR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(scan_select_kernel<MM, CC>),                             \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)scan_select_lds(MM, CC, 512)));
    IVFR_SS_ALL(IVFR_SS)
#undef IVFR_SS
    return IVFR_OK;
}
