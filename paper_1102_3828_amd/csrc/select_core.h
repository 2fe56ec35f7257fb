// Exact selection by 64-bit key inside one workgroup of SEL_T threads: the device routines behind the kernels of
// select.hip, shared with the kernels that select from keys they hold in LDS.
//
// Method: the K-th smallest key (the pivot) is found by narrowing a range of distance words.  One sweep takes the
// minimum and maximum word of the segment; each further sweep histograms the words inside the current range
// into up to 1024 equal power-of-two bins (LDS atomics), a workgroup scan finds the bin that holds the K-th
// smallest, and the range shrinks to that bin.  Starting at the minimum and maximum skips the leading bits that
// all estimates of a query share, so one histogram sweep usually leaves a handful of keys; at most four are ever
// needed for 32 bits.  The few keys left in the range are gathered into LDS with their index words and ranked by
// counting.  Only if more than 512 keys share one distance word does the same narrowing go on over their index
// words.  A last sweep by the caller emits every key <= pivot.  For short-list records the index word (the
// vector id) is fetched from the record array only for the gathered keys.  When few keys are wanted out of many
// (K <= 256 of more than 4096: the bound from the sample, the visited lists, the final top-k) the range comes from
// one sweep instead of two: the K-th smallest of the 512 per-thread minima is an upper bound with few keys below it.
#pragma once

#include "ivfr_internal.h"

#define SEL_T 512
#define SEL_BINS (2 * SEL_T)
#define SEL_RC 512        // keys ranked by counting
#define SEL_RANK_SORT 256 // results sorted by counting rather than by a bitonic network

// One sweep of the workgroup over n elements: body(distance word, reference) for every element, thread tid taking
// elements tid, tid + SEL_T, ...  at(i, body) calls the body for an element already loaded by load(i).  Four loads are
// issued before the first is used (a sweep is a chain of load latencies otherwise: a segment of 50000 sampled
// estimates is 98 elements per thread).
template <class L, class A, class B>
__device__ __forceinline__ void sweep4(int64_t n, L load, A at, B body) {
    int64_t i = threadIdx.x;
    for (; i + 3 * SEL_T < n; i += 4 * SEL_T) {
        const auto a = load(i), b = load(i + SEL_T), c = load(i + 2 * SEL_T), d = load(i + 3 * SEL_T);
        at(a, i, body); at(b, i + SEL_T, body); at(c, i + 2 * SEL_T, body); at(d, i + 3 * SEL_T, body);
    }
    for (; i < n; i += SEL_T) at(load(i), i, body);
}

// Sources of a selection: n elements, each a distance word and a reference; lo(reference) is the index word that
// breaks ties and makes every key distinct.
struct ValsSrc {   // bare distance words; the element index is the low half of the key
    const uint32_t* v;
    int64_t n;
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return ref; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep4(n, [&](int64_t i) { return v[i]; }, [](uint32_t x, int64_t i, B& f) { f(x, (uint32_t)i); }, body);
    }
};
struct KeysSrc {   // 64-bit keys
    const uint64_t* v;
    int64_t n;
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return ref; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep4(n, [&](int64_t i) { return v[i]; }, [](uint64_t x, int64_t, B& f) { f((uint32_t)(x >> 32), (uint32_t)x); }, body);
    }
};
struct RecsSrc {   // (estimate bits, entry position); ids[pos * id_stride] is the id of the entry at position pos
    const uint2* v;
    int64_t n;
    const int32_t* ids;
    uint32_t id_stride;
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return (uint32_t)ids[(size_t)ref * id_stride]; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep4(n, [&](int64_t i) { return v[i]; }, [](const uint2& x, int64_t, B& f) { f(x.x, x.y); }, body);
    }
};

struct SelShared {
    uint32_t hist[SEL_BINS];
    uint64_t cand[SEL_RC];
    uint32_t wa[SEL_T / 64], wb[SEL_T / 64];
    uint32_t bin, need, cnt, fill;
    uint64_t pivot;
};

// Narrows [lo, hi] around the need-th smallest of the words that word(f) feeds to f (one call sweeps this thread's
// share of them), until at most `stop` words are left in the range or the range is a single value.  count is the
// number of words on entry and in the final range on return; need becomes the rank inside the final range.  All
// threads call.
template <class F>
__device__ void narrow_range(SelShared& sh, F word, uint32_t& lo, uint32_t& hi, uint32_t& need,
                             uint64_t& count, uint32_t stop = SEL_RC) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    word([&](uint32_t v) { mn = v < mn ? v : mn; mx = v > mx ? v : mx; });
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t a = __shfl_xor(mn, off, 64), b = __shfl_xor(mx, off, 64);
        mn = a < mn ? a : mn;
        mx = b > mx ? b : mx;
    }
    if (lane == 0) { sh.wa[wv] = mn; sh.wb[wv] = mx; }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SEL_T / 64; ++i) {
        mn = sh.wa[i] < mn ? sh.wa[i] : mn;
        mx = sh.wb[i] > mx ? sh.wb[i] : mx;
    }
    __syncthreads();   // wa is used again below
    lo = mn;
    hi = mx;
    // each pass leaves a span below 2^shift <= span / 512: four passes reach a single value from any 32-bit span
    for (int pass = 0; pass < 4 && count > stop && hi > lo; ++pass) {
        const uint32_t span = hi - lo;
        int shift = 0;
        while ((span >> shift) >= SEL_BINS) ++shift;
        for (int i = tid; i < SEL_BINS; i += SEL_T) sh.hist[i] = 0;
        __syncthreads();
        word([&](uint32_t v) {
            if (v >= lo && v <= hi) atomicAdd(&sh.hist[(v - lo) >> shift], 1u);
        });
        __syncthreads();
        // two bins per thread; inclusive scan over the workgroup
        const uint32_t a = sh.hist[2 * tid], b = sh.hist[2 * tid + 1];
        uint32_t inc = a + b;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(inc, off, 64);
            if (lane >= off) inc += o;
        }
        if (lane == 63) sh.wa[wv] = inc;
        __syncthreads();
        uint32_t exc = inc - (a + b);
        for (int i = 0; i < wv; ++i) exc += sh.wa[i];
        if (exc < need && need <= exc + a) {
            sh.bin = 2u * tid; sh.need = need - exc; sh.cnt = a;
        } else if (exc + a < need && need <= exc + a + b) {
            sh.bin = 2u * tid + 1u; sh.need = need - exc - a; sh.cnt = b;
        }
        __syncthreads();
        const uint32_t nlo = lo + (sh.bin << shift);
        const uint64_t nhi = (uint64_t)nlo + ((1ull << shift) - 1ull);
        hi = nhi < (uint64_t)hi ? (uint32_t)nhi : hi;
        lo = nlo;
        need = sh.need;
        count = sh.cnt;
        __syncthreads();
    }
}

// Returns the K-th smallest key of the segment (1 <= K <= n).  All threads must call; ends with a barrier.  sh: LDS scratch.
template <class S>
__device__ uint64_t kth_key(SelShared& sh, const S& s, uint32_t K) {
    const int tid = threadIdx.x;
    // keys with distance word in [lo, hi] (and, with by_index, index word in [lo2, hi2]) go to LDS; returns how many
    // there were (only the first SEL_RC are kept)
    auto gather = [&](uint32_t lo, uint32_t hi, bool by_index, uint32_t lo2, uint32_t hi2) -> uint32_t {
        if (tid == 0) sh.fill = 0;
        __syncthreads();
        s.sweep([&](uint32_t h, uint32_t pos) {
            if (h < lo || h > hi) return;
            const uint32_t l = s.lo(pos);
            if (by_index && (l < lo2 || l > hi2)) return;
            const uint32_t slot = atomicAdd(&sh.fill, 1u);
            if (slot < SEL_RC) sh.cand[slot] = ((uint64_t)h << 32) | l;
        });
        __syncthreads();
        const uint32_t got = sh.fill;
        __syncthreads();
        return got;
    };
    // the need-th smallest of the got <= SEL_RC gathered keys, by counting: the key with fewer than `need` keys below
    // it and at least `need` at or below it (equal keys agree)
    auto ranked = [&](uint32_t got, uint32_t need) -> uint64_t {
        if ((uint32_t)tid < got) {
            const uint64_t key = sh.cand[tid];
            uint32_t lt = 0, le = 0;
            for (uint32_t j = 0; j < got; ++j) {
                const uint64_t kj = sh.cand[j];
                lt += kj < key ? 1u : 0u;
                le += kj <= key ? 1u : 0u;
            }
            if (lt < need && need <= le) sh.pivot = key;
        }
        __syncthreads();
        const uint64_t pivot = sh.pivot;
        __syncthreads();
        return pivot;
    };
    if (K <= SEL_T / 2 && s.n > 8 * SEL_T) {
        // Few of many: every thread takes the minimum distance word of its strided share; the K-th smallest of those
        // SEL_T minima bounds the K-th smallest key from above, and at least K keys (a few more as a rule) lie at or
        // below it.  One sweep for the minima, one to gather those keys; the bound itself is found by narrowing over
        // the minima in LDS.
        uint32_t* mins = reinterpret_cast<uint32_t*>(sh.cand);
        uint32_t mn = 0xFFFFFFFFu;
        s.sweep([&](uint32_t h, uint32_t) { mn = h < mn ? h : mn; });
        mins[tid] = mn;
        __syncthreads();
        auto min_words = [&](auto f) { f(mins[tid]); };   // one minimum per thread
        uint32_t mlo = 0u, bound = 0xFFFFFFFFu, mneed = K;
        uint64_t mcount = SEL_T;
        narrow_range(sh, min_words, mlo, bound, mneed, mcount, 1u);   // ends with a barrier: mins may be overwritten
        const uint32_t got = gather(0u, bound, false, 0u, 0u);
        if (got <= SEL_RC) return ranked(got, K);
        // a crowd of equal distance words at the bound: the general way
    }
    uint32_t need = K;
    uint64_t count = (uint64_t)s.n;
    uint32_t lo = 0u, hi = 0xFFFFFFFFu, lo2 = 0u, hi2 = 0xFFFFFFFFu;
    bool by_index = false;
    if (count > SEL_RC) {
        auto dist_words = [&](auto f) { s.sweep([&](uint32_t h, uint32_t) { f(h); }); };
        narrow_range(sh, dist_words, lo, hi, need, count);
        if (count > SEL_RC) {   // lo == hi: that many keys share the distance word, their index words decide
            by_index = true;
            const uint32_t fixed = lo;
            auto index_words = [&](auto f) {
                s.sweep([&](uint32_t h, uint32_t pos) { if (h == fixed) f(s.lo(pos)); });
            };
            narrow_range(sh, index_words, lo2, hi2, need, count);
            if (count > SEL_RC) return ((uint64_t)fixed << 32) | lo2;   // equal keys throughout
        }
    }
    uint32_t got = gather(lo, hi, by_index, lo2, hi2);
    got = got < SEL_RC ? got : SEL_RC;
    return ranked(got, need);
}

// The m_have keys in sk (LDS, at most a few hundred) to their sorted places: every key counts the keys before it.  The
// first m_out of them are written to lo / hi (index word and distance), places m_out .. K - 1 get index -1 and
// distance +inf.  sk must be complete (barrier) before the call.
__device__ __forceinline__ void write_ranked(const uint64_t* sk, int m_have, int m_out, int K, int32_t* lo, float* hi) {
    for (int i = threadIdx.x; i < m_have; i += SEL_T) {
        const uint64_t key = sk[i];
        int r = 0;
        for (int j = 0; j < m_have; ++j) {
            const uint64_t kj = sk[j];
            r += (kj < key || (kj == key && j < i)) ? 1 : 0;
        }
        if (r < m_out) {
            lo[r] = (int32_t)(uint32_t)key;
            hi[r] = __uint_as_float((uint32_t)(key >> 32));
        }
    }
    for (int i = m_out + threadIdx.x; i < K; i += SEL_T) {
        lo[i] = -1;
        hi[i] = INFINITY;
    }
}
