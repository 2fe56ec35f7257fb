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
// words.  A last sweep by the caller emits every key <= pivot.  The index words (for short-list records the vector
// ids, in memory) are looked at only where distance words tie at the pivot.  When few keys are wanted out of many
// (K <= 256 of more than 4096: the bound from the sample, the visited lists, the final top-k) the range comes from
// one sweep instead of two: the K-th smallest of the 512 per-thread minima is an upper bound with few keys below it.
//
// Bound: latency.  A selection is a chain of barriers, reductions over the lanes and LDS round trips, so those were cut: sums and
// prefixes over the lanes inside the vector unit instead of through LDS, three barriers a pass instead of five, segments that fit in
// registers read once, counts with several LDS reads in flight, no id read without a tie.  Measured (one MI355X): 500 keys, k = 50
// 15.3 -> 5.5 us; k' = 10000 of 12000 records, 1000 queries 92 -> 50 us; k = 100 of 10000 keys 43 -> 30 us; k = 100 of 1000 keys inside
// the re-rank 9.8 -> 3.6 us; 64 of 8192 24.6 -> 23.
#pragma once

#include "ivfr_internal.h"

#define SEL_T 512
#define SEL_BINS (2 * SEL_T)
#define SEL_BIN_BITS 10    // of 1024 bins
#define SEL_RC 512        // keys ranked by counting
#define SEL_STOP_REGS 96   // where a sweep costs little, one more is shorter than a count over this many keys
#define SEL_RANK_SORT 256 // results sorted by counting rather than by a bitonic network

// One sweep of the workgroup over n elements: body(distance word, reference) for every element, thread tid taking
// elements tid, tid + SEL_T, ...  at(i, body) calls the body for an element already loaded by load(i).  U loads are
// issued before the first is used: a sweep is a chain of load latencies otherwise (a segment of 50000 sampled
// estimates is 98 elements per thread).  Four are enough for the LDS; SEL_AHEAD for memory, whose latency one workgroup's 2 KB
// a load hide badly (the short-list of 10000 out of 78750 records 73 -> 61 us, the bound from some 40000 samples 46 -> 41).
#define SEL_AHEAD 12
template <int U, class L, class A, class B>
__device__ __forceinline__ void sweep_ahead(int64_t n, L load, A at, B body) {
    int64_t i = threadIdx.x;
    for (; i + (U - 1) * SEL_T < n; i += U * SEL_T) {
        decltype(load(i)) x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = load(i + u * SEL_T);
#pragma unroll
        for (int u = 0; u < U; ++u) at(x[u], i + u * SEL_T, body);
    }
    if constexpr (U > 4) {
        for (; i + 3 * SEL_T < n; i += 4 * SEL_T) {
            decltype(load(i)) x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = load(i + u * SEL_T);
#pragma unroll
            for (int u = 0; u < 4; ++u) at(x[u], i + u * SEL_T, body);
        }
    }
    for (; i < n; i += SEL_T) at(load(i), i, body);
}
template <class L, class A, class B>
__device__ __forceinline__ void sweep4(int64_t n, L load, A at, B body) { sweep_ahead<4>(n, load, at, body); }

// Sources of a selection: n elements, each a distance word and a reference; lo(reference) is the index word that
// breaks ties and makes every key distinct.
struct ValsSrc {   // bare distance words; the element index is the low half of the key
    const uint32_t* v;
    int64_t n;
    static constexpr uint32_t stop = SEL_RC;   // keys left in the range when the narrowing ends
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return ref; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep_ahead<SEL_AHEAD>(n, [&](int64_t i) { return v[i]; }, [](uint32_t x, int64_t i, B& f) { f(x, (uint32_t)i); }, body);
    }
};
struct KeysSrc {   // 64-bit keys
    const uint64_t* v;
    int64_t n;
    static constexpr uint32_t stop = SEL_RC;   // keys left in the range when the narrowing ends
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return ref; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep_ahead<SEL_AHEAD>(n, [&](int64_t i) { return v[i]; }, [](uint64_t x, int64_t, B& f) { f((uint32_t)(x >> 32), (uint32_t)x); }, body);
    }
};
template <int U>   // loads in flight
struct RecordsSrc {   // (estimate bits, entry position); ids[pos * id_stride] is the id of the entry at position pos
    const uint2* v;
    int64_t n;
    const int32_t* ids;
    uint32_t id_stride;
    static constexpr uint32_t stop = SEL_RC;
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return (uint32_t)ids[(size_t)ref * id_stride]; }
    __device__ __forceinline__ uint32_t ref(uint32_t i) const { return v[i].y; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        sweep_ahead<U>(n, [&](int64_t i) { return v[i]; }, [](const uint2& x, int64_t, B& f) { f(x.x, x.y); }, body);
    }
};
using RecsSrc = RecordsSrc<4>;   // in LDS
using MemRecsSrc = RecordsSrc<SEL_AHEAD>;

// Records or bare words of a segment that fits the workgroup's registers, NR per thread: loaded once, every sweep after that is
// arithmetic.  (The selection of k' = 10000 from some 12000 records of a query used to read them from L2 four times.)
template <int NR>
struct RegRecsSrc {
    uint2 r[NR];
    int64_t n;
    const int32_t* ids;
    uint32_t id_stride;
    static constexpr uint32_t stop = SEL_STOP_REGS;
    __device__ __forceinline__ void load(const uint2* v) {
#pragma unroll
        for (int i = 0; i < NR; ++i) r[i] = (int64_t)threadIdx.x + SEL_T * i < n ? v[threadIdx.x + SEL_T * i] : make_uint2(0u, 0u);
    }
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return (uint32_t)ids[(size_t)ref * id_stride]; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if ((int64_t)threadIdx.x + SEL_T * i < n) body(r[i].x, r[i].y);
    }
};
template <int NR, class S>   // words of a source whose references are the element numbers
struct RegValsSrc {
    uint32_t v[NR];
    int64_t n;
    const S& base;
    static constexpr uint32_t stop = SEL_STOP_REGS;
    __device__ __forceinline__ RegValsSrc(const S& b) : n(b.n), base(b) {
#pragma unroll
        for (int i = 0; i < NR; ++i) v[i] = (int64_t)threadIdx.x + SEL_T * i < n ? b.v[threadIdx.x + SEL_T * i] : 0u;
    }
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return base.lo(ref); }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if ((int64_t)threadIdx.x + SEL_T * i < n) body(v[i], threadIdx.x + SEL_T * i);
    }
};
template <int NR>
struct RegKeysSrc {   // 64-bit keys
    uint64_t v[NR];
    int64_t n;
    static constexpr uint32_t stop = SEL_STOP_REGS;
    __device__ __forceinline__ RegKeysSrc(const KeysSrc& b) : n(b.n) {
#pragma unroll
        for (int i = 0; i < NR; ++i) v[i] = (int64_t)threadIdx.x + SEL_T * i < n ? b.v[threadIdx.x + SEL_T * i] : 0ull;
    }
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return ref; }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if ((int64_t)threadIdx.x + SEL_T * i < n) body((uint32_t)(v[i] >> 32), (uint32_t)v[i]);
    }
};

// Reductions and prefixes over the 64 lanes by moves between lanes inside the vector unit: a step takes a few cycles, where one
// through the LDS (__shfl) takes its latency, and a selection is a chain of a dozen of them.
template <class F>
__device__ __forceinline__ uint32_t wave_fold(uint32_t v, uint32_t identity, F f) {   // prefix over the lanes; lane 63 holds the whole
#define SEL_DPP(CTRL, ROWS) v = f(v, (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)v, CTRL, ROWS, 0xf, false))
    SEL_DPP(0x111, 0xf); SEL_DPP(0x112, 0xf); SEL_DPP(0x114, 0xf); SEL_DPP(0x118, 0xf);   // inside rows of sixteen
    SEL_DPP(0x142, 0xa); SEL_DPP(0x143, 0xc);                                             // over the rows
#undef SEL_DPP
    return v;
}
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) { return wave_fold(v, 0u, [](uint32_t a, uint32_t b) { return a + b; }); }

struct alignas(16) SelShared {
    uint32_t hist[SEL_BINS];
    uint32_t word[SEL_RC], low[SEL_RC];   // gathered keys
    uint32_t wa[SEL_T / 64], wb[SEL_T / 64], wc[SEL_T / 64];
    uint32_t bin, need, cnt, fill, tie;
    uint64_t pivot;
};

// Narrows [lo, hi] around the need-th smallest of the words that word(f) feeds to f (one call sweeps this thread's
// share of them), until at most `stop` words are left in the range or the range is a single value.  count is the
// number of words on entry and in the final range on return; need becomes the rank inside the final range.  All
// threads call.
template <class F>
__device__ __forceinline__ void narrow_range(SelShared& sh, F word, uint32_t& lo, uint32_t& hi, uint32_t& need,
                                             uint64_t& count, uint32_t stop = SEL_RC) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    sh.hist[2 * tid] = 0;
    sh.hist[2 * tid + 1] = 0;
    word([&](uint32_t v) { mn = v < mn ? v : mn; mx = v > mx ? v : mx; });
    mn = wave_fold(mn, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
    mx = wave_fold(mx, 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
    if (lane == 63) { sh.wa[wv] = mn; sh.wb[wv] = mx; }
    __syncthreads();
    mn = sh.wa[0];
    mx = sh.wb[0];
#pragma unroll
    for (int i = 1; i < SEL_T / 64; ++i) {
        mn = sh.wa[i] < mn ? sh.wa[i] : mn;
        mx = sh.wb[i] > mx ? sh.wb[i] : mx;
    }
    lo = mn;
    hi = mx;
    // each pass leaves a span below 2^shift <= span / 512: four passes reach a single value from any 32-bit span
    for (int pass = 0; pass < 4 && count > stop && hi > lo; ++pass) {
        const uint32_t span = hi - lo;
        const int bits = 32 - __clz((int)span);                     // span > 0
        const int shift = bits > SEL_BIN_BITS ? bits - SEL_BIN_BITS : 0;
        word([&](uint32_t v) {
            if (v >= lo && v <= hi) atomicAdd(&sh.hist[(v - lo) >> shift], 1u);
        });
        __syncthreads();
        // two bins per thread, left at zero for the next pass; inclusive scan over the workgroup
        const uint32_t a = sh.hist[2 * tid], b = sh.hist[2 * tid + 1];
        sh.hist[2 * tid] = 0;
        sh.hist[2 * tid + 1] = 0;
        const uint32_t inc = wave_prefix(a + b);
        if (lane == 63) sh.wc[wv] = inc;
        __syncthreads();
        uint32_t exc = inc - (a + b);
#pragma unroll
        for (int i = 0; i < SEL_T / 64; ++i) exc += i < wv ? sh.wc[i] : 0u;
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
    }
}

// Returns the K-th smallest key of the segment (1 <= K <= n), or, where exactly K keys have a distance word up to that key's
// word, the largest key with that word (index word 0xFFFFFFFF): either way exactly the K smallest keys lie at or below what is
// returned (more only where keys are equal).  The index words, for short-list records a random read of memory, are only looked
// at where words tie there.  All threads must call; ends with a barrier.  sh: LDS scratch.
template <class S>
__device__ __forceinline__ uint64_t kth_key(SelShared& sh, const S& s, uint32_t K) {
    const int tid = threadIdx.x;
    // keys with distance word in [lo, hi] (and, with by_index, index word in [lo2, hi2]) go to LDS, words and references (with
    // by_index: index words); returns how many there were (only the first SEL_RC are kept)
    auto gather = [&](uint32_t lo, uint32_t hi, bool by_index, uint32_t lo2, uint32_t hi2) -> uint32_t {
        if (tid == 0) sh.fill = 0;
        __syncthreads();
        s.sweep([&](uint32_t h, uint32_t ref) {
            if (h < lo || h > hi) return;
            if (by_index) {
                ref = s.lo(ref);
                if (ref < lo2 || ref > hi2) return;
            }
            const uint32_t slot = atomicAdd(&sh.fill, 1u);
            if (slot < SEL_RC) { sh.word[slot] = h; sh.low[slot] = ref; }
        });
        __syncthreads();
        return sh.fill;
    };
    // the need-th smallest of the got <= SEL_RC gathered keys, by counting: the word with fewer than `need` words below
    // it and at least `need` at or below it, then, if not all of the latter are wanted, the same over their index words
    auto ranked = [&](uint32_t got, uint32_t need, bool by_index) -> uint64_t {
        if (tid < 4 && got + tid < SEL_RC) sh.word[got + tid] = 0xFFFFFFFFu;   // the count below goes four at a time
        __syncthreads();
        if ((uint32_t)tid < got) {
            const uint32_t word = sh.word[tid];
            uint32_t lt = 0, le = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < got; j += 4) {
                const uint4 v = *reinterpret_cast<const uint4*>(sh.word + j);
                lt += (v.x < word ? 1u : 0u) + (v.y < word ? 1u : 0u) + (v.z < word ? 1u : 0u) + (v.w < word ? 1u : 0u);
                le += (v.x <= word ? 1u : 0u) + (v.y <= word ? 1u : 0u) + (v.z <= word ? 1u : 0u) + (v.w <= word ? 1u : 0u);
            }
            // (the words behind the last only add to le where `word` is the largest there is: the index words decide then)
            if (lt < need && need <= le) { sh.pivot = word; sh.need = need - lt; sh.tie = by_index || le != need ? 1u : 0u; }
        }
        __syncthreads();
        const uint32_t word = (uint32_t)sh.pivot;
        if (!sh.tie) {   // uniform
            __syncthreads();
            return ((uint64_t)word << 32) | 0xFFFFFFFFu;
        }
        need = sh.need;
        const bool mine = (uint32_t)tid < got && sh.word[tid] == word;
        uint32_t low = 0;
        if (mine) {
            low = by_index ? sh.low[tid] : s.lo(sh.low[tid]);
            sh.low[tid] = low;
        }
        __syncthreads();   // (pivot, need and tie have been read)
        if (mine) {
            uint32_t lt = 0, le = 0;
            for (uint32_t j = 0; j < got; ++j) {
                const bool eq = sh.word[j] == word;
                lt += eq && sh.low[j] < low ? 1u : 0u;
                le += eq && sh.low[j] <= low ? 1u : 0u;
            }
            if (lt < need && need <= le) sh.pivot = ((uint64_t)word << 32) | low;
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
        // the minima.
        uint32_t mn = 0xFFFFFFFFu;
        s.sweep([&](uint32_t h, uint32_t) { mn = h < mn ? h : mn; });
        auto min_words = [&](auto f) { f(mn); };   // one minimum per thread
        uint32_t mlo = 0u, bound = 0xFFFFFFFFu, mneed = K;
        uint64_t mcount = SEL_T;
        narrow_range(sh, min_words, mlo, bound, mneed, mcount, 1u);
        const uint32_t got = gather(0u, bound, false, 0u, 0u);
        if (got <= SEL_RC) return ranked(got, K, false);
        // a crowd of equal distance words at the bound: the general way
    }
    uint32_t need = K;
    uint64_t count = (uint64_t)s.n;
    uint32_t lo = 0u, hi = 0xFFFFFFFFu, lo2 = 0u, hi2 = 0xFFFFFFFFu;
    bool by_index = false;
    if (count > S::stop) {
        auto dist_words = [&](auto f) { s.sweep([&](uint32_t h, uint32_t) { f(h); }); };
        narrow_range(sh, dist_words, lo, hi, need, count, S::stop);
        if (count > SEL_RC) {   // lo == hi: that many keys share the distance word, their index words decide
            by_index = true;
            const uint32_t fixed = lo;
            auto index_words = [&](auto f) {
                s.sweep([&](uint32_t h, uint32_t pos) { if (h == fixed) f(s.lo(pos)); });
            };
            __syncthreads();   // the last pass's result has been read
            narrow_range(sh, index_words, lo2, hi2, need, count);
            if (count > SEL_RC) {   // equal keys throughout
                __syncthreads();
                return ((uint64_t)fixed << 32) | lo2;
            }
        }
    }
    uint32_t got = gather(lo, hi, by_index, lo2, hi2);
    got = got < SEL_RC ? got : SEL_RC;
    return ranked(got, need, by_index);
}

// Whether a key at or below the pivot: the index word is only fetched where the distance words are equal and the pivot is a key
template <class L>
__device__ __forceinline__ bool within(uint32_t word, uint64_t pivot, L low) {
    const uint32_t p_hi = (uint32_t)(pivot >> 32), p_lo = (uint32_t)pivot;
    return word < p_hi || (word == p_hi && (p_lo == 0xFFFFFFFFu || low() <= p_lo));
}

// The m_have keys in sk (LDS, at most a few hundred) to their sorted places: every key counts the keys before it, four lanes
// a key, eight reads in flight (one thread a key and one read at a time took 6 us for 100 keys: a chain of LDS latencies).  The
// first m_out of them are written to lo / hi (index word and distance), places m_out .. K - 1 get index -1 and
// distance +inf.  sk must be complete (barrier) before the call.
__device__ __forceinline__ void write_ranked(const uint64_t* sk, int m_have, int m_out, int K, int32_t* lo, float* hi) {
    const int part = threadIdx.x & 3;
    for (int i0 = 0; i0 < m_have; i0 += SEL_T / 4) {
        const int i = i0 + (int)(threadIdx.x >> 2);
        const uint64_t key = sk[i < m_have ? i : 0];
        int r = 0;
#pragma unroll 8
        for (int j = part; j < m_have; j += 4) {
            const uint64_t kj = sk[j];
            r += (kj < key || (kj == key && j < i)) ? 1 : 0;
        }
        r += __builtin_amdgcn_update_dpp(0, r, 0xB1, 0xf, 0xf, false);   // over the four lanes
        r += __builtin_amdgcn_update_dpp(0, r, 0x4E, 0xf, 0xf, false);
        if (part == 0 && i < m_have && r < m_out) {
            lo[r] = (int32_t)(uint32_t)key;
            hi[r] = __uint_as_float((uint32_t)(key >> 32));
        }
    }
    for (int i = m_out + threadIdx.x; i < K; i += SEL_T) {
        lo[i] = -1;
        hi[i] = INFINITY;
    }
}
