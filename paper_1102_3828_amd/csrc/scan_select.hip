// Steps a3 and a4 of a query in one workgroup: ADC scan of its visited lists (Eq. (5)) and the exact k' smallest estimates
// (gfx950).
//
// For visits of some 10^4 entries the general way - plan, sample, bound, scan, selection - is a chain of eight kernels that
// spend more time starting and draining than working, and writes every estimate to memory to read it back three times.
// Here a workgroup walks over its query's lists, the tables of several in LDS at a time (the next ones on their way in
// registers, or computed by the workgroup), and keeps what it finds in LDS:
//  - a visit that fits (twice CAP entries) keeps the bare estimates, entry e of the r-th list at its place in visit order;
//  - a longer one keeps records (estimate, position).  When fewer than a pass's worth of places are left, the k' smallest
//    so far are selected, the rest is dropped and the k'-th smallest becomes the bound for what follows.  Any k' entries at
//    or below a bound make it valid, so nothing can be missed, whatever the order of the entries; with entries in
//    no particular order k' ln(visit / CAP) of them pass the first bound.
// The selection is the one of select_core.h, on LDS.  Estimates are the sums of adc_sum in the scan kernels, the short-list
// is the one the general way finds.
#include "select_core.h"

#include <algorithm>

#define PASS (4 * SEL_T)   // entries per pass at the most: two slots of two per thread

// bare estimates in visit order; an element's id is found through its list's place in the visit
struct PlacedSrc {
    const uint32_t* v;
    int64_t n;
    const uint32_t* pre;     // [w + 1] entries before each list that was scanned
    const uint32_t* start;   // [w] position of each of them
    int w;
    const int32_t* ids;
    uint32_t id_stride;
    static constexpr uint32_t stop = SEL_STOP_REGS;
    __device__ __forceinline__ uint32_t position(uint32_t i) const {
        int lo = 0, hi = w;   // last list with pre[list] <= i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= i) lo = mid; else hi = mid;
        }
        return start[lo] + (i - pre[lo]);
    }
    __device__ __forceinline__ uint32_t lo(uint32_t i) const { return (uint32_t)ids[(size_t)position(i) * id_stride]; }
    __device__ __forceinline__ uint32_t ref(uint32_t i) const { return i; }   // of element i
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

// Look-up tables of G lists of a query (Eq. (5)), computed by the workgroup: the entries of lut_mfma_kernel (the matrix
// instruction accumulates like a chain of fused multiply-adds, here in the order in which it takes the dimensions: 0, 4,
// 1, 5, 2, 6, 3, 7 of every eight) or of lut_direct_kernel, bit for bit.  A wavefront works on one sub-quantizer at a time, or on
// half of one: I of its values per lane, so that a residual read from LDS (the same address in all lanes: what such a read costs
// is the way of its 16 bytes to 64 lanes) serves I of them.  The codebook is read from a copy that has the same four components of
// consecutive values side by side (pq_cols): a load is 1 KB in a row, where rows of 64 bytes cost four times the address cycles.
// Measured (8 lists for one query alone): 8.2 -> 5.1 us.
template <int M, int G, int I>
__device__ __forceinline__ void own_tables(const ScanSelectArgs& a, int q, const int (&lists)[G], float* s_res, float* s_lut) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, d = a.d, dsub = d / M;
    constexpr int PARTS = 4 / I, UNITS = M * PARTS;   // (sub-quantizer, 64 I of its values), dealt to the wavefronts in turn
    static_assert(UNITS % (SEL_T / 64) == 0, "every wavefront has as many");
    float4 u[I], v[I];   // components e .. e + 3 and e + 4 .. e + 7 of the values
    auto load_values = [&](int unit, int e) {
        const float4* p = a.pq_cols + (unit / PARTS * (dsub / 4) + e / 4) * IVFR_KS + unit % PARTS * (64 * I) + lane;
#pragma unroll
        for (int x = 0; x < I; ++x) { u[x] = p[64 * x]; v[x] = p[IVFR_KS + 64 * x]; }
    };
    // the residuals, on their way while the previous tables may still be read
    constexpr int RR = (G * 512 / 4 + SEL_T - 1) / SEL_T;   // pieces per thread, d <= 512
    float4 res[RR];
#pragma unroll
    for (int i = 0; i < RR; ++i) {
        const int piece = tid + SEL_T * i, g = piece / (d / 4), e = 4 * (piece % (d / 4));
        res[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        int l = -1;
#pragma unroll
        for (int x = 0; x < G; ++x) l = g == x ? lists[x] : l;
        if (l >= 0) {
            const float4 x = *reinterpret_cast<const float4*>(a.queries + (int64_t)q * d + e);
            const float4 c = *reinterpret_cast<const float4*>(a.coarse + (int64_t)l * d + e);
            res[i] = make_float4(x.x - c.x, x.y - c.y, x.z - c.z, x.w - c.w);
        }
    }
    if (dsub % 8 == 0) load_values(wave, 0);
    __syncthreads();   // the previous tables and residuals are no longer read
#pragma unroll
    for (int i = 0; i < RR; ++i)
        if (tid + SEL_T * i < G * (d / 4)) reinterpret_cast<float4*>(s_res)[tid + SEL_T * i] = res[i];
    __syncthreads();
    if (dsub % 8 == 0) {
        for (int unit = wave; unit < UNITS; unit += SEL_T / 64) {
            const int j = unit / PARTS;
            // ||r^j||^2 of list g in lane g
            float rn = 0.f;
            for (int e = 0; e < dsub; e += 8) {
                const float4* r = reinterpret_cast<const float4*>(s_res + (lane % G) * d + j * dsub + e);
                const float4 y = r[0], z = r[1];
                rn = fmaf(y.x, y.x, rn); rn = fmaf(y.y, y.y, rn); rn = fmaf(y.z, y.z, rn); rn = fmaf(y.w, y.w, rn);
                rn = fmaf(z.x, z.x, rn); rn = fmaf(z.y, z.y, rn); rn = fmaf(z.z, z.z, rn); rn = fmaf(z.w, z.w, rn);
            }
            float acc[I][G];
#pragma unroll
            for (int x = 0; x < I; ++x)
#pragma unroll
                for (int g = 0; g < G; ++g) acc[x][g] = 0.f;
            for (int e = 0; e < dsub; e += 8) {
                float4 cu[I], cv[I];
#pragma unroll
                for (int x = 0; x < I; ++x) { cu[x] = u[x]; cv[x] = v[x]; }
                if (e + 8 < dsub) load_values(unit, e + 8);
                else if (unit + SEL_T / 64 < UNITS) load_values(unit + SEL_T / 64, 0);
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    const float4 y = *reinterpret_cast<const float4*>(s_res + g * d + j * dsub + e);
                    const float4 z = *reinterpret_cast<const float4*>(s_res + g * d + j * dsub + e + 4);
#pragma unroll
                    for (int x = 0; x < I; ++x) {
                        float t = acc[x][g];
                        t = fmaf(y.x, cu[x].x, t); t = fmaf(z.x, cv[x].x, t); t = fmaf(y.y, cu[x].y, t); t = fmaf(z.y, cv[x].y, t);
                        t = fmaf(y.z, cu[x].z, t); t = fmaf(z.z, cv[x].z, t); t = fmaf(y.w, cu[x].w, t); t = fmaf(z.w, cv[x].w, t);
                        acc[x][g] = t;
                    }
                }
            }
#pragma unroll
            for (int x = 0; x < I; ++x) {
                const int k = j * IVFR_KS + unit % PARTS * (64 * I) + 64 * x + lane;
                const float pn = a.pq_norm[k];
#pragma unroll
                for (int g = 0; g < G; ++g)
                    s_lut[g * (M * IVFR_KS) + k] = fmaxf(0.f, fmaf(-2.f, acc[x][g], __uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(rn), g)) + pn));
            }
        }
    } else {   // 1, 2 or 4 dimensions per sub-quantizer
        for (int i = tid; i < M * IVFR_KS; i += SEL_T) {
            const int j = i >> 8;
            float p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = e < dsub ? a.pq[(int64_t)i * dsub + e] : 0.f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float s = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < dsub) { const float df = s_res[g * d + j * dsub + e] - p[e]; s = fmaf(df, df, s); }
                s_lut[g * (M * IVFR_KS) + i] = s;
            }
        }
    }
}

// GM: KB of tables in LDS at a time (a multiple of M, or M where that is larger): the tables of G lists, whose entries are
// scanned as one stream, so that short lists and the ends of long ones do not leave lanes idle.
// TAB: where the tables come from: loaded whole, the sum of two loaded terms (split tables), or
// OWN: the workgroup computes the tables itself instead of loading them.  It can then also leave lists out: given a lower bound on
// the estimates of every pair (a.low, from the pair-bound kernel), a group takes the next G lists that may hold something within
// the k' smallest so far: the bound of the last cut, or the largest estimate while k' entries or more have been met and not cut.
enum { TAB_LOADED = 0, TAB_SPLIT = 1, TAB_OWN = 2 };
template <int M, int GM, int CAP, int TAB>
__global__ __launch_bounds__(SEL_T, CAP > 4096 ? 2 : 4) void scan_select_kernel(
    const uint8_t* __restrict__ codes, ScanSelectArgs a, const uint32_t* __restrict__ list_start,
    const uint32_t* __restrict__ list_len, const int32_t* __restrict__ ids, uint32_t id_stride) {
    constexpr bool OWN = TAB == TAB_OWN, split = TAB == TAB_SPLIT;
    constexpr int G = GM / M > 0 ? GM / M : 1;
    constexpr int T4 = M * IVFR_KS / 4;                      // 16-byte pieces of a table
    constexpr int TR = (G * T4 + SEL_T - 1) / SEL_T;         // pieces of a group's tables per thread
    constexpr bool AHEAD = M <= 16;                          // a pass's codes are loaded one pass ahead
    constexpr int U = M <= 16 ? 2 : 1;                       // slots per thread and pass
    // (16-byte reads: without the alignment the array starts right behind the static ones, and they take four times as long)
    extern __shared__ __align__(16) float s_dyn[];
    float* const s_lut = s_dyn;                              // [G][M * 256]
    uint2* const s_rec = reinterpret_cast<uint2*>(s_lut + G * M * IVFR_KS);   // [CAP]
    uint32_t* const s_val = reinterpret_cast<uint32_t*>(s_rec);          // [2 CAP]
    const int q = blockIdx.x, w = a.w;
    uint32_t* const s_list = s_val + 2 * CAP;                // [w] the visited lists: number, start, entries, lower bound
    uint32_t* const s_start = s_list + w;                    // [w]
    uint32_t* const s_len = s_start + w;                     // [w]
    float* const s_low = reinterpret_cast<float*>(s_len + w);   // [w]
    uint32_t* const s_first = reinterpret_cast<uint32_t*>(s_low + w);   // [w] those that were scanned, in order: start,
    uint32_t* const s_pre = s_first + w;                     // [w + 1] and entries before each
    float* const s_res = s_dyn + ((size_t)(reinterpret_cast<float*>(s_pre + w + 1) - s_dyn) + 3) / 4 * 4;   // OWN: residuals [G][d], 16-byte aligned
    __shared__ SelShared sh;
    __shared__ uint32_t s_fill, s_cut;   // records kept so far; of a cut to the k' best
    __shared__ uint32_t s_total;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int r = tid; r < w; r += SEL_T) {
        const int l = a.probe[(int64_t)q * w + r];
        s_list[r] = (uint32_t)l;
        s_start[r] = list_start[l];
        s_len[r] = list_len[l];
        s_low[r] = OWN && a.low ? a.low[(int64_t)q * w + r] : 0.f;
    }
    if (tid == 0) s_fill = 0;
    __syncthreads();
    if (wave == 0) {
        uint32_t sum = 0;
        if constexpr (OWN) {
            for (int r = lane; r < w; r += 64) sum += s_len[r];
            sum = wave_prefix(sum);
        } else {   // every list is scanned, in order
            for (int r0 = 0; r0 < w; r0 += 64) {
                const uint32_t v = r0 + lane < w ? s_len[r0 + lane] : 0u, inc = wave_prefix(v);
                if (r0 + lane < w) s_pre[r0 + lane] = sum + inc - v;
                sum += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
            }
            if (lane == 0) s_pre[w] = sum;
        }
        if (lane == 63) s_total = sum;
    }
    __syncthreads();
    const uint32_t total = s_total;   // below 2^32: the launcher bounds w times the longest list
    if (tid == 0) atomicAdd(a.counter, (unsigned long long)total);   // nothing waits for it; the re-rank tells the host the sum
    const bool placed = total <= 2u * CAP;
    const uint32_t K = (uint32_t)a.kprime;
    // Records: at most n_top are kept now (uniform).  Waves reserve places with an LDS atomic and run on; the true count is
    // only looked at when another pass might not fit.
    uint32_t n_top = 0;
    float tau = INFINITY, largest = 0.f;   // largest: of this thread's estimates
    // A group: the ranks (by distance) of up to G lists that are not empty and may hold something at or below `bound`, the next
    // ones from rank `next`, which moves behind them.  Uniform.
    struct Group {   // len: 0 without a list
        int r[OWN ? G : 1];   // loaded tables: the first of consecutive ones
        uint32_t len[G];
        int n;
        __device__ __forceinline__ int rank(int x) const { return OWN ? r[OWN ? x : 0] : (x < n ? r[0] + x : -1); }
    };
    int next = 0;
    auto form = [&](float bound) {
        Group g;
        g.n = 0;
        if constexpr (!OWN) {   // the next G lists as they come
#pragma unroll
            for (int x = 0; x < G; ++x) {
                if (next + x < w) g.n = x + 1;
                g.len[x] = __builtin_amdgcn_readfirstlane(next + x < w ? s_len[next + x] : 0u);
            }
            g.r[0] = next;
            next += G;
            return g;
        }
        int base = next & ~63;
        auto may = [&](int from) { return __ballot(from + lane < w && s_len[from + lane < w ? from + lane : 0] > 0 && !(s_low[from + lane < w ? from + lane : 0] > bound)); };
        uint64_t mask = next < w ? may(base) & (~0ull << (next & 63)) : 0ull;
#pragma unroll
        for (int x = 0; x < G; ++x) {
            while (!mask && base + 64 < w) { base += 64; mask = may(base); }
            g.r[OWN ? x : 0] = mask ? base + __builtin_ctzll(mask) : -1;
            if (mask) { g.n = x + 1; next = g.rank(x) + 1; mask &= mask - 1; }
            else next = w;
            g.len[x] = __builtin_amdgcn_readfirstlane(g.rank(x) >= 0 ? s_len[g.rank(x)] : 0u);
        }
        return g;
    };
    // The next group's tables on their way.  Split tables are summed when they go to LDS: summed on arrival, the wait for the list's term
    // would stand before the scan that hides it.  A thread's pieces of the query's term are the same for every list.  (501 queries, 13 lists
    // of 777 entries, m = 16: 84 -> 75 us, and 67 with the wavefronts without a slot left out below; 700 queries, 24 lists of 100: the
    // call 1.26 times as fast at m = 16 and 8, 1.12 at m = 4.  With 16 KB of tables at m = 16 and 32 that spills 4 of the 128 registers of
    // two workgroups a compute unit, 20 bytes a lane, in these figures.)
    constexpr int QR = T4 > SEL_T ? T4 / SEL_T : 1;          // different pieces of a table per thread
    float4 ahead_tab[TR], query_term[QR];
    float ahead_base[TR];
    if constexpr (split) {
#pragma unroll
        for (int i = 0; i < QR; ++i) query_term[i] = *reinterpret_cast<const float4*>(a.ts.lut + (int64_t)q * (M * IVFR_KS) + 4 * ((tid + SEL_T * i) % T4));
    }
    auto fetch = [&](const Group& grp) {   // the group's tables
#pragma unroll
        for (int i = 0; i < TR; ++i) {
            const int piece = tid + SEL_T * i, g = piece / T4, e = 4 * (piece % T4);   // a power of two
            if (g < grp.n) {
                const int64_t pair = (int64_t)q * w + grp.r[0] + g;
                const float* t = split ? a.ts.list_term + (int64_t)s_list[grp.r[0] + g] * (M * IVFR_KS) : a.ts.lut + pair * (M * IVFR_KS);
                ahead_tab[i] = *reinterpret_cast<const float4*>(t + e);
                if (split) ahead_base[i] = a.ts.pbase[pair * M + (e >> 8)];
            }
        }
    };
    auto table_piece = [&](int i) {   // as PairTable::get
        const float4 va = ahead_tab[i], vb = query_term[i % QR];
        const float s = ahead_base[i];
        if (!split) return va;
        return make_float4(fmaxf(0.f, (va.x + vb.x) + s), fmaxf(0.f, (va.y + vb.y) + s), fmaxf(0.f, (va.z + vb.z) + s), fmaxf(0.f, (va.w + vb.w) + s));
    };
    // A pass: U SEL_T slots of two consecutive entries of one list, counted over the group's lists.
    struct Pass { uint32_t wds[U][2][M / 4]; uint32_t e[U]; int g[U]; int have[U]; uint32_t start[U]; };   // have: entries in the slot, 0 to 2
    auto slots = [&](const Group& grp) {
        uint32_t s = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) s += (grp.len[g] + 1u) / 2u;
        return s;
    };
    auto load_pass = [&](const Group& grp, uint32_t base) {
        Pass p;
        uint32_t s[U], len[U];
        bool found[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { s[u] = base + tid + SEL_T * u; len[u] = 0; found[u] = false; p.g[u] = 0; p.start[u] = 0; }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const uint32_t l = grp.len[g], k = (l + 1u) / 2u;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool here = !found[u] && s[u] < k;
                if (here) { p.g[u] = g; len[u] = l; if (OWN) p.start[u] = s_start[grp.rank(g)]; }
                found[u] = found[u] || here;
                if (!found[u]) s[u] -= k;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            p.e[u] = 2u * s[u];
            if (!OWN && found[u]) p.start[u] = s_start[grp.r[0] + p.g[u]];
            p.have[u] = found[u] ? (p.e[u] + 1 < len[u] ? 2 : 1) : 0;
            if (found[u]) {   // lists start at multiples of 32 entries and end in padding: both codes are there to read
                const uint32_t* src = reinterpret_cast<const uint32_t*>(codes + ((uint64_t)p.start[u] + p.e[u]) * M);
#pragma unroll
                for (int t = 0; t < M / 4; ++t) { p.wds[u][0][t] = src[t]; p.wds[u][1][t] = src[M / 4 + t]; }
            } else {
#pragma unroll
                for (int t = 0; t < M / 4; ++t) p.wds[u][0][t] = p.wds[u][1][t] = 0;
            }
        }
        return p;
    };
    Group now = form(INFINITY);
    if (!OWN) fetch(now);
    Pass ahead;
    if (AHEAD && now.n) ahead = load_pass(now, 0);
    int scanned = 0;            // lists behind s_first
    uint32_t met = 0;           // their entries
    while (now.n) {             // uniform
        Group then;
        if constexpr (OWN) {
            int lists[G];
#pragma unroll
            for (int g = 0; g < G; ++g) lists[g] = now.rank(g) >= 0 ? (int)s_list[now.rank(g)] : -1;
            own_tables<M, G, (CAP > 4096 && M >= 8 ? 4 : 2)>(a, q, lists, s_res, s_lut);   // (begins with a barrier)
        } else {
            __syncthreads();   // the previous tables are no longer read
#pragma unroll
            for (int i = 0; i < TR; ++i)
                if (TR * SEL_T == G * T4 || tid + SEL_T * i < G * T4) reinterpret_cast<float4*>(s_lut)[tid + SEL_T * i] = table_piece(i);
        }
        __syncthreads();
        // where the group's entries begin among those that were met
        uint32_t place0[G], sum = met;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            place0[g] = sum;
            if (OWN && tid == 0 && now.rank(g) >= 0) { s_first[scanned + g] = s_start[now.rank(g)]; s_pre[scanned + g] = sum; }   // (read at the end)
            sum += now.len[g];
        }
        if (!OWN) {
            then = form(INFINITY);
            if (then.n) fetch(then);
        }
        const uint32_t n_slots = slots(now);
        // (loaded tables: a group without entries still takes one pass, of idle lanes, in which the next one's codes are loaded)
        for (uint32_t base = 0; base < n_slots || (!OWN && base == 0); base += U * SEL_T) {
            Pass p;
            if (AHEAD) {
                p = ahead;
                const bool more = base + U * SEL_T < n_slots;
                if constexpr (OWN) {
                    if (more) ahead = load_pass(now, base + U * SEL_T);
                } else {   // (one call for both: with two the compiler copies, and waits for, what has just been requested)
                    Group from = now;
                    if (!more) from = then;
                    if (more || then.n) ahead = load_pass(from, more ? base + U * SEL_T : 0u);
                }
            } else {
                p = load_pass(now, base);
            }
            if (!placed && n_top + U * PASS / 2 > CAP) {   // uniform: is there really no room for another pass?
                __syncthreads();
                const uint32_t n = s_fill;
                __syncthreads();   // everyone has read it
                n_top = n;
                if (n + U * PASS / 2 > CAP) {   // then n > CAP - PASS >= k': the k' smallest are among the n records
                    const RecsSrc all{s_rec, n, ids, id_stride};
                    const uint64_t pivot = kth_key(sh, all, K);
                    uint2 rec[CAP / SEL_T];
#pragma unroll
                    for (int i = 0; i < CAP / SEL_T; ++i) rec[i] = (uint32_t)(tid + SEL_T * i) < n ? s_rec[tid + SEL_T * i] : make_uint2(0xFFFFFFFFu, 0u);
                    // K are stored.  (Where ids repeat more than K keys lie at or below the pivot: they are counted apart, so that the
                    // next places follow what is stored, whatever the ids are.)
                    if (tid == 0) { s_fill = K; s_cut = 0; }
                    __syncthreads();   // everything is in registers
#pragma unroll
                    for (int i = 0; i < CAP / SEL_T; ++i) {
                        const bool keep = (uint32_t)(tid + SEL_T * i) < n && within(rec[i].x, pivot, [&]() { return all.lo(rec[i].y); });
                        const uint64_t mk = __ballot(keep);
                        uint32_t first = 0;
                        if (lane == 0 && mk) first = atomicAdd(&s_cut, (uint32_t)__popcll(mk));
                        first = __builtin_amdgcn_readfirstlane(first);
                        const uint32_t slot = first + __popcll(mk & ((1ull << lane) - 1ull));
                        if (keep && slot < K) s_rec[slot] = rec[i];   // exactly k' of them
                    }
                    tau = __uint_as_float((uint32_t)(pivot >> 32));
                    n_top = K;
                    __syncthreads();
                }
            }
            float est[U][2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // Loaded tables, often of one list: wavefronts without a slot leave the LDS to the others (777 entries fill 389 of 1024 slots).
                // Own tables are of four lists or more, and the test cost what it saved (8 lists of 977 entries 1 %).
                if (!OWN && U > 1) {
                    est[u][0] = est[u][1] = 0.f;
                    if (base + SEL_T * u + 64 * __builtin_amdgcn_readfirstlane(wave) >= n_slots) continue;
                }
                const float* lut = s_lut + p.g[u] * (M * IVFR_KS);
                est[u][0] = table_sum<M>(lut, p.wds[u][0]);
                est[u][1] = table_sum<M>(lut, p.wds[u][1]);
                if (OWN) largest = fmaxf(largest, fmaxf(p.have[u] > 0 ? est[u][0] : 0.f, p.have[u] > 1 ? est[u][1] : 0.f));
            }
            if (placed) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    uint32_t at = 0;
#pragma unroll
                    for (int g = 0; g < G; ++g) at = p.g[u] == g ? place0[g] : at;
                    uint32_t* v = s_val + at + p.e[u];
                    if (p.have[u] > 0) v[0] = __float_as_uint(est[u][0]);
                    if (p.have[u] > 1) v[1] = __float_as_uint(est[u][1]);
                }
                continue;
            }
            uint64_t mk[U][2];
            uint32_t cnt = 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    mk[u][x] = __ballot(p.have[u] > x && est[u][x] <= tau);
                    cnt += __popcll(mk[u][x]);
                }
            if (cnt) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&s_fill, cnt);
                at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        const uint64_t m = mk[u][x];
                        if ((m >> lane) & 1ull)
                            s_rec[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                                make_uint2(__float_as_uint(est[u][x]), p.start[u] + p.e[u] + x);
                        at += __popcll(m);
                    }
            }
            n_top += U * PASS / 2;
        }
        scanned += now.n;
        met = sum;
        if constexpr (OWN) {
            float bound = tau;
            if (a.low && next < w && met >= K) {   // uniform
                const uint32_t l = wave_fold(__float_as_uint(largest), 0u, [](uint32_t x, uint32_t y) { return x > y ? x : y; });
                if (lane == 63) sh.wa[wave] = l;
                __syncthreads();
                uint32_t m = sh.wa[0];
#pragma unroll
                for (int i = 1; i < SEL_T / 64; ++i) m = sh.wa[i] > m ? sh.wa[i] : m;
                bound = fminf(bound, __uint_as_float(m));
                // (the next writes to sh.wa lie behind a barrier: of the tables, or the one below)
            }
            then = form(bound);
            if (AHEAD && then.n) ahead = load_pass(then, 0u);
        }
        now = then;
    }
    if (OWN && tid == 0) s_pre[scanned] = met;
    __syncthreads();
    uint32_t* const op = a.out_pos + (int64_t)q * K;
    float* const oe = a.out_est ? a.out_est + (int64_t)q * K : nullptr;
    const uint32_t n = placed ? met : s_fill;   // (a barrier lies behind the last reservation)
    __syncthreads();
    if (tid == 0) {
        a.out_n[q] = (int32_t)(n < K ? n : K);
        s_fill = 0;
    }
    // Output: a thread counts what it keeps, a prefix over the lanes and one LDS atomic per wavefront give the places in an LDS list
    // of what is kept, which all threads then turn into positions (where each looked up its own as it came, nearly every step
    // of the loop waited for some lane's search: 4.9 us for 1000 of 7800).
    uint32_t* const s_kept = sh.hist;   // [K], K <= SEL_BINS (the launcher's limit); the selection is done with it
    auto emit = [&](const auto& src, auto word, auto position) {
        uint64_t pivot = ~0ull;
        if (n > K) pivot = kth_key(sh, src, K);
        else __syncthreads();   // (the selection ends with a barrier)
        uint32_t mine = 0;
#pragma unroll 4
        for (uint32_t i = tid; i < n; i += SEL_T) mine += within(word(i), pivot, [&]() { return src.lo(src.ref(i)); }) ? 1u : 0u;
        const uint32_t inc = wave_prefix(mine);
        uint32_t at = 0;
        if (lane == 63 && inc) at = atomicAdd(&s_fill, inc);
        uint32_t slot = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + inc - mine;
#pragma unroll 4
        for (uint32_t i = tid; i < n; i += SEL_T) {
            if (!within(word(i), pivot, [&]() { return src.lo(src.ref(i)); })) continue;
            if (slot < K) s_kept[slot] = i;
            ++slot;
        }
        __syncthreads();
        const uint32_t have = n < K ? n : K;
        for (uint32_t t = tid; t < have; t += SEL_T) {
            const uint32_t i = s_kept[t];
            op[t] = position(i);
            if (oe) oe[t] = __uint_as_float(word(i));
        }
    };
    if (placed) {
        const PlacedSrc s{s_val, n, s_pre, OWN ? s_first : s_start, OWN ? scanned : w, ids, id_stride};
        emit(s, [&](uint32_t i) { return s.v[i]; }, [&](uint32_t i) { return s.position(i); });
    } else {
        const RecsSrc s{s_rec, n, ids, id_stride};
        emit(s, [&](uint32_t i) { return s.v[i].x; }, [&](uint32_t i) { return s.v[i].y; });
    }
    if (OWN && tid == 0 && met < total) atomicAdd(a.counter + IVFR_COUNTER_LEFT(q % IVFR_LEFT_LINES), (unsigned long long)(total - met));
}

static size_t scan_select_lds(int m, int gm, int cap, int w, int d, bool own) {
    const size_t g = (size_t)std::max(1, gm / m);
    return g * m * IVFR_KS * sizeof(float) + (size_t)cap * sizeof(uint2) + (6 * (size_t)w + 1) * sizeof(uint32_t) +
           (own ? (4 + g * d) * sizeof(float) : 0);
}

#define IVFR_SS_STATIC (9 * 1024)     // the kernel's static LDS, rounded up
#define IVFR_SS_LDS (160 * 1024)

// Whether many queries' own tables are the faster ones where no list is left out, against loaded ones (written by another kernel, on
// their way while the lists before are scanned).  Measured (us of a call own / loaded; 300 to 1000 queries, d = 32 to 256):
//  - long lists hide the loading: 8 or 16 lists of 4000 entries, m = 8, 0.97 to 1.02 times as long at d = 128 and 1.02 to 1.09 at 256;
//    of 1000 entries 0.81 to 1.04; 1 list, half a group or more without a use, 500 queries 0.93 to 1.00, 1000 0.91 to 1.05, 2000 0.97 to
//    1.17; 2 lists 0.85 to 0.98, 0.89 to 1.04 and 0.94 to 1.13;
//  - sub-vectors of 32 dimensions take the longest to tabulate: lists of 1000 entries, m = 8, 16 to 64 of them 1.01 to 1.09, 8 1.00; of
//    100 entries 0.88 to 0.97; 2 lists, 300 queries 0.97, 1000 1.05, 3454 1.15; d = 512, 8 to 64 lists 1.04 to 1.14, 2 lists and 300
//    queries 0.91;
//  - m = 4, where a group is eight lists and their scan is short: 64 lists of 1000 entries 1.00 to 1.11, 32 0.95 to 1.05, 100 entries
//    0.82 to 1.02; 2 lists, three quarters of a group without a use, 1.00 to 1.11;
//  - m = 32, where every list reads the whole codebook, d = 256, 8 to 32 lists: 300 queries 1.01 to 1.13, 600 0.91 to 1.08, 1000 0.85
//    to 1.06.
static bool own_pays(const ivfr_index* ix, int nq, int w) {
    const double len = ix->wmean_len;
    const int m = ix->p.m, d = ix->p.d;
    if (m == 4 && 3 * w < 2 * ((w + 7) / 8 * 8)) return false;   // more than a third of the groups' places without a list
    if (w < 4) return nq <= (w == 1 || ix->dsub == 32 || d > 256 ? 2 : 4) * ix->n_cu;
    if (d > 256) return false;
    if (m == 32) return w < 8 || 2 * nq > 5 * ix->n_cu;
    return len < (ix->dsub == 32 && w >= 16 ? 500.0 : 2000.0) && (m != 4 || w * len < 4.0e4);
}

// What a call is launched with.  Few queries have a compute unit each: 64 KB of tables, of many lists at a time, computed where
// they are used (another kernel costs more than the workgroup that needs them waits), and 8192 places; 32 KB at m = 4, where that is
// eight lists already (sixteen take more scalar registers than there are: 8 lists for one query alone 27 us against 18, 1 list 19
// and 13.5), and where 32 KB hold all lists (m = 8, 1 list 18.8 us against 14.1, 4 lists of 3900 entries 36.8 and 31.4; m = 16, 2 lists
// 14.0 and 12.3): a group's tables are computed whole.  Many queries share the compute units, two at a time (a third would need the
// kernel to spill: 58 -> 75 us per 1000 queries), with 4096 places and 32 KB of tables, computed as well where sub-vectors have 8
// dimensions or more: a group of four lists (m = 8) reads the 128 KB codebook once, and the lists that a bound leaves out cost nothing
// (1000 queries, tables and scan: 8 lists of 977 entries 78 -> 61 us, 16 of 1220 146 -> 57, and 8 to 11 us for the bounds).  Else
// 16 KB of tables (32 at m = 32), loaded.
struct SelectShape { int gm, cap; int tab; size_t lds; };
static bool select_shape(const ivfr_index* ix, int nq, int w, int kprime, bool split, bool bounds, SelectShape* out) {
    const int m = ix->p.m;
    const bool shared = nq > ix->n_cu;
    const size_t room = (size_t)IVFR_SS_LDS / (shared ? 2 : 1);
    SelectShape s;
    const bool own = !split && ix->p.d <= 512 && (!shared || (ix->dsub % 8 == 0 && m <= 32 && (bounds || own_pays(ix, nq, w))));
    s.cap = shared ? 4096 : 8192;
    s.gm = shared || m == 4 || (m <= 16 && w * m <= 32) ? 32 : 64;
    s.lds = scan_select_lds(m, s.gm, s.cap, w, ix->p.d, own);
    s.tab = split ? TAB_SPLIT : (own ? TAB_OWN : TAB_LOADED);
    if (shared && (!own || s.lds + IVFR_SS_STATIC > room)) {
        if (own) s.tab = TAB_LOADED;
        s.gm = 16;
        s.lds = scan_select_lds(m, s.gm, s.cap, w, ix->p.d, false);
    }
    *out = s;
    return !(shared && m > 32) && kprime <= SEL_BINS && kprime + PASS <= s.cap && s.lds + IVFR_SS_STATIC <= room;
}

bool ivfr_scan_select_supported(const ivfr_index* ix, int nq, int w, int kprime, bool split) {
    SelectShape s;   // (loaded tables take less of the LDS: with a shape for bounds there is one without)
    return (uint64_t)w * ix->max_len < 0xFFFFFFF0ull && select_shape(ix, nq, w, kprime, split, true, &s);
}

bool ivfr_scan_select_own_tables(const ivfr_index* ix, int nq, int w, int kprime, bool split, bool bounds) {
    SelectShape s;
    return select_shape(ix, nq, w, kprime, split, bounds, &s) && s.tab == TAB_OWN;
}

// The kernels by select_shape's results.  (A compute unit per query loads tables of more than 512 dimensions only, which m = 4, 8 and 16
// do not have.)
#define IVFR_SS_FEW(F, MM, GG) F(MM, GG, 8192, TAB_SPLIT) F(MM, GG, 8192, TAB_OWN)
#define IVFR_SS_MANY(F, MM) F(MM, 16, 4096, TAB_LOADED) F(MM, 16, 4096, TAB_SPLIT) F(MM, 32, 4096, TAB_OWN)
#define IVFR_SS_ALL(F)                                                                                                 \
    IVFR_SS_FEW(F, 4, 32) IVFR_SS_FEW(F, 8, 32) IVFR_SS_FEW(F, 16, 32) IVFR_SS_FEW(F, 8, 64) IVFR_SS_FEW(F, 16, 64)     \
    IVFR_SS_FEW(F, 32, 64) IVFR_SS_FEW(F, 64, 64) F(32, 64, 8192, TAB_LOADED) F(64, 64, 8192, TAB_LOADED)               \
    IVFR_SS_MANY(F, 4) IVFR_SS_MANY(F, 8) IVFR_SS_MANY(F, 16) IVFR_SS_MANY(F, 32)

int ivfr_launch_scan_select(const ivfr_index* ix, ScanSelectArgs a, bool split, bool bounds, hipStream_t st) {
    if (a.nq <= 0) return IVFR_OK;
    SelectShape s;
    if (!select_shape(ix, a.nq, a.w, a.kprime, split, bounds, &s)) { ivfr_set_error("internal: no launch shape for w = %d, k' = %d", a.w, a.kprime); return IVFR_ERR_STATE; }
    a.d = ix->p.d;
    a.coarse = ix->coarse;
    a.pq = ix->pq;
    a.pq_norm = ix->pq_norm;
    a.pq_cols = reinterpret_cast<const float4*>(ix->pq_cols);
    const int m = ix->p.m;
    bool launched = false;
#define IVFR_SS(MM, GG, CC, OO)                                                                                                \
    if (m == MM && s.gm == GG && s.cap == CC && s.tab == OO) {                                                                 \
        hipLaunchKernelGGL((scan_select_kernel<MM, GG, CC, OO>), dim3((unsigned)a.nq), dim3(SEL_T), s.lds, st, ix->codes, a,   \
                           ix->list_start, ix->list_len, reinterpret_cast<const int32_t*>(ix->rec), (uint32_t)(ix->rec_stride / 4)); \
        launched = true;                                                                                                       \
    }
    IVFR_SS_ALL(IVFR_SS)
#undef IVFR_SS
    if (!launched) {   // the re-rank would read what an earlier call left
        ivfr_set_error("internal: no kernel for m = %d, %d KB of tables, %d places", m, s.gm, s.cap);
        return IVFR_ERR_STATE;
    }
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Dynamic LDS beyond 48 KB has to be allowed per kernel and device.
int ivfr_scan_select_init() {
#define IVFR_SS(MM, GG, CC, OO)                                                                                             \
    IVFR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(scan_select_kernel<MM, GG, CC, OO>),                         \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, IVFR_SS_LDS - IVFR_SS_STATIC));
    IVFR_SS_ALL(IVFR_SS)
#undef IVFR_SS
    return IVFR_OK;
}
