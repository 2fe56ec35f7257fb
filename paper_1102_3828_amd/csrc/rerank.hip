// Query step 2 of section 3.2 (gfx950): for each short-list entry, rebuild the refined
// approximation  y^ = coarse[l] + decode(q_c code) + decode(q_r code)  of Eq. (9) explicitly and
// compute the squared distance ||x - y^||^2 of Eq. (10).  No full database vector is read:
// an entry costs m + m' + 4 gathered bytes; the codebooks and the coarse centroids are small
// enough to be served from cache.
//
// The general kernel (any shape): eight lanes share one entry and interleave its dimensions in 16-byte pieces (lane t takes
// dimensions 4t..4t+3 of every group of 32), so that one load instruction of the eight lanes
// covers 128 contiguous bytes of the query and the coarse centroid and whole codebook rows (few
// cache lines per instruction); the partial sums are combined with three xor-shuffles.
// Everything that is fetched per candidate - id, list, code and refinement code - sits in one
// record that never straddles a 128-byte line, so the random gather from HBM costs one line per
// candidate.  Output per entry: the 64-bit key (distance bits << 32 | id) consumed by the final
// top-k selection.
#include "select_core.h"

template <int VEC>
__global__ __launch_bounds__(256) void rerank_kernel(const float* __restrict__ queries, int d, int c, int m, int mr,
                                                     int dsub, int dsub_r, const float* __restrict__ coarse,
                                                     const float* __restrict__ pq, const float* __restrict__ rq,
                                                     const uint8_t* __restrict__ rec, int rec_stride,
                                                     int kprime,
                                                     const uint32_t* __restrict__ short_pos,
                                                     const int32_t* __restrict__ short_n, uint64_t* __restrict__ keys,
                                                     float* __restrict__ refined_out, int32_t* __restrict__ ids_out,
                                                     StatusToHost tell) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) tell.publish();
    const int q = blockIdx.y;
    const int n = short_n[q];
    const int slot = blockIdx.x * 32 + (threadIdx.x >> 3);
    const int t = threadIdx.x & 7;
    const bool live = slot < n;   // uniform over the 8 lanes of an entry
    float acc = 0.f;
    int32_t id = -1;
    if (live) {
        const uint32_t pos = short_pos[(int64_t)q * kprime + slot];
        const uint8_t* r = rec + (uint64_t)pos * rec_stride;
        id = *reinterpret_cast<const int32_t*>(r);
        const uint32_t l = *reinterpret_cast<const uint32_t*>(r + 4);
        const uint8_t* code = r + 8;
        const uint8_t* rcode = r + 8 + m;
        const float* x = queries + (int64_t)q * d;
        const float* cl = coarse + (int64_t)l * d;
        if (VEC == 4) {
            for (int e = 4 * t; e < d; e += 32) {
                const int j = e / dsub;
                float4 y = *reinterpret_cast<const float4*>(cl + e);
                float4 pv = *reinterpret_cast<const float4*>(pq + ((int64_t)j * IVFR_KS + code[j]) * dsub + (e - j * dsub));
                y.x += pv.x; y.y += pv.y; y.z += pv.z; y.w += pv.w;
                if (mr > 0) {
                    const int jr = e / dsub_r;
                    float4 rv = *reinterpret_cast<const float4*>(rq + ((int64_t)jr * IVFR_KS + rcode[jr]) * dsub_r +
                                                                 (e - jr * dsub_r));
                    y.x += rv.x; y.y += rv.y; y.z += rv.z; y.w += rv.w;
                }
                float4 xv = *reinterpret_cast<const float4*>(x + e);
                float a = xv.x - y.x, b = xv.y - y.y, cc = xv.z - y.z, dd = xv.w - y.w;
                acc = fmaf(a, a, acc); acc = fmaf(b, b, acc); acc = fmaf(cc, cc, acc); acc = fmaf(dd, dd, acc);
            }
        } else {
            for (int e = t; e < d; e += 8) {
                const int j = e / dsub;
                float y = cl[e] + pq[((int64_t)j * IVFR_KS + code[j]) * dsub + (e - j * dsub)];
                if (mr > 0) {
                    const int jr = e / dsub_r;
                    y += rq[((int64_t)jr * IVFR_KS + rcode[jr]) * dsub_r + (e - jr * dsub_r)];
                }
                float a = x[e] - y;
                acc = fmaf(a, a, acc);
            }
        }
    }
    acc += __shfl_xor(acc, 4, 64);
    acc += __shfl_xor(acc, 2, 64);
    acc += __shfl_xor(acc, 1, 64);
    if (t == 0 && slot < kprime) {
        const int64_t o = (int64_t)q * kprime + slot;
        if (live) {
            keys[o] = ((uint64_t)__float_as_uint(acc) << 32) | (uint32_t)id;
            if (refined_out) refined_out[o] = acc;
            if (ids_out) ids_out[o] = id;
        } else {
            keys[o] = ~0ull;
            if (refined_out) refined_out[o] = INFINITY;
            if (ids_out) ids_out[o] = -1;
        }
    }
}

// ------------------------------------------------------------------------------------------
// The common shapes (d = 32, 64, 128 or 256, sub-vectors of 4 to 32 dimensions in both stages).
//
// Four lanes share an entry, and a workgroup works on its up to 128 R entries slice by slice: 16 dimensions of all of
// them, then the next 16.  Of a slice the decode needs 256 rows of each codebook (32 KB together) and the same 64 bytes
// of each visited centroid, so the rows are staged in LDS once per slice and the centroid pieces stay in the vector
// cache, where an entry-by-entry walk gathers a 128-byte line from L2 for every 32 or 64 bytes it uses (3 KB per entry).
// The rows of both codebooks lie side by side (book_rows: [slice][256][16 first-stage | 16 refinement floats], written
// when the codebooks are set): row k holds, for each dimension of the slice, value k of the sub-quantizer that covers
// it, so a lane's column is fixed and only the row depends on the code.  Even entries read the first-stage half first,
// odd entries the refinement half, so that the eight lanes that the LDS serves together always meet eight different
// bank groups.  What a lane needs of an entry's code is one byte per slice, packed into words when the record
// arrives.  ||x - y^||^2 is summed as ((x - c) - (p + r))^2 in two chains per lane (even and odd slices).
// Bound: the vector cache's address path (records and staging, 60 % busy) and latency at 16 wavefronts per compute
// unit; three 16-byte LDS reads per lane and slice (43 % busy; profiles/rerank_cfg3_counters.txt).  Measured: 10^7 entries of 1000 queries,
// d = 128, m' = 16, 726 -> 448 us; 10^6 entries 75.7 (and 13.6 for the final selection, now inside) -> 52 us, against a
// kernel that kept the refinement codebook in LDS and gathered the rest entry by entry.  Of a workgroup's 23 us at 10^6 entries the
// records take 6 (13 with m' = 32: random lines), the slices 12 (at the rate of their LDS reads), the selection 3.6.  Centroid pieces read from memory
// instead of residuals in LDS: 560 us.
// ------------------------------------------------------------------------------------------
#define RR_T SEL_T        // threads; 128 entries per round
#define RR_ROW4 8         // 16-byte pieces per codebook row of a slice
typedef float f4 __attribute__((ext_vector_type(4)));

#define RR_SLICE (IVFR_KS * RR_ROW4 * 16u)   // bytes of a slice's rows
#define RR_RSRC 0x00027000                   // raw 32-bit data, offsets in bytes, reads past the end return zero

__device__ __forceinline__ f4 load16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(f4, (u4)__builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}

struct RerankArgs {
    const float* queries;
    const float* coarse;
    const f4* rows;       // [d / 16][256][RR_ROW4]
    const uint8_t* rec;
    const uint32_t* short_pos;
    const int32_t* short_n;
    uint64_t* keys;
    float* refined_out;
    int32_t* ids_out;
    int32_t* top_ids;     // FINAL: the k best, sorted
    float* top_dist;
    const int32_t* probe;
    int w, c, m, dsub, dsub_r, rec_stride, kprime, k, chunks;
    StatusToHost tell;
};

// Byte strings of R entries: byte s of a lane's string is the code byte of the sub-quantizer that covers dimensions
// 16 s + 4 t .. + 3, for W dimensions per sub-quantizer; code points at the code inside the first record, off[r] is
// the byte offset of record r.  (At d = 32 a string has two bytes of the four; what is read behind the code is still the
// record's: 32 bytes, the code at 8, 12 or 16, at most 16 read.)
template <int NSW, int R>
__device__ __forceinline__ void slice_bytes(const uint8_t* code, const uint64_t (&off)[R], int W, uint32_t t,
                                            uint32_t (&out)[R][NSW]) {
    if (W == 16) {   // (one load for all words of a code: what counts is the number of loads, each a gather of 16 lines)
#pragma unroll
        for (int r = 0; r < R; ++r) __builtin_memcpy(out[r], __builtin_assume_aligned(code + off[r], 4), 4 * NSW);
    } else if (W == 8) {
        const uint32_t sel = (t >> 1) ? 0x07050301u : 0x06040200u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t v[2 * NSW];
            __builtin_memcpy(v, __builtin_assume_aligned(code + off[r], 4), 8 * NSW);
#pragma unroll
            for (int w = 0; w < NSW; ++w) out[r][w] = __builtin_amdgcn_perm(v[2 * w + 1], v[2 * w], sel);
        }
    } else if (W == 4) {
        const uint32_t sel = 0x0c0c0400u + 0x0101u * t;   // byte t of the low word, byte t of the high word
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int w = 0; w < NSW; ++w) {
                uint32_t v[4];
                __builtin_memcpy(v, __builtin_assume_aligned(code + off[r] + 16 * w, 4), 16);
                out[r][w] = __builtin_amdgcn_perm(v[1], v[0], sel) | (__builtin_amdgcn_perm(v[3], v[2], sel) << 16);
            }
    } else {   // 32
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int w = 0; w < NSW; ++w) {
                const uint32_t v = *reinterpret_cast<const uint32_t*>(code + off[r] + 4 * (w >> 1));
                out[r][w] = __builtin_amdgcn_perm(v, v, (w & 1) ? 0x03030202u : 0x01010000u);
            }
    }
}

// NS: slices (d / 16); R: rounds of 128 entries per workgroup; STAGE: rows through LDS; RESID: so are the query's
// residuals x - c to its visited centroids (the entry's rank among them from a byte map over the lists);
// FINAL: the workgroup holds all entries of its query and writes the k best itself.
template <int NS, int R, bool STAGE, bool RESID, bool FINAL>
__global__ __launch_bounds__(RR_T, 4) void rerank_rows_kernel(RerankArgs a) {
    extern __shared__ f4 s_rows[];                         // STAGE: [256][RR_ROW4]; RESID: then residuals and the map
    f4* const s_res = s_rows + IVFR_KS * RR_ROW4;          // [w][2][4]: two copies, for even and for odd entries
    uint8_t* const s_rank = reinterpret_cast<uint8_t*>(s_res + 8 * a.w);   // [c]
    __shared__ uint64_t s_keys[FINAL ? R * 128 : 1];
    __shared__ uint64_t s_top[FINAL ? SEL_RANK_SORT : 1];
    __shared__ uint32_t s_slot;
    __shared__ int32_t s_id[R * 128];   // ids wait here for the sums: reading the records again at the end cost a second line each
    const int tid = threadIdx.x;
    const uint32_t t = tid & 3;
    const int g = tid >> 2;
    const bool odd = g & 1;
    if (blockIdx.x == 0 && tid == 0) a.tell.publish();
    const int q = FINAL ? (int)blockIdx.x : (int)(blockIdx.x / (uint32_t)a.chunks);
    const int chunk0 = FINAL ? 0 : (int)(blockIdx.x % (uint32_t)a.chunks) * (R * 128);   // first slot of the workgroup
    const int n = a.short_n[q] - chunk0;                       // its entries (may be negative)
    const int room = a.kprime - chunk0;                        // its slots
    const uint32_t* spos = a.short_pos + ((int64_t)q * a.kprime + chunk0);
    constexpr int NSW = NS < 4 ? 1 : NS / 4;   // words of an entry's byte string
    constexpr int D = 16 * NS;
    const bool has_r = a.dsub_r > 0;
    if (!FINAL && n <= 0 && !a.refined_out && !a.ids_out) return;   // uniform: nothing of this chunk is there
    // buffer descriptors: one register of address per load in flight
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<f4*>(a.rows), 0, NS * RR_SLICE, RR_RSRC);
    const __amdgpu_buffer_rsrc_t coarse =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.coarse), 0, (int)((uint32_t)a.c * (uint32_t)(4 * D)), RR_RSRC);
    f4 pre[4];
    if (STAGE) {
#pragma unroll
        for (int i = 0; i < 4; ++i) pre[i] = load16(rows, 16u * tid + 16u * RR_T * i, 0u);
    }
    // RESID: this thread's piece of the residuals (list tid / 4 of the query), one slice ahead
    f4 res_pre = {0.f, 0.f, 0.f, 0.f}, x_pre = {0.f, 0.f, 0.f, 0.f};
    uint32_t res_off = 16u * t;
    const bool has_res = RESID && g < a.w;
    const float* x = a.queries + (int64_t)q * D + 4 * t;
    if constexpr (RESID) {
        if (has_res) {
            const uint32_t l = (uint32_t)a.probe[(int64_t)q * a.w + g];
            if (t == 0) s_rank[l] = (uint8_t)g;
            res_off += l * (uint32_t)(4 * D);
            res_pre = load16(coarse, res_off, 0u);
            x_pre = *reinterpret_cast<const f4*>(x);
        }
    }
    uint32_t first[R][NSW], second[R][NSW], cl[R];   // cl: byte offset of the lane's piece of the centroid, or its place in s_res
    float acc[R][2];
    {
        // A slot without an entry decodes the record of position 0: in bounds, and never looked at.
        uint64_t off[R];
#pragma unroll
        for (int r = 0; r < R; ++r) off[r] = (uint64_t)(g + 128 * r < n ? spos[g + 128 * r] : 0u) * (uint32_t)a.rec_stride;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc[r][0] = acc[r][1] = 0.f;
            const uint2 head = *reinterpret_cast<const uint2*>(a.rec + off[r]);   // id and list
            const uint32_t l = head.y;
            if (t == 0) s_id[g + 128 * r] = (int32_t)head.x;   // (read by the same lane)
            cl[r] = g + 128 * r < n ? l : 0u;   // byte offsets fit: ivfr_book_rows_floats
            if (!RESID) cl[r] = cl[r] * (uint32_t)(4 * D) + 16u * t;
        }
        slice_bytes<NSW, R>(a.rec + 8, off, a.dsub, t, first);
        if (has_r) {
            slice_bytes<NSW, R>(a.rec + 8 + a.m, off, a.dsub_r, t, second);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int w = 0; w < NSW; ++w) {
                    const uint32_t u = first[r][w], v = second[r][w];
                    first[r][w] = odd ? v : u;
                    second[r][w] = odd ? u : v;
                }
        } else {   // the rows' second halves are zero: any row will do
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int w = 0; w < NSW; ++w) second[r][w] = first[r][w];
        }
    }
    if constexpr (RESID) {
        __syncthreads();   // the map is complete
#pragma unroll
        for (int r = 0; r < R; ++r) cl[r] = 128u * (g + 128 * r < n ? s_rank[cl[r]] : 0u) + (odd ? 64u : 0u) + 16u * t;
    }
    const uint32_t col1 = (odd ? 4u : 0u) + t, col2 = (odd ? 0u : 4u) + t;
    constexpr int G = R < 2 ? R : 2;   // rounds whose loads are in flight together
    // One slice: byte `shift` of the strings' first words, accumulator `chain`.  A real loop over pairs of slices: unrolled
    // altogether the compiler issues the loads of all slices up front and spills.
    auto slice = [&](int s, int shift, int chain) {
        if (STAGE) {
            if (s) __syncthreads();   // the previous slice's rows are no longer read
#pragma unroll
            for (int i = 0; i < 4; ++i) s_rows[tid + RR_T * i] = pre[i];
            if (has_res) s_res[8 * g + t] = s_res[8 * g + 4 + t] = x_pre - res_pre;
            __syncthreads();
            const uint32_t next = (uint32_t)(s + 1 < NS ? s + 1 : s) * RR_SLICE;   // the last slice reads its own rows again
#pragma unroll
            for (int i = 0; i < 4; ++i) pre[i] = load16(rows, 16u * tid + 16u * RR_T * i, next);
            if (has_res) {
                const int sn = s + 1 < NS ? s + 1 : s;
                res_pre = load16(coarse, res_off, 64u * sn);
                x_pre = *reinterpret_cast<const f4*>(x + 16 * sn);
            }
        }
        f4 xv = {0.f, 0.f, 0.f, 0.f};
        if (!RESID) xv = *reinterpret_cast<const f4*>(x + 16 * s);
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += G) {
            f4 c[G], v[G];
#pragma unroll
            for (int i = 0; i < G; ++i) c[i] = RESID ? *reinterpret_cast<const f4*>(reinterpret_cast<const char*>(s_res) + cl[r0 + i]) : xv - load16(coarse, cl[r0 + i], 64u * s);
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const uint32_t k1 = (first[r0 + i][0] >> shift) & 0xffu, k2 = (second[r0 + i][0] >> shift) & 0xffu;
                v[i] = STAGE ? s_rows[k1 * RR_ROW4 + col1] + s_rows[k2 * RR_ROW4 + col2]
                             : load16(rows, 16u * (k1 * RR_ROW4 + col1), (uint32_t)s * RR_SLICE) +
                                   load16(rows, 16u * (k2 * RR_ROW4 + col2), (uint32_t)s * RR_SLICE);
            }
#pragma unroll
            for (int i = 0; i < G; ++i) {
                const f4 e = c[i] - v[i];
                float s0 = acc[r0 + i][chain];
                s0 = fmaf(e.x, e.x, s0); s0 = fmaf(e.y, e.y, s0); s0 = fmaf(e.z, e.z, s0); s0 = fmaf(e.w, e.w, s0);
                // the sums are taken here: otherwise the compiler moves them behind the next slice's barrier and keeps what
                // they are made of, 12 registers an entry
                asm volatile("" : "+v"(s0));
                acc[r0 + i][chain] = s0;
            }
        }
    };
#pragma unroll 1
    for (int s = 0; s < NS; s += 2) {
        slice(s, 0, 0);
        slice(s + 1, 8, 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {   // the strings move on by two bytes
#pragma unroll
            for (int w = 0; w < NSW; ++w) {
                first[r][w] = w + 1 < NSW ? __builtin_amdgcn_alignbit(first[r][w + 1 < NSW ? w + 1 : w], first[r][w], 16) : first[r][w] >> 16;
                second[r][w] = w + 1 < NSW ? __builtin_amdgcn_alignbit(second[r][w + 1 < NSW ? w + 1 : w], second[r][w], 16) : second[r][w] >> 16;
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        // the eight chains are added in double precision: their sums would be the largest roundings of all
        double v8 = (double)acc[r][0] + (double)acc[r][1];
        v8 += __shfl_xor(v8, 1, 64);
        v8 += __shfl_xor(v8, 2, 64);
        const float v = (float)v8;
        const int slot = g + 128 * r;
        const bool live = slot < n;
        if (t == 0 && slot < room) {
            const int64_t o = (int64_t)q * a.kprime + chunk0 + slot;
            const int32_t id = live ? s_id[slot] : -1;
            const uint64_t key = ((uint64_t)__float_as_uint(v) << 32) | (uint32_t)id;
            if (FINAL) s_keys[slot] = live ? key : ~0ull;
            else if (live) a.keys[o] = key;
            if (a.refined_out) a.refined_out[o] = live ? v : INFINITY;
            if (a.ids_out) a.ids_out[o] = id;
        }
    }
    if constexpr (FINAL) {
        __shared__ SelShared sh;
        if (tid == 0) s_slot = 0;
        __syncthreads();
        int m_out = n, m_have = n;
        const uint64_t* top = s_keys;
        if (n > a.k) {
            const uint64_t pivot = kth_key(sh, RegKeysSrc<(R + 3) / 4>(KeysSrc{s_keys, n}), (uint32_t)a.k);
            for (int i = tid; i < n; i += RR_T) {
                const uint64_t key = s_keys[i];
                if (key <= pivot) {
                    const uint32_t slot = atomicAdd(&s_slot, 1u);
                    if (slot < SEL_RANK_SORT) s_top[slot] = key;
                }
            }
            __syncthreads();
            m_out = a.k;
            m_have = (int)(s_slot < SEL_RANK_SORT ? s_slot : SEL_RANK_SORT);
            top = s_top;
        }
        write_ranked(top, m_have, m_out, a.k, a.top_ids + (int64_t)q * a.k, a.top_dist + (int64_t)q * a.k);
    }
}

// Rows of both codebooks by slice (see above); without a refinement stage its half is zero.
__global__ __launch_bounds__(256) void book_rows_kernel(const float* __restrict__ pq, const float* __restrict__ rq, int d,
                                                        int dsub, int dsub_r, float* __restrict__ rows) {
    const int i = blockIdx.x * 256 + threadIdx.x;   // (slice, k, column of 32)
    if (i >= d / 16 * IVFR_KS * 32) return;
    const int col = i & 31, k = (i >> 5) & (IVFR_KS - 1), s = i >> 13;
    const int e = 16 * s + (col & 15);
    const int W = col < 16 ? dsub : dsub_r;
    const float* book = col < 16 ? pq : rq;
    rows[i] = W > 0 ? book[((int64_t)(e / W) * IVFR_KS + k) * W + e % W] : 0.f;
}

__global__ __launch_bounds__(256) void pq_cols_kernel(const float* __restrict__ pq, int m, int dsub, float* __restrict__ cols) {
    const int i = blockIdx.x * 256 + threadIdx.x;   // (j, k, component)
    if (i >= m * IVFR_KS * dsub) return;
    const int e = i % dsub, k = (i / dsub) & (IVFR_KS - 1), j = i / dsub / IVFR_KS;
    cols[((j * (dsub / 4) + e / 4) * IVFR_KS + k) * 4 + (e & 3)] = pq[i];
}

__global__ __launch_bounds__(256) void coarse_cols_kernel(const float* __restrict__ coarse, int c, int d, float* __restrict__ cols) {
    const int i = blockIdx.x * 256 + threadIdx.x;   // (centroid, component)
    if (i >= c * d) return;
    const int e = i % d, l = i / d;
    cols[(e / 4 * c + l) * 4 + (e & 3)] = coarse[i];
}

int ivfr_launch_book_rows(const ivfr_index* ix, hipStream_t st) {
    if (ix->coarse_cols) {
        hipLaunchKernelGGL(coarse_cols_kernel, dim3((unsigned)((ix->p.c * ix->p.d + 255) / 256)), dim3(256), 0, st, ix->coarse, ix->p.c, ix->p.d,
                           ix->coarse_cols);
        IVFR_HIP(hipGetLastError());
    }
    if (ix->pq_cols) {
        const int total = ix->p.m * IVFR_KS * ix->dsub;
        hipLaunchKernelGGL(pq_cols_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, ix->pq, ix->p.m, ix->dsub, ix->pq_cols);
        IVFR_HIP(hipGetLastError());
    }
    if (!ix->book_rows) return IVFR_OK;
    hipLaunchKernelGGL(book_rows_kernel, dim3((unsigned)(ix->p.d / 16 * IVFR_KS * 32 / 256)), dim3(256), 0, st, ix->pq, ix->rq,
                       ix->p.d, ix->dsub, ix->dsub_r, ix->book_rows);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

template <int NS, int R>
static void launch_rows(const RerankArgs& a, int nq, bool resid, bool final, hipStream_t st) {
    constexpr bool STAGE = R > 1;
    const size_t lds = STAGE ? (IVFR_KS * RR_ROW4 + (resid ? 8 * (size_t)a.w : 0)) * sizeof(f4) + (resid ? (size_t)a.c : 0) : 0;
    const dim3 grid((unsigned)nq * (unsigned)a.chunks);
#define IVFR_ROWS(RES, F) hipLaunchKernelGGL((rerank_rows_kernel<NS, R, STAGE, RES, F>), grid, dim3(RR_T), lds, st, a)
    if (STAGE && resid) { if (final) IVFR_ROWS(STAGE, true); else IVFR_ROWS(STAGE, false); }
    else { if (final) IVFR_ROWS(false, true); else IVFR_ROWS(false, false); }
#undef IVFR_ROWS
}

// Returns whether the launch also wrote the k best of every query (top_ids, top_dist).
int ivfr_launch_rerank(const ivfr_index* ix, const float* queries, const int32_t* probe, int nq, int w, int kprime, int k,
                       const uint32_t* short_pos, const int32_t* short_n, uint64_t* keys, float* refined_out,
                       int32_t* ids_out, int32_t* top_ids, float* top_dist, bool* wrote_top, StatusToHost tell, hipStream_t st) {
    *wrote_top = false;
    if (nq <= 0) return IVFR_OK;
    if (ix->book_rows) {
        RerankArgs a;
        a.queries = queries; a.coarse = ix->coarse; a.rows = reinterpret_cast<const f4*>(ix->book_rows); a.rec = ix->rec;
        a.short_pos = short_pos; a.short_n = short_n; a.keys = keys; a.refined_out = refined_out; a.ids_out = ids_out;
        a.top_ids = top_ids; a.top_dist = top_dist;
        a.probe = probe; a.w = w; a.c = ix->p.c; a.m = ix->p.m; a.dsub = ix->dsub; a.dsub_r = ix->dsub_r; a.rec_stride = ix->rec_stride;
        a.kprime = kprime; a.k = k; a.tell = tell;
        // Rounds per workgroup: one workgroup holds a whole short-list of up to 1024 entries (and then also selects the
        // k best); a workgroup that has one round to decode reads the rows directly.  Up to 256 entries per compute unit
        // it is one round everywhere: the decode spreads over more workgroups, which outweighs the second kernel for the
        // k best.  Measured (call, d = 128, m' = 32, one round against as many as fit): 2 queries, k' = 5000 121 and 134 us;
        // 16 x 1000 162 and 169; 64 x 1000 161 and 164; 128 x 1000 170 and 161; 256 x 1000 191 and 174.
        const int r_max = ix->p.d > 128 ? 4 : 8;
        int R = 1;
        while ((int64_t)nq * kprime > 256ll * ix->n_cu && R < r_max && 128 * R < kprime) R *= 2;
        a.chunks = (kprime + 128 * R - 1) / (128 * R);
        // residuals in LDS: one thread per piece, 128 bytes per visited list and a byte per list of the index
        const bool resid = w <= RR_T / 4 && ix->p.c <= 16384;
        const bool final = a.chunks == 1 && k <= SEL_RANK_SORT;
#define IVFR_ROWS_R(NS)                                                      \
        switch (R) {                                                         \
            case 1: launch_rows<NS, 1>(a, nq, resid, final, st); break;        \
            case 2: launch_rows<NS, 2>(a, nq, resid, final, st); break;        \
            case 4: launch_rows<NS, 4>(a, nq, resid, final, st); break;        \
            default: launch_rows<NS, NS == 16 ? 4 : 8>(a, nq, resid, final, st); break; \
        }
        if (ix->p.d == 32) { IVFR_ROWS_R(2) }
        else if (ix->p.d == 64) { IVFR_ROWS_R(4) }
        else if (ix->p.d == 128) { IVFR_ROWS_R(8) }
        else { IVFR_ROWS_R(16) }
#undef IVFR_ROWS_R
        IVFR_HIP(hipGetLastError());
        *wrote_top = final;
        return IVFR_OK;
    }
    dim3 grid((kprime + 31) / 32, nq);
    const bool vec = (ix->dsub % 4 == 0) && (ix->p.m_refine == 0 || ix->dsub_r % 4 == 0) && ((ix->p.d / 8) % 4 == 0);
#define IVFR_RERANK_ARGS                                                                                       \
    queries, ix->p.d, ix->p.c, ix->p.m, ix->p.m_refine, ix->dsub, ix->dsub_r, ix->coarse, ix->pq, ix->rq,      \
        ix->rec, ix->rec_stride, kprime, short_pos, short_n, keys, refined_out, ids_out, tell
    if (vec) hipLaunchKernelGGL(rerank_kernel<4>, grid, dim3(256), 0, st, IVFR_RERANK_ARGS);
    else hipLaunchKernelGGL(rerank_kernel<1>, grid, dim3(256), 0, st, IVFR_RERANK_ARGS);
#undef IVFR_RERANK_ARGS
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}
