// fp32 MFMA distance GEMM for gfx950: rows X [n, d] against centroids C [c, d].
//
// Used for the coarse-quantizer distances of the search (section 3.3: the w nearest of c
// reproduction values) and for nearest-centroid assignment when vectors are encoded or a
// k-means iteration runs (offline steps 1-2 of section 3.2).  ||x - c||^2 is expanded as
// ||x||^2 + ||c||^2 - 2 x.c so that the O(n c d) part is a dense contraction on the matrix
// cores; fp32 inputs and fp32 accumulation (v_mfma_f32_32x32x2_f32) keep the result within
// a few ulp of the direct form.
//
// Tiling: a 256-thread workgroup (4 wavefronts, 2x2) owns a 128x128 output tile; each
// wavefront owns 64x64 = 2x2 MFMA tiles of 32x32 (64 accumulator VGPRs).  K is consumed in
// slabs of 32 staged through LDS (rows padded to 36 floats so that 16-byte fragment reads of
// 8 consecutive rows cover all 32 banks).  A lane reads one float4 per 32-row fragment and
// k-group of 8: lanes 0-31 take k+0..3, lanes 32-63 take k+4..7, and the four MFMAs of the
// group pair element t of A's float4 with element t of B's, so both operands see the same k.
#include "ivfr_internal.h"

typedef float floatx16 __attribute__((ext_vector_type(16)));

#define TM 128
#define TN 128
#define KT 32
#define LDS_STRIDE (KT + 4)

// bad (optional, zero on entry): raised to row + 1 of a row whose squared norm is not a finite number (the last such row)
__global__ __launch_bounds__(256) void row_norms_kernel(const float* __restrict__ X, int64_t n, int dim,
                                                        float* __restrict__ out, uint32_t* __restrict__ bad) {
    int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= n) return;
    const float* x = X + row * dim;
    float s = 0.f;
    for (int e = 0; e < dim; ++e) s = fmaf(x[e], x[e], s);
    out[row] = s;
    if (bad && !(s <= 3.0e38f)) atomicMax(bad, (uint32_t)row + 1u);
}

// out[j] = max over the `per` rows of group j of sqrt(norm2[j * per + k])
__global__ __launch_bounds__(256) void group_max_norm_kernel(const float* __restrict__ norm2, int per,
                                                             float* __restrict__ out) {
    __shared__ float red[256];
    float m = 0.f;
    for (int k = threadIdx.x; k < per; k += 256) m = fmaxf(m, norm2[(int64_t)blockIdx.x * per + k]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = sqrtf(red[0]);
}

int ivfr_launch_group_max_norm(const float* norm2, int groups, int per, float* out, hipStream_t st) {
    hipLaunchKernelGGL(group_max_norm_kernel, dim3(groups), dim3(256), 0, st, norm2, per, out);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Rows of at least 32 floats: eight lanes per row, 16 bytes per lane and step (coalesced), partial sums combined
// with three xor-shuffles.
__global__ __launch_bounds__(256) void row_norms8_kernel(const float* __restrict__ X, int64_t n, int dim,
                                                         float* __restrict__ out, uint32_t* __restrict__ bad) {
    const int64_t row = (int64_t)blockIdx.x * 32 + (threadIdx.x >> 3);
    const int t = threadIdx.x & 7;
    float s = 0.f;
    if (row < n) {
        const float* x = X + row * dim;
        for (int e = 4 * t; e < dim; e += 32) {
            const float4 v = *reinterpret_cast<const float4*>(x + e);
            s = fmaf(v.x, v.x, s); s = fmaf(v.y, v.y, s); s = fmaf(v.z, v.z, s); s = fmaf(v.w, v.w, s);
        }
    }
    s += __shfl_xor(s, 4, 64);
    s += __shfl_xor(s, 2, 64);
    s += __shfl_xor(s, 1, 64);
    if (row < n && t == 0) {
        out[row] = s;
        if (bad && !(s <= 3.0e38f)) atomicMax(bad, (uint32_t)row + 1u);
    }
}

int ivfr_launch_row_norms(const float* X, int64_t n, int dim, float* out, hipStream_t st, uint32_t* bad) {
    if (n <= 0) return IVFR_OK;
    if (dim >= 32 && dim % 4 == 0) {
        hipLaunchKernelGGL(row_norms8_kernel, dim3((unsigned)((n + 31) / 32)), dim3(256), 0, st, X, n, dim, out, bad);
        IVFR_HIP(hipGetLastError());
        return IVFR_OK;
    }
    hipLaunchKernelGGL(row_norms_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, X, n, dim, out, bad);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// four consecutive components of a row, k0 a multiple of 4
__device__ __forceinline__ float4 load4(const float* row, int k0) { return *reinterpret_cast<const float4*>(row + k0); }
__device__ __forceinline__ float4 load4(const uint8_t* row, int k0) {
    const uint32_t v = *reinterpret_cast<const uint32_t*>(row + k0);
    return make_float4((float)(v & 0xff), (float)((v >> 8) & 0xff), (float)((v >> 16) & 0xff), (float)(v >> 24));
}

// Stage a [128 x KT] slab of a row-major [rows, d] matrix into LDS (zero fill past `rows` and past d;
// d % 4 == 0).
template <class T>
__device__ __forceinline__ void stage_slab(const T* __restrict__ M, int64_t rows, int d, int64_t row0, int k0,
                                           float* lds) {
    const int tid = threadIdx.x;
    const int kc = (tid & 7) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int r = (tid >> 3) + 32 * i;
        int64_t gr = row0 + r;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (gr < rows && k0 + kc < d) v = load4(M + gr * d, k0 + kc);
        *reinterpret_cast<float4*>(lds + r * LDS_STRIDE + kc) = v;
    }
}

// Accumulate one KT slab: acc[a][b] += A(rows 64*wm + 32a ..) . B(cols 64*wn + 32b ..)
__device__ __forceinline__ void mma_slab(const float* As, const float* Bs, int wm, int wn, floatx16 acc[2][2]) {
    const int lane = threadIdx.x & 63;
    const int r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < KT / 8; ++kk) {
        float4 a[2], b[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            a[t] = *reinterpret_cast<const float4*>(As + (64 * wm + 32 * t + r) * LDS_STRIDE + kk * 8 + 4 * h);
            b[t] = *reinterpret_cast<const float4*>(Bs + (64 * wn + 32 * t + r) * LDS_STRIDE + kk * 8 + 4 * h);
        }
#pragma unroll
        for (int ta = 0; ta < 2; ++ta)
#pragma unroll
            for (int tb = 0; tb < 2; ++tb) {
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].x, b[tb].x, acc[ta][tb], 0, 0, 0);
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].y, b[tb].y, acc[ta][tb], 0, 0, 0);
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].z, b[tb].z, acc[ta][tb], 0, 0, 0);
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].w, b[tb].w, acc[ta][tb], 0, 0, 0);
            }
    }
}

// Accumulator element v of a 32x32 MFMA tile sits at row 8*(v/4) + 4*(lane/32) + v%4, col lane%32.
__device__ __forceinline__ int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

// The same accumulation for a workgroup tile of (64 T) x (64 T) outputs, T = 1 or 2: each of the
// 2x2 wavefronts owns T x T MFMA tiles.  The k order per output element does not depend on T, so both tile sizes
// give the same bits.
template <int T>
__device__ __forceinline__ void mma_tiles(const float* As, const float* Bs, int wm, int wn, floatx16 (&acc)[T][T]) {
    const int lane = threadIdx.x & 63;
    const int r = lane & 31, h = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < KT / 8; ++kk) {
        float4 a[T], b[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            a[t] = *reinterpret_cast<const float4*>(As + (32 * T * wm + 32 * t + r) * LDS_STRIDE + kk * 8 + 4 * h);
            b[t] = *reinterpret_cast<const float4*>(Bs + (32 * T * wn + 32 * t + r) * LDS_STRIDE + kk * 8 + 4 * h);
        }
#pragma unroll
        for (int ta = 0; ta < T; ++ta)
#pragma unroll
            for (int tb = 0; tb < T; ++tb) {
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].x, b[tb].x, acc[ta][tb], 0, 0, 0);
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].y, b[tb].y, acc[ta][tb], 0, 0, 0);
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].z, b[tb].z, acc[ta][tb], 0, 0, 0);
                acc[ta][tb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ta].w, b[tb].w, acc[ta][tb], 0, 0, 0);
            }
    }
}

// Distance words (bits of max(0, ||x||^2 + ||c||^2 - 2 x.c)) of n rows against c centroids.  The rows' squared norms come
// with the slabs that are staged anyway (xnorm == nullptr; the eight threads of a row hold the pieces and the order of
// row_norms8_kernel), and a row whose norm is not a finite number raises bad to row + 1.
template <int T>
__global__ __launch_bounds__(256) void dist_words_kernel(const float* __restrict__ X, const float* __restrict__ xnorm,
                                                         int64_t n, const float* __restrict__ C,
                                                         const float* __restrict__ cnorm, int c, int d,
                                                         uint32_t* __restrict__ words, uint32_t* __restrict__ bad) {
    __shared__ float As[64 * T * LDS_STRIDE];
    __shared__ float Bs[64 * T * LDS_STRIDE];
    __shared__ float xn[64 * T];
    const int64_t row0 = (int64_t)blockIdx.x * (64 * T);
    const int64_t col0 = (int64_t)blockIdx.y * (64 * T);
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = wave >> 1, wn = wave & 1;
    const int kc = (tid & 7) * 4;
    float sq[2 * T];
#pragma unroll
    for (int i = 0; i < 2 * T; ++i) sq[i] = 0.f;
    floatx16 acc[T][T];
#pragma unroll
    for (int a = 0; a < T; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    // the next slab's loads are issued before the matrix instructions of the current one
    float4 pa[2 * T], pb[2 * T];
    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2 * T; ++i) {
            const int r = (tid >> 3) + 32 * i;
            pa[i] = pb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k0 + kc < d) {
                if (row0 + r < n) pa[i] = *reinterpret_cast<const float4*>(X + (row0 + r) * d + k0 + kc);
                if (col0 + r < c) pb[i] = *reinterpret_cast<const float4*>(C + (col0 + r) * d + k0 + kc);
            }
        }
    };
    load(0);
    for (int k0 = 0; k0 < d; k0 += KT) {
        if (k0) __syncthreads();
#pragma unroll
        for (int i = 0; i < 2 * T; ++i) {
            const int r = (tid >> 3) + 32 * i;
            *reinterpret_cast<float4*>(As + r * LDS_STRIDE + kc) = pa[i];
            *reinterpret_cast<float4*>(Bs + r * LDS_STRIDE + kc) = pb[i];
            sq[i] = fmaf(pa[i].x, pa[i].x, sq[i]); sq[i] = fmaf(pa[i].y, pa[i].y, sq[i]);
            sq[i] = fmaf(pa[i].z, pa[i].z, sq[i]); sq[i] = fmaf(pa[i].w, pa[i].w, sq[i]);
        }
        __syncthreads();
        if (k0 + KT < d) load(k0 + KT);
        mma_tiles<T>(As, Bs, wm, wn, acc);
    }
#pragma unroll
    for (int i = 0; i < 2 * T; ++i) {
        float s = sq[i];
        s += __shfl_xor(s, 4, 64);
        s += __shfl_xor(s, 2, 64);
        s += __shfl_xor(s, 1, 64);
        const int r = (tid >> 3) + 32 * i;
        if ((tid & 7) == 0) {
            if (xnorm) s = row0 + r < n ? xnorm[row0 + r] : 0.f;
            xn[r] = s;
            if (!xnorm && blockIdx.y == 0 && row0 + r < n && !(s <= 3.0e38f)) atomicMax(bad, (uint32_t)(row0 + r) + 1u);
        }
    }
    __syncthreads();
#pragma unroll
    for (int ta = 0; ta < T; ++ta)
#pragma unroll
        for (int tb = 0; tb < T; ++tb) {
            int64_t col = col0 + 32 * T * wn + 32 * tb + (lane & 31);
            float cn = (col < c) ? cnorm[col] : 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 32 * T * wm + 32 * ta + acc_row(v, lane);
                if (row0 + r < n && col < c)
                    words[(row0 + r) * c + col] = __float_as_uint(fmaxf(0.f, fmaf(-2.f, acc[ta][tb][v], xn[r] + cn)));
            }
        }
}

int ivfr_launch_dist_words(const float* X, float* xnorm, int64_t n, const float* C, const float* cnorm, int c, int d,
                           uint32_t* words, uint32_t* bad, hipStream_t st) {
    if (n <= 0) return IVFR_OK;
    // rows too short for the norms of the staged pieces have a kernel of their own
    const bool inside = d >= 32 && d % 4 == 0;
    if (!inside) IVFR_TRY(ivfr_launch_row_norms(X, n, d, xnorm, st, bad));
    const float* xnp = inside ? nullptr : xnorm;
    // 128 x 128 tiles unless they would leave most compute units without a workgroup
    const int64_t big = ((n + TM - 1) / TM) * ((c + TN - 1) / TN);
    if (big >= 256) {
        dim3 grid((unsigned)((n + TM - 1) / TM), (unsigned)((c + TN - 1) / TN));
        hipLaunchKernelGGL(dist_words_kernel<2>, grid, dim3(256), 0, st, X, xnp, n, C, cnorm, c, d, words, bad);
    } else {
        dim3 grid((unsigned)((n + 63) / 64), (unsigned)((c + 63) / 64));
        hipLaunchKernelGGL(dist_words_kernel<1>, grid, dim3(256), 0, st, X, xnp, n, C, cnorm, c, d, words, bad);
    }
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Nearest centroid of each row: one workgroup per 128 rows walks all column tiles and keeps,
// per accumulator slot, the best (value, col) seen; columns are visited in increasing order
// so a strict '<' keeps the lowest index among equal values.  ||x||^2 is the same for every
// column of a row and is left out.
__global__ __launch_bounds__(256) void assign_kernel(const uint8_t* __restrict__ X, int64_t n,
                                                     const float* __restrict__ C, const float* __restrict__ cnorm,
                                                     int c, int d, int32_t* __restrict__ assign) {
    __shared__ float As[TM * LDS_STRIDE];
    __shared__ float Bs[TN * LDS_STRIDE];
    __shared__ float red_v[2][TM];
    __shared__ int red_i[2][TM];
    const int64_t row0 = (int64_t)blockIdx.x * TM;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;
    float best_v[2][16];
    int best_i[2][16];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int v = 0; v < 16; ++v) { best_v[a][v] = INFINITY; best_i[a][v] = 0x7fffffff; }

    for (int64_t col0 = 0; col0 < c; col0 += TN) {
        floatx16 acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
        for (int k0 = 0; k0 < d; k0 += KT) {
            __syncthreads();
            stage_slab(X, n, d, row0, k0, As);
            stage_slab(C, c, d, col0, k0, Bs);
            __syncthreads();
            mma_slab(As, Bs, wm, wn, acc);
        }
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            int col = (int)col0 + 64 * wn + 32 * tb + (lane & 31);
            bool ok = col < c;
            float cn = ok ? cnorm[col] : 0.f;
#pragma unroll
            for (int ta = 0; ta < 2; ++ta)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float val = fmaf(-2.f, acc[ta][tb][v], cn);
                    if (ok && val < best_v[ta][v]) { best_v[ta][v] = val; best_i[ta][v] = col; }
                }
        }
    }
    // reduce over the 32 lanes that share a row (same lane/32), then over the two column waves
#pragma unroll
    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float bv = best_v[ta][v];
            int bi = best_i[ta][v];
#pragma unroll
            for (int off = 16; off >= 1; off >>= 1) {
                float ov = __shfl_xor(bv, off, 64);
                int oi = __shfl_xor(bi, off, 64);
                if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            if ((lane & 31) == 0) {
                int r = 64 * wm + 32 * ta + acc_row(v, lane);
                red_v[wn][r] = bv;
                red_i[wn][r] = bi;
            }
        }
    __syncthreads();
    if (threadIdx.x < TM) {
        int r = threadIdx.x;
        int64_t row = row0 + r;
        if (row < n) {
            float v0 = red_v[0][r], v1 = red_v[1][r];
            int i0 = red_i[0][r], i1 = red_i[1][r];
            assign[row] = (v1 < v0 || (v1 == v0 && i1 < i0)) ? i1 : i0;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Nearest centroid of byte vectors on the 8-bit matrix cores.
//
// x' = x - 128 is a signed byte, and a centroid component is rounded to a 16-bit multiple q of a unit, taken apart into two signed
// bytes q = 256 hi + lo, so x . c is two v_mfma_i32_32x32x32_i8 products, exact, at twice the rate of the bf16 instruction.  The
// scores x . c - ||c||^2 / 2, whole numbers of units that fit 32 bits, are a filter: a row whose best score leads the second best by
// more than both arithmetics can be off keeps its column; the others (some per cent of the rows as a rule; exact ties among them) are
// decided by the fp32 kernel below with the arithmetic, column order and ties of assign_kernel.  The result is that kernel's, bit
// for bit.
//
// The columns are the rows of the product, so a lane has 16 scores of one row a tile: the low four bits of a score are replaced by its
// register's number, and best and second best and a tile's number are all there is to keep: four vector instructions a score (shift and
// add, insert, median, maximum).  (With the rows as the rows of the product every register was another row: 64 registers of
// best and second best, the tile's number in the score, and a reduction over 32 lanes at the end.)
//
// A wavefront keeps RT x 32 rows in registers for the whole walk over the columns and looks at the scores of one of its tiles while the
// products of the next are formed, an instruction of the matrix cores to nine of the vector unit; the workgroup's four wavefronts
// share the centroid fragments, which lie in the order the lanes read them (split_rows_kernel) and go from memory to LDS
// without passing through registers, one stage ahead.  128 rows a wavefront where that gives every compute unit two workgroups, 64 with
// fewer rows (10^6 rows, c = 1024: 0.278 and 0.310 ms).  Adds of 2^18 to 2^20 vectors, 64 / 128 rows: c = 8192 1.06 to 1.09 at d = 128
// (2^20: 2896 / 2695 us), 1.05 to 1.09 at 64, 1.00 to 1.04 at 8 to 32, where a wavefront of occupancy goes for it; c = 1024 1.03 at 128, 0.97
// to 1.03 below; fewer columns within the scatter (0.94 to 1.06, an add of 0.2 ms).  At d = 256 128 rows would take every register.
// Bound: matrix cores plus vector instructions, 256 and 272 cycles a tile; the two
// take turns rather than overlap (525 measured), also of different wavefronts.
// Measured (2^20 rows, d = 128): c = 8192 2.05 ms (2.47 before) and 0.43 ms for the unsure rows, c = 1024 0.29 (0.53; 0.46 from bytes) and 0.08;
// with bf16 pairs of each component 3.69 and 0.61, 0.66 and 0.11, on the fp32 instruction 18.5 and 3.1; c = 8192 with almost every row
// unsure 1.0 and 19.1 ms.  10^5 rows, c = 1024: 62 -> 41 us.
// ------------------------------------------------------------------------------------------
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef int int4v __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));

// fragment of (32-column tile, k-step of 32, part): 64 lanes x 16 bytes; lane l holds column l % 32, k = 16 (l / 32) ..
#define FRAG_BYTES 1024
#define SCORE_PAD 16
#define NO_SCORE (-0x7f000000)   // below every score (their limit is 2^30)

// What the centroids are like: [0] largest norm, [1] largest component (bits of non-negative floats; zero on entry); and of
// every column the sum of its components and its squared norm.  Eight lanes a column, from 32 components on with the pieces and the order of
// row_norms8_kernel: cnorm (optional) is then what that kernel writes.
// The launch also starts the counts of its assignment.  filtered: rows that went through the filter (low word; of one workgroup in 17) and
// those it left unsure (high word), kept from one assignment on the same scratch to the next (the iterations of a training, the
// batches of an add) and scaled down so that the latest weigh most.
__global__ __launch_bounds__(256) void centroid_stats_kernel(const float* __restrict__ C, int c, int d, double2* __restrict__ sums,
                                                             float* __restrict__ cnorm, uint32_t* __restrict__ stats,
                                                             uint32_t* __restrict__ n_unsure, unsigned long long* __restrict__ filtered,
                                                             int fresh) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        uint32_t rows = fresh ? 0u : (uint32_t)*filtered, open = fresh ? 0u : (uint32_t)(*filtered >> 32);
        while (rows > 65536u) { rows >>= 1; open >>= 1; }
        *n_unsure = 0u;
        *filtered = ((unsigned long long)open << 32) | rows;
    }
    const int col = blockIdx.x * 32 + (threadIdx.x >> 3), t = threadIdx.x & 7;
    double sum = 0.0, norm = 0.0;
    float big = 0.f, s = 0.f;
    bool odd = false;   // something that is no number: infinite statistics, no row is sure
    if (col < c) {
        const float* x = C + (int64_t)col * d;
        const bool wide = d >= 32;   // uniform
        for (int e = wide ? 4 * t : t; e < d; e += wide ? 32 : 8) {
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (wide) v = *reinterpret_cast<const float4*>(x + e);
            else v.x = x[e];
            s = fmaf(v.x, v.x, s); s = fmaf(v.y, v.y, s); s = fmaf(v.z, v.z, s); s = fmaf(v.w, v.w, s);
            const float f[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                sum += f[i];
                norm += (double)f[i] * f[i];
                big = fmaxf(big, fabsf(f[i]));
                odd = odd || !(fabsf(f[i]) < INFINITY);
            }
        }
    }
    if (cnorm) {
        s += __shfl_xor(s, 4, 64);
        s += __shfl_xor(s, 2, 64);
        s += __shfl_xor(s, 1, 64);
        if (col < c && t == 0) cnorm[col] = s;
    }
#pragma unroll
    for (int off = 4; off >= 1; off >>= 1) {
        sum += __shfl_xor(sum, off, 64);
        norm += __shfl_xor(norm, off, 64);
        big = fmaxf(big, __shfl_xor(big, off, 64));
    }
    if (col < c && t == 0) sums[col] = make_double2(sum, norm);
    float len = odd ? INFINITY : sqrtf((float)norm) * 1.000001f;   // (never below the norm)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        big = fmaxf(big, __shfl_xor(big, off, 64));
        len = fmaxf(len, __shfl_xor(len, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&stats[0], __float_as_uint(len));
        atomicMax(&stats[1], __float_as_uint(odd ? INFINITY : big));
    }
}

// The unit: components reach 32000 of it at the most, and a score |x . c - ||c||^2 / 2| 2^30.
__device__ __forceinline__ float score_unit(const uint32_t* stats, int d) {
    const float cmax = __uint_as_float(stats[0]), big = __uint_as_float(stats[1]);
    const float u = fmaxf(big * (1.f / 32000.f), (255.f * sqrtf((float)d) * cmax + 0.5f * cmax * cmax) * (1.01f / 1073741824.f));
    return u > 1e-30f ? u : 1e-30f;
}

// frag[tile][k-step][2 parts][64 lanes][16], a workgroup per tile; score0[2][score_stride(tiles)]: -||c||^2 / 2 and 128 times the sum of the
// components q, or of c itself, in units; NO_SCORE for columns past c
__host__ __device__ inline int score_stride(int tiles) { return (tiles + SCORE_PAD) * 32; }

__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ C, const double2* __restrict__ sums,
                                                         const uint32_t* __restrict__ stats, int c, int d, int ksteps,
                                                         uint4v* __restrict__ frag, int* __restrict__ score0) {
    __shared__ int s_sum[4][32];
    const int tiles = (int)gridDim.x, tile = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col = tile * 32 + (lane & 31);
    const float unit = score_unit(stats, d), inv = 1.f / unit;
    int sum = 0;
    for (int ks = wave; ks < ksteps; ks += 4) {
        const int k0 = ks * 32 + 16 * (lane >> 5);
        uint4v h = {0, 0, 0, 0}, l = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float v = col < c && k0 + e < d ? C[(int64_t)col * d + k0 + e] : 0.f;
            const int q = (int)rintf(fminf(fmaxf(v * inv, -32000.f), 32000.f));
            const int lo = (int)(int8_t)(q & 0xff), hi = (q - lo) >> 8;
            h[e >> 2] |= (uint32_t)(hi & 0xff) << (8 * (e & 3));
            l[e >> 2] |= (uint32_t)(lo & 0xff) << (8 * (e & 3));
            sum += q;
        }
        uint4v* o = frag + ((int64_t)tile * ksteps + ks) * 128 + lane;
        o[0] = h;
        o[64] = l;
    }
    sum += __shfl_xor(sum, 32, 64);
    if (lane < 32) s_sum[wave][lane] = sum;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int z = lane >> 5;   // which of the two scores
        int s = NO_SCORE;
        if (col < c) {
            const double q = z ? sums[col].x / (double)unit : (double)(s_sum[0][lane & 31] + s_sum[1][lane & 31] + s_sum[2][lane & 31] + s_sum[3][lane & 31]);
            const double v = 128.0 * q - 0.5 * sums[col].y / (double)unit;
            // (x' . c is below 2^30 units as well; beyond, with infinite statistics, no row is sure)
            s = v > -2.0e9 && v < 2.0e9 ? (int)rint(v) : NO_SCORE;
        }
        score0[z * score_stride(tiles) + col] = s;
    }
    if (tile == tiles - 1)   // the stages reach up to SCORE_PAD tiles past the last column
        for (int j = threadIdx.x; j < SCORE_PAD * 32; j += 256) score0[tiles * 32 + j] = score0[score_stride(tiles) + tiles * 32 + j] = NO_SCORE;
}

// KS k-steps of 32 (d <= 32 KS), RT tiles of 32 rows per wavefront (even), TC column tiles per stage
template <int KS, int RT, int TC>
__global__ __launch_bounds__(256, 2) void assign_bytes_kernel(const uint8_t* __restrict__ X, int64_t n, int d,
                                                              const uint4v* __restrict__ frag,
                                                              const int* __restrict__ score0, int tiles,
                                                              const uint32_t* __restrict__ stats, float margin_rel,
                                                              int32_t* __restrict__ assign, uint32_t* __restrict__ unsure,
                                                              uint32_t* __restrict__ n_unsure,
                                                              unsigned long long* __restrict__ filtered,
                                                              unsigned long long* __restrict__ best_key) {
    constexpr int STAGE = TC * KS * 2;   // fragments per stage
    extern __shared__ uint4v s_frag[];   // 2 x [STAGE][64]
    __shared__ __align__(16) int s_first[2][2][TC * 32];   // the columns' constants of a stage, both forms
    __shared__ uint32_t s_place, s_open;
    __shared__ uint16_t s_list[128 * RT];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t block0 = (int64_t)blockIdx.x * (128 * RT);
    const uint32_t here = (uint32_t)(n - block0 < 128 * RT ? n - block0 : 128 * RT);
    unsigned long long seen = 0;
    if (tid == 0) seen = __hip_atomic_load(filtered, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * (32 * RT);
    const int r = lane & 31, h = lane >> 5;
    const int stages = (tiles + TC - 1) / TC;
    // a stage's fragments: 256 threads x 16 bytes per step, straight to LDS (past the last tile: the last tile again)
    auto load_stage = [&](int s, int buf) {
#pragma unroll
        for (int i = 0; i < STAGE / 4; ++i) {
            const int f = 4 * i + wave;
            int tile = s * TC + f / (2 * KS);
            tile = tile < tiles ? tile : tiles - 1;
            const uint4v* src = frag + ((int64_t)tile * (2 * KS) + f % (2 * KS)) * 64 + lane;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(s_frag + ((size_t)buf * STAGE + f) * 64), 16, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < (TC + 3) / 4; ++i) {   // 64 constants a wavefront (they are padded by a stage)
            const int f = 4 * i + wave, form = f / (TC / 2), at = f % (TC / 2) * 64;
            if (f >= TC) break;   // uniform
            const int* src = score0 + form * score_stride(tiles) + s * TC * 32 + at + lane;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                             (__attribute__((address_space(3))) void*)(&s_first[buf][form][at]), 4, 0, 0);
        }
    };
    load_stage(0, 0);
    uint4v A[RT][KS];
    float xn[RT], x1[RT], x0[RT];   // norm of the row, sum of |x'|, sum of x
    float more = 0.f;               // of the rows' sums of |x'|, less those of x
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int64_t row = row0 + 32 * t + r;
        uint32_t s = 0, s1 = 0, s0 = 0;   // (sums of whole numbers, below 2^24)
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int e = 32 * k + 16 * h + 8 * i;
                uint2 v = make_uint2(0u, 0u), x = v;
                if (row < n && e < d) {   // d is a multiple of 8
                    v = *reinterpret_cast<const uint2*>(X + row * d + e);
                    x = make_uint2(v.x ^ 0x80808080u, v.y ^ 0x80808080u);
                    s = __builtin_amdgcn_udot4(v.x, v.x, s, false); s = __builtin_amdgcn_udot4(v.y, v.y, s, false);
                    s1 = __builtin_amdgcn_sad_u8(v.x, 0x80808080u, s1); s1 = __builtin_amdgcn_sad_u8(v.y, 0x80808080u, s1);
                    s0 = __builtin_amdgcn_sad_u8(v.x, 0u, s0); s0 = __builtin_amdgcn_sad_u8(v.y, 0u, s0);
                }
                A[t][k][2 * i] = x.x;
                A[t][k][2 * i + 1] = x.y;
            }
        xn[t] = sqrtf((float)(s + __shfl_xor(s, 32, 64)));
        x1[t] = (float)(s1 + __shfl_xor(s1, 32, 64));
        x0[t] = (float)(s0 + __shfl_xor(s0, 32, 64));
        more += x1[t] - x0[t];
    }
    // A centroid's rounding makes a score wrong by half a unit per unit of |x'| where the constant has the sum of c, and per unit of x where
    // it has the sum of q (x' . q + 128 sum q is x . q): the wavefront takes what is less for its rows.  (Components of 0 to 3, c = 1024,
    // an add of 2^20: 3.27 ms with x' for all, most rows unsure, 2.20 so; with two bf16 parts of each component 2.61.)
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) more += __shfl_xor(more, off, 64);
    const bool whole = more > 0.f;   // uniform: of whole numbers, exact
#pragma unroll
    for (int t = 0; t < RT; ++t) x1[t] = whole ? x0[t] : x1[t];
    // The filter costs about a fifth of what the fp32 kernel takes for all rows.  Where it has left more than three rows in four
    // unsure so far (centroids that are all but equal, or norms far larger than the distances between them), the rows go
    // straight to that kernel; one workgroup in 17 goes on looking (an odd number: neighbours in the grid run on different
    // XCDs, and every sixteenth would keep one XCD busy).  Which way a row goes does not change its result.
    if (tid == 0) {
        s_open = 0;
        const uint32_t rows = (uint32_t)seen, open = (uint32_t)(seen >> 32);
        const bool leave = blockIdx.x % 17u && rows >= 4096u && 4ull * open > 3ull * rows;
        s_place = leave ? atomicAdd(n_unsure, here) : 0xFFFFFFFFu;
    }
    __syncthreads();
    if (s_place != 0xFFFFFFFFu) {   // uniform
        for (uint32_t i = tid; i < here; i += 256) {
            best_key[block0 + i] = ~0ull;
            unsure[s_place + i] = (uint32_t)(block0 + i);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the stage under way is in LDS
        return;
    }
    // A lane has one row of each tile: 16 scores of it a column tile, a row's other 16 in the other half of the wavefront.
    int best[RT], second[RT], bt[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) { best[t] = INT32_MIN; second[t] = INT32_MIN; bt[t] = 0; }
    // The scores of a tile are looked at while the products of the next are formed.
    intx16 H[2], L[2];
    auto look = [&](int t, int tile, const intx16& hi, const intx16& lo) {
        const int before = best[t];
        int b = before, s2 = second[t];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int x = ((int)(((uint32_t)hi[v] << 8) + (uint32_t)lo[v]) & ~15) | v;
            const int lo2 = b < s2 ? b : s2, hi2 = b < s2 ? s2 : b, lo3 = hi2 < x ? hi2 : x;
            s2 = lo2 < lo3 ? lo3 : lo2;   // the median of the three, one instruction
            b = x > b ? x : b;
        }
        best[t] = b;
        second[t] = s2;
        bt[t] = b != before ? tile : bt[t];
    };
#pragma unroll
    for (int v = 0; v < 16; ++v) { H[1][v] = 0; L[1][v] = NO_SCORE; }   // before the first: nothing
    for (int s = 0; s < stages; ++s) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's part of the stage is in LDS
        __syncthreads();                                   // so are the others', and the other buffer is no longer read
        if (s + 1 < stages) load_stage(s + 1, (s + 1) & 1);
        const uint4v* F = s_frag + (size_t)(s & 1) * STAGE * 64 + lane;
#pragma unroll
        for (int tc = 0; tc < TC; ++tc) {
            const int tile = s * TC + tc;
            if (tile >= tiles) break;   // uniform (the stage repeats the last tile, whose products on top of NO_SCORE could wrap)
            intx16 c0;
#pragma unroll
            for (int g = 0; g < 4; ++g) {   // of the columns in this lane's registers
                const int4v f = *reinterpret_cast<const int4v*>(&s_first[s & 1][whole ? 0 : 1][tc * 32 + 8 * g + 4 * h]);
                c0[4 * g] = f.x; c0[4 * g + 1] = f.y; c0[4 * g + 2] = f.z; c0[4 * g + 3] = f.w;
            }
            int4v fh[KS], fl[KS];
#pragma unroll
            for (int k = 0; k < KS; ++k) { fh[k] = __builtin_bit_cast(int4v, F[(2 * k) * 64]); fl[k] = __builtin_bit_cast(int4v, F[(2 * k + 1) * 64]); }
            F += 2 * KS * 64;
#pragma unroll
            for (int t = 0; t < RT; ++t) {
                const int now = t & 1, prev = now ^ 1;
                intx16 hi = intx16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}, lo = c0;
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    hi = __builtin_amdgcn_mfma_i32_32x32x32_i8(fh[k], __builtin_bit_cast(int4v, A[t][k]), hi, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_i32_32x32x32_i8(fl[k], __builtin_bit_cast(int4v, A[t][k]), lo, 0, 0, 0);
                }
                H[now] = hi;
                L[now] = lo;
                if (t == 0) look(RT - 1, tile - 1, H[prev], L[prev]);
                else look(t - 1, tile, H[prev], L[prev]);
#pragma unroll
                for (int k = 0; k < 2 * KS; ++k) {
                    __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x2, 72 / (2 * KS), 0);
                }
            }
        }
    }
    look(RT - 1, tiles - 1, H[1], L[1]);
    // The halves of the wavefront have other columns of the same rows; then lane l has row l of every 64.
    const float cm = __uint_as_float(stats[0]), unit = score_unit(stats, d);
#pragma unroll
    for (int t = 0; t < RT; t += 2) {
        auto column = [&](int u) { const int x = best[u] & 15; return 32 * bt[u] + 8 * (x >> 2) + (x & 3) + 4 * h; };
        int b = (h ? best[t + 1] : best[t]) & ~15, s2 = (h ? second[t + 1] : second[t]) & ~15, ci = h ? column(t + 1) : column(t);
        const int ob = __shfl_xor((h ? best[t] : best[t + 1]) & ~15, 32, 64), os = __shfl_xor((h ? second[t] : second[t + 1]) & ~15, 32, 64);
        const int oc = __shfl_xor(h ? column(t) : column(t + 1), 32, 64);
        const int least = b < ob ? b : ob;
        s2 = s2 > os ? s2 : os;
        s2 = least > s2 ? least : s2;
        if (ob > b || (ob == b && oc < ci)) { b = ob; ci = oc; }
        const int64_t row = row0 + 32 * t + lane;
        if (row < n) {
            assign[row] = ci;
            // (a lead that is no number - an infinite or missing norm somewhere - is no lead)
            const float lead = (float)((int64_t)b - (int64_t)s2) * unit;
            const float margin = margin_rel * cm * ((h ? xn[t + 1] : xn[t]) + cm) + 2.02f * unit * (0.5f * (h ? x1[t + 1] : x1[t]) + 17.f);
            if (!(lead > margin)) {
                best_key[row] = ~0ull;
                s_list[atomicAdd(&s_open, 1u)] = (uint16_t)(row - block0);
            }
        }
    }
    __syncthreads();
    // one place in the list for the workgroup's rows; those that always look count them (if all did, the counter's 28 ns an
    // addition would show: 0.23 ms for 8192 workgroups)
    if (tid == 0) {
        s_place = s_open ? atomicAdd(n_unsure, s_open) : 0u;
        if (blockIdx.x % 17u == 0) atomicAdd(filtered, ((unsigned long long)s_open << 32) | here);
    }
    __syncthreads();
    for (uint32_t i = tid; i < s_open; i += 256) unsure[s_place + i] = (uint32_t)(block0 + s_list[i]);
}

// The rows left unsure, with the arithmetic of assign_kernel: an item is 128 listed rows against a range of the columns, 128
// x 256 outputs per step (8 wavefronts, 2 x 4), slabs of both operands double-buffered and loaded one ahead.  All columns in
// one item where that is four items per workgroup, else up to 4 gridDim.x items; the ranges of a row meet in a 64-bit minimum
// of (ordered score, column), so the lowest column wins among equal scores whatever their order.  Every row of a call can end
// up here (see assign_bytes_kernel).  Bound: the fp32 matrix instruction.  Measured (2^20 rows of d = 128, c = 8192, every
// row unsure): 19.1 ms; the same on 128 x 128 tiles with a reduction per tile 41.7; a kernel over all rows without a list 18.5.
//
// Few rows (some hundred of a training set, against 1024 columns) would be some thirty such items, each as long as its chain of loads and
// products: 37 us.  Up to four items of 32 rows x 256 columns per workgroup are therefore done in those: the rows in LDS whole, a wavefront's 32 columns
// straight from memory to registers, 64 of its components in flight at a time: 18 us.
#define UN 256
__global__ __launch_bounds__(512) void assign_unsure_kernel(const uint8_t* __restrict__ X, const float* __restrict__ C,
                                                            const float* __restrict__ cnorm, int c, int d,
                                                            const uint32_t* __restrict__ unsure,
                                                            const uint32_t* __restrict__ n_unsure,
                                                            unsigned long long* __restrict__ best_key) {
    __shared__ float As[2][TM * LDS_STRIDE];
    __shared__ float Bs[2][UN * LDS_STRIDE];
    __shared__ float red_v[4][TM];
    __shared__ int red_i[4][TM];
    __shared__ uint32_t rows[TM];
    const uint32_t n = *n_unsure;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3;
    // a best value and column, below everything that is not a number: the ordered score above the column
    auto take = [&](uint32_t row, float bv, int bi) {
        if (bv < INFINITY) {   // as assign_kernel: never an infinite or missing value
            const uint32_t bits = __float_as_uint(bv + 0.f);   // no negative zero
            const uint32_t ord = bits ^ ((bits >> 31) ? 0xffffffffu : 0x80000000u);
            atomicMin(&best_key[row], ((unsigned long long)ord << 32) | (uint32_t)bi);
        }
    };
    {
        const uint32_t row_tiles = (n + 31u) / 32u, col_tiles = ((uint32_t)c + UN - 1) / UN;
        if (row_tiles <= 4u * gridDim.x && row_tiles * (unsigned long long)col_tiles <= 4u * gridDim.x) {   // uniform
            float* const rs = &As[0][0];
            const int stride = d + 4;   // (d <= 256: 33 KB of As)
            const int r = lane & 31, h = lane >> 5;
            for (uint32_t item = blockIdx.x; item < row_tiles * col_tiles; item += gridDim.x) {
                const uint32_t first = item / col_tiles * 32;
                const int col = (int)(item % col_tiles) * UN + 32 * wave + r;
                const float* const cp = C + (int64_t)(col < c ? col : c - 1) * d + 4 * h;
                floatx16 acc;
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[v] = 0.f;
                float4 b[8];   // 64 components ahead
                auto load_b = [&](int k0) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) b[i] = k0 + 8 * i < d ? *reinterpret_cast<const float4*>(cp + k0 + 8 * i) : make_float4(0.f, 0.f, 0.f, 0.f);
                };
                load_b(0);
                __syncthreads();   // the previous item's rows and results are no longer read
                if (tid < 32) rows[tid] = unsure[first + tid < n ? first + tid : n - 1];
                __syncthreads();
                for (int i = tid; i < 32 * (d / 4); i += 512) {
                    const int row = i / (d / 4), k = 4 * (i % (d / 4));
                    *reinterpret_cast<float4*>(rs + row * stride + k) = load4(X + (int64_t)rows[row] * d, k);
                }
                __syncthreads();
                for (int k0 = 0; k0 < d; k0 += 64) {
                    float4 now[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) now[i] = b[i];
                    if (k0 + 64 < d) load_b(k0 + 64);
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        if (k0 + 8 * i >= d) break;   // uniform
                        const float4 a = *reinterpret_cast<const float4*>(rs + r * stride + k0 + 8 * i + 4 * h);
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, now[i].x, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, now[i].y, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, now[i].z, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, now[i].w, acc, 0, 0, 0);
                    }
                }
                const float cn = col < c ? cnorm[col] : 0.f;
                // over the 32 lanes that share a row, then over the eight wavefronts
                float* const rv = &Bs[0][0];                                   // [8][32]
                int* const ri = reinterpret_cast<int*>(&Bs[0][0]) + 8 * 32;    // [8][32]
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float bv = fmaf(-2.f, acc[v], cn);
                    int bi = col;
                    if (!(col < c && bv < INFINITY)) { bv = INFINITY; bi = 0x7fffffff; }
#pragma unroll
                    for (int off = 16; off >= 1; off >>= 1) {
                        const float ov = __shfl_xor(bv, off, 64);
                        const int oi = __shfl_xor(bi, off, 64);
                        if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
                    }
                    if (r == 0) { rv[wave * 32 + acc_row(v, lane)] = bv; ri[wave * 32 + acc_row(v, lane)] = bi; }
                }
                __syncthreads();
                if (tid < 32 && first + tid < n) {
                    float bv = rv[tid];
                    int bi = ri[tid];
#pragma unroll
                    for (int x = 1; x < 8; ++x) {
                        const float ov = rv[x * 32 + tid];
                        const int oi = ri[x * 32 + tid];
                        if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
                    }
                    take(rows[tid], bv, bi);
                }
            }
            return;
        }
    }
    const int kc = (tid & 7) * 4, sr = tid >> 3;   // staging: 64 rows x 8 float4 per pass
    const int ks = (d + KT - 1) / KT;
    const uint32_t nt = ((uint32_t)c + UN - 1) / UN, nb = n / TM + (n % TM ? 1u : 0u), wanted = 4u * gridDim.x;
    uint32_t ranges = 1;
    if (nb < wanted && nb > 0) { ranges = (wanted + nb - 1) / nb; ranges = ranges < nt ? ranges : nt; }
    // item, n and ranges are uniform: every barrier is reached by all threads
    for (uint32_t item = blockIdx.x; item < nb * ranges; item += gridDim.x) {
        const uint32_t first = item / ranges * TM, range = item % ranges;
        const int col_begin = (int)(nt * range / ranges) * UN, steps = (int)(nt * (range + 1) / ranges - nt * range / ranges) * ks;
        __syncthreads();   // the previous item's rows and results are no longer read
        if (tid < TM) rows[tid] = unsure[first + tid < n ? first + tid : n - 1];
        __syncthreads();
        float4 pa[2], pb[4];
        auto load = [&](int s) {
            const int col0 = col_begin + s / ks * UN, k = s % ks * KT + kc;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                pa[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (k < d) pa[i] = load4(X + (int64_t)rows[sr + 64 * i] * d, k);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int col = col0 + sr + 64 * i;
                pb[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (col < c && k < d) pb[i] = *reinterpret_cast<const float4*>(C + (int64_t)col * d + k);
            }
        };
        auto store = [&](int buf) {
#pragma unroll
            for (int i = 0; i < 2; ++i) *reinterpret_cast<float4*>(&As[buf][(sr + 64 * i) * LDS_STRIDE + kc]) = pa[i];
#pragma unroll
            for (int i = 0; i < 4; ++i) *reinterpret_cast<float4*>(&Bs[buf][(sr + 64 * i) * LDS_STRIDE + kc]) = pb[i];
        };
        float best_v[2][16];
        int best_i[2][16];
        floatx16 acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                best_v[a][v] = INFINITY; best_i[a][v] = 0x7fffffff;
                acc[a][0][v] = 0.f; acc[a][1][v] = 0.f;
            }
        load(0);
        store(0);
        __syncthreads();
        for (int s = 0; s < steps; ++s) {
            if (s + 1 < steps) load(s + 1);
            mma_slab(As[s & 1], Bs[s & 1], wm, wn, acc);
            if (s % ks == ks - 1) {
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
                    const int col = col_begin + s / ks * UN + 64 * wn + 32 * tb + (lane & 31);
                    const bool ok = col < c;
                    const float cn = ok ? cnorm[col] : 0.f;
#pragma unroll
                    for (int ta = 0; ta < 2; ++ta)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const float val = fmaf(-2.f, acc[ta][tb][v], cn);
                            if (ok && val < best_v[ta][v]) { best_v[ta][v] = val; best_i[ta][v] = col; }
                            acc[ta][tb][v] = 0.f;
                        }
                }
            }
            if (s + 1 < steps) store((s + 1) & 1);
            __syncthreads();
        }
        // over the 32 lanes that share a row, then over the four column wavefronts
#pragma unroll
        for (int ta = 0; ta < 2; ++ta)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                float bv = best_v[ta][v];
                int bi = best_i[ta][v];
#pragma unroll
                for (int off = 16; off >= 1; off >>= 1) {
                    const float ov = __shfl_xor(bv, off, 64);
                    const int oi = __shfl_xor(bi, off, 64);
                    if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
                }
                if ((lane & 31) == 0) {
                    const int r = 64 * wm + 32 * ta + acc_row(v, lane);
                    red_v[wn][r] = bv;
                    red_i[wn][r] = bi;
                }
            }
        __syncthreads();
        if (tid < TM && first + tid < n) {
            float bv = red_v[0][tid];
            int bi = red_i[0][tid];
#pragma unroll
            for (int x = 1; x < 4; ++x) {
                const float ov = red_v[x][tid];
                const int oi = red_i[x][tid];
                if (ov < bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
            }
            take(rows[tid], bv, bi);
        }
    }
}

__global__ __launch_bounds__(256) void assign_take_kernel(const uint32_t* __restrict__ unsure, const uint32_t* __restrict__ n_unsure,
                                                          const unsigned long long* __restrict__ best_key,
                                                          int32_t* __restrict__ assign, uint32_t* __restrict__ stats) {
    if (blockIdx.x == 0 && threadIdx.x < 2) stats[threadIdx.x] = 0u;   // for the next assignment
    const uint32_t n = *n_unsure;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const unsigned long long key = best_key[unsure[i]];
        assign[unsure[i]] = key == ~0ull ? 0 : (int32_t)(uint32_t)key;
    }
}

// Scratch of ivfr_launch_assign for n rows: fragments and scores of the c centroids, a key and a list entry per row.
struct AssignScratch {
    size_t frag, score0, sums, stats, count, filtered, unsure, key, bytes;
};
static AssignScratch assign_scratch(int64_t n, int c, int d) {
    AssignScratch s;
    size_t off = 0;
    auto take = [&](size_t b) { const size_t o = off; off += (b + 255) / 256 * 256; return o; };
    const size_t tiles = ((size_t)c + 31) / 32, ksteps = ((size_t)d + 31) / 32;
    s.frag = take(tiles * ksteps * 2 * FRAG_BYTES);
    s.score0 = take(2 * (size_t)score_stride((int)tiles) * sizeof(int));
    s.sums = take((size_t)c * sizeof(double2));
    s.stats = take(2 * sizeof(uint32_t));
    s.count = take(sizeof(uint32_t));
    s.filtered = take(sizeof(unsigned long long));   // (a cache line of its own: every workgroup reads it)
    s.unsure = take((size_t)n * sizeof(uint32_t));
    s.key = take((size_t)n * sizeof(unsigned long long));
    s.bytes = off;
    return s;
}

// Widths the 8-bit kernel covers; wider vectors (their rows do not fit a wavefront's registers) go to assign_kernel.
static bool assign_on_bytes(int d) { return d <= 256; }

size_t ivfr_assign_scratch_bytes(int64_t n, int c, int d) { return assign_on_bytes(d) ? assign_scratch(n, c, d).bytes : 0; }

int ivfr_launch_assign(const uint8_t* X, int64_t n, const float* C, float* cnorm, bool norms, int c, int d, int32_t* assign,
                       void* scratch, bool fresh, hipStream_t st) {
    const bool inside = norms && assign_on_bytes(d) && d >= 32 && n > 0;   // the norms come with the centroids' statistics
    if (norms && !inside) IVFR_TRY(ivfr_launch_row_norms(C, c, d, cnorm, st));
    if (n <= 0) return IVFR_OK;
    if (!assign_on_bytes(d)) {
        hipLaunchKernelGGL(assign_kernel, dim3((unsigned)((n + TM - 1) / TM)), dim3(256), 0, st, X, n, C, cnorm, c, d, assign);
        IVFR_HIP(hipGetLastError());
        return IVFR_OK;
    }
    const AssignScratch s = assign_scratch(n, c, d);
    char* p = static_cast<char*>(scratch);
    uint4v* frag = reinterpret_cast<uint4v*>(p + s.frag);
    int* score0 = reinterpret_cast<int*>(p + s.score0);
    double2* sums = reinterpret_cast<double2*>(p + s.sums);
    uint32_t* stats = reinterpret_cast<uint32_t*>(p + s.stats);
    uint32_t* count = reinterpret_cast<uint32_t*>(p + s.count);
    uint32_t* unsure = reinterpret_cast<uint32_t*>(p + s.unsure);
    unsigned long long* key = reinterpret_cast<unsigned long long*>(p + s.key);
    const int tiles = (c + 31) / 32;
    const int ksteps = d <= 32 ? 1 : d / 32;
    unsigned long long* filtered = reinterpret_cast<unsigned long long*>(p + s.filtered);
    if (fresh) IVFR_HIP(hipMemsetAsync(stats, 0, 2 * sizeof(uint32_t), st));
    hipLaunchKernelGGL(centroid_stats_kernel, dim3((unsigned)((c + 31) / 32)), dim3(256), 0, st, C, c, d, sums, inside ? cnorm : nullptr,
                       stats, count, filtered, fresh ? 1 : 0);
    hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)tiles), dim3(256), 0, st, C, sums, stats, c,
                       d, ksteps, frag, score0);
    // What two scores can be off together, and two fp32 values of assign_kernel, halved: those by |x| |c| d 2^-24 and two roundings
    // each, with |x| |c| + ||c||^2 <= cmax (|x| + cmax); a score by half a unit per unit of |x'| or x (the centroid's rounding), half a
    // unit (its constant's) and the four bits that the register's number takes: 15 units and two for roundings, the last term of the
    // kernel's margin.
    const float margin_rel = 2.f * ((float)d * 5.9605e-8f + 4.7684e-7f) * 1.01f;
    const bool wide = n >= 1024 * 256;   // two workgroups of 512 rows for every compute unit
#define IVFR_ASSIGN(KS, RT, TC)                                                                                       \
    hipLaunchKernelGGL((assign_bytes_kernel<KS, RT, TC>), dim3((unsigned)((n + 128 * RT - 1) / (128 * RT))), dim3(256),  \
                       (size_t)2 * TC * KS * 2 * FRAG_BYTES, st, X, n, d, frag, score0, tiles, stats, margin_rel, assign, \
                       unsure, count, filtered, key)
    switch (ksteps) {
        case 1: if (wide) IVFR_ASSIGN(1, 4, 8); else IVFR_ASSIGN(1, 2, 8); break;
        case 2: if (wide) IVFR_ASSIGN(2, 4, 8); else IVFR_ASSIGN(2, 2, 8); break;
        case 4: if (wide) IVFR_ASSIGN(4, 4, 4); else IVFR_ASSIGN(4, 2, 4); break;
        case 8: IVFR_ASSIGN(8, 2, 2); break;
        default:
            ivfr_set_error("assignment supports d = 8 .. 256 in powers of two and larger d; got %d", d);
            return IVFR_ERR_INVALID_ARG;
    }
#undef IVFR_ASSIGN
    IVFR_HIP(hipGetLastError());
    // a workgroup per compute unit, which walk over however many items there are
    hipLaunchKernelGGL(assign_unsure_kernel, dim3(256), dim3(512), 0, st, X, C, cnorm, c, d, unsure, count, key);
    hipLaunchKernelGGL(assign_take_kernel, dim3(512), dim3(256), 0, st, unsure, count, key, assign, stats);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}
