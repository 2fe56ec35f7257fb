// Offline stage of section 3.2 (gfx950): residuals, product-quantizer encoding (Eq. (4), (8)),
// stable placement of encoded vectors into inverted lists, and the k-means updates used to
// learn the quantizers (step 1).
#include "select_core.h"

#include <algorithm>
#include <math.h>

// R[i] = X[i] - C[assign[i]]   (Eq. (7) with the coarse quantizer: residual to the list's centroid)
__global__ __launch_bounds__(256) void residual_kernel(const uint8_t* __restrict__ X, int64_t n, int d4,
                                                       const float* __restrict__ C,
                                                       const int32_t* __restrict__ assign, float* __restrict__ R) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * d4) return;
    int64_t row = i / d4;
    int e = (int)(i % d4);
    const uint32_t x = reinterpret_cast<const uint32_t*>(X)[i];
    float4 c = reinterpret_cast<const float4*>(C)[(int64_t)assign[row] * d4 + e];
    reinterpret_cast<float4*>(R)[i] = make_float4((float)(x & 0xff) - c.x, (float)((x >> 8) & 0xff) - c.y,
                                                  (float)((x >> 16) & 0xff) - c.z, (float)(x >> 24) - c.w);
}

int ivfr_launch_residual(const uint8_t* X, int64_t n, int d, const float* C, const int32_t* assign, float* R, hipStream_t st) {
    if (n <= 0) return IVFR_OK;
    int64_t total = n * (d / 4);
    hipLaunchKernelGGL(residual_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X, n, d / 4, C,
                       assign, R);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// code[i][j] = argmin_k || r_i^j - book[j][k] ||^2 (ties to the lowest k) for vectors r that are there in fp32 (training) or are what
// centroid and first-stage value leave of bytes (EncSrc): an add never writes a residual to memory.  With `subtract` (fp32 only)
// the chosen reproduction value is removed in place, leaving the next-level residual.
//
// The scores r . p_k - ||p_k||^2 / 2 of 32 vectors against the 256 values of a sub-quantizer come from the bf16 matrix
// cores: r and p are split into two bf16 parts each and the three products that matter are laid along the contraction,
// K' = [r_hi | r_lo | r_hi] . [p_hi | p_hi | p_lo], padded to steps of 16 (three v_mfma_f32_32x32x16_bf16 per 32 x 32 scores
// at 16 dimensions, one at 4 or fewer).  The reproduction values are the rows of the product, so a lane holds 16
// scores of one vector and keeps best, second best and index in two registers and a tile number.  The scores are a filter: where
// the best does not lead by more than both arithmetics can be off (about 0.1 % of the codes) the wavefront evaluates
// all 256 distances as sum (r - p)^2 in fp32, which is also what decides ties; the codes are those of that arithmetic
// throughout.
//
// A wavefront takes 64 vectors a step, so that the fragments of the values and their norms are read from LDS once for two products,
// and fetches a step's components while the step before is scored.  Bound: the vector unit's three instructions per score and the
// matrix cores beside it, which add up here rather than overlap (10^6 vectors, m = 16: 0.31 ms and 0.11 of 0.62; without the
// insertion of the index, one of the three, 0.52).  Measured (10^6 vectors, d = 128, c = 1024): the first stage of m = 8 from bytes 0.32 ms, from
// fp32 vectors 0.60 and 0.26 for writing them and their residuals; the second, m' = 16, 0.62 and 0.77 ms.
//
// A code that is left unsure costs the wavefront about what 1.1 (16 dimensions) to 2 (2 dimensions) codes cost in fp32 with a
// lane each (less since its components come from registers and the values from LDS), so where the first step of a wavefront leaves many
// unsure (a codebook that has values twice, vectors that share sub-vectors) all its steps are done in fp32, 64 vectors at a time against
// reproduction values from scalar registers.
// At one dimension a score costs as much as a distance and many codes would be unsure: fp32 throughout.  Measured (ms for an add
// of 2^20 vectors, c = 1; one thread per code in fp32 / filter and one code at a time / now): d = 64, m = 64 3.8 / 8.0 / 2.9;
// every value twice, d = 128: m = 64 5.2 / 12.0 / 4.1, m = 16 4.3 / 4.5 / 2.6, m = 8 4.3 / 3.7 / 2.6; d = 256, m = 8 6.3 / 6.8 / 5.2.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

#define ENC_STEPS 4   // 64-vector steps per wavefront

__device__ __forceinline__ uint32_t bf16_near(float v) {   // nearest, ties to even
    const uint32_t b = __float_as_uint(v);
    return (b + 0x7fffu + ((b >> 16) & 1u)) >> 16;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// two values to bf16, nearest, ties to even: one instruction
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
}

// The larger of two numbers in one instruction.  (For fmaxf the compiler first quiets an operand that might be a signalling NaN: a
// fourth instruction a score.  Scores that are no numbers come with a norm that is none, and then no lead counts.)
__device__ __forceinline__ float max_plain(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Where the vectors come from.  MODE 0: fp32 rows R; 1: bytes less their list's centroid; 2 and 3: that less the first-stage value, the
// vectors of the refinement stage (3: where its sub-vectors are the wider ones, so that a run of components has several first-stage
// values).  Differences are rounded one after the other, as if each were written to memory.
// In mode 3 a component's code and value are fetched one by one and nothing is fetched ahead, and at 32 dimensions 28 registers are
// spilled (116 bytes a lane): that stage takes up to 1.6 times as long as from residuals in memory, which the first stage no longer writes.
// 2^18 vectors, from residuals / from bytes: d = 128, m = 32, m' = 8 131 / 133 us, m' = 4 95 / 149; d = 256, m = 64, m' = 8 189 / 286; but
// first stage 354 / 264 and 701 / 509, conversion and first residuals 65 and 136 / 0, and the whole add 907 / 514, 849 / 524 and 1417 / 955 us.
struct EncSrc {
    float* R;
    const uint8_t* X;
    const int32_t* list;
    const float* C;
    const uint8_t* code1;   // first stage: codes [n, m1], values [m1][256][1 << lg1]
    const float* book1;
    int m1, lg1;
};

// A run of SW consecutive components on its way: bytes, centroid, first-stage value (MODE 0: the components themselves in c).
template <int SW, int MODE>
struct EncRun {
    uint32_t w[MODE ? (SW + 3) / 4 : 1];
    float c[SW];
    float p[MODE >= 2 ? SW : 1];
    // components e .. e + SW - 1 of vector i, of list l; k: its first-stage code there (MODE 2)
    __device__ __forceinline__ void fetch(const EncSrc& s, int64_t i, int d, int e, uint32_t l, uint32_t k) {
        if constexpr (MODE == 0) {
            __builtin_memcpy(c, __builtin_assume_aligned(s.R + i * d + e, SW >= 4 ? 16 : 4 * SW), 4 * SW);
        } else {
            __builtin_memcpy(w, __builtin_assume_aligned(s.X + i * d + e, SW), SW);
            __builtin_memcpy(c, __builtin_assume_aligned(s.C + (int64_t)l * d + e, SW >= 4 ? 16 : 4 * SW), 4 * SW);
            if constexpr (MODE == 2)
                __builtin_memcpy(p, __builtin_assume_aligned(s.book1 + ((((int64_t)(e >> s.lg1) * IVFR_KS + k) << s.lg1) + (e & ((1 << s.lg1) - 1))), SW >= 4 ? 16 : 4 * SW), 4 * SW);
            if constexpr (MODE == 3) {
#pragma unroll
                for (int t = 0; t < SW; ++t) {
                    const int j1 = (e + t) >> s.lg1;
                    p[t] = s.book1[(((int64_t)j1 * IVFR_KS + s.code1[i * s.m1 + j1]) << s.lg1) + ((e + t) & ((1 << s.lg1) - 1))];
                }
            }
        }
    }
    __device__ __forceinline__ float value(int t) const {
        if constexpr (MODE == 0) return c[t];
        float v = (float)((w[t >> 2] >> (8 * (t & 3))) & 0xffu) - c[t];
        if constexpr (MODE >= 2) v -= p[t];
        return v;
    }
};

template <int DS, int MODE>
__global__ __launch_bounds__(256, DS == 32 ? 2 : 3) void pq_encode_kernel(EncSrc src, int64_t n, int d, const float* __restrict__ book,
                                                                         int parts, uint8_t* __restrict__ codes, int subtract,
                                                                         int64_t vec_blocks) {
    constexpr int KM = (3 * DS + 15) / 16;
    constexpr int SW = DS >= 16 ? 8 : DS, SEG = DS >= 16 ? DS / 16 : 1;   // with 16 dimensions or more, the halves of a wavefront share them
    constexpr int ND = SW * SEG;
    __shared__ uint4v s_frag[8 * KM * 64];
    __shared__ float s_score[IVFR_KS];
    __shared__ float s_max[4];
    constexpr int BV = DS < 4 ? DS : 4;            // the values in fp32, BV components of all 256 side by side
    constexpr bool BOOK = DS > 1 && DS <= 16;      // (at 32 dimensions a second workgroup would not fit a compute unit)
    typedef float bookv __attribute__((ext_vector_type(BV)));
    __shared__ bookv s_book[BOOK ? DS / BV * IVFR_KS : 1];
    // the workgroups of all sub-quantizers of some vectors run on one XCD (dealt round-robin): they share its lines of the vectors
    const int64_t b = blockIdx.x >> 3;
    const int j = (int)(b % parts);
    const int64_t vb = (b / parts) * 8 + (blockIdx.x & 7);
    if (vb >= vec_blocks) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5;
    const float* cb = book + (int64_t)j * IVFR_KS * DS;
    const int64_t first = vb * (256 * ENC_STEPS) + wave * 64;   // the wavefront's 64 vectors of step s: 256 s behind
    auto codes_of = [&](int64_t i, int e) { return MODE == 2 ? (uint32_t)src.code1[i * src.m1 + (e >> src.lg1)] : 0u; };
    auto whole = [&](int64_t i, float (&y)[DS]) {   // all components of vector i
        const uint32_t l = MODE ? (uint32_t)src.list[i] : 0u;
#pragma unroll
        for (int t = 0; t < DS; t += SW) {
            EncRun<SW, MODE> run;
            run.fetch(src, i, d, j * DS + t, l, codes_of(i, j * DS + t));
#pragma unroll
            for (int x = 0; x < SW; ++x) y[t + x] = run.value(x);
        }
    };
    // the vectors from a step on in fp32, a lane per vector
    auto exact_from = [&](int step) {
        for (; step < ENC_STEPS && first + step * 256 < n; ++step) {
            const int64_t i = first + step * 256 + lane;
            float y[DS];
            whole(i < n ? i : n - 1, y);
            float best = INFINITY;
            int bi = 0;
#pragma unroll 4
            for (int k = 0; k < IVFR_KS; ++k) {
                float s = 0.f;
#pragma unroll
                for (int t = 0; t < DS; ++t) { const float df = y[t] - cb[k * DS + t]; s = fmaf(df, df, s); }
                if (s < best) { best = s; bi = k; }
            }
            if (i >= n) continue;
            if (codes) codes[i * parts + j] = (uint8_t)bi;
            if (MODE == 0 && subtract) {
#pragma unroll
                for (int t = 0; t < DS; ++t) src.R[i * d + j * DS + t] = y[t] - cb[bi * DS + t];
            }
        }
    };
    if constexpr (DS == 1) {
        exact_from(0);
        return;
    }
    // A step's components are fetched a step ahead (not where they fill the registers), what says where they are two steps ahead.
    constexpr bool AHEAD = DS < 16 ? MODE < 3 : (DS == 16 && MODE < 2);
    struct Where { uint32_t l[2]; uint32_t k[2][SEG]; } ahead2;
    EncRun<SW, MODE> ahead[2][SEG];
    auto vector = [&](int step, int u) {   // this lane's vector of tile u
        const int64_t i = first + (int64_t)step * 256 + 32 * u + (lane & 31);
        return i < n ? i : n - 1;
    };
    auto place = [&](int s) { return j * DS + (DS >= 16 ? 16 * s + 8 * h : 0); };
    auto look = [&](int step) {
        if constexpr (MODE != 0) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int64_t i = vector(step, u);
                ahead2.l[u] = (uint32_t)src.list[i];
#pragma unroll
                for (int s = 0; s < SEG; ++s) ahead2.k[u][s] = codes_of(i, place(s));
            }
        }
    };
    auto fetch = [&](int step) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t i = vector(step, u);
#pragma unroll
            for (int s = 0; s < SEG; ++s) ahead[u][s].fetch(src, i, d, place(s), MODE ? ahead2.l[u] : 0u, MODE == 2 ? ahead2.k[u][s] : 0u);
        }
    };
    look(0);
    {
        float p[DS];
        float norm = 0.f;
#pragma unroll
        for (int t = 0; t < DS; ++t) { p[t] = cb[tid * DS + t]; norm = fmaf(p[t], p[t], norm); }
        s_score[tid] = -0.5f * norm;
        if constexpr (BOOK) {
#pragma unroll
            for (int t = 0; t < DS; t += BV)
#pragma unroll
                for (int x = 0; x < BV; ++x) reinterpret_cast<float*>(&s_book[t / BV * IVFR_KS + tid])[x] = p[t + x];
        }
        uint32_t hi[DS], lo[DS];
#pragma unroll
        for (int t = 0; t < DS; ++t) { hi[t] = bf16_near(p[t]); lo[t] = bf16_near(p[t] - __uint_as_float(hi[t] << 16)); }
#pragma unroll
        for (int ks = 0; ks < KM; ++ks)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                uint4v o;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t w[2];
#pragma unroll
                    for (int x = 0; x < 2; ++x) {
                        const int k = 16 * ks + 8 * hh + 2 * e + x;
                        w[x] = k < 2 * DS ? hi[k % DS] : (k < 3 * DS ? lo[k % DS] : 0u);
                    }
                    o[e] = w[0] | (w[1] << 16);
                }
                s_frag[((tid >> 5) * KM + ks) * 64 + hh * 32 + (tid & 31)] = o;
            }
        float mx = norm;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) { const float o = __shfl_xor(mx, off, 64); mx = mx >= o ? mx : o; }
        if (lane == 0) s_max[wave] = mx;
    }
    if (AHEAD) {
        fetch(0);
        look(1);
    }
    __syncthreads();
    const float pmax = sqrtf(fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3])));
    // Two scores, each off by at most M = (||r|| + max ||p||)^2 times: 3 2^-18 / 4 (split), 3 DS 2^-23 / 2 (additions, a whole
    // ulp each), DS 2^-25 (norm), 15 2^-24 (the low bits: a score is at most M / 2); and (DS + 2) 2^-25 for the fp32 distance they
    // are compared with, halved.
    constexpr float margin_rel = 2.f * 1.01f * (2.8611e-6f + 3.f * DS * 5.9605e-8f + (2.f * DS + 2.f) * 2.9803e-8f + 8.9407e-7f);
    for (int step = 0; step < ENC_STEPS; ++step) {
        const int64_t base = first + (int64_t)step * 256;
        if (base >= n) break;   // uniform over the wavefront
        if (!AHEAD) {
            fetch(step);
            if (step + 1 < ENC_STEPS) look(step + 1);
        }
        float v[2][ND];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int t = 0; t < ND; ++t) v[u][t] = ahead[u][t / SW].value(t % SW);
        if (AHEAD && step + 1 < ENC_STEPS) {   // (past the last vector: the last one again)
            fetch(step + 1);
            look(step + 2);
        }
        float r2[2] = {0.f, 0.f};
        uint4v B[2][KM];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int t = 0; t < ND; ++t) r2[u] = fmaf(v[u][t], v[u][t], r2[u]);
            if constexpr (DS >= 16) {   // a step of the contraction lies inside one part, and this half's eight dimensions of it are the lane's
                uint32_t hi[ND / 2], lo[ND / 2];
#pragma unroll
                for (int t = 0; t < ND; t += 2) {
                    hi[t / 2] = bf16_pair(v[u][t], v[u][t + 1]);
                    lo[t / 2] = bf16_pair(v[u][t] - __uint_as_float(hi[t / 2] << 16), v[u][t + 1] - __uint_as_float(hi[t / 2] & 0xffff0000u));
                }
#pragma unroll
                for (int ks = 0; ks < KM; ++ks) {
                    const int s = ks % (DS / 16), part = ks / (DS / 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e) B[u][ks][e] = part == 1 ? lo[4 * s + e] : hi[4 * s + e];
                }
            } else {
                uint32_t hi[ND], lo[ND];
#pragma unroll
                for (int t = 0; t < ND; t += 2) {
                    const uint32_t hp = bf16_pair(v[u][t], v[u][t + 1]);
                    hi[t] = hp & 0xffffu; hi[t + 1] = hp >> 16;
                    const uint32_t lp = bf16_pair(v[u][t] - __uint_as_float(hp << 16), v[u][t + 1] - __uint_as_float(hp & 0xffff0000u));
                    lo[t] = lp & 0xffffu; lo[t + 1] = lp >> 16;
                }
#pragma unroll
                for (int ks = 0; ks < KM; ++ks)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        uint32_t w[2][2];   // [half][value]
#pragma unroll
                        for (int hh = 0; hh < 2; ++hh)
#pragma unroll
                            for (int x = 0; x < 2; ++x) {
                                const int k = 16 * ks + 8 * hh + 2 * e + x, part = k / DS;
                                w[hh][x] = part == 1 ? lo[k % DS] : (part == 0 || part == 2 ? hi[k % DS] : 0u);
                            }
                        B[u][ks][e] = h ? (w[1][0] | (w[1][1] << 16)) : (w[0][0] | (w[0][1] << 16));
                    }
            }
        }
        // The low four bits of a score are replaced by its register's number, so that best and second best are all there is to keep:
        // three instructions a score, and three more per 32 values for the number of their tile.
        float best[2] = {-INFINITY, -INFINITY}, second[2] = {-INFINITY, -INFINITY};
        int bt[2] = {0, 0};
#pragma unroll 2
        for (int T = 0; T < 8; ++T) {
            floatx16 acc[2];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 f = *reinterpret_cast<const float4*>(s_score + 32 * T + 8 * g + 4 * h);
#pragma unroll
                for (int u = 0; u < 2; ++u) { acc[u][4 * g] = f.x; acc[u][4 * g + 1] = f.y; acc[u][4 * g + 2] = f.z; acc[u][4 * g + 3] = f.w; }
            }
#pragma unroll
            for (int ks = 0; ks < KM; ++ks) {
                const bf16x8 A = __builtin_bit_cast(bf16x8, s_frag[(T * KM + ks) * 64 + lane]);
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, __builtin_bit_cast(bf16x8, B[u][ks]), acc[u], 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float before = best[u];
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const float sc = __uint_as_float((__float_as_uint(acc[u][x]) & 0xfffffff0u) | (uint32_t)x);
                    second[u] = __builtin_amdgcn_fmed3f(best[u], second[u], sc);   // second <= best throughout
                    best[u] = max_plain(best[u], sc);
                }
                bt[u] = best[u] != before ? T : bt[u];
            }
        }
        // The halves of the wavefront have different values of the same vectors; from here on lane l has vector base + l.
        const float send_b = h ? best[0] : best[1], send_s = h ? second[0] : second[1], send_r = h ? r2[0] : r2[1];
        float top = h ? best[1] : best[0], next = h ? second[1] : second[0], rr = h ? r2[1] : r2[0];
        auto index = [&](float bb, int tile) { const int x = (int)(__float_as_uint(bb) & 15u); return 32 * tile + 8 * (x >> 2) + (x & 3) + 4 * h; };
        int bi = index(top, h ? bt[1] : bt[0]);
        {
            const float ob = __shfl_xor(send_b, 32, 64), os = __shfl_xor(send_s, 32, 64);
            const int oi = __shfl_xor(index(send_b, h ? bt[0] : bt[1]), 32, 64);
            if (DS >= 16) rr += __shfl_xor(send_r, 32, 64);
            next = fmaxf(fminf(top, ob), fmaxf(next, os));
            if (ob > top || (ob == top && oi < bi)) { top = ob; bi = oi; }
        }
        const int64_t i = base + lane;
        const bool live = i < n;
        const float reach = sqrtf(rr) + pmax;
        // (no lead, or one that is no number, or one of the size of fp32's smallest values, of which the low bits are a large part: the
        // fp32 distances decide)
        uint64_t unsure = __ballot(live && !(top - next > margin_rel * reach * reach + 1.17549435e-38f));
        if (step == 0 && __popcll(unsure) >= (DS >= 16 ? 44 : (DS == 8 ? 32 : (DS == 4 ? 24 : 12)))) {   // uniform over the wavefront
            exact_from(0);
            break;
        }
        while (unsure) {   // the wavefront evaluates all distances of one vector, whose components come from the lanes that hold them
            const int w = __builtin_ctzll(unsure);
            unsure &= unsure - 1;
            float y[DS];
#pragma unroll
            for (int t = 0; t < DS; ++t) {
                const int x = DS >= 16 ? t / 16 * 8 + t % 8 : t, from = (w & 31) + (DS >= 16 ? t / 8 % 2 * 32 : 0);
                const int y0 = __builtin_amdgcn_readlane((int)__float_as_uint(v[0][x]), from), y1 = __builtin_amdgcn_readlane((int)__float_as_uint(v[1][x]), from);
                y[t] = __uint_as_float(w >> 5 ? y1 : y0);
            }
            float s[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int k = 64 * g + lane;
                s[g] = 0.f;
#pragma unroll
                for (int t = 0; t < DS; t += BV) {
                    const bookv p = BOOK ? s_book[t / BV * IVFR_KS + k] : *reinterpret_cast<const bookv*>(cb + k * DS + t);
#pragma unroll
                    for (int x = 0; x < BV; ++x) { const float df = y[t + x] - reinterpret_cast<const float*>(&p)[x]; s[g] = fmaf(df, df, s[g]); }
                }
                s[g] = s[g] < INFINITY ? s[g] : INFINITY;   // nothing below infinity: value 0
            }
            const uint32_t least = (uint32_t)__builtin_amdgcn_readlane(
                (int)wave_fold(__float_as_uint(fminf(fminf(s[0], s[1]), fminf(s[2], s[3]))), 0x7f800000u, [](uint32_t a, uint32_t b) { return a < b ? a : b; }), 63);
            int k = 0;
#pragma unroll
            for (int g = 3; g >= 0; --g) {
                const uint64_t here = __ballot(__float_as_uint(s[g]) == least);
                k = here ? 64 * g + __builtin_ctzll(here) : k;
            }
            if (lane == w) bi = k;
        }
        if (codes && live) codes[i * parts + j] = (uint8_t)bi;
        if (MODE == 0 && subtract) {
            if constexpr (DS >= 16) {
                const int other = __shfl_xor(bi, 32, 64);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int64_t iu = base + 32 * u + (lane & 31);
                    const float* p = cb + (u == h ? bi : other) * DS;
                    if (iu < n) {
#pragma unroll
                        for (int s = 0; s < SEG; ++s)
#pragma unroll
                            for (int e = 0; e < 8; e += 4) {
                                const int o = 16 * s + 8 * h + e, t = 8 * s + e;
                                const float4 f = *reinterpret_cast<const float4*>(p + o);
                                *reinterpret_cast<float4*>(src.R + iu * d + j * DS + o) =
                                    make_float4(v[u][t] - f.x, v[u][t + 1] - f.y, v[u][t + 2] - f.z, v[u][t + 3] - f.w);
                            }
                    }
                }
            } else if (live) {
                float y[DS];
                whole(i, y);
#pragma unroll
                for (int t = 0; t < DS; ++t) src.R[i * d + j * DS + t] = y[t] - cb[bi * DS + t];
            }
        }
    }
}

template <int MODE>
static int launch_encode(const EncSrc& src, int64_t n, int d, const float* book, int parts, uint8_t* codes, bool subtract, hipStream_t st) {
    if (n <= 0 || parts <= 0) return IVFR_OK;
    const int dsub = d / parts;
    const int64_t vec_blocks = (n + 256 * ENC_STEPS - 1) / (256 * ENC_STEPS);
    const dim3 grid((unsigned)((vec_blocks + 7) / 8 * 8 * parts));
#define IVFR_ENC_CASE(D)                                                                                       \
    case D:                                                                                                    \
        if constexpr (D > 1 || MODE != 3) /* no first stage is narrower than one dimension */                  \
            hipLaunchKernelGGL((pq_encode_kernel<D, MODE>), grid, dim3(256), 0, st, src, n, d, book, parts, codes, \
                               subtract ? 1 : 0, vec_blocks);                                                  \
        break
    switch (dsub) {
        IVFR_ENC_CASE(1);
        IVFR_ENC_CASE(2);
        IVFR_ENC_CASE(4);
        IVFR_ENC_CASE(8);
        IVFR_ENC_CASE(16);
        IVFR_ENC_CASE(32);
        default:
            ivfr_set_error("sub-vector width d/m = %d not supported (1, 2, 4, 8, 16, 32)", dsub);
            return IVFR_ERR_INVALID_ARG;
    }
#undef IVFR_ENC_CASE
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// fp32 vectors; with `subtract` the chosen values are taken off in place
int ivfr_launch_pq_encode(float* R, int64_t n, int d, const float* book, int parts, uint8_t* codes, bool subtract,
                          hipStream_t st) {
    EncSrc src = {};
    src.R = R;
    return launch_encode<0>(src, n, d, book, parts, codes, subtract, st);
}

// Both codes of bytes whose lists are known: of what the centroid leaves, and of what the first code leaves of that.
int ivfr_launch_encode_bytes(const ivfr_index* ix, const uint8_t* X, int64_t n, const int32_t* list, uint8_t* codes, uint8_t* rcodes,
                             hipStream_t st) {
    EncSrc src = {};
    src.X = X; src.list = list; src.C = ix->coarse; src.code1 = codes; src.book1 = ix->pq; src.m1 = ix->p.m;
    src.lg1 = __builtin_ctz((unsigned)ix->dsub);
    IVFR_TRY(launch_encode<1>(src, n, ix->p.d, ix->pq, ix->p.m, codes, false, st));
    if (ix->p.m_refine == 0) return IVFR_OK;
    // a run is 8 components at the most
    if (ix->dsub >= std::min(8, ix->dsub_r)) return launch_encode<2>(src, n, ix->p.d, ix->rq, ix->p.m_refine, rcodes, false, st);
    return launch_encode<3>(src, n, ix->p.d, ix->rq, ix->p.m_refine, rcodes, false, st);
}

// ---- stable rank of each vector inside its list ----------------------------------------------
// Insertion order, hence ascending id order, is kept.  The batch is cut into runs of consecutive vectors, cnt is a [runs, c] matrix:
// (1) each run's vectors are ranked and counted per list, (2) a column scan turns the counts into each run's first rank in the list
// (continuing from the entries already in it), (3) the first rank is added to what a vector has inside its run.
//
// Up to RANK_LDS_LISTS lists a run is RANK_RUN vectors and one wavefront, whose counters are in LDS: 64 vectors at a time, a vector's
// equals among the 64 found by a ballot per bit of the list's number.  Bound: the chain of one wavefront's steps, and the matrix.
// Measured (three kernels, with 4096 runs and counters in memory before): 10^6 vectors, c = 1024 141 -> 34 us; 2^20, c = 8192 245 -> 58.
// Beyond, a run is one thread's and its counters are its row of the matrix (4096 of them, cleared first): it counts its run,
// and after the column scan hands out consecutive ranks on a second walk.
#define RANK_RUN 2048
#define RANK_LDS_LISTS 16384
__global__ __launch_bounds__(64) void rank_runs_kernel(const int32_t* __restrict__ list, int64_t n, int c, int bits,
                                                       uint32_t* __restrict__ cnt, uint32_t* __restrict__ rank) {
    extern __shared__ uint32_t s_cnt[];   // [c]
    const int lane = threadIdx.x;
    const int64_t a = (int64_t)blockIdx.x * RANK_RUN, b = a + RANK_RUN < n ? a + RANK_RUN : n;
    uint32_t next = a + lane < b ? (uint32_t)list[a + lane] : 0u;
    for (int l = lane; l < c; l += 64) s_cnt[l] = 0;
    __syncthreads();
    for (int64_t i = a + lane; i - lane < b; i += 64) {   // uniform
        const uint32_t l = next;
        next = i + 64 < b ? (uint32_t)list[i + 64] : 0u;
        const bool live = i < b;
        uint64_t same = __ballot(live);
        for (int x = 0; x < bits; ++x) {
            const bool one = (l >> x) & 1u;
            const uint64_t m = __ballot(one);
            same &= one ? m : ~m;
        }
        const uint32_t before = s_cnt[l];   // (l < c, also where there is no vector)
        if (live) {
            rank[i] = before + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
            if (__builtin_ctzll(same) == lane) s_cnt[l] = before + (uint32_t)__popcll(same);
        }
        __syncthreads();   // one wavefront: the order of its LDS accesses
    }
    for (int l = lane; l < c; l += 64) cnt[(int64_t)blockIdx.x * c + l] = s_cnt[l];
}

__global__ __launch_bounds__(256) void rank_add_kernel(const int32_t* __restrict__ list, int64_t n, int c,
                                                       const uint32_t* __restrict__ cnt, uint32_t* __restrict__ rank) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) rank[i] += cnt[i / RANK_RUN * c + list[i]];
}

__global__ void rank_count_kernel(const int32_t* __restrict__ list, int64_t n, int64_t run, int c,
                                  uint32_t* __restrict__ cnt) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t a = t * run, b = a + run < n ? a + run : n;
    uint32_t* row = cnt + t * c;
    // (additions without a result: nothing waits for them.  Read, add and write, a chain of memory latencies, took 0.16 ms per 2^20.)
#pragma unroll 8
    for (int64_t i = a; i < b; ++i) atomicAdd(&row[list[i]], 1u);
}

// Columns are scanned by 64 x 16 threads: thread (s, l) sums its sixteenth of column l, the sixteen sums are
// prefixed in LDS, and a second walk writes the run's first ranks.  (One thread per column, a chain of T dependent
// steps on c threads, took 0.91 ms per 2^20 vectors at c = 1024.)
#define COLSCAN_SEGS 16
__global__ __launch_bounds__(64 * COLSCAN_SEGS) void rank_colscan_kernel(uint32_t* __restrict__ cnt, int T, int c,
                                                                         unsigned long long* __restrict__ list_fill) {
    __shared__ uint32_t sums[COLSCAN_SEGS][64];
    const int x = threadIdx.x & 63, seg = threadIdx.x >> 6;
    const int l = blockIdx.x * 64 + x;
    const int t0 = (int)((int64_t)T * seg / COLSCAN_SEGS), t1 = (int)((int64_t)T * (seg + 1) / COLSCAN_SEGS);
    uint32_t sum = 0;
    if (l < c) {
        int t = t0;
        for (; t + 8 <= t1; t += 8) {   // eight loads in flight
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = cnt[(int64_t)(t + u) * c + l];
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += v[u];
        }
        for (; t < t1; ++t) sum += cnt[(int64_t)t * c + l];
    }
    sums[seg][x] = sum;
    const unsigned long long fill = l < c ? list_fill[l] : 0ull;
    __syncthreads();   // the sums are there, and every thread has read the old fill
    if (l >= c) return;
    uint32_t running = (uint32_t)fill;   // ranks are 32-bit
    for (int s = 0; s < seg; ++s) running += sums[s][x];
    if (seg == COLSCAN_SEGS - 1) list_fill[l] = fill + (running + sum - (uint32_t)fill);
    {
        int t = t0;
        for (; t + 8 <= t1; t += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = cnt[(int64_t)(t + u) * c + l];
#pragma unroll
            for (int u = 0; u < 8; ++u) { cnt[(int64_t)(t + u) * c + l] = running; running += v[u]; }
        }
        for (; t < t1; ++t) { const uint32_t v = cnt[(int64_t)t * c + l]; cnt[(int64_t)t * c + l] = running; running += v; }
    }
}

__global__ void rank_assign_kernel(const int32_t* __restrict__ list, int64_t n, int64_t run, int c,
                                   uint32_t* __restrict__ cnt, uint32_t* __restrict__ rank) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t a = t * run, b = a + run < n ? a + run : n;
    uint32_t* row = cnt + t * c;
    // Eight additions in flight: a thread's additions to one address take effect in its order, and no other thread adds to its row.
    int64_t i = a;
    for (; i + 8 <= b; i += 8) {
        uint32_t r[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = (uint32_t)list[i + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) r[u] = atomicAdd(&row[r[u]], 1u);
#pragma unroll
        for (int u = 0; u < 8; ++u) rank[i + u] = r[u];
    }
    for (; i < b; ++i) rank[i] = atomicAdd(&row[list[i]], 1u);
}

// runs of a batch of n vectors: rows of the matrix of counts
static int rank_runs(int64_t n, int c) {
    if (c <= RANK_LDS_LISTS) return (int)((n + RANK_RUN - 1) / RANK_RUN);
    int T = 4096;
    while ((int64_t)T * c > (1ll << 27) && T > 64) T >>= 1;
    return T;
}
size_t ivfr_rank_scratch_bytes(int64_t n, int c) { return (size_t)rank_runs(n, c) * c * sizeof(uint32_t); }

int ivfr_launch_list_ranks(const int32_t* list, int64_t n, int c, unsigned long long* list_fill, void* scratch, uint32_t* rank, hipStream_t st) {
    if (n <= 0) return IVFR_OK;
    const int T = rank_runs(n, c);
    uint32_t* cnt = static_cast<uint32_t*>(scratch);
    const dim3 scan_grid((unsigned)((c + 63) / 64));
    if (c <= RANK_LDS_LISTS) {
        int bits = 0;
        while ((1 << bits) < c) ++bits;
        const size_t lds = (size_t)c * sizeof(uint32_t);
        hipLaunchKernelGGL(rank_runs_kernel, dim3((unsigned)T), dim3(64), lds, st, list, n, c, bits, cnt, rank);
        hipLaunchKernelGGL(rank_colscan_kernel, scan_grid, dim3(64 * COLSCAN_SEGS), 0, st, cnt, T, c, list_fill);
        hipLaunchKernelGGL(rank_add_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, list, n, c, cnt, rank);
        IVFR_HIP(hipGetLastError());
        return IVFR_OK;
    }
    int64_t run = (n + T - 1) / T;
    IVFR_HIP(hipMemsetAsync(cnt, 0, (size_t)T * c * sizeof(uint32_t), st));
    hipLaunchKernelGGL(rank_count_kernel, dim3((T + 63) / 64), dim3(64), 0, st, list, n, run, c, cnt);
    hipLaunchKernelGGL(rank_colscan_kernel, scan_grid, dim3(64 * COLSCAN_SEGS), 0, st, cnt, T, c, list_fill);
    hipLaunchKernelGGL(rank_assign_kernel, dim3((T + 63) / 64), dim3(64), 0, st, list, n, run, c, cnt, rank);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Move one staged batch into the finished, list-sorted arrays: the dense code stream of the list scan and the
// per-entry record (id, list, code, refinement code) that the re-rank and the tie-breaks by id read.
__global__ __launch_bounds__(256) void scatter_kernel(const int32_t* __restrict__ list,
                                                      const uint32_t* __restrict__ rank,
                                                      int64_t id_base,
                                                      const uint8_t* __restrict__ codes_in,
                                                      const uint8_t* __restrict__ rcodes_in, int64_t n, int m, int mr,
                                                      const uint32_t* __restrict__ list_start,
                                                      uint8_t* __restrict__ codes, uint8_t* __restrict__ rec,
                                                      int rec_stride) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int l = list[i];
    uint64_t dst = (uint64_t)list_start[l] + rank[i];
    const uint32_t* s = reinterpret_cast<const uint32_t*>(codes_in + i * m);
    uint32_t* o = reinterpret_cast<uint32_t*>(codes + dst * m);
    uint32_t* r = reinterpret_cast<uint32_t*>(rec + dst * rec_stride);
    r[0] = (uint32_t)(id_base + i);
    r[1] = (uint32_t)l;
    for (int t = 0; t < m / 4; ++t) { o[t] = s[t]; r[2 + t] = s[t]; }
    if (mr > 0) {
        const uint32_t* sr = reinterpret_cast<const uint32_t*>(rcodes_in + i * mr);
        for (int t = 0; t < mr / 4; ++t) r[2 + m / 4 + t] = sr[t];
    }
}

int ivfr_launch_scatter(const StagedChunk& ch, int m, int mr, const uint32_t* list_start, uint8_t* codes,
                        uint8_t* rec, int rec_stride, hipStream_t st) {
    if (ch.n <= 0) return IVFR_OK;
    hipLaunchKernelGGL(scatter_kernel, dim3((unsigned)((ch.n + 255) / 256)), dim3(256), 0, st, ch.list, ch.rank,
                       ch.id_base, ch.codes, ch.rcodes, ch.n, m, mr, list_start, codes, rec, rec_stride);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// The index's dense arrays (ids, codes or refinement codes of entries i0 .. i0 + n - 1 in list order, `words` 32-bit words
// per entry) <-> the padded code stream and the per-entry records, for import and export.  One thread per word, so that
// a wavefront reads and writes runs of consecutive words on the dense side and whole codes on the other.  An entry's list
// is the last one that starts at or before it: the workgroup's first and last entries are searched for in all
// offsets, the others only between those two.
enum { ARR_IDS = 0, ARR_CODES = 1, ARR_RCODES = 2 };
template <bool IMPORT>
__global__ __launch_bounds__(256) void entry_words_kernel(int which, int64_t i0, int64_t n, int words, int m, int c,
                                                          const int64_t* __restrict__ offsets,
                                                          const uint32_t* __restrict__ list_start,
                                                          uint8_t* __restrict__ codes, uint8_t* __restrict__ rec,
                                                          int rec_stride, uint32_t* __restrict__ dense) {
    __shared__ int ends[2];
    const int64_t w0 = (int64_t)blockIdx.x * 256;
    const int64_t i_first = i0 + w0 / words;
    const int64_t w_last = w0 + 255 < n * words ? w0 + 255 : n * words - 1;
    const int64_t i_last = i0 + w_last / words;
    auto find = [&](int64_t i, int lo, int hi) {   // last list in [lo, hi) with offsets[list] <= i
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (offsets[mid] <= i) lo = mid; else hi = mid;
        }
        return lo;
    };
    if (threadIdx.x < 2) ends[threadIdx.x] = find(threadIdx.x ? i_last : i_first, 0, c);
    __syncthreads();
    const int64_t w = w0 + threadIdx.x;
    if (w >= n * words) return;
    const int64_t i = i0 + w / words;
    const int k = (int)(w % words);
    const int l = find(i, ends[0], ends[1] + 1);
    const uint64_t slot = (uint64_t)list_start[l] + (uint64_t)(i - offsets[l]);
    uint32_t* r = reinterpret_cast<uint32_t*>(rec + slot * rec_stride);
    uint32_t* stream = reinterpret_cast<uint32_t*>(codes + slot * m);
    if (IMPORT) {
        const uint32_t v = dense[w];
        if (which == ARR_IDS) { r[0] = v; r[1] = (uint32_t)l; }
        else if (which == ARR_CODES) { stream[k] = v; r[2 + k] = v; }
        else r[2 + m / 4 + k] = v;
    } else {
        dense[w] = which == ARR_IDS ? r[0] : (which == ARR_CODES ? stream[k] : r[2 + m / 4 + k]);
    }
}

int ivfr_launch_entry_words(const ivfr_index* ix, bool import, int which, int64_t i0, int64_t n, const int64_t* offsets,
                            uint32_t* dense, hipStream_t st) {
    const int words = which == ARR_IDS ? 1 : (which == ARR_CODES ? ix->p.m : ix->p.m_refine) / 4;
    if (n <= 0 || words <= 0) return IVFR_OK;
    const dim3 grid((unsigned)((n * words + 255) / 256));
#define IVFR_WORDS(IMP)                                                                                            \
    hipLaunchKernelGGL(entry_words_kernel<IMP>, grid, dim3(256), 0, st, which, i0, n, words, ix->p.m, ix->p.c, offsets, \
                       ix->list_start, ix->codes, ix->rec, ix->rec_stride, dense)
    if (import) IVFR_WORDS(true);
    else IVFR_WORDS(false);
#undef IVFR_WORDS
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// ---- k-means update (Lloyd): centroid = mean of its assigned points ---------------------------
// Sums are accumulated as 64-bit fixed point (2^-20 resolution) with integer atomics, so the
// result does not depend on the order in which threads arrive.
#define KM_SCALE 1048576.0f

// Rows by centroid: every row takes its place among its centroid's rows (km_count), the centroids' rows follow one another
// (km_offsets, km_place), and groups of threads walk over runs of KM_RUN rows in that order, four dimensions a thread, with one
// global addition per centroid and run.  (An addition per component queued up at the c d sums: 10^5 rows, c = 1024, d = 128
// 100 us, now 33 with all four kernels.)
#define KM_RUN 32
//
// The counting: the workgroup ranks its KM_COUNT rows per centroid in LDS and takes their places with one addition per centroid that
// occurs (an addition per row: 24 us for 10^5 rows, now 5).  More centroids than LDS counters: an addition per row.
#define KM_COUNT 2048
#define KM_LDS_LISTS 16384
template <bool LDS>
__global__ __launch_bounds__(1024) void km_count_kernel(const int32_t* __restrict__ assign, int64_t n, int c, uint32_t* __restrict__ cnt,
                                                        uint32_t* __restrict__ rank) {
    extern __shared__ uint32_t s_list[];   // [c]
    const int64_t i0 = (int64_t)blockIdx.x * KM_COUNT + threadIdx.x;
    if constexpr (!LDS) {
#pragma unroll
        for (int u = 0; u < KM_COUNT / 1024; ++u)
            if (i0 + 1024 * u < n) rank[i0 + 1024 * u] = atomicAdd(&cnt[assign[i0 + 1024 * u]], 1u);
        return;
    }
    int l[KM_COUNT / 1024];
    uint32_t r[KM_COUNT / 1024];
#pragma unroll
    for (int u = 0; u < KM_COUNT / 1024; ++u) l[u] = i0 + 1024 * u < n ? assign[i0 + 1024 * u] : -1;
    for (int x = threadIdx.x; x < c; x += 1024) s_list[x] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KM_COUNT / 1024; ++u) r[u] = l[u] >= 0 ? atomicAdd(&s_list[l[u]], 1u) : 0u;
    __syncthreads();
    for (int x = threadIdx.x; x < c; x += 1024) {
        const uint32_t here = s_list[x];
        if (here) s_list[x] = atomicAdd(&cnt[x], here);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < KM_COUNT / 1024; ++u)
        if (l[u] >= 0) rank[i0 + 1024 * u] = s_list[l[u]] + r[u];
}

// one workgroup: exclusive prefix of the c counters; they are left at zero for the next iteration
__global__ __launch_bounds__(1024) void km_offsets_kernel(uint32_t* __restrict__ cnt, int c, uint32_t* __restrict__ off,
                                                          unsigned long long* __restrict__ counts) {
    __shared__ uint32_t wtot[16];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t carry = 0;
    for (int base = 0; base < c; base += 1024) {
        const int l = base + tid;
        const uint32_t v = l < c ? cnt[l] : 0u;
        const uint32_t inc = wave_prefix(v);
        if (lane == 63) wtot[wv] = inc;
        __syncthreads();
        uint32_t before = carry, all = 0;
#pragma unroll
        for (int x = 0; x < 16; ++x) { before += x < wv ? wtot[x] : 0u; all += wtot[x]; }
        if (l < c) { off[l] = before + inc - v; counts[l] = v; cnt[l] = 0; }
        carry += all;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void km_place_kernel(const int32_t* __restrict__ assign, int64_t n, const uint32_t* __restrict__ off,
                                                       const uint32_t* __restrict__ rank, uint2* __restrict__ order) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t l = (uint32_t)assign[i];
    order[off[l] + rank[i]] = make_uint2((uint32_t)i, l);
}

__global__ __launch_bounds__(256) void km_sum_rows_kernel(const uint8_t* __restrict__ X, int64_t n, int d,
                                                          const uint2* __restrict__ order,
                                                          unsigned long long* __restrict__ sums) {
    const int per = d < 1024 ? d / 4 : 256, walkers = 256 / per;   // blockIdx.y: 1024 dimensions
    const int e = 4 * ((int)threadIdx.x % per) + 1024 * (int)blockIdx.y, walker = (int)threadIdx.x / per;
    if (walker >= walkers || e >= d) return;
    const int64_t i0 = ((int64_t)blockIdx.x * walkers + walker) * KM_RUN;
    const int64_t i1 = i0 + KM_RUN < n ? i0 + KM_RUN : n;
    if (i0 >= i1) return;
    uint32_t list = order[i0].y;
    uint32_t s[4] = {0, 0, 0, 0};
    auto flush = [&]() {
#pragma unroll
        for (int t = 0; t < 4; ++t) { atomicAdd(&sums[(int64_t)list * d + e + t], (unsigned long long)s[t] * (unsigned long long)KM_SCALE); s[t] = 0; }
    };
    for (int64_t i = i0; i < i1; i += 4) {
        uint2 o[4];
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) o[u] = order[i + u < i1 ? i + u : i1 - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const uint32_t*>(X + (int64_t)o[u].x * d + e);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i + u >= i1) break;
            if (o[u].y != list) { flush(); list = o[u].y; }
            s[0] += v[u] & 0xff; s[1] += (v[u] >> 8) & 0xff; s[2] += (v[u] >> 16) & 0xff; s[3] += v[u] >> 24;
        }
    }
    flush();
}

// Product-quantizer variant: point i, sub-quantizer j is assigned to centroid codes[i][j].  A workgroup sums a run of
// points for one sub-quantizer in LDS (256 centroids x dsub 64-bit sums, 32 KB at 16 dimensions) and adds its sums to the
// global ones at the end: 4096 points per 256 dsub global atomics instead of 4096 dsub of them, which queued up at the
// 256 dsub addresses.  Eight points of a thread are in flight at a time.  Measured (10^5 points, d = 128): 157 -> 31 us (44 one at a time).
#define KM_POINTS 4096
__global__ __launch_bounds__(512) void km_accum_pq_kernel(const float* __restrict__ R, int64_t n, int d, int parts,
                                                          const uint8_t* __restrict__ codes,
                                                          unsigned long long* __restrict__ sums,
                                                          unsigned long long* __restrict__ counts) {
    extern __shared__ unsigned long long s_sum[];   // [256][dsub], then counts [256]
    const int j = blockIdx.x % parts, dsub = d / parts;
    const int64_t i0 = (int64_t)(blockIdx.x / parts) * KM_POINTS;
    const int64_t i1 = i0 + KM_POINTS < n ? i0 + KM_POINTS : n;
    unsigned long long* s_cnt = s_sum + IVFR_KS * dsub;
    for (int k = threadIdx.x; k < IVFR_KS * (dsub + 1); k += 512) s_sum[k] = 0ull;
    __syncthreads();
    // dsub (a power of two up to 32) neighbouring threads take one point
    const int t = threadIdx.x % dsub, step = 512 / dsub;
    constexpr int B = 8;   // points in flight
    for (int64_t i = i0 + threadIdx.x / dsub; i < i1; i += (int64_t)B * step) {
        int k[B];
        float v[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            const int64_t p = i + (int64_t)u * step < i1 ? i + (int64_t)u * step : i;
            k[u] = codes[p * parts + j];
            v[u] = R[p * d + j * dsub + t];
        }
#pragma unroll
        for (int u = 0; u < B; ++u) {
            if (i + (int64_t)u * step >= i1) break;
            atomicAdd(&s_sum[k[u] * dsub + t], (unsigned long long)__float2ll_rn(v[u] * KM_SCALE));
            if (t == 0) atomicAdd(&s_cnt[k[u]], 1ull);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < IVFR_KS * dsub; k += 512)
        if (s_sum[k]) atomicAdd(&sums[(int64_t)j * IVFR_KS * dsub + k], s_sum[k]);
    for (int k = threadIdx.x; k < IVFR_KS; k += 512)
        if (s_cnt[k]) atomicAdd(&counts[j * IVFR_KS + k], s_cnt[k]);
}

// cent[g][t] = sums / counts where counts > 0 (an empty cluster keeps its centroid); width = floats per centroid.  Sums and counts
// are left at zero for the next iteration; a workgroup has whole centroids, so that a count is read by all before it is cleared.
__global__ __launch_bounds__(256) void km_update_kernel(float* __restrict__ cent, int64_t groups, int width,
                                                        unsigned long long* __restrict__ sums,
                                                        unsigned long long* __restrict__ counts) {
    const int per = width < 256 ? 256 / width : 1;   // centroids per workgroup
    const int64_t g0 = (int64_t)blockIdx.x * per;
    const int64_t g1 = g0 + per < groups ? g0 + per : groups;
    for (int64_t i = g0 * width + threadIdx.x; i < g1 * width; i += 256) {
        const unsigned long long cn = counts[i / width];
        if (cn == 0) continue;
        const double s = (double)(long long)sums[i] / (double)KM_SCALE;
        cent[i] = (float)(s / (double)cn);
        sums[i] = 0ull;
    }
    __syncthreads();
    for (int64_t g = g0 + threadIdx.x; g < g1; g += 256) counts[g] = 0ull;
}

// scratch of the launch below (n < 2^32): the order of the rows, their ranks, offsets and counters of the centroids;
// the counters, at the start, have to be zero at first
size_t ivfr_km_scratch_bytes(int64_t n, int c) { return (size_t)c * 8 + (size_t)n * 12; }

int ivfr_launch_km_accum_rows(const uint8_t* X, int64_t n, int d, int c, const int32_t* assign, unsigned long long* sums,
                              unsigned long long* counts, void* scratch, hipStream_t st) {
    uint32_t* cnt = static_cast<uint32_t*>(scratch);
    uint32_t* off = cnt + c;
    uint2* order = reinterpret_cast<uint2*>(off + c);
    uint32_t* rank = reinterpret_cast<uint32_t*>(order + n);
    const dim3 rows((unsigned)((n + 255) / 256));
    const dim3 count_grid((unsigned)((n + KM_COUNT - 1) / KM_COUNT));
    if (c <= KM_LDS_LISTS) {
        const size_t lds = (size_t)c * sizeof(uint32_t);
        hipLaunchKernelGGL(km_count_kernel<true>, count_grid, dim3(1024), lds, st, assign, n, c, cnt, rank);
    } else {
        hipLaunchKernelGGL(km_count_kernel<false>, count_grid, dim3(1024), 0, st, assign, n, c, cnt, rank);
    }
    hipLaunchKernelGGL(km_offsets_kernel, dim3(1), dim3(1024), 0, st, cnt, c, off, counts);
    hipLaunchKernelGGL(km_place_kernel, rows, dim3(256), 0, st, assign, n, off, rank, order);
    const int64_t per_block = (int64_t)(d < 1024 ? 256 / (d / 4) : 1) * KM_RUN;
    hipLaunchKernelGGL(km_sum_rows_kernel, dim3((unsigned)((n + per_block - 1) / per_block), (unsigned)((d + 1023) / 1024)), dim3(256),
                       0, st, X, n, d, order, sums);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

static size_t km_accum_pq_lds(int dsub) { return (size_t)IVFR_KS * (dsub + 1) * sizeof(unsigned long long); }   // 66 KB at 32 dimensions

int ivfr_launch_km_accum_pq(const float* R, int64_t n, int d, int parts, const uint8_t* codes,
                            unsigned long long* sums, unsigned long long* counts, hipStream_t st) {
    const int64_t runs = (n + KM_POINTS - 1) / KM_POINTS;
    const size_t lds = km_accum_pq_lds(d / parts);
    hipLaunchKernelGGL(km_accum_pq_kernel, dim3((unsigned)(runs * parts)), dim3(512), lds, st, R, n, d, parts, codes, sums, counts);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

int ivfr_launch_km_update(float* cent, int64_t groups, int width, unsigned long long* sums, unsigned long long* counts,
                          hipStream_t st) {
    const int64_t per = width < 256 ? 256 / width : 1;
    hipLaunchKernelGGL(km_update_kernel, dim3((unsigned)((groups + per - 1) / per)), dim3(256), 0, st, cent, groups, width,
                       sums, counts);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Initial centroids: rows of X selected by idx -> out; part p (of `parts`) takes columns p * width .. of its own
// `count` rows idx[p * count ..].
template <class T>
__global__ __launch_bounds__(256) void gather_rows_kernel(const T* __restrict__ X, int d, int width, int parts,
                                                          const int64_t* __restrict__ idx, int count,
                                                          float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)parts * count * width) return;
    const int t = (int)(i % width);
    const int64_t r = i / width;   // p * count + row of the part
    out[i] = (float)X[idx[r] * d + (r / count) * width + t];
}

template <class T>
static int gather_rows(const T* X, int d, int width, int parts, const int64_t* idx, int count, float* out, hipStream_t st) {
    const int64_t total = (int64_t)parts * count * width;
    hipLaunchKernelGGL(gather_rows_kernel<T>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, X, d, width, parts,
                       idx, count, out);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}
int ivfr_launch_gather_rows(const float* X, int d, int width, int parts, const int64_t* idx, int count, float* out, hipStream_t st) {
    return gather_rows(X, d, width, parts, idx, count, out, st);
}
int ivfr_launch_gather_byte_rows(const uint8_t* X, int d, const int64_t* idx, int count, float* out, hipStream_t st) {
    return gather_rows(X, d, d, 1, idx, count, out, st);
}

// ---- initial draws ------------------------------------------------------------------------------------------------
// Part p draws `count` distinct rows of [0, n): those with the smallest hashes of (seed, salt0 + p, row), equal hashes by
// row, written in ascending order.
//
// Hashes are spread evenly, so the rows whose hash lies below (count + 8 sqrt(count) + 16) / n of the range hold the wanted ones
// except by a chance beyond eight deviations: draw_candidates_kernel lists them by runs of rows, on the whole chip, and one
// workgroup per part selects among them, the count-th smallest as in every other selection, and writes them in order by a running prefix.
// Where a run lists more than its place takes, fewer than `count` are listed in all, or more than half of the rows are wanted, that
// workgroup looks at all rows instead.  Bound: latency; the sweeps of one workgroup over 10^5 hashes were the whole time.  Measured
// (1024 of 10^5 rows): 143 us with one workgroup for everything, 4 + 12 us now.
__host__ __device__ inline uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__device__ __forceinline__ uint64_t draw_key(uint64_t seed, uint64_t salt) { return mix64(seed * 0x9E3779B97F4A7C15ull + salt); }
__device__ __forceinline__ uint64_t draw_hash(uint64_t key, int64_t row) { return mix64(key + (uint64_t)(row + 1) * 0x9E3779B97F4A7C15ull); }

#define DRAW_RUNS (2 * SEL_T)   // runs of rows at the most

// How the rows are cut up; runs == 0: no candidates are listed.
struct DrawPlan {
    uint64_t below;    // hashes looked for
    int run, runs, room;   // rows per run, runs, places per run
};

static DrawPlan draw_plan(int64_t n, int count, double surplus) {
    DrawPlan p = {0, 0, 0, 0};
    const double share = ((double)count + surplus * sqrt((double)count) + 2.0 * surplus) / (double)n;
    if (share > 0.5 || n >= 0xFFFFFFFFll) return p;
    p.below = (uint64_t)(share * 18446744073709551616.0);
    p.run = (int)((std::max<int64_t>(1024, (n + DRAW_RUNS - 1) / DRAW_RUNS) + 255) / 256 * 256);
    p.runs = (int)((n + p.run - 1) / p.run);
    const double each = share * p.run;
    p.room = (int)(each + surplus * sqrt(each) + 2.0 * surplus);
    return p;
}

// per part: counts [runs], candidates [runs][room], the same without gaps [runs * room]
static size_t draw_words(const DrawPlan& p) { return (size_t)p.runs * (1 + 2 * (size_t)p.room); }
size_t ivfr_draw_scratch_bytes(int parts, int64_t n, int count, double surplus) { return parts * draw_words(draw_plan(n, count, surplus)) * sizeof(uint32_t); }

__global__ __launch_bounds__(256) void draw_candidates_kernel(uint64_t seed, uint64_t salt0, int64_t n, DrawPlan p, size_t words,
                                                              uint32_t* __restrict__ scratch) {
    __shared__ uint32_t s_cnt[2][4];
    const int part = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t* const out = scratch + part * words;
    const uint64_t key = draw_key(seed, salt0 + part);
    const int64_t r0 = (int64_t)blockIdx.x * p.run;
    uint32_t before = 0;
    for (int t = 0; t < p.run; t += 256) {   // uniform
        const int64_t row = r0 + t + tid;
        const bool hit = row < n && draw_hash(key, row) < p.below;
        const uint64_t mask = __ballot(hit);
        const int parity = (t >> 8) & 1;
        if (lane == 0) s_cnt[parity][wave] = __popcll(mask);
        __syncthreads();   // (one barrier a step: the next one but one writes here again behind the next)
        uint32_t at = before;
#pragma unroll
        for (int w = 0; w < 4; ++w) { at += w < wave ? s_cnt[parity][w] : 0u; before += s_cnt[parity][w]; }
        at += __popcll(mask & ((1ull << lane) - 1ull));
        if (hit && at < (uint32_t)p.room) out[p.runs + (size_t)blockIdx.x * p.room + at] = (uint32_t)row;
    }
    if (tid == 0) out[blockIdx.x] = before;
}

struct HashSrc {   // of all rows, or of those listed
    uint64_t key;
    int64_t n;
    const uint32_t* rows;
    static constexpr uint32_t stop = SEL_RC;
    __device__ __forceinline__ int64_t row(int64_t i) const { return rows ? (int64_t)rows[i] : i; }
    __device__ __forceinline__ uint64_t hash(int64_t i) const { return draw_hash(key, row(i)); }
    __device__ __forceinline__ uint32_t lo(uint32_t ref) const { return (uint32_t)hash(ref); }
    template <class B> __device__ __forceinline__ void sweep(B body) const {
        for (int64_t i = threadIdx.x; i < n; i += SEL_T) body((uint32_t)(hash(i) >> 32), (uint32_t)i);
    }
};

__global__ __launch_bounds__(SEL_T) void draw_rows_kernel(uint64_t seed, uint64_t salt0, int64_t n, int count, DrawPlan p, size_t words,
                                                          uint32_t* __restrict__ scratch, int64_t* __restrict__ out) {
    __shared__ SelShared sh;
    __shared__ uint32_t s_less, s_over;
    __shared__ uint32_t s_cnt[2][2][SEL_T / 64];
    __shared__ uint32_t s_pre[DRAW_RUNS + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    HashSrc s{draw_key(seed, salt0 + blockIdx.x), n, nullptr};
    out += (int64_t)blockIdx.x * count;
    if (tid == 0) { s_less = 0; s_over = 0; }
    __syncthreads();
    if (p.runs > 0) {   // uniform
        const uint32_t* listed = scratch + blockIdx.x * words;
        const uint32_t a = 2 * tid < p.runs ? listed[2 * tid] : 0u, b = 2 * tid + 1 < p.runs ? listed[2 * tid + 1] : 0u;
        if (a > (uint32_t)p.room || b > (uint32_t)p.room) s_over = 1;
        const uint32_t inc = wave_prefix(a + b);
        if (lane == 63) s_cnt[0][0][wave] = inc;
        __syncthreads();
        uint32_t at = inc - a - b;
#pragma unroll
        for (int w = 0; w < SEL_T / 64; ++w) at += w < wave ? s_cnt[0][0][w] : 0u;
        s_pre[2 * tid] = at;
        s_pre[2 * tid + 1] = at + a;
        if (tid == SEL_T - 1) s_pre[DRAW_RUNS] = at + a + b;
        __syncthreads();
        const uint32_t total = s_pre[DRAW_RUNS];
        if (!s_over && total >= (uint32_t)count) {   // uniform
            uint32_t* rows = scratch + blockIdx.x * words + p.runs + (size_t)p.runs * p.room;
            for (uint32_t i = tid; i < total; i += SEL_T) {
                int lo = 0, hi = p.runs;   // last run with s_pre[run] <= i
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (s_pre[mid] <= i) lo = mid; else hi = mid;
                }
                rows[i] = listed[p.runs + (size_t)lo * p.room + (i - s_pre[lo])];
            }
            s.n = total;
            s.rows = rows;
        }
        __syncthreads();
    }
    const uint64_t pivot = count < s.n ? kth_key(sh, s, (uint32_t)count) : ~0ull;
    uint32_t less = 0;
    for (int64_t i = tid; i < s.n; i += SEL_T) less += s.hash(i) < pivot ? 1u : 0u;
    if (less) atomicAdd(&s_less, less);
    __syncthreads();
    const uint32_t equal = (uint32_t)count - s_less;   // rows with the pivot's hash that are still wanted
    uint32_t before_less = 0, before_equal = 0, parity = 0;
    for (int64_t i0 = 0; i0 < s.n; i0 += SEL_T) {
        const uint64_t h = i0 + tid < s.n ? s.hash(i0 + tid) : 0ull;
        const bool is_less = i0 + tid < s.n && h < pivot, is_equal = i0 + tid < s.n && h == pivot;
        const uint64_t ml = __ballot(is_less), me = __ballot(is_equal);
        if (lane == 0) { s_cnt[parity][0][wave] = __popcll(ml); s_cnt[parity][1][wave] = __popcll(me); }
        __syncthreads();
        uint32_t l = before_less, e = before_equal;
#pragma unroll
        for (int w = 0; w < SEL_T / 64; ++w) {
            const uint32_t cl = s_cnt[parity][0][w], ce = s_cnt[parity][1][w];
            l += w < wave ? cl : 0u;
            e += w < wave ? ce : 0u;
            before_less += cl;
            before_equal += ce;
        }
        parity ^= 1u;
        const uint64_t below = (1ull << lane) - 1ull;
        l += __popcll(ml & below);
        e += __popcll(me & below);
        const uint32_t at = l + (e < equal ? e : equal);
        if (is_less || (is_equal && e < equal)) out[at] = s.row(i0 + tid);
    }
}

// scratch: ivfr_draw_scratch_bytes(parts, n, count, surplus); surplus: deviations by which candidates and places exceed what is expected
int ivfr_launch_draw_rows(uint64_t seed, uint64_t salt0, int parts, int64_t n, int count, int64_t* out, void* scratch, hipStream_t st,
                          double surplus) {
    const DrawPlan p = draw_plan(n, count, surplus);
    const size_t words = draw_words(p);
    if (p.runs > 0)
        hipLaunchKernelGGL(draw_candidates_kernel, dim3((unsigned)p.runs, (unsigned)parts), dim3(256), 0, st, seed, salt0, n, p, words,
                           static_cast<uint32_t*>(scratch));
    hipLaunchKernelGGL(draw_rows_kernel, dim3((unsigned)parts), dim3(SEL_T), 0, st, seed, salt0, n, count, p, words,
                       static_cast<uint32_t*>(scratch), out);
    IVFR_HIP(hipGetLastError());
    return IVFR_OK;
}

// Dynamic LDS beyond 48 KB has to be allowed per kernel and device: for the largest counters, so that no index takes away what another
// one's call, in another thread, is about to launch with.
int ivfr_encode_init() {
    IVFR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(rank_runs_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 RANK_LDS_LISTS * (int)sizeof(uint32_t)));
    IVFR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(km_count_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 KM_LDS_LISTS * (int)sizeof(uint32_t)));
    IVFR_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(km_accum_pq_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)km_accum_pq_lds(32)));
    return IVFR_OK;
}
