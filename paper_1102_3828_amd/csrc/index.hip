// Index lifetime, codebooks, offline stage (train / add / finalize) and import / export.
#include "ivfr_internal.h"

#include <algorithm>
#include <string.h>

// launchers defined in encode.hip and rerank.hip
int ivfr_launch_book_rows(const ivfr_index* ix, hipStream_t st);
size_t ivfr_rank_scratch_bytes(int64_t n, int c);
int ivfr_launch_list_ranks(const int32_t* list, int64_t n, int c, unsigned long long* list_fill, void* scratch, uint32_t* rank, hipStream_t st);
int ivfr_launch_scatter(const StagedChunk& ch, int m, int mr, const uint32_t* list_start, uint8_t* codes,
                        uint8_t* rec, int rec_stride, hipStream_t st);
int ivfr_launch_entry_words(const ivfr_index* ix, bool import, int which, int64_t i0, int64_t n, const int64_t* offsets,
                            uint32_t* dense, hipStream_t st);
size_t ivfr_km_scratch_bytes(int64_t n, int c);
int ivfr_launch_km_accum_rows(const uint8_t* X, int64_t n, int d, int c, const int32_t* assign, unsigned long long* sums,
                              unsigned long long* counts, void* scratch, hipStream_t st);
int ivfr_launch_km_accum_pq(const float* R, int64_t n, int d, int parts, const uint8_t* codes,
                            unsigned long long* sums, unsigned long long* counts, hipStream_t st);
int ivfr_launch_km_update(float* cent, int64_t groups, int width, unsigned long long* sums, unsigned long long* counts,
                          hipStream_t st);
int ivfr_launch_gather_rows(const float* X, int d, int width, int parts, const int64_t* idx, int count, float* out,
                            hipStream_t st);
int ivfr_launch_gather_byte_rows(const uint8_t* X, int d, const int64_t* idx, int count, float* out, hipStream_t st);
size_t ivfr_draw_scratch_bytes(int parts, int64_t n, int count, double surplus = 8.0);
int ivfr_launch_draw_rows(uint64_t seed, uint64_t salt0, int parts, int64_t n, int count, int64_t* out, void* scratch, hipStream_t st,
                          double surplus = 8.0);

static thread_local char g_err[512] = "";

void ivfr_set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

extern "C" const char* ivfr_last_error(void) { return g_err; }

#define ADD_SUB 1048576   // vectors encoded per internal batch

static int use_device(const ivfr_index* ix) {
    IVFR_HIP(hipSetDevice(ix->p.device));
    return IVFR_OK;
}

template <class T>
static int dev_alloc(T** p, size_t count) {
    *p = nullptr;
    if (count == 0) count = 1;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(p), count * sizeof(T));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
        ivfr_set_error("device allocation of %zu bytes failed: %s", count * sizeof(T), hipGetErrorString(e));
        return IVFR_ERR_OOM;
    }
    return IVFR_OK;
}

template <class T>
static void dev_free(T*& p) {
    if (p) (void)hipFree(p);
    p = nullptr;
}

extern "C" int ivfr_create(const ivfr_params* params, ivfr_index** out) {
    IVFR_REQUIRE(params && out, "ivfr_create: null argument");
    const ivfr_params& p = *params;
    IVFR_REQUIRE(p.d > 0 && p.d % 8 == 0, "d = %d must be a positive multiple of 8", p.d);
    IVFR_REQUIRE(p.c >= 1, "c = %d must be >= 1", p.c);
    IVFR_REQUIRE(p.m == 4 || p.m == 8 || p.m == 16 || p.m == 32 || p.m == 64, "m = %d must be 4, 8, 16, 32 or 64", p.m);
    IVFR_REQUIRE(p.d % p.m == 0, "d = %d is not a multiple of m = %d", p.d, p.m);
    IVFR_REQUIRE(p.d / p.m <= 32, "d/m = %d exceeds 32", p.d / p.m);
    IVFR_REQUIRE(p.m_refine >= 0 && p.m_refine % 4 == 0, "m_refine = %d must be a non-negative multiple of 4", p.m_refine);
    if (p.m_refine) {
        IVFR_REQUIRE(p.d % p.m_refine == 0, "d = %d is not a multiple of m_refine = %d", p.d, p.m_refine);
        IVFR_REQUIRE(p.d / p.m_refine <= 32, "d/m_refine = %d exceeds 32", p.d / p.m_refine);
        int ds = p.d / p.m_refine;
        IVFR_REQUIRE((ds & (ds - 1)) == 0, "d/m_refine = %d must be a power of two", ds);
    }
    {
        int ds = p.d / p.m;
        IVFR_REQUIRE((ds & (ds - 1)) == 0, "d/m = %d must be a power of two", ds);
    }
    int ndev = 0;
    IVFR_HIP(hipGetDeviceCount(&ndev));
    IVFR_REQUIRE(p.device >= 0 && p.device < ndev, "device %d out of range (%d devices)", p.device, ndev);
    ivfr_index* ix = new (std::nothrow) ivfr_index();
    if (!ix) { ivfr_set_error("host allocation failed"); return IVFR_ERR_OOM; }
    ix->p = p;
    ix->dsub = p.d / p.m;
    ix->dsub_r = p.m_refine ? p.d / p.m_refine : 0;
    int r = use_device(ix);
    if (r == IVFR_OK) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, p.device) == hipSuccess) ix->n_cu = prop.multiProcessorCount;
        // function attributes are per device: set with this index's device current, every time
        r = ivfr_select_init();
        if (r == IVFR_OK) r = ivfr_scan_init();
        if (r == IVFR_OK) r = ivfr_scan_select_init();
        if (r == IVFR_OK) r = ivfr_encode_init();
    }
    if (r == IVFR_OK) {
        hipError_t e = hipHostMalloc(reinterpret_cast<void**>(&ix->h_slots), IVFR_STATUS_SLOTS * sizeof(DevStatus),
                                     hipHostMallocDefault);
        if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void**>(&ix->h_redo), (16 + IVFR_REDO_CHUNK) * sizeof(uint32_t), hipHostMallocDefault);
        if (e != hipSuccess) { ivfr_set_error("pinned host allocation failed"); r = IVFR_ERR_OOM; }
        else memset(ix->h_slots, 0, IVFR_STATUS_SLOTS * sizeof(DevStatus));
    }
    if (r == IVFR_OK) r = dev_alloc(&ix->counter, IVFR_COUNTER_WORDS);
    if (r == IVFR_OK && hipMemset(ix->counter, 0, IVFR_COUNTER_WORDS * sizeof(unsigned long long)) != hipSuccess) {
        ivfr_set_error("clearing the counter failed");
        r = IVFR_ERR_HIP;
    }
    if (r == IVFR_OK) r = ivfr_static_scratch_address(p.device, &ix->static_ws);
    for (int i = 0; i < 4 && r == IVFR_OK; ++i) {
        if (hipStreamCreateWithFlags(&ix->side[i], hipStreamNonBlocking) != hipSuccess) {
            ivfr_set_error("stream creation failed");
            r = IVFR_ERR_HIP;
        }
    }
    for (int sl = 0; sl < IVFR_STATUS_SLOTS && r == IVFR_OK; ++sl) {
        bool ok = hipEventCreateWithFlags(&ix->ev_fork[sl], hipEventDisableTiming) == hipSuccess;
        for (int i = 0; i < 4 && ok; ++i)
            ok = hipEventCreateWithFlags(&ix->ev_join[sl][i], hipEventDisableTiming) == hipSuccess;
        for (int i = 0; i < 2 && ok; ++i)
            ok = hipEventCreateWithFlags(&ix->ev_group[sl][i], hipEventDisableTiming) == hipSuccess;
        if (!ok) { ivfr_set_error("event creation failed"); r = IVFR_ERR_HIP; }
    }
    if (r != IVFR_OK) { ivfr_destroy(ix); return r; }
    *out = ix;
    return IVFR_OK;
}

static void free_staged(ivfr_index* ix) {
    for (auto& ch : ix->staged) dev_free(ch.list);
    ix->staged.clear();
}

static void free_books(ivfr_index* ix) {
    dev_free(ix->coarse); dev_free(ix->coarse_norm); dev_free(ix->coarse_cols); dev_free(ix->pq); dev_free(ix->pq_norm);
    dev_free(ix->pq_maxnorm); dev_free(ix->rq); dev_free(ix->book_rows); dev_free(ix->pq_cols);
}

extern "C" int ivfr_destroy(ivfr_index* ix) {
    if (!ix) return IVFR_OK;
    (void)hipSetDevice(ix->p.device);
    (void)hipDeviceSynchronize();
    free_staged(ix);
    free_books(ix);
    dev_free(ix->list_term);
    dev_free(ix->list_fill); dev_free(ix->list_start); dev_free(ix->list_len);
    dev_free(ix->codes);
    dev_free(ix->counter);
    ix->search_ws.release(); ix->cand_ws.release(); ix->encode_ws.release(); ix->dense_ws.release();
    if (ix->h_slots) (void)hipHostFree(ix->h_slots);
    if (ix->h_redo) (void)hipHostFree(ix->h_redo);
    for (int i = 0; i < 4; ++i)
        if (ix->side[i]) (void)hipStreamDestroy(ix->side[i]);
    for (int sl = 0; sl < IVFR_STATUS_SLOTS; ++sl) {
        if (ix->ev_fork[sl]) (void)hipEventDestroy(ix->ev_fork[sl]);
        for (int i = 0; i < 4; ++i)
            if (ix->ev_join[sl][i]) (void)hipEventDestroy(ix->ev_join[sl][i]);
        for (int i = 0; i < 2; ++i)
            if (ix->ev_group[sl][i]) (void)hipEventDestroy(ix->ev_group[sl][i]);
    }
    for (hipEvent_t e : ix->prof_events) (void)hipEventDestroy(e);
    ix->prof_events.clear();
    delete ix;
    return IVFR_OK;
}

static int alloc_books_inner(ivfr_index* ix) {
    const ivfr_params& p = ix->p;
    IVFR_TRY(dev_alloc(&ix->coarse, (size_t)p.c * p.d));
    IVFR_TRY(dev_alloc(&ix->coarse_norm, (size_t)p.c));
    if (ivfr_coarse_cols(p)) IVFR_TRY(dev_alloc(&ix->coarse_cols, (size_t)p.c * p.d));
    IVFR_TRY(dev_alloc(&ix->pq, (size_t)p.m * IVFR_KS * ix->dsub));
    IVFR_TRY(dev_alloc(&ix->pq_norm, (size_t)p.m * IVFR_KS));
    IVFR_TRY(dev_alloc(&ix->pq_maxnorm, (size_t)p.m));
    if (p.m_refine) IVFR_TRY(dev_alloc(&ix->rq, (size_t)p.m_refine * IVFR_KS * ix->dsub_r));
    if (ix->dsub % 8 == 0) IVFR_TRY(dev_alloc(&ix->pq_cols, (size_t)p.m * IVFR_KS * ix->dsub));
    if (ivfr_book_rows_floats(p)) IVFR_TRY(dev_alloc(&ix->book_rows, ivfr_book_rows_floats(p)));
    return IVFR_OK;
}

// all of them or, after a failure, none: a call made again starts anew
static int alloc_books(ivfr_index* ix) {
    if (ix->coarse) return IVFR_OK;
    const int r = alloc_books_inner(ix);
    if (r != IVFR_OK) free_books(ix);
    return r;
}

// what is derived from the codebooks: norms, and copies of them in the order in which kernels read them
static int refresh_derived(ivfr_index* ix, hipStream_t st) {
    IVFR_TRY(ivfr_launch_row_norms(ix->coarse, ix->p.c, ix->p.d, ix->coarse_norm, st));
    IVFR_TRY(ivfr_launch_row_norms(ix->pq, (int64_t)ix->p.m * IVFR_KS, ix->dsub, ix->pq_norm, st));
    IVFR_TRY(ivfr_launch_group_max_norm(ix->pq_norm, ix->p.m, IVFR_KS, ix->pq_maxnorm, st));
    IVFR_TRY(ivfr_launch_book_rows(ix, st));
    return IVFR_OK;
}

extern "C" int ivfr_set_codebooks(ivfr_index* ix, const float* coarse, const float* pq, const float* rq) {
    IVFR_REQUIRE(ix && coarse && pq, "ivfr_set_codebooks: null argument");
    IVFR_REQUIRE(ix->p.m_refine == 0 || rq, "ivfr_set_codebooks: rq is required when m_refine > 0");
    if (ix->n_added > 0 || ix->finalized) { ivfr_set_error("codebooks cannot change after vectors were added"); return IVFR_ERR_STATE; }
    IVFR_TRY(use_device(ix));
    IVFR_TRY(alloc_books(ix));
    const ivfr_params& p = ix->p;
    IVFR_HIP(hipMemcpy(ix->coarse, coarse, (size_t)p.c * p.d * sizeof(float), hipMemcpyHostToDevice));
    IVFR_HIP(hipMemcpy(ix->pq, pq, (size_t)p.m * IVFR_KS * ix->dsub * sizeof(float), hipMemcpyHostToDevice));
    if (p.m_refine)
        IVFR_HIP(hipMemcpy(ix->rq, rq, (size_t)p.m_refine * IVFR_KS * ix->dsub_r * sizeof(float), hipMemcpyHostToDevice));
    IVFR_TRY(refresh_derived(ix, nullptr));
    IVFR_HIP(hipDeviceSynchronize());
    dev_free(ix->list_term);   // belongs to the previous codebooks
    ix->has_books = true;
    return IVFR_OK;
}

extern "C" int ivfr_get_codebooks(const ivfr_index* ix, float* coarse, float* pq, float* rq) {
    IVFR_REQUIRE(ix && coarse && pq, "ivfr_get_codebooks: null argument");
    if (!ix->has_books) { ivfr_set_error("no codebooks yet"); return IVFR_ERR_STATE; }
    IVFR_TRY(use_device(ix));
    const ivfr_params& p = ix->p;
    IVFR_HIP(hipMemcpy(coarse, ix->coarse, (size_t)p.c * p.d * sizeof(float), hipMemcpyDeviceToHost));
    IVFR_HIP(hipMemcpy(pq, ix->pq, (size_t)p.m * IVFR_KS * ix->dsub * sizeof(float), hipMemcpyDeviceToHost));
    if (p.m_refine && rq)
        IVFR_HIP(hipMemcpy(rq, ix->rq, (size_t)p.m_refine * IVFR_KS * ix->dsub_r * sizeof(float), hipMemcpyDeviceToHost));
    return IVFR_OK;
}

static bool is_device_ptr(const void* p) {
    hipPointerAttribute_t attr;
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) { (void)hipGetLastError(); return false; }
    return attr.type == hipMemoryTypeDevice;
}

// Vectors are read in place where they are in device memory and start at a multiple of eight bytes (the kernels' loads); others are
// copied to a device buffer, `stage`, first.
struct ByteRows {
    const uint8_t* src;
    bool on_device, in_place;
    explicit ByteRows(const uint8_t* x) : src(x), on_device(is_device_ptr(x)), in_place(on_device && reinterpret_cast<uintptr_t>(x) % 8 == 0) {}
    // rows [a, a + n) as the kernels take them
    int get(int64_t a, int64_t n, int d, uint8_t* stage, const uint8_t** rows, hipStream_t st) const {
        *rows = in_place ? src + a * d : stage;
        if (!in_place)
            IVFR_HIP(hipMemcpyAsync(stage, src + a * d, (size_t)n * d, on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice, st));
        return IVFR_OK;
    }
};

// ---- training -----------------------------------------------------------------------------
// Lloyd iterations for the `parts` sub-quantizers of a product quantizer on the rows of R [n, d], from the rows d_idx; sums and counts
// are zero before and after
static int train_pq(ivfr_index* ix, float* R, int64_t n, int parts, float* book, int iters, uint8_t* codes_tmp,
                    unsigned long long* sums, unsigned long long* counts, const int64_t* d_idx, hipStream_t st) {
    const int d = ix->p.d, dsub = d / parts;
    IVFR_TRY(ivfr_launch_gather_rows(R, d, dsub, parts, d_idx, IVFR_KS, book, st));
    for (int it = 0; it < iters; ++it) {
        IVFR_TRY(ivfr_launch_pq_encode(R, n, d, book, parts, codes_tmp, false, st));
        IVFR_TRY(ivfr_launch_km_accum_pq(R, n, d, parts, codes_tmp, sums, counts, st));
        IVFR_TRY(ivfr_launch_km_update(book, (int64_t)parts * IVFR_KS, dsub, sums, counts, st));
    }
    return IVFR_OK;
}

extern "C" int ivfr_train(ivfr_index* ix, const uint8_t* train, int64_t n, int32_t iters, uint64_t seed) {
    IVFR_REQUIRE(ix && train, "ivfr_train: null argument");
    IVFR_REQUIRE(iters >= 0, "iters = %d must be >= 0", iters);
    IVFR_REQUIRE(n >= ix->p.c && n >= IVFR_KS, "training set of %lld rows is smaller than max(c, 256)", (long long)n);
    if (ix->n_added > 0 || ix->finalized) { ivfr_set_error("codebooks cannot change after vectors were added"); return IVFR_ERR_STATE; }
    IVFR_TRY(use_device(ix));
    IVFR_TRY(alloc_books(ix));
    const ivfr_params& p = ix->p;
    const int d = p.d, c = p.c;
    hipStream_t st = nullptr;
    const ByteRows from(train);

    float* T = nullptr;
    uint8_t* stage = nullptr;
    int32_t* assign = nullptr;
    uint8_t* codes_tmp = nullptr;
    unsigned long long *sums = nullptr, *counts = nullptr;
    int64_t* d_idx = nullptr;
    char *assign_ws = nullptr, *km_ws = nullptr;
    const int max_parts = std::max(p.m, p.m_refine);
    const size_t sum_elems = std::max((size_t)c * d, (size_t)IVFR_KS * d);
    const size_t cnt_elems = std::max((size_t)c, (size_t)max_parts * IVFR_KS);
    int r = IVFR_OK;
    auto cleanup = [&]() {
        dev_free(T); dev_free(stage); dev_free(assign); dev_free(codes_tmp); dev_free(sums); dev_free(counts);
        dev_free(d_idx); dev_free(assign_ws); dev_free(km_ws);
    };
#define TR(expr) do { r = (expr); if (r != IVFR_OK) { cleanup(); return r; } } while (0)
#define TRH(expr) do { hipError_t e_ = (expr); if (e_ != hipSuccess) { ivfr_set_error("%s failed: %s", #expr, hipGetErrorString(e_)); cleanup(); return IVFR_ERR_HIP; } } while (0)
    TR(dev_alloc(&T, (size_t)n * d));
    if (!from.in_place) TR(dev_alloc(&stage, (size_t)n * d));
    TR(dev_alloc(&assign, (size_t)n));
    TR(dev_alloc(&codes_tmp, (size_t)n * max_parts));
    TR(dev_alloc(&sums, sum_elems));
    TR(dev_alloc(&counts, cnt_elems));
    // the drawn rows, and behind them the scratch of the draws (the three run side by side)
    const size_t n_idx = (size_t)c + (size_t)IVFR_KS * (p.m + p.m_refine);
    const size_t draw_c = (ivfr_draw_scratch_bytes(1, n, c) + 7) / 8, draw_pq = (ivfr_draw_scratch_bytes(p.m, n, IVFR_KS) + 7) / 8;
    const size_t draw_rq = p.m_refine ? (ivfr_draw_scratch_bytes(p.m_refine, n, IVFR_KS) + 7) / 8 : 0;
    TR(dev_alloc(&d_idx, n_idx + draw_c + draw_pq + draw_rq));
    TR(dev_alloc(&assign_ws, ivfr_assign_scratch_bytes(n, c, d)));
    TR(dev_alloc(&km_ws, ivfr_km_scratch_bytes(n, c)));
    TRH(hipMemsetAsync(km_ws, 0, (size_t)c * sizeof(uint32_t), st));
    TRH(hipMemsetAsync(sums, 0, sum_elems * sizeof(unsigned long long), st));
    TRH(hipMemsetAsync(counts, 0, cnt_elems * sizeof(unsigned long long), st));
    const uint8_t* X = nullptr;
    TR(from.get(0, n, d, stage, &X, st));

    // coarse quantizer: initial centroids = c distinct training rows
    // (the draws depend on nothing but seed and n: those of the product quantizers run on a side stream while the
    // coarse quantizer is learned; the event is waited for before they are read)
    int64_t* const idx_pq = d_idx + c;
    int64_t* const idx_rq = idx_pq + (size_t)IVFR_KS * p.m;
    TR(ivfr_launch_draw_rows(seed, 100, p.m, n, IVFR_KS, idx_pq, d_idx + n_idx + draw_c, ix->side[0]));
    if (p.m_refine) TR(ivfr_launch_draw_rows(seed, 200, p.m_refine, n, IVFR_KS, idx_rq, d_idx + n_idx + draw_c + draw_pq, ix->side[0]));
    TRH(hipEventRecord(ix->ev_group[0][0], ix->side[0]));
    TR(ivfr_launch_draw_rows(seed, 1, 1, n, c, d_idx, d_idx + n_idx, st));
    TR(ivfr_launch_gather_byte_rows(X, d, d_idx, c, ix->coarse, st));
    for (int it = 0; it < iters; ++it) {
        TR(ivfr_launch_assign(X, n, ix->coarse, ix->coarse_norm, true, c, d, assign, assign_ws, it == 0, st));
        TR(ivfr_launch_km_accum_rows(X, n, d, c, assign, sums, counts, km_ws, st));
        TR(ivfr_launch_km_update(ix->coarse, c, d, sums, counts, st));
    }
    // residuals to the coarse centroid, then q_c on them, then q_r on what q_c leaves
    TR(ivfr_launch_assign(X, n, ix->coarse, ix->coarse_norm, true, c, d, assign, assign_ws, iters == 0, st));
    TR(ivfr_launch_residual(X, n, d, ix->coarse, assign, T, st));
    TRH(hipStreamWaitEvent(st, ix->ev_group[0][0], 0));
    TR(train_pq(ix, T, n, p.m, ix->pq, iters, codes_tmp, sums, counts, idx_pq, st));
    if (p.m_refine) {
        TR(ivfr_launch_pq_encode(T, n, d, ix->pq, p.m, nullptr, true, st));
        TR(train_pq(ix, T, n, p.m_refine, ix->rq, iters, codes_tmp, sums, counts, idx_rq, st));
    }
    TR(refresh_derived(ix, st));
    TRH(hipStreamSynchronize(st));
    dev_free(ix->list_term);   // belongs to the previous codebooks
#undef TR
#undef TRH
    cleanup();
    ix->has_books = true;
    return IVFR_OK;
}

// ---- add / finalize ---------------------------------------------------------------------------
extern "C" int64_t ivfr_ntotal(const ivfr_index* ix) {
    if (!ix) { ivfr_set_error("ivfr_ntotal: null index"); return IVFR_ERR_INVALID_ARG; }
    return ix->finalized ? ix->N : ix->n_added;
}

extern "C" int ivfr_add(ivfr_index* ix, const uint8_t* x, int64_t n, int64_t id_base) {
    IVFR_REQUIRE(ix && (x || n == 0), "ivfr_add: null argument");
    IVFR_REQUIRE(n >= 0, "n = %lld must be >= 0", (long long)n);
    if (!ix->has_books) { ivfr_set_error("ivfr_add before codebooks were trained or set"); return IVFR_ERR_STATE; }
    if (ix->finalized) { ivfr_set_error("ivfr_add after ivfr_finalize"); return IVFR_ERR_STATE; }
    IVFR_REQUIRE(id_base >= 0 && id_base + n <= 2147483647LL, "ids %lld..%lld do not fit int32", (long long)id_base,
                 (long long)(id_base + n));
    IVFR_REQUIRE(ix->next_id == INT64_MIN || id_base >= ix->next_id, "id ranges must increase: id_base %lld < %lld",
                 (long long)id_base, (long long)ix->next_id);
    IVFR_REQUIRE(ix->n_added + n <= 4000000000LL, "index is limited to 4e9 entries");
    if (n == 0) return IVFR_OK;
    IVFR_TRY(use_device(ix));
    const ivfr_params& p = ix->p;
    const int d = p.d, c = p.c, m = p.m, mr = p.m_refine;
    hipStream_t st = nullptr;
    if (!ix->list_fill) {
        IVFR_TRY(dev_alloc(&ix->list_fill, (size_t)c));
        IVFR_HIP(hipMemset(ix->list_fill, 0, (size_t)c * sizeof(unsigned long long)));
    }
    const ByteRows from(x);
    const int64_t sub = std::min<int64_t>(n, ADD_SUB);
    // workspace: staged bytes, rank counters
    size_t off_stage = 0;
    size_t off_cnt = off_stage + (from.in_place ? 0 : ((size_t)sub * d + 255) / 256 * 256);
    size_t off_assign = off_cnt + (ivfr_rank_scratch_bytes(sub, c) + 255) / 256 * 256;
    size_t total = off_assign + ivfr_assign_scratch_bytes(sub, c, d);
    IVFR_TRY(ix->encode_ws.reserve(total));
    char* ws = ix->encode_ws.as<char>();
    uint8_t* stage = reinterpret_cast<uint8_t*>(ws + off_stage);

    StagedChunk ch;
    ch.n = n;
    int r = IVFR_OK;
    auto fail = [&](int code) {
        dev_free(ch.list);
        return code;
    };
    ch.id_base = id_base;
    {   // (one allocation: each takes about 40 us to get and to give back)
        const size_t words = ((size_t)n * sizeof(int32_t) + 255) / 256 * 256, first = ((size_t)n * m + 255) / 256 * 256;
        char* base = nullptr;
        if ((r = dev_alloc(&base, 2 * words + first + (size_t)n * mr)) != IVFR_OK) return fail(r);
        ch.list = reinterpret_cast<int32_t*>(base);
        ch.rank = reinterpret_cast<uint32_t*>(base + words);
        ch.codes = reinterpret_cast<uint8_t*>(base + 2 * words);
        ch.rcodes = ch.codes + first;
    }
#define AD(expr) do { r = (expr); if (r != IVFR_OK) { (void)hipDeviceSynchronize(); return fail(r); } } while (0)
    for (int64_t a = 0; a < n; a += sub) {
        const int64_t nb = std::min(sub, n - a);
        const uint8_t* X = nullptr;
        AD(from.get(a, nb, d, stage, &X, st));
        AD(ivfr_launch_assign(X, nb, ix->coarse, ix->coarse_norm, false, c, d, ch.list + a, ws + off_assign, a == 0, st));
        AD(ivfr_launch_encode_bytes(ix, X, nb, ch.list + a, ch.codes + a * m, ch.rcodes + a * mr, st));
        AD(ivfr_launch_list_ranks(ch.list + a, nb, c, ix->list_fill, ws + off_cnt, ch.rank + a, st));
    }
    hipError_t e = hipStreamSynchronize(st);
    if (e != hipSuccess) { ivfr_set_error("ivfr_add: %s", hipGetErrorString(e)); return fail(IVFR_ERR_HIP); }
#undef AD
    ix->staged.push_back(ch);
    ix->n_added += n;
    ix->next_id = id_base + n;
    return IVFR_OK;
}

int ivfr_check_room(const ivfr_index* ix, size_t more) {
    if (more == 0) return IVFR_OK;
    if (ix->mem_limit > 0) {
        const size_t held = ix->index_bytes + ix->search_ws.bytes + ix->cand_ws.bytes + ix->dense_ws.bytes + ix->encode_ws.bytes;
        if (held + more > (size_t)ix->mem_limit) {
            ivfr_set_error("%zu more device bytes on top of the %zu held exceed the index's memory limit of %lld",
                           more, held, (long long)ix->mem_limit);
            return IVFR_ERR_OOM;
        }
    }
    size_t free_b = 0, total_b = 0;
    if (hipMemGetInfo(&free_b, &total_b) == hipSuccess) {
        if (more > free_b) {
            ivfr_set_error("%zu more device bytes needed, %zu free of %zu", more, free_b, total_b);
            return IVFR_ERR_OOM;
        }
    } else {
        (void)hipGetLastError();
    }
    return IVFR_OK;
}

static void free_layout(ivfr_index* ix) {
    dev_free(ix->list_start); dev_free(ix->list_len);
    dev_free(ix->codes);
    ix->rec = nullptr;
    ix->index_bytes = 0;
}

static int install_layout_inner(ivfr_index* ix, const std::vector<int64_t>& offsets);

// logical offsets -> padded layout on the device; a failure leaves nothing allocated, so the call can be repeated
static int install_layout(ivfr_index* ix, const std::vector<int64_t>& offsets) {
    free_layout(ix);
    const int r = install_layout_inner(ix, offsets);
    if (r != IVFR_OK) free_layout(ix);
    return r;
}

static int install_layout_inner(ivfr_index* ix, const std::vector<int64_t>& offsets) {
    const int c = ix->p.c;
    ix->h_offsets = offsets;
    ix->h_start.assign((size_t)c + 1, 0);
    std::vector<uint32_t> len((size_t)c);
    uint64_t pos = 0;
    for (int l = 0; l < c; ++l) {
        ix->h_start[(size_t)l] = (uint32_t)pos;
        uint64_t n = (uint64_t)(offsets[(size_t)l + 1] - offsets[(size_t)l]);
        len[(size_t)l] = (uint32_t)n;
        pos += (n + IVFR_LIST_ALIGN - 1) / IVFR_LIST_ALIGN * IVFR_LIST_ALIGN;
    }
    if (pos + IVFR_TAIL_PAD >= 0xFFFFFFFFull) { ivfr_set_error("index too large for 32-bit entry positions"); return IVFR_ERR_INVALID_ARG; }
    ix->h_start[(size_t)c] = (uint32_t)pos;
    ix->n_slots = pos + IVFR_TAIL_PAD;
    ix->N = offsets[(size_t)c];
    {
        // a query lands in a list with a probability proportional to its size: expected visited-list length
        double s2 = 0.0;
        for (int l = 0; l < c; ++l) s2 += (double)len[(size_t)l] * (double)len[(size_t)l];
        ix->wmean_len = ix->N > 0 ? s2 / (double)ix->N : 0.0;
        ix->max_len = c > 0 ? *std::max_element(len.begin(), len.end()) : 0u;
    }
    IVFR_TRY(ivfr_check_room(ix, ivfr_index_bytes(ix->p, ix->n_slots)));
    ix->index_bytes = ivfr_index_bytes(ix->p, ix->n_slots);
    IVFR_TRY(dev_alloc(&ix->list_start, (size_t)c + 1));
    IVFR_TRY(dev_alloc(&ix->list_len, (size_t)c));
    IVFR_HIP(hipMemcpy(ix->list_start, ix->h_start.data(), ((size_t)c + 1) * sizeof(uint32_t), hipMemcpyHostToDevice));
    IVFR_HIP(hipMemcpy(ix->list_len, len.data(), (size_t)c * sizeof(uint32_t), hipMemcpyHostToDevice));
    ix->rec_stride = ivfr_record_stride(ix->p);
    const size_t code_bytes = ((size_t)ix->n_slots * ix->p.m + 255) / 256 * 256;
    IVFR_TRY(dev_alloc(&ix->codes, code_bytes + (size_t)ix->n_slots * ix->rec_stride));   // the records behind the codes
    ix->rec = ix->codes + code_bytes;
    IVFR_HIP(hipMemset(ix->codes, 0, (size_t)ix->n_slots * ix->p.m));
    IVFR_HIP(hipMemset(ix->rec, 0xff, (size_t)ix->n_slots * ix->rec_stride));   // padding slots: id -1
    return IVFR_OK;
}

extern "C" int ivfr_finalize(ivfr_index* ix) {
    IVFR_REQUIRE(ix, "ivfr_finalize: null index");
    if (ix->finalized) { ivfr_set_error("index already finalized"); return IVFR_ERR_STATE; }
    if (!ix->has_books) { ivfr_set_error("ivfr_finalize before codebooks were trained or set"); return IVFR_ERR_STATE; }
    IVFR_TRY(use_device(ix));
    const int c = ix->p.c;
    std::vector<unsigned long long> fill((size_t)c, 0ull);
    if (ix->list_fill)
        IVFR_HIP(hipMemcpy(fill.data(), ix->list_fill, (size_t)c * sizeof(unsigned long long), hipMemcpyDeviceToHost));
    std::vector<int64_t> offsets((size_t)c + 1, 0);
    for (int l = 0; l < c; ++l) offsets[(size_t)l + 1] = offsets[(size_t)l] + (int64_t)fill[(size_t)l];
    if (offsets[(size_t)c] != ix->n_added) { ivfr_set_error("internal: list fill %lld != added %lld", (long long)offsets[(size_t)c], (long long)ix->n_added); return IVFR_ERR_STATE; }
    IVFR_TRY(install_layout(ix, offsets));
    for (auto& ch : ix->staged)
        IVFR_TRY(ivfr_launch_scatter(ch, ix->p.m, ix->p.m_refine, ix->list_start, ix->codes, ix->rec, ix->rec_stride, nullptr));
    IVFR_HIP(hipDeviceSynchronize());
    free_staged(ix);
    ix->encode_ws.release();
    ix->finalized = true;
    return IVFR_OK;
}

// The host's dense arrays (ids, codes, refinement codes in list order) into the finished layout, or out of it.  Each
// array goes through a device buffer in a few large copies, entry by entry spread over (or gathered from) the padded
// lists by a kernel; a copy per list and array costs about 12 us each (24576 of them at 8192 lists).
static int move_entries(ivfr_index* ix, bool import, uint8_t* ids, uint8_t* codes, uint8_t* rcodes) {
    const size_t c = (size_t)ix->p.c, m = (size_t)ix->p.m, mr = (size_t)ix->p.m_refine, N = (size_t)ix->N;
    if (N == 0) return IVFR_OK;
    const size_t table = ((c + 1) * sizeof(int64_t) + 255) / 256 * 256;
    size_t buf = std::min(N * std::max<size_t>(4, std::max(m, mr)), (size_t)(64u << 20));
    // where room is short a smaller buffer does (more copies): a thousand bytes are enough, as little as a list of a few entries
    // would need by itself
    while (ivfr_check_room(ix, table + buf > ix->encode_ws.bytes ? table + buf : 0) != IVFR_OK) {
        if (buf <= 1024) return IVFR_ERR_OOM;
        buf /= 2;
    }
    IVFR_TRY(ix->encode_ws.reserve(table + buf));
    int64_t* offsets = ix->encode_ws.as<int64_t>();
    uint32_t* dense = reinterpret_cast<uint32_t*>(ix->encode_ws.as<char>() + table);
    IVFR_HIP(hipMemcpy(offsets, ix->h_offsets.data(), (c + 1) * sizeof(int64_t), hipMemcpyHostToDevice));
    uint8_t* const host[3] = {ids, codes, rcodes};
    const size_t width[3] = {4, m, mr};
    for (int which = 0; which < 3; ++which) {
        if (width[which] == 0) continue;
        const size_t run = std::max<size_t>(1, buf / width[which]);
        for (size_t i = 0; i < N; i += run) {
            const size_t n = std::min(run, N - i);
            uint8_t* h = host[which] + i * width[which];
            if (import) IVFR_HIP(hipMemcpy(dense, h, n * width[which], hipMemcpyHostToDevice));
            IVFR_TRY(ivfr_launch_entry_words(ix, import, which, (int64_t)i, (int64_t)n, offsets, dense, nullptr));
            if (import) IVFR_HIP(hipDeviceSynchronize());   // the next copy overwrites the buffer
            else IVFR_HIP(hipMemcpy(h, dense, n * width[which], hipMemcpyDeviceToHost));
        }
    }
    ix->encode_ws.release();
    return IVFR_OK;
}

extern "C" int ivfr_export(const ivfr_index* ix, int64_t* list_offsets, int32_t* ids, uint8_t* codes, uint8_t* rcodes) {
    IVFR_REQUIRE(ix && list_offsets && ids && codes, "ivfr_export: null argument");
    IVFR_REQUIRE(ix->p.m_refine == 0 || rcodes, "ivfr_export: rcodes is required when m_refine > 0");
    if (!ix->finalized) { ivfr_set_error("ivfr_export before ivfr_finalize"); return IVFR_ERR_STATE; }
    IVFR_TRY(use_device(ix));
    memcpy(list_offsets, ix->h_offsets.data(), ((size_t)ix->p.c + 1) * sizeof(int64_t));
    return move_entries(const_cast<ivfr_index*>(ix), false, reinterpret_cast<uint8_t*>(ids), codes, rcodes);
}

extern "C" int ivfr_import(ivfr_index* ix, int64_t N, const int64_t* list_offsets, const int32_t* ids,
                           const uint8_t* codes, const uint8_t* rcodes) {
    IVFR_REQUIRE(ix && list_offsets && (N == 0 || (ids && codes)), "ivfr_import: null argument");
    IVFR_REQUIRE(ix->p.m_refine == 0 || N == 0 || rcodes, "ivfr_import: rcodes is required when m_refine > 0");
    if (!ix->has_books) { ivfr_set_error("ivfr_import before codebooks were set"); return IVFR_ERR_STATE; }
    if (ix->finalized || ix->n_added > 0) { ivfr_set_error("ivfr_import into a non-empty index"); return IVFR_ERR_STATE; }
    const int c = ix->p.c;
    IVFR_REQUIRE(N >= 0 && N <= 2147483647LL, "N = %lld out of range", (long long)N);
    IVFR_REQUIRE(list_offsets[0] == 0 && list_offsets[c] == N, "list_offsets must run from 0 to N");
    for (int l = 0; l < c; ++l)
        IVFR_REQUIRE(list_offsets[l + 1] >= list_offsets[l], "list_offsets must be non-decreasing (list %d)", l);
    for (int64_t i = 0; i < N; ++i)
        IVFR_REQUIRE(ids[i] >= 0, "ids must be >= 0 (entry %lld has id %d)", (long long)i, (int)ids[i]);
    IVFR_TRY(use_device(ix));
    std::vector<int64_t> offsets(list_offsets, list_offsets + c + 1);
    IVFR_TRY(install_layout(ix, offsets));
    // (the arrays are only read)
    IVFR_TRY(move_entries(ix, true, reinterpret_cast<uint8_t*>(const_cast<int32_t*>(ids)), const_cast<uint8_t*>(codes),
                          const_cast<uint8_t*>(rcodes)));
    ix->n_added = N;
    ix->finalized = true;
    return IVFR_OK;
}

extern "C" int ivfr_set_tuning(ivfr_index* ix, int32_t full_mult, int32_t cap_mult, int32_t min_cap, int32_t batch,
                               int32_t scan_groups) {
    IVFR_REQUIRE(ix, "ivfr_set_tuning: null index");
    IVFR_REQUIRE(full_mult >= 0 && cap_mult >= 0 && min_cap >= 0 && batch >= 0 && scan_groups >= 0,
                 "tuning values must be >= 0");
    IVFR_REQUIRE(batch <= 65535, "batch = %d exceeds 65535", batch);
    if (full_mult) ix->full_mult = full_mult;
    if (cap_mult) ix->cap_mult = cap_mult;
    if (min_cap) ix->min_cap = min_cap;
    if (batch) ix->batch = batch;
    ix->scan_groups = scan_groups;
    return IVFR_OK;
}

int ivfr_ensure_list_terms(ivfr_index* ix, hipStream_t st) {
    if (ix->list_term) return IVFR_OK;
    const size_t count = (size_t)ix->p.c * ix->p.m * IVFR_KS;
    IVFR_TRY(ivfr_check_room(ix, count * sizeof(float)));
    IVFR_TRY(dev_alloc(&ix->list_term, count));
    ix->index_bytes += count * sizeof(float);
    const int r = ivfr_launch_list_terms(ix, ix->list_term, st);
    if (r != IVFR_OK) { dev_free(ix->list_term); ix->index_bytes -= count * sizeof(float); }
    return r;
}

extern "C" int ivfr_set_table_mode(ivfr_index* ix, int32_t mode) {
    IVFR_REQUIRE(ix, "ivfr_set_table_mode: null index");
    IVFR_REQUIRE(mode == 0 || mode == 1, "table mode %d must be 0 (one table per pair) or 1 (split tables)", mode);
    ix->split_tables = mode;
    return IVFR_OK;
}

extern "C" int ivfr_set_memory_limit(ivfr_index* ix, int64_t bytes) {
    IVFR_REQUIRE(ix, "ivfr_set_memory_limit: null index");
    IVFR_REQUIRE(bytes >= 0, "memory limit %lld must be >= 0", (long long)bytes);
    ix->mem_limit = bytes;
    return IVFR_OK;
}

extern "C" int ivfr_workspace_info(const ivfr_index* ix, int64_t* index_bytes, int64_t* workspace_bytes,
                                   int64_t* pool_bytes, int64_t* batch_reruns) {
    IVFR_REQUIRE(ix, "ivfr_workspace_info: null index");
    if (index_bytes) *index_bytes = (int64_t)ix->index_bytes;
    if (workspace_bytes) *workspace_bytes = (int64_t)(ix->search_ws.bytes + ix->dense_ws.bytes);
    if (pool_bytes) *pool_bytes = (int64_t)ix->cand_ws.bytes;
    if (batch_reruns) *batch_reruns = ix->st_reruns;
    return IVFR_OK;
}

extern "C" int ivfr_set_profiling(ivfr_index* ix, int32_t enable) {
    IVFR_REQUIRE(ix, "ivfr_set_profiling: null index");
    IVFR_REQUIRE(enable >= 0 && enable <= 2, "profiling level %d must be 0, 1 or 2", enable);
    ix->profiling = enable;
    return IVFR_OK;
}

extern "C" int ivfr_stage_times(const ivfr_index* ix, double* ms, int32_t* scan_launches) {
    IVFR_REQUIRE(ix && ms, "ivfr_stage_times: null argument");
    for (int i = 0; i < IVFR_N_STAGES; ++i) ms[i] = ix->prof_ms[i];
    if (scan_launches) *scan_launches = ix->prof_scan_launches;
    return IVFR_OK;
}

extern "C" int ivfr_search_stats(const ivfr_index* ix, int64_t* codes_scanned, int64_t* pairs, int64_t* dense_fallbacks,
                                 int64_t* codes_streamed, int64_t* codes_scanned_shared,
                                 int64_t* codes_scanned_shared2, int64_t* codes_scanned_shared8,
                                 int64_t* bound_retries, int64_t* codes_scanned_shared64) {
    IVFR_REQUIRE(ix, "ivfr_search_stats: null index");
    if (codes_scanned) *codes_scanned = ix->st_codes;
    if (pairs) *pairs = ix->st_pairs;
    if (dense_fallbacks) *dense_fallbacks = ix->st_dense;
    if (codes_streamed) *codes_streamed = ix->st_streamed;
    if (codes_scanned_shared) *codes_scanned_shared = ix->st_shared_codes;
    if (codes_scanned_shared2) *codes_scanned_shared2 = ix->st_shared2_codes;
    if (codes_scanned_shared8) *codes_scanned_shared8 = ix->st_shared8_codes;
    if (bound_retries) *bound_retries = ix->st_retries;
    if (codes_scanned_shared64) *codes_scanned_shared64 = ix->st_shared64_codes;
    return IVFR_OK;
}

extern "C" int ivfr_set_list_sharing(ivfr_index* ix, int32_t mode) {
    IVFR_REQUIRE(ix, "ivfr_set_list_sharing: null index");
    IVFR_REQUIRE(mode >= -1 && mode <= 3, "list sharing mode %d must be -1 (automatic), 0, 1, 2 or 3", mode);
    ix->share_lists = mode;
    return IVFR_OK;
}
