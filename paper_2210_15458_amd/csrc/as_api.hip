// extern "C" entry points: argument checks on the host, then kernel launches on
// the context's stream.  No entry point synchronises the device except
// as_ctx_destroy and as_model_create_bigram / as_model_destroy.
#include <math.h>
#include <stdlib.h>

#include <mutex>
#include <new>

#include "as_common.hpp"

// Workspace of as_step_static, the entry point for callers that cannot allocate: the per-row keep thresholds
// that the threshold kernel hands to the sampling kernel.  Every GPU the library runs on holds its own copy
// (256 KiB) until the process ends.  In host code this name is only a handle for hipGetSymbolAddress; the
// address the kernels are given is looked up once per device (static_scratch below).
constexpr int64_t kStaticMaxRows = AS_STATIC_MAX_ROWS;
static __device__ __align__(256) float scratch[kStaticMaxRows];

namespace as {

static thread_local std::string g_err;

as_status fail(as_ctx *ctx, as_status code, const std::string &msg)
{
    if (ctx) ctx->err = msg;
    else g_err = msg;
    return code;
}

as_status hip_fail(as_ctx *ctx, hipError_t e, const char *what)
{
    return fail(ctx, AS_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

bool profile_acquire(as_ctx *ctx, int kid, hipEvent_t *start, hipEvent_t *stop)
{
    Profile &p = ctx->prof;
    if (p.used[kid] >= kProfileCapacity) {
        ++p.dropped[kid];
        return false;
    }
    if (p.used[kid] == p.slots[kid].size()) {
        ProfileSlot s;
        if (hipEventCreate(&s.start) != hipSuccess || hipEventCreate(&s.stop) != hipSuccess) {
            (void)hipGetLastError();
            ++p.dropped[kid];
            return false;
        }
        p.slots[kid].push_back(s);
    }
    *start = p.slots[kid][p.used[kid]].start;
    *stop = p.slots[kid][p.used[kid]].stop;
    ++p.used[kid];
    return true;
}

static bool device_alloc(const as_ctx *ctx, void **p, size_t bytes)
{
    *p = nullptr;
    if (ctx->workspace_mib > 0 && bytes > (size_t)ctx->workspace_mib << 20) return false;
    if (hipMalloc(p, bytes) == hipSuccess) return true;
    *p = nullptr;
    (void)hipGetLastError();
    return false;
}

static as_status grow(as_ctx *ctx, DeviceBuf &b, size_t bytes)
{
    if (b.bytes >= bytes) return AS_OK;
    if (b.ptr) {
        AS_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        AS_HIP_TRY(ctx, hipFree(b.ptr));
        b.ptr = nullptr;
        b.bytes = 0;
    }
    if (!device_alloc(ctx, &b.ptr, bytes)) return fail(ctx, AS_ERR_ALLOC, "device allocation of the workspace failed");
    b.bytes = bytes;
    return AS_OK;
}

// The same for a buffer that the call can do without, or with `less` bytes of it.  The old one is given up only when the new
// one is there; what could not be had once is not asked for again (the next call would wait for the stream and move the
// buffer in vain, each time); and nothing is allocated under a capture, which it would end.
static bool grow_if_possible(as_ctx *ctx, DeviceBuf &b, size_t bytes, size_t less = 0)
{
    if (b.bytes >= bytes) return true;
    if (b.refused) return false;
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return false;
    }
    void *p = nullptr;
    if (!device_alloc(ctx, &p, bytes)) {
        b.refused = true;
        if (b.bytes >= less || !device_alloc(ctx, &p, bytes = less)) return false;
    }
    if (b.ptr && (hipStreamSynchronize(ctx->stream) != hipSuccess || hipFree(b.ptr) != hipSuccess)) {
        (void)hipFree(p);          // (an earlier launch failed: the call's own launches report it)
        return false;
    }
    b.ptr = p;
    b.bytes = bytes;
    return true;
}

// Row indices handed in by the caller, as the kernels use them: a copy in the context's workspace with every
// index brought into [0, logits_rows) (an index outside is a caller's error that no call can report, since
// none reads device data back; it must not send a kernel outside the logits).
__global__ void row_ids_in_range_kernel(const int32_t *in, int32_t *out, int64_t n, int64_t logits_rows)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t v = in[i];
    out[i] = (int32_t)(v < 0 ? 0 : (v > logits_rows - 1 ? logits_rows - 1 : v));
}

static as_status row_ids_in_range(as_ctx *ctx, const int32_t *&row_ids, int64_t rows, int64_t logits_rows)
{
    if (!row_ids) return AS_OK;
    const int64_t top = logits_rows < 0x7fffffffLL ? logits_rows : 0x7fffffffLL;
    hipLaunchKernelGGL(row_ids_in_range_kernel, dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, ctx->stream,
                       row_ids, ctx->rid, rows, top);
    AS_HIP_TRY(ctx, hipGetLastError());
    row_ids = ctx->rid;
    return AS_OK;
}

// Device address of `scratch` on the current device, looked up on the first call made with that device current.
constexpr int kMaxDevices = 64;
static std::mutex g_static_mu;
static float *g_static_ptr[kMaxDevices] = {};
static int g_static_cus[kMaxDevices] = {};

static as_status static_scratch(int *device_out, float **ptr_out, int *cus_out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(nullptr, e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(nullptr, AS_ERR_UNSUPPORTED, "device ordinal beyond 63");
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return hip_fail(nullptr, e, "hipGetSymbolAddress(scratch)");
        }
        e = hipDeviceGetAttribute(&g_static_cus[dev], hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return hip_fail(nullptr, e, "hipDeviceGetAttribute");
        g_static_ptr[dev] = static_cast<float *>(p);
    }
    *device_out = dev;
    *ptr_out = g_static_ptr[dev];
    *cus_out = g_static_cus[dev];
    return AS_OK;
}

static bool truncation_on(int32_t V, int32_t top_k, float top_p)
{
    return (top_k > 0 && top_k < V) || (top_p > 0.f && top_p < 1.f);
}

static as_status check_step(as_ctx *ctx, const void *logits, int64_t rows, int64_t ld, const float *codes,
                            float temp, const int32_t *tokens_out, const float *codes_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (rows < 0 || rows > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "rows outside [0, max_rows]");
    if (rows == 0) return AS_OK;
    if (!logits || !codes || !tokens_out || !codes_out)
        return fail(ctx, AS_ERR_INVALID_ARG, "logits, codes, tokens_out and codes_out must not be NULL");
    if (ld < ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "ld is smaller than the vocabulary");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    const size_t esz = ctx->dtype == AS_BF16 ? 2 : 4;
    if (reinterpret_cast<uintptr_t>(logits) % esz != 0)
        return fail(ctx, AS_ERR_INVALID_ARG, "logits pointer is not aligned to its element type");
    return AS_OK;
}

}  // namespace as

using namespace as;

extern "C" {

as_status as_ctx_create(as_ctx **out, int64_t max_rows, int32_t V, as_dtype logits_dtype, void *hip_stream)
{
    if (!out) return fail(nullptr, AS_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (max_rows < 1 || max_rows > 0x7fffffffLL) return fail(nullptr, AS_ERR_INVALID_ARG, "max_rows outside [1, 2^31)");
    if (V < 1 || V > AS_MAX_VOCAB) return fail(nullptr, AS_ERR_INVALID_ARG, "V outside [1, AS_MAX_VOCAB]");
    if (logits_dtype != AS_F32 && logits_dtype != AS_BF16)
        return fail(nullptr, AS_ERR_INVALID_ARG, "unknown logits dtype");
    as_ctx *c = new (std::nothrow) as_ctx();
    if (!c) return fail(nullptr, AS_ERR_ALLOC, "host allocation failed");
    hipError_t e = hipGetDevice(&c->device);
    if (e != hipSuccess) {
        delete c;
        return hip_fail(nullptr, e, "hipGetDevice");
    }
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->max_rows = max_rows;
    c->V = V;
    c->dtype = logits_dtype;
    e = hipDeviceGetAttribute(&c->num_cus, hipDeviceAttributeMultiprocessorCount, c->device);
    if (e != hipSuccess) {
        delete c;
        return hip_fail(nullptr, e, "hipDeviceGetAttribute");
    }
    e = hipMalloc(reinterpret_cast<void **>(&c->thr), (size_t)max_rows * sizeof(float));
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&c->rid), (size_t)max_rows * sizeof(int32_t));
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (c->thr) (void)hipFree(c->thr);
        delete c;
        return fail(nullptr, AS_ERR_ALLOC, "device allocation of the context workspace failed");
    }
    *out = c;
    return AS_OK;
}

as_status as_ctx_destroy(as_ctx *ctx)
{
    if (!ctx) return AS_OK;
    (void)hipStreamSynchronize(ctx->stream);
    if (ctx->thr) (void)hipFree(ctx->thr);
    if (ctx->rid) (void)hipFree(ctx->rid);
    if (ctx->logits.ptr) (void)hipFree(ctx->logits.ptr);
    if (ctx->state.ptr) (void)hipFree(ctx->state.ptr);
    if (ctx->encode_logits.ptr) (void)hipFree(ctx->encode_logits.ptr);
    if (ctx->encode_state.ptr) (void)hipFree(ctx->encode_state.ptr);
    for (auto &v : ctx->prof.slots)
        for (auto &s : v) {
            (void)hipEventDestroy(s.start);
            (void)hipEventDestroy(s.stop);
        }
    delete ctx;
    return AS_OK;
}

const char *as_last_error(const as_ctx *ctx) { return ctx ? ctx->err.c_str() : g_err.c_str(); }

as_status as_ctx_set_tuning(as_ctx *ctx, as_tuning knob, int32_t value)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (value < 0) return fail(ctx, AS_ERR_INVALID_ARG, "a tuning value is >= 0");
    switch (knob) {
    case AS_TUNE_STEP_SHAPE: ctx->step_shape = value; return AS_OK;
    case AS_TUNE_GEMM_SHAPE: ctx->gemm_shape = value; return AS_OK;
    case AS_TUNE_THR_PATH: ctx->thr_path = value; return AS_OK;
    case AS_TUNE_GEMM_GM: ctx->gemm_gm = value; return AS_OK;
    case AS_TUNE_KEPT_ROWS: ctx->kept_rows = value; return AS_OK;
    case AS_TUNE_WORKSPACE_MIB: ctx->workspace_mib = value; return AS_OK;
    }
    return fail(ctx, AS_ERR_INVALID_ARG, "unknown tuning knob");
}

as_status as_ctx_profile(as_ctx *ctx, int enable)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    ctx->prof.on = enable != 0;
    return AS_OK;
}

as_status as_ctx_profile_read(as_ctx *ctx, int kernel, double *total_ms, int64_t *launches, int64_t *untimed)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (kernel < 0 || kernel >= kKernelCount) return fail(ctx, AS_ERR_INVALID_ARG, "unknown kernel id");
    AS_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    Profile &p = ctx->prof;
    double ms = 0.0;
    for (size_t i = 0; i < p.used[kernel]; ++i) {
        float t = 0.f;
        AS_HIP_TRY(ctx, hipEventElapsedTime(&t, p.slots[kernel][i].start, p.slots[kernel][i].stop));
        ms += t;
    }
    if (total_ms) *total_ms = ms;
    if (launches) *launches = (int64_t)p.used[kernel];
    if (untimed) *untimed = (int64_t)p.dropped[kernel];
    p.used[kernel] = 0;
    p.dropped[kernel] = 0;
    return AS_OK;
}

as_status as_ctx_profile_samples(as_ctx *ctx, int kernel, float *ms_out, int64_t capacity, int64_t *count)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (kernel < 0 || kernel >= kKernelCount) return fail(ctx, AS_ERR_INVALID_ARG, "unknown kernel id");
    if (capacity < 0 || (capacity > 0 && !ms_out)) return fail(ctx, AS_ERR_INVALID_ARG, "ms_out is NULL");
    AS_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    Profile &p = ctx->prof;
    const int64_t n = (int64_t)p.used[kernel] < capacity ? (int64_t)p.used[kernel] : capacity;
    for (int64_t i = 0; i < n; ++i)
        AS_HIP_TRY(ctx, hipEventElapsedTime(&ms_out[i], p.slots[kernel][i].start, p.slots[kernel][i].stop));
    if (count) *count = (int64_t)p.used[kernel];
    return AS_OK;
}

as_status as_step_ex(as_ctx *ctx, const void *logits, int64_t rows, int64_t ld, const float *codes, float temp,
                     int32_t top_k, float top_p, int32_t *tokens_out, float *codes_out,
                     const uint8_t *finished_in, int32_t eos_id, uint8_t *finished_out, float *prob_out,
                     float *flo_out, const int32_t *row_ids, int64_t logits_rows)
{
    as_status st = check_step(ctx, logits, rows, ld, codes, temp, tokens_out, codes_out);
    if (st != AS_OK || rows == 0) return st;
    if (row_ids && logits_rows < 1) return fail(ctx, AS_ERR_INVALID_ARG, "row_ids given but logits_rows < 1");
    if (finished_in && eos_id < 0)
        return fail(ctx, AS_ERR_INVALID_ARG, "finished_in given without an eos_id to emit");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    if (isnan(top_p)) return fail(ctx, AS_ERR_INVALID_ARG, "top_p is NaN");
    st = row_ids_in_range(ctx, row_ids, rows, logits_rows);
    if (st != AS_OK) return st;

    StepArgs a{};
    a.logits = logits; a.rows = rows; a.ld = ld; a.V = ctx->V; a.dtype = ctx->dtype;
    a.codes = codes; a.temp = temp; a.k = 1.44269504088896340736f / temp; a.thr = nullptr;
    a.tokens_out = tokens_out; a.tok_stride = 1; a.codes_out = codes_out;
    a.finished_in = finished_in; a.eos_id = eos_id; a.finished_out = finished_out;
    a.prob_out = prob_out; a.flo_out = flo_out; a.row_ids = row_ids; a.prev_out = nullptr;
    if (truncation_on(ctx->V, top_k, top_p)) {
        // top-k rows that fit the resident kernel are finished there; otherwise threshold, then step
        if (launch_topk_step(ctx, a, top_k, top_p, &st)) return st;
        st = launch_threshold(ctx, logits, rows, ld, finished_in, row_ids, temp, top_k, top_p, ctx->thr);
        if (st != AS_OK) return st;
        a.thr = ctx->thr;
    }
    return launch_step(ctx, a);
}

as_status as_step(as_ctx *ctx, const void *logits, int64_t rows, int64_t ld, const float *codes, float temp,
                  int32_t top_k, float top_p, int32_t *tokens_out, float *codes_out)
{
    return as_step_ex(ctx, logits, rows, ld, codes, temp, top_k, top_p, tokens_out, codes_out, nullptr, -1,
                      nullptr, nullptr, nullptr, nullptr, 0);
}

as_status as_step_static(const void *logits, as_dtype logits_dtype, int64_t rows, int64_t ld, int32_t V,
                         const float *codes, float temp, int32_t top_k, float top_p, int32_t *tokens_out,
                         float *codes_out, void *hip_stream)
{
    if (V < 1 || V > AS_MAX_VOCAB) return fail(nullptr, AS_ERR_INVALID_ARG, "V outside [1, AS_MAX_VOCAB]");
    if (logits_dtype != AS_F32 && logits_dtype != AS_BF16)
        return fail(nullptr, AS_ERR_INVALID_ARG, "unknown logits dtype");
    if (rows < 0) return fail(nullptr, AS_ERR_INVALID_ARG, "rows is negative");
    if (rows > kStaticMaxRows)
        return fail(nullptr, AS_ERR_INVALID_ARG,
                    "rows exceeds AS_STATIC_MAX_ROWS (65536), the size of the static workspace of as_step_static");
    if (isnan(top_p)) return fail(nullptr, AS_ERR_INVALID_ARG, "top_p is NaN");
    // a context that lives for this call only and owns nothing: its threshold workspace is the static array
    as_ctx c;
    as_status st = static_scratch(&c.device, &c.thr, &c.num_cus);
    if (st != AS_OK) return st;
    c.stream = static_cast<hipStream_t>(hip_stream);
    c.max_rows = kStaticMaxRows;
    c.V = V;
    c.dtype = logits_dtype;
    st = check_step(&c, logits, rows, ld, codes, temp, tokens_out, codes_out);
    if (st == AS_OK && rows > 0) {
        StepArgs a{};
        a.logits = logits; a.rows = rows; a.ld = ld; a.V = V; a.dtype = logits_dtype;
        a.codes = codes; a.temp = temp; a.k = 1.44269504088896340736f / temp; a.thr = nullptr;
        a.tokens_out = tokens_out; a.tok_stride = 1; a.codes_out = codes_out;
        a.finished_in = nullptr; a.eos_id = -1; a.finished_out = nullptr;
        a.prob_out = nullptr; a.flo_out = nullptr; a.row_ids = nullptr; a.prev_out = nullptr;
        bool done = false;
        if (truncation_on(V, top_k, top_p)) {
            done = launch_topk_step(&c, a, top_k, top_p, &st);
            if (!done) {
                st = launch_threshold(&c, logits, rows, ld, nullptr, nullptr, temp, top_k, top_p, c.thr);
                a.thr = c.thr;
            }
        }
        if (!done && st == AS_OK) st = launch_step(&c, a);
    }
    if (st != AS_OK) g_err = c.err;
    return st;
}

as_status as_lattice(as_ctx *ctx, const float *u, int32_t B, int32_t N, float *codes_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (B < 0 || N < 1) return fail(ctx, AS_ERR_INVALID_ARG, "B must be >= 0 and N >= 1");
    if ((int64_t)B * N > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "B*N exceeds max_rows");
    if (B == 0) return AS_OK;
    if (!u || !codes_out) return fail(ctx, AS_ERR_INVALID_ARG, "u and codes_out must not be NULL");
    return launch_lattice(ctx, u, B, N, codes_out, nullptr, nullptr, nullptr);
}

as_status as_model_create_bigram(as_model **out, const void *E, const void *U, int32_t V, int32_t d, float scale,
                                 as_dtype wdtype)
{
    if (!out) return fail(nullptr, AS_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!E || !U) return fail(nullptr, AS_ERR_INVALID_ARG, "E and U must not be NULL");
    if (V < 1 || V > AS_MAX_VOCAB || d < 1) return fail(nullptr, AS_ERR_INVALID_ARG, "V or d out of range");
    if (wdtype != AS_F32 && wdtype != AS_BF16) return fail(nullptr, AS_ERR_INVALID_ARG, "unknown weight dtype");
    if (!isfinite(scale)) return fail(nullptr, AS_ERR_INVALID_ARG, "scale must be finite");
    as_model *m = new (std::nothrow) as_model();
    if (!m) return fail(nullptr, AS_ERR_ALLOC, "host allocation failed");
    (void)hipGetDevice(&m->device);
    m->V = V; m->d = d; m->scale = scale; m->wdtype = wdtype; m->E = E;
    const size_t esz = wdtype == AS_BF16 ? 2 : 4;
    // rows of Ut are padded with zeros to a whole number of the logits kernel's 256-column tiles, so that its
    // loader needs no bounds on the rows it requests
    const size_t vpad = ((size_t)V + 255) / 256 * 256;
    if (hipMalloc(&m->Ut, vpad * d * esz) != hipSuccess) {
        (void)hipGetLastError();
        delete m;
        return fail(nullptr, AS_ERR_ALLOC, "device allocation of the transposed weights failed");
    }
    as_status st = AS_OK;
    if (vpad > (size_t)V &&
        hipMemset(static_cast<unsigned char *>(m->Ut) + (size_t)V * d * esz, 0, (vpad - V) * d * esz) != hipSuccess) {
        (void)hipGetLastError();
        st = fail(nullptr, AS_ERR_DEVICE, "clearing the padding of the transposed weights failed");
    }
    if (st == AS_OK) st = launch_transpose(U, m->Ut, d, V, wdtype);
    if (st != AS_OK) {
        (void)hipFree(m->Ut);
        delete m;
        return st;
    }
    *out = m;
    return AS_OK;
}

as_status as_model_destroy(as_model *model)
{
    if (!model) return AS_OK;
    (void)hipDeviceSynchronize();
    if (model->Ut) (void)hipFree(model->Ut);
    delete model;
    return AS_OK;
}

as_status as_bigram_logits(as_ctx *ctx, const as_model *model, const int32_t *prev, int64_t rows,
                           void *logits_out, int64_t ld)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (!model) return fail(ctx, AS_ERR_INVALID_ARG, "model is NULL");
    if (model->V != ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "model and context disagree on V");
    if (rows < 0 || rows > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "rows outside [0, max_rows]");
    if (rows == 0) return AS_OK;
    if (!prev || !logits_out) return fail(ctx, AS_ERR_INVALID_ARG, "prev and logits_out must not be NULL");
    if (ld < ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "ld is smaller than the vocabulary");
    return launch_bigram_logits(ctx, model, prev, rows, logits_out, ld);
}

// The state of a running decode in the context's workspace: per row the code, the conditioning token and the
// finished flag, and the tables of shared logits rows where those pay.
struct DecodeState {
    float *codes;
    int32_t *prev;
    uint8_t *fin;
    bool share;
    RowShare tables;
    int64_t logits_rows;         // rows of the table of logits (or group masses) that the decode works on
    float *sums;                 // kept rows whose steps work from sums: [logits_rows, kRowSums], else null
    // a table of every token's logits row, made before the first step:
    bool table;
    unsigned char *records;      // [V, kTableRecord], where steps work from records
    int32_t *token;              // [V] the rows' tokens
    int32_t *prev_next;          // [R] the other half of prev (steps that read it as row_ids)
    // the same of the tokens that codes come to alone, made as they do
    bool demand;
    Demand rows;
};

// What a decode of `rows` rows asks for (as_workspace.hpp): `few` a table of kept rows that only a first call of its size may
// make room for, 0 for any other call.  A decode of logits leaves room for group masses, not the other way round.
static DecodeSizes decode_asks(as_ctx *ctx, int64_t rows, int32_t T, bool masses, size_t &few)
{
    const int64_t V = ctx->V, esz = ctx->dtype == AS_BF16 ? 2 : 4;
    const int64_t row_bytes = masses ? mass_row_bytes(V) : logits_row_bytes(V, esz);
    const bool covered = ctx->seen[0].covers(rows, T) || (masses && ctx->seen[1].covers(rows, T));
    few = covered ? 0 : (size_t)(kept_rows_few(V, rows, T, row_bytes) * row_bytes);
    ctx->seen[masses ? 1 : 0].add(rows, T);
    return decode_sizes(V, esz, rows, T, masses);
}

// Its table: the largest that it may want, or if that cannot be had the kept rows' alone
static void reserve_table(as_ctx *ctx, const DecodeSizes &z, size_t few)
{
    (void)grow_if_possible(ctx, ctx->logits, few > z.preferred ? few : z.preferred, few > z.kept ? few : z.kept);
}

// Makes the workspace of a decode.  A table, of kept rows or of every token's, or its records that cannot be had are done
// without.
static as_status reserve_decode(as_ctx *ctx, int64_t rows, int32_t T, bool masses)
{
    size_t few;
    const DecodeSizes z = decode_asks(ctx, rows, T, masses, few);
    reserve_table(ctx, z, few);
    const as_status st = grow(ctx, ctx->logits, z.needed);
    if (st != AS_OK) return st;
    if (ctx->logits.bytes >= z.preferred) (void)grow_if_possible(ctx, ctx->state, z.state_preferred, z.state);
    return grow(ctx, ctx->state, z.state);
}

// The same for a call that needs none of it
static void reserve_decode_if_possible(as_ctx *ctx, int64_t rows, int32_t T)
{
    size_t few;
    const DecodeSizes z = decode_asks(ctx, rows, T, false, few);
    reserve_table(ctx, z, few);
    (void)grow_if_possible(ctx, ctx->state, ctx->logits.bytes >= z.preferred ? z.state_preferred : z.state, z.state);
}

// Lays a decode's state out and takes its table of logits: rows of row_bytes, `masses` if they are group masses.  by_sums:
// kept rows are stepped from their sums.  form: what steps from a table of every token's row work from.
static as_status decode_state(as_ctx *ctx, const as_model *model, int32_t B, int32_t N, int32_t T, int64_t row_bytes,
                              bool masses, bool by_sums, TableForm form, DecodeState &s)
{
    const int64_t R = (int64_t)B * N, V = ctx->V;
    as_status st = reserve_decode(ctx, R, T, masses);
    if (st != AS_OK) return st;
    const int64_t kept_rows = smaller(V, R * larger((int64_t)T - 1, 0) + B);
    bool keep = (kept_rows_most(V, R, T, row_bytes) > 0 || kept_rows_few(V, R, T, row_bytes) > 0) &&
                keeping_pays(ctx, model, R, T, by_sums) && (size_t)(kept_rows * row_bytes) <= ctx->logits.bytes;
    const bool room = table_rows(V, R, T, row_bytes) > 0 && (size_t)(V * row_bytes) <= ctx->logits.bytes &&
                      table_state(V, R, form != kTableRows) <= ctx->state.bytes;
    const TableChoice choice = room ? table_pays(ctx, model, R, T, form, keep, by_sums) : kNoTable;
    s.table = choice != kNoTable;
    s.demand = choice == kTableDemand;
    if (s.table) {
        keep = false;
        unsigned char *w = static_cast<unsigned char *>(ctx->state.ptr);
        s.records = w;
        if (form != kTableRows) w += V * kTableRecord;
        s.codes = reinterpret_cast<float *>(w);
        s.prev = reinterpret_cast<int32_t *>(w) + R;
        s.prev_next = s.prev + R;
        s.token = s.prev_next + R;
        s.fin = reinterpret_cast<uint8_t *>(s.token + V);
        if (s.demand) {
            int32_t *const q = s.token + V;
            s.rows = Demand{q, q + V, s.prev_next, s.token, q + 2 * V};
            static_assert((kRounds + 3) * Demand::kNumbers <= 48, "table_state");
            s.fin = reinterpret_cast<uint8_t *>(q + 2 * V + 48);
            st = launch_demand_clear(ctx, s.rows, R);
            if (st != AS_OK) return st;
        }
        s.share = false;
        s.tables = RowShare{};
        s.sums = nullptr;
        s.logits_rows = V;
        return AS_OK;
    }
    s.share = keep || sharing_pays(ctx, model, R, T);
    s.logits_rows = keep ? kept_rows : R;
    const int64_t filled = keep ? s.logits_rows : V;
    const size_t sums = keep && by_sums ? (size_t)s.logits_rows * kRowSums : 0;
    int32_t *w = static_cast<int32_t *>(ctx->state.ptr);
    s.sums = sums ? reinterpret_cast<float *>(w) : nullptr;
    w += sums;
    s.codes = reinterpret_cast<float *>(w);
    s.prev = w + R;
    w += 2 * R;
    s.tables = RowShare{};
    if (s.share) {
        s.tables.kept = keep ? (int32_t)s.logits_rows : 0;
        s.tables.token = w;
        s.tables.mark = w + s.logits_rows;
        s.tables.slot = s.tables.mark + V;
        s.tables.count = s.tables.slot + V;
        s.tables.fill = s.tables.count + T + 1;
        s.tables.order = s.tables.fill + filled;
        w = s.tables.order + R;
        if (sums) s.tables.fill = nullptr;                    // (no order is made)
        st = launch_share_clear(ctx, s.tables, T + 1);
    }
    s.fin = reinterpret_cast<uint8_t *>(w);
    return st;
}

// The rows of the model's output that step t of a decode needs: in the first step one per prompt (its N codes condition
// on the same token; ctx->rid already says so), later one per row, or one per token in use where that pays, or, where
// rows are kept, those of the tokens that are new.  `rows` is their largest number, `range` says which they are where
// only the device knows.
struct StepRows {
    const int32_t *prev;
    int64_t rows;
    RowRange range;
    const int32_t *row_ids;
    int64_t src_rows;
    const int32_t *order;        // the rows sorted by logits row, where those are read from memory rather than caches
};

static as_status step_rows(as_ctx *ctx, const DecodeState &s, const int32_t *prompts, int32_t B, int32_t N, int32_t t,
                           bool sorted, StepRows &o)
{
    const int64_t R = (int64_t)B * N;
    if (s.table) {                                            // (its rows are there)
        o = StepRows{nullptr, 0, RowRange{}, s.prev, s.logits_rows, nullptr};
        return AS_OK;
    }
    if (s.tables.kept) {
        // (the first step's prompts are claimed as such: R rows on a few tokens would queue for them)
        const int64_t most = t == 0 ? B : (R < s.logits_rows ? R : s.logits_rows);
        o = StepRows{s.tables.token, most, RowRange{t > 0 ? s.tables.count + t - 1 : nullptr, s.tables.count + t}, ctx->rid,
                     s.logits_rows, sorted && t > 0 ? s.tables.order : nullptr};
        const as_status st = launch_claim(ctx, s.tables, t, t == 0 ? prompts : s.prev, t == 0 ? B : R);
        if (st != AS_OK || s.sums) return st;
        return launch_share_map(ctx, s.tables, t, s.prev, R, ctx->rid, o.order != nullptr);
    }
    if (t == 0 && N > 1) {
        o = StepRows{prompts, B, RowRange{}, ctx->rid, B, nullptr};
        return AS_OK;
    }
    if (t == 0 || !s.share) {
        o = StepRows{s.prev, R, RowRange{}, nullptr, 0, nullptr};
        return AS_OK;
    }
    o = StepRows{s.tables.token, R, RowRange{nullptr, s.tables.count + t}, ctx->rid, 0, sorted ? s.tables.order : nullptr};
    return launch_share(ctx, s.tables, t, s.prev, R, ctx->rid, sorted);
}

// The rows of a table of every token's logits, and the records that its steps work from: each in one launch (1024 / 2048 /
// 4096 / 8192 / 16384 / all 32128 rows, d = 512, at a time, so that the records find them in the caches: 1708 / 1642 / 1589 /
// 1693 / 1591 / 1542 us a decode of 1024 codes x 64).
static as_status fill_table(as_ctx *ctx, const as_model *model, const DecodeState &s, int64_t ldw, TableForm form, float temp,
                            int32_t top_k, float top_p)
{
    const as_status st = launch_bigram_logits(ctx, model, s.token, ctx->V, ctx->logits.ptr, ldw);
    if (st != AS_OK || form == kTableRows) return st;
    return launch_table_records(ctx, form, ctx->logits.ptr, ldw, temp, top_k, top_p, s.records, ctx->V, RowRange{});
}

// What its steps are given; they share one launch.
static WalkArgs walk_args(as_ctx *ctx, const DecodeState &s, int64_t ldw, int64_t R, int32_t T, const float *uniforms, float temp,
                          int32_t eos_id, int32_t *tokens_out)
{
    WalkArgs a{};
    a.logits = ctx->logits.ptr; a.records = s.records; a.ld = ldw; a.V = ctx->V; a.dtype = ctx->dtype;
    a.k = 1.44269504088896340736f / temp; a.rows = R; a.T = T; a.eos_id = eos_id; a.uniforms = uniforms;
    a.codes = s.codes; a.prev = s.prev; a.finished = s.fin; a.tokens = tokens_out;
    return a;
}

// Steps from rows made on demand, in rounds: rows for the tokens that codes wait for (the prompts at first; which those are and
// how many only the device knows), their records, and every code through its steps until it meets a token without a row.  A
// round takes each code a step at least, so T of them are enough; if codes still wait after kRounds, or tokens turn out to
// come evenly, the rows of all tokens that are missing are made (demand_claim_kernel).
static as_status decode_on_demand(as_ctx *ctx, const as_model *model, const DecodeState &s, TableForm form, int32_t B, float temp,
                                  int32_t top_k, float top_p, WalkArgs a)
{
    a.slot = s.rows.slot; a.wanted = s.rows.wanted; a.at = s.rows.at;
    for (a.every = 0; a.rows > 64 * ((int64_t)a.every + 1); a.every = 2 * a.every + 1) {}
    const int32_t rounds = a.T <= kRounds + 1 ? a.T : kRounds + 1;
    for (int32_t i = 0; i < rounds; ++i) {
        const int64_t most = i == 0 ? smaller(B, ctx->V) : i == 1 ? smaller(a.rows, ctx->V) : ctx->V;
        a.round = s.rows.round + i * Demand::kNumbers;
        const RowRange range{a.round + Demand::kMade, a.round + Demand::kNumbers + Demand::kMade};
        as_status st = launch_demand_claim(ctx, s.rows, i, a.T, a.every + 1, i == kRounds && a.T > rounds);
        if (st == AS_OK) st = launch_bigram_logits(ctx, model, s.token, most, ctx->logits.ptr, a.ld, range);
        if (st == AS_OK)
            st = launch_table_records(ctx, form, ctx->logits.ptr, a.ld, temp, top_k, top_p, s.records, most, range);
        if (st == AS_OK) st = launch_walk(ctx, form, a);
        if (st != AS_OK) return st;
    }
    return AS_OK;
}

// as_decode and as_decode_ancestral: with `uniforms` the code of row r at step t is uniforms[t*R + r] and
// the rescaled code is dropped, otherwise codes start on the lattice of u and are carried from step to step.
static as_status decode_impl(as_ctx *ctx, const as_model *model, const int32_t *prompts, int32_t B, int32_t N,
                             int32_t T, const float *u, const float *uniforms, float temp, int32_t top_k,
                             float top_p, int32_t eos_id, int32_t *tokens_out, float *codes_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (!model) return fail(ctx, AS_ERR_INVALID_ARG, "model is NULL");
    if (model->V != ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "model and context disagree on V");
    if (B < 0 || N < 1 || T < 0) return fail(ctx, AS_ERR_INVALID_ARG, "B, T must be >= 0 and N >= 1");
    const int64_t R = (int64_t)B * N;
    if (R > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "B*N exceeds max_rows");
    if (R == 0) return AS_OK;
    if (!prompts || (!u && !uniforms)) return fail(ctx, AS_ERR_INVALID_ARG, "prompts and u must not be NULL");
    if (T > 0 && !tokens_out) return fail(ctx, AS_ERR_INVALID_ARG, "tokens_out must not be NULL");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    if (isnan(top_p)) return fail(ctx, AS_ERR_INVALID_ARG, "top_p is NaN");

    const bool trunc = truncation_on(ctx->V, top_k, top_p);
    if (!trunc && T > 0 && small_decode_applies(ctx, model, R, T, temp)) {
        SmallArgs a{};
        a.temp = temp; a.prompts = prompts; a.u = uniforms ? nullptr : u; a.uniforms = uniforms;
        a.rows = R; a.N = N; a.T = T; a.eos_id = eos_id; a.tokens = tokens_out; a.codes_out = codes_out;
        // (it takes no workspace, but the same call with a truncation, or over one step, does and may be captured)
        reserve_decode_if_possible(ctx, R, T);
        return launch_small_decode(ctx, model, a);
    }
    const size_t esz = ctx->dtype == AS_BF16 ? 2 : 4;
    const int64_t ldw = ((int64_t)ctx->V + 7) / 8 * 8;        // rows start 16-byte aligned
    DecodeState state;
    const TableForm form = table_form(ctx, R, temp, top_k, top_p);
    as_status st = decode_state(ctx, model, B, N, T, ldw * (int64_t)esz, false, !trunc && step_by_sums(ctx, temp), form, state);
    if (st != AS_OK) return st;
    float *const codes = state.codes;
    uint8_t *const fin = state.fin;

    st = launch_lattice(ctx, u, B, N, uniforms ? nullptr : codes, prompts, state.prev, fin, ctx->rid,
                        state.table && !state.demand ? state.token : nullptr, state.demand ? state.rows.wanted : nullptr);
    if (st == AS_OK && state.table && !state.demand) st = fill_table(ctx, model, state, ldw, form, temp, top_k, top_p);
    if (st != AS_OK) return st;
    const bool walk = state.table && form != kTableRows;
    if (walk) {
        const WalkArgs a = walk_args(ctx, state, ldw, R, T, uniforms, temp, eos_id, tokens_out);
        st = state.demand ? decode_on_demand(ctx, model, state, form, B, temp, top_k, top_p, a) : launch_walk(ctx, form, a);
    }
    if (st != AS_OK) return st;
    for (int32_t t = 0; t < T && !walk; ++t) {
        StepRows sr;
        st = step_rows(ctx, state, prompts, B, N, t, !trunc && stream_rows(R, ldw, esz), sr);
        if (st != AS_OK) return st;
        if (!state.table) st = launch_bigram_logits(ctx, model, sr.prev, sr.rows, ctx->logits.ptr, ldw, sr.range);
        if (st != AS_OK) return st;
        // (the tokens of the step before are read as row_ids: those of this step go to the other half)
        if (state.table) { int32_t *const half = state.prev; state.prev = state.prev_next; state.prev_next = half; }
        int32_t *const prev = state.prev;
        StepArgs a{};
        a.logits = ctx->logits.ptr; a.rows = R; a.ld = ldw; a.V = ctx->V; a.dtype = ctx->dtype;
        a.codes = uniforms ? uniforms + (int64_t)t * R : codes; a.temp = temp; a.k = 1.44269504088896340736f / temp; a.thr = nullptr;
        a.tokens_out = tokens_out + t; a.tok_stride = T; a.codes_out = codes;
        a.finished_in = eos_id >= 0 ? fin : nullptr; a.eos_id = eos_id;
        a.finished_out = eos_id >= 0 ? fin : nullptr;
        a.prob_out = nullptr; a.flo_out = nullptr; a.row_ids = sr.row_ids; a.src_rows = sr.src_rows; a.prev_out = prev;
        a.order = sr.order;
        if (state.sums) {
            RowSumsArgs q{};
            q.logits = a.logits; q.ld = ldw; q.V = ctx->V; q.dtype = ctx->dtype; q.k = a.k; q.sums = state.sums;
            q.range = sr.range;
            st = launch_row_sums(ctx, kKernelStep, q, sr.rows);
            if (st != AS_OK) return st;
            SelectArgs sel{};
            sel.step = a; sel.prev = prev; sel.slot = state.tables.slot; sel.sums = state.sums;
            sel.count = state.tables.count + t;
            st = launch_row_select(ctx, sel);
            if (st != AS_OK) return st;
            continue;
        }
        if (trunc) {
            if (launch_topk_step(ctx, a, top_k, top_p, &st)) {
                if (st != AS_OK) return st;
                continue;
            }
            st = launch_threshold(ctx, ctx->logits.ptr, R, ldw, eos_id >= 0 ? fin : nullptr, sr.row_ids, temp,
                                  top_k, top_p, ctx->thr);
            if (st != AS_OK) return st;
            a.thr = ctx->thr;
        }
        st = launch_step(ctx, a);
        if (st != AS_OK) return st;
    }
    if (codes_out)
        AS_HIP_TRY(ctx, hipMemcpyAsync(codes_out, codes, (size_t)R * sizeof(float), hipMemcpyDeviceToDevice,
                                       ctx->stream));
    return AS_OK;
}

as_status as_decode(as_ctx *ctx, const as_model *model, const int32_t *prompts, int32_t B, int32_t N, int32_t T,
                    const float *u, float temp, int32_t top_k, float top_p, int32_t eos_id, int32_t *tokens_out,
                    float *codes_out)
{
    if (ctx && !u) return fail(ctx, AS_ERR_INVALID_ARG, "prompts and u must not be NULL");
    return decode_impl(ctx, model, prompts, B, N, T, u, nullptr, temp, top_k, top_p, eos_id, tokens_out, codes_out);
}

as_status as_decode_ancestral(as_ctx *ctx, const as_model *model, const int32_t *prompts, int32_t B, int32_t N,
                              int32_t T, const float *uniforms, float temp, int32_t top_k, float top_p,
                              int32_t eos_id, int32_t *tokens_out)
{
    if (ctx && !uniforms && (int64_t)B * N * T > 0)
        return fail(ctx, AS_ERR_INVALID_ARG, "uniforms must not be NULL");
    return decode_impl(ctx, model, prompts, B, N, T, nullptr, uniforms, temp, top_k, top_p, eos_id, tokens_out,
                       nullptr);
}

as_status as_bigram_group_mass(as_ctx *ctx, const as_model *model, const int32_t *prev, int64_t rows, float temp,
                               float *mass_out, int64_t ldp)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (!model) return fail(ctx, AS_ERR_INVALID_ARG, "model is NULL");
    if (model->V != ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "model and context disagree on V");
    if (rows < 0 || rows > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "rows outside [0, max_rows]");
    if (rows == 0) return AS_OK;
    if (!prev || !mass_out) return fail(ctx, AS_ERR_INVALID_ARG, "prev and mass_out must not be NULL");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    const int64_t ngroups = ((int64_t)ctx->V + 31) / 32;
    if (ldp < ngroups || ldp % 16 != 0 || reinterpret_cast<uintptr_t>(mass_out) % 16 != 0)
        return fail(ctx, AS_ERR_INVALID_ARG, "ldp must be a multiple of 16 covering ceil(V/32) groups, mass_out 16-byte aligned");
    if (!fused_path_applies(ctx, model))
        return fail(ctx, AS_ERR_UNSUPPORTED,
                    "group masses need bf16 weights, a rank that is a multiple of 64 and at least 128, "
                    "and operands below 4 GB");
    return launch_bigram_partials(ctx, model, prev, rows, temp, reinterpret_cast<float2 *>(mass_out), ldp);
}

as_status as_step_fused(as_ctx *ctx, const as_model *model, const float *mass, int64_t ldp, const int32_t *prev,
                        int64_t rows, const float *codes, float temp, int32_t *tokens_out, float *codes_out,
                        const uint8_t *finished_in, int32_t eos_id, uint8_t *finished_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (!model) return fail(ctx, AS_ERR_INVALID_ARG, "model is NULL");
    if (model->V != ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "model and context disagree on V");
    if (rows < 0 || rows > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "rows outside [0, max_rows]");
    if (rows == 0) return AS_OK;
    if (!mass || !prev || !codes || !tokens_out || !codes_out)
        return fail(ctx, AS_ERR_INVALID_ARG, "mass, prev, codes, tokens_out and codes_out must not be NULL");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    if (finished_in && eos_id < 0) return fail(ctx, AS_ERR_INVALID_ARG, "finished_in given without an eos_id to emit");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    const int64_t ngroups = ((int64_t)ctx->V + 31) / 32;
    if (ldp < ngroups || ldp % 16 != 0 || ldp > 65536 || reinterpret_cast<uintptr_t>(mass) % 16 != 0)
        return fail(ctx, AS_ERR_INVALID_ARG,
                    "ldp must be a multiple of 16, at most 65536, covering ceil(V/32) groups; mass 16-byte aligned");
    if (!fused_path_applies(ctx, model))
        return fail(ctx, AS_ERR_UNSUPPORTED, "the fused step needs bf16 weights and a rank that is a multiple of 64");
    FusedArgs a{};
    a.part = reinterpret_cast<const float2 *>(mass); a.ldp = ldp; a.ngroups = (int32_t)ngroups; a.rows = rows;
    a.V = ctx->V; a.d = model->d;
    a.E = static_cast<const uint16_t *>(model->E); a.Ut = static_cast<const uint16_t *>(model->Ut);
    a.alpha = (float)((double)model->scale / sqrt((double)model->d) * 1.44269504088896340736 / (double)temp);
    a.codes = codes; a.codes_out = codes_out; a.tokens_out = tokens_out; a.tok_stride = 1;
    a.finished_in = finished_in; a.eos_id = eos_id; a.finished_out = finished_out; a.prev = prev; a.prev_out = nullptr;
    return launch_fused_sample(ctx, a);
}

as_status as_decode_fused(as_ctx *ctx, const as_model *model, const int32_t *prompts, int32_t B, int32_t N, int32_t T,
                          const float *u, float temp, int32_t eos_id, int32_t *tokens_out, float *codes_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (!model) return fail(ctx, AS_ERR_INVALID_ARG, "model is NULL");
    if (model->V != ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "model and context disagree on V");
    if (B < 0 || N < 1 || T < 0) return fail(ctx, AS_ERR_INVALID_ARG, "B, T must be >= 0 and N >= 1");
    const int64_t R = (int64_t)B * N;
    if (R > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "B*N exceeds max_rows");
    if (R == 0) return AS_OK;
    if (!prompts || !u) return fail(ctx, AS_ERR_INVALID_ARG, "prompts and u must not be NULL");
    if (T > 0 && !tokens_out) return fail(ctx, AS_ERR_INVALID_ARG, "tokens_out must not be NULL");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    if (!fused_path_applies(ctx, model))
        return fail(ctx, AS_ERR_UNSUPPORTED,
                    "the fused decode needs bf16 weights, a rank that is a multiple of 64 and at least 128, "
                    "and operands below 4 GB");

    const int32_t ngroups = (ctx->V + 31) / 32;
    const int64_t ldp = ((int64_t)ngroups + 15) / 16 * 16;
    DecodeState state;
    as_status st = decode_state(ctx, model, B, N, T, ldp * (int64_t)sizeof(float2), true, false, kTableRows, state);
    if (st != AS_OK) return st;
    float *const codes = state.codes;
    uint8_t *const fin = state.fin;
    float2 *part = static_cast<float2 *>(ctx->logits.ptr);

    st = launch_lattice(ctx, u, B, N, codes, prompts, state.prev, fin, ctx->rid,
                        state.table ? state.token : nullptr);
    if (st == AS_OK && state.table) st = launch_bigram_partials(ctx, model, state.token, ctx->V, temp, part, ldp);
    if (st != AS_OK) return st;
    for (int32_t t = 0; t < T; ++t) {
        StepRows sr;
        st = step_rows(ctx, state, prompts, B, N, t, false, sr);
        if (st != AS_OK) return st;
        if (!state.table) st = launch_bigram_partials(ctx, model, sr.prev, sr.rows, temp, part, ldp, sr.range);
        if (st != AS_OK) return st;
        const int32_t *const prev = state.prev;
        if (state.table) { state.prev = state.prev_next; state.prev_next = const_cast<int32_t *>(prev); }
        FusedArgs a{};
        a.part = part; a.row_ids = sr.row_ids; a.ldp = ldp; a.ngroups = ngroups; a.rows = R; a.V = ctx->V; a.d = model->d;
        a.E = static_cast<const uint16_t *>(model->E); a.Ut = static_cast<const uint16_t *>(model->Ut);
        a.alpha = (float)((double)model->scale / sqrt((double)model->d) * 1.44269504088896340736 / (double)temp);
        a.codes = codes; a.codes_out = codes; a.tokens_out = tokens_out + t; a.tok_stride = T;
        a.finished_in = eos_id >= 0 ? fin : nullptr; a.eos_id = eos_id;
        a.finished_out = eos_id >= 0 ? fin : nullptr; a.prev = prev; a.prev_out = state.prev;
        st = launch_fused_sample(ctx, a);
        if (st != AS_OK) return st;
    }
    if (codes_out)
        AS_HIP_TRY(ctx, hipMemcpyAsync(codes_out, codes, (size_t)R * sizeof(float), hipMemcpyDeviceToDevice,
                                       ctx->stream));
    return AS_OK;
}

as_status as_estimate_mean(as_ctx *ctx, const int32_t *tokens, int32_t B, int32_t N, int32_t T, const float *score,
                           int32_t eos_id, double *est_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (B < 0 || N < 1 || T < 0) return fail(ctx, AS_ERR_INVALID_ARG, "B, T must be >= 0 and N >= 1");
    if (B == 0) return AS_OK;
    if (!score || !est_out || (T > 0 && !tokens))
        return fail(ctx, AS_ERR_INVALID_ARG, "tokens, score and est_out must not be NULL");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    return launch_estimate(ctx, tokens, B, N, T, score, eos_id, est_out);
}

as_status as_interval_step(as_ctx *ctx, const void *logits, int64_t rows, int64_t ld, const int32_t *tokens,
                           float temp, int32_t top_k, float top_p, double *lo, double *width,
                           const uint8_t *finished_in, int32_t eos_id, uint8_t *finished_out,
                           const int32_t *row_ids, int64_t logits_rows)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (rows < 0 || rows > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "rows outside [0, max_rows]");
    if (rows == 0) return AS_OK;
    if (!logits || !tokens || !lo || !width)
        return fail(ctx, AS_ERR_INVALID_ARG, "logits, tokens, lo and width must not be NULL");
    if (ld < ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "ld is smaller than the vocabulary");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    if (row_ids && logits_rows < 1) return fail(ctx, AS_ERR_INVALID_ARG, "row_ids given but logits_rows < 1");
    if (finished_in && eos_id < 0)
        return fail(ctx, AS_ERR_INVALID_ARG, "finished_in given without an eos_id");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    if (isnan(top_p)) return fail(ctx, AS_ERR_INVALID_ARG, "top_p is NaN");
    if (as_status st = row_ids_in_range(ctx, row_ids, rows, logits_rows); st != AS_OK) return st;

    const float *thr = nullptr;
    if (truncation_on(ctx->V, top_k, top_p)) {
        as_status st = launch_threshold(ctx, logits, rows, ld, finished_in, row_ids, temp, top_k, top_p, ctx->thr);
        if (st != AS_OK) return st;
        thr = ctx->thr;
    }
    IntervalArgs a{};
    a.logits = logits; a.rows = rows; a.ld = ld; a.V = ctx->V; a.dtype = ctx->dtype;
    a.tokens = tokens; a.tok_stride = 1; a.k = 1.44269504088896340736f / temp; a.thr = thr;
    a.finished_in = finished_in; a.eos_id = eos_id; a.finished_out = finished_out;
    a.lo = lo; a.width = width; a.row_ids = row_ids;
    return launch_interval(ctx, a);
}

// Whether an encode of n positions gives every token in use one logits row (otherwise every position has its own, the
// first column's one per prompt).  With tokens spread evenly n - V(1 - exp(-n/V)) rows of product and of sums are spared;
// the tables take five launches, 20 us.
static bool claiming_pays(const as_ctx *ctx, const as_model *m, int64_t n)
{
    if (!rows_on_device(ctx, m)) return false;
    const double spared = (double)n - (double)m->V * (1.0 - exp(-(double)n / (double)m->V));
    const double row = (double)m->V * ((double)m->d * 2.0 / 1e15 + (ctx->dtype == AS_BF16 ? 2.0 : 4.0) / 4e12);
    return spared * row > 30e-6;
}

static as_status encode_windows(as_ctx *ctx, const as_model *model, const int32_t *prompts, int64_t R, int32_t N, int32_t T,
                                const int32_t *tokens, float temp, int32_t top_k, float top_p, int32_t eos_id,
                                double *lo_out, double *width_out)
{
    const size_t esz = ctx->dtype == AS_BF16 ? 2 : 4;
    const int64_t ldw = ((int64_t)ctx->V + 7) / 8 * 8;        // rows start 16-byte aligned
    // its own workspace, or where that cannot be had (memory, a first call under a capture) that of a decode of its size,
    // a column at a time
    const EncodeSizes sizes = encode_sizes(ctx->V, esz, R, T);
    const bool own = grow_if_possible(ctx, ctx->encode_logits, sizes.logits) &&
                     grow_if_possible(ctx, ctx->encode_state, sizes.state);
    as_status st = own ? AS_OK : reserve_decode(ctx, R, T, false);
    if (st != AS_OK) return st;
    void *const logits = own ? ctx->encode_logits.ptr : ctx->logits.ptr;
    unsigned char *const base = static_cast<unsigned char *>(own ? ctx->encode_state.ptr : ctx->state.ptr);

    const int32_t window = own ? (int32_t)encode_window(R, T) : 1;
    const int64_t most = R * window;                          // positions of a window
    const bool claimed = own && claiming_pays(ctx, model, most);
    const int64_t max_rows = claimed ? smaller(ctx->V, most) : most;
    const int64_t chunk = smaller(own ? encode_chunk(ldw * (int64_t)esz) : kPlainChunk, max_rows);
    const bool trunc = truncation_on(ctx->V, top_k, top_p), by_sums = step_by_sums(ctx, temp);

    Positions w{};
    w.tokens = tokens; w.prompts = prompts; w.R = R; w.N = N; w.T = T; w.V = ctx->V; w.eos_id = eos_id;
    w.dtype = ctx->dtype; w.chunk = chunk;
    const EncodeTables at = encode_tables(ctx->V, esz, R, most, max_rows, chunk, claimed);
    auto words = [&](size_t o) { return reinterpret_cast<int32_t *>(base + o); };
    w.f_lo = reinterpret_cast<double *>(base + at.f_lo); w.p = reinterpret_cast<double *>(base + at.p);
    w.slot = words(at.slot); w.order = words(at.order); w.token = words(at.token); w.ends = words(at.ends);
    w.idle = base + at.idle; w.ended = base + at.ended; w.cond = words(at.cond); w.count = words(at.count);
    w.chunk_rows = claimed ? words(at.chunks) : nullptr;
    float *const sums = reinterpret_cast<float *>(base + at.sums), *const thr = reinterpret_cast<float *>(base + at.thr);
    RowShare tables{};
    tables.mark = words(at.mark); tables.slot = words(at.claim); tables.token = w.token; tables.count = w.count;
    tables.fill = w.ends;

    for (int32_t t0 = 0; t0 < T; t0 += window) {
        w.t0 = t0;
        w.Tw = T - t0 < window ? T - t0 : window;
        const int64_t n = R * w.Tw;
        st = launch_positions(ctx, w, claimed);
        if (st == AS_OK && claimed) st = launch_claim_positions(ctx, tables, w.cond, n, w.slot);
        const int64_t own = t0 == 0 && N > 1 ? R / N + R * (w.Tw - 1) : n;
        const int64_t rows = claimed ? (n < max_rows ? n : max_rows) : own;
        if (st == AS_OK && claimed) st = launch_positions_order(ctx, w, rows);
        if (st != AS_OK) return st;
        for (int64_t s0 = 0, c = 0; s0 < rows; s0 += chunk, ++c) {
            const int64_t here = rows - s0 < chunk ? rows - s0 : chunk;
            const RowRange range{nullptr, claimed ? w.chunk_rows + c : nullptr};
            st = launch_bigram_logits(ctx, model, w.token + s0, here, logits, ldw, range);
            if (st == AS_OK && trunc)
                st = launch_threshold(ctx, logits, here, ldw, w.idle + s0, nullptr, temp, top_k, top_p, thr);
            if (st != AS_OK) return st;
            ChunkArgs a{};
            a.w = w; a.logits = logits; a.s0 = s0; a.rows = here; a.ld = ldw; a.V = ctx->V;
            a.k = 1.44269504088896340736f / temp; a.thr = trunc ? thr : nullptr; a.sums = sums;
            if (by_sums) {
                RowSumsArgs q{};
                q.logits = a.logits; q.ld = ldw; q.V = ctx->V; q.dtype = ctx->dtype; q.k = a.k; q.thr = a.thr; q.sums = sums;
                q.range = range;
                st = launch_row_sums(ctx, kKernelInterval, q, here);
                if (st != AS_OK) return st;
            }
            st = launch_interval_chunk(ctx, a, by_sums);
            if (st != AS_OK) return st;
        }
        st = launch_fold(ctx, w, lo_out, width_out);
        if (st != AS_OK) return st;
    }
    return T > 0 ? AS_OK : launch_fold(ctx, w, lo_out, width_out);      // (no column: the whole interval)
}

as_status as_encode(as_ctx *ctx, const as_model *model, const int32_t *prompts, int32_t B, int32_t N, int32_t T,
                    const int32_t *tokens, float temp, int32_t top_k, float top_p, int32_t eos_id,
                    double *lo_out, double *width_out)
{
    if (!ctx) return fail(nullptr, AS_ERR_INVALID_ARG, "ctx is NULL");
    if (!model) return fail(ctx, AS_ERR_INVALID_ARG, "model is NULL");
    if (model->V != ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "model and context disagree on V");
    if (B < 0 || N < 1 || T < 0) return fail(ctx, AS_ERR_INVALID_ARG, "B, T must be >= 0 and N >= 1");
    const int64_t R = (int64_t)B * N;
    if (R > ctx->max_rows) return fail(ctx, AS_ERR_INVALID_ARG, "B*N exceeds max_rows");
    if (R == 0) return AS_OK;
    if (!prompts || !lo_out || !width_out)
        return fail(ctx, AS_ERR_INVALID_ARG, "prompts, lo_out and width_out must not be NULL");
    if (T > 0 && !tokens) return fail(ctx, AS_ERR_INVALID_ARG, "tokens must not be NULL");
    if (!(temp > 0.f) || !isfinite(temp)) return fail(ctx, AS_ERR_INVALID_ARG, "temp must be finite and > 0");
    if (eos_id >= ctx->V) return fail(ctx, AS_ERR_INVALID_ARG, "eos_id outside the vocabulary");
    if (isnan(top_p)) return fail(ctx, AS_ERR_INVALID_ARG, "top_p is NaN");

    return encode_windows(ctx, model, prompts, R, N, T, tokens, temp, top_k, top_p, eos_id, lo_out, width_out);
}

}  // extern "C"
