// Shared declarations of the HIP library: context, model, error plumbing and
// the wave-level primitives (DPP scans/reductions for 64-wide wavefronts).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/arith_sampling.h"
#include "as_workspace.hpp"

namespace as {

constexpr int kWave = 64;

// ---------------------------------------------------------------- host state

struct DeviceBuf {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool refused = false;          // a larger one that the context can do without could not be had: not asked for again
};

// Optional per-kernel timing: when switched on, every launch of a profiled
// kernel carries its own start/stop events (taken from the dispatch itself,
// not from separate stream markers), read back by as_ctx_profile_read.
enum KernelId { kKernelStep = 0, kKernelLogits = 1, kKernelThreshold = 2, kKernelInterval = 3, kKernelCount = 4 };
constexpr size_t kProfileCapacity = 16384;      // timed launches per kernel between reads

struct ProfileSlot {
    hipEvent_t start = nullptr, stop = nullptr;
};
struct Profile {
    bool on = false;
    std::vector<ProfileSlot> slots[kKernelCount];   // created on demand, reused after a read
    size_t used[kKernelCount] = {};
    size_t dropped[kKernelCount] = {};
};

}  // namespace as

struct as_ctx {
    int device = 0;
    hipStream_t stream = nullptr;
    int64_t max_rows = 0;
    int32_t V = 0;
    as_dtype dtype = AS_BF16;
    // fixed workspace (allocated at creation): per-row truncation thresholds
    float *thr = nullptr;          // [max_rows]
    int32_t *rid = nullptr;        // [max_rows] the caller's row_ids brought into range
    // decode workspace (grown on demand)
    as::DeviceBuf logits;          // [rows, ld]
    as::DeviceBuf state;           // codes, prev, tables and sums of shared rows, finished flags
    as::RowsSeen seen[2];          // by decodes of logits, of group masses
    // encode workspace: the logits of a chunk of rows, the tables of a window of positions.  Its own, since encodes want
    // many rows where decodes of their size have few, and neither is to move the other's
    as::DeviceBuf encode_logits, encode_state;
    as::Profile prof;
    int step_shape = 0;            // work-group shape of the sampling kernel (tuning knob, 0 = default)
    // choices of a kernel (tuning knobs, 0 = by the rules on sizes)
    int gemm_shape = 0;            // logits: 1 = tile kernel, 2 = persistent also for few rows
    int thr_path = 0;              // truncation: 1 = radix select, 2 = resident where the row fits, 3 = wide for every row
    int gemm_gm = 0;               // logits kernel, many row tiles: workers of an XCD along the rows (tuning knob: 0 = default)
    int kept_rows = 0;             // decodes: 1 = no logits rows kept from step to step, 2 / 3 = kept / a table of all wherever there is room,
                                   // 4 = no table of all, 5 = one of the tokens that come
    int workspace_mib = 0;         // largest buffer of the workspace, in MiB (tuning knob: 0 = as large as the device gives)
    int num_cus = 0;               // compute units of the device (the persistent logits kernel runs one block on each)
    std::string err;
};

struct as_model {
    int device = 0;
    int32_t V = 0;
    int32_t d = 0;
    float scale = 0.f;
    as_dtype wdtype = AS_BF16;
    const void *E = nullptr;       // borrowed [V, d]
    void *Ut = nullptr;            // owned    [V, d]  (U transposed: K contiguous)
};

namespace as {

as_status fail(as_ctx *ctx, as_status code, const std::string &msg);
as_status hip_fail(as_ctx *ctx, hipError_t e, const char *what);

#define AS_HIP_TRY(ctx, expr)                                        \
    do {                                                             \
        hipError_t _e = (expr);                                      \
        if (_e != hipSuccess) return ::as::hip_fail((ctx), _e, #expr); \
    } while (0)

// Launch on the context's stream; with profiling on, attach dispatch events.
bool profile_acquire(as_ctx *ctx, int kid, hipEvent_t *start, hipEvent_t *stop);

template <class K, class... A>
inline void launch(as_ctx *ctx, int kid, K kernel, dim3 grid, dim3 block, size_t lds, A... args)
{
    hipEvent_t s = nullptr, e = nullptr;
    if (ctx->prof.on && profile_acquire(ctx, kid, &s, &e))
        hipExtLaunchKernelGGL(kernel, grid, block, (unsigned)lds, ctx->stream, s, e, 0, args...);
    else
        hipLaunchKernelGGL(kernel, grid, block, (unsigned)lds, ctx->stream, args...);
}

// -------------------------------------------------------------- launch entry
// (implemented in as_step.hip / as_model.hip; called only from as_api.hip)

// How the one-tile kernels load a row.  Logits that the logits kernel has just written are partly still in the
// caches when the whole tensor fits them: ordinary loads then (0.5 us of 13.4 per launch at 1024 x 32128 bf16
// inside a decode).  A tensor beyond the caches is streamed with the non-temporal hint (65536 rows: 651 us
// against 718 with ordinary loads).
inline bool stream_rows(int64_t rows, int64_t ld, size_t esz)
{
    return (double)rows * (double)ld * (double)esz > 128.0 * 1024.0 * 1024.0;
}

// Rows begin .. end of a table, read on the device where only that knows them (end null: not so; begin null: 0).
struct RowRange {
    const int32_t *begin = nullptr, *end = nullptr;
};

struct StepArgs {
    const void *logits;
    int64_t rows;
    int64_t src_rows;            // rows of logits that row_ids can name (0: as many as rows)
    int64_t ld;
    int32_t V;
    as_dtype dtype;
    const float *codes;
    float temp;
    float k;                     // log2(e)/temp, computed once on the host
    const float *thr;            // per-row keep threshold on raw logits, or null
    int32_t *tokens_out;
    int64_t tok_stride;          // tokens_out[r * tok_stride]
    float *codes_out;
    const uint8_t *finished_in;
    int32_t eos_id;
    uint8_t *finished_out;
    float *prob_out;
    float *flo_out;
    const int32_t *row_ids;
    int32_t *prev_out;           // decode state: next step's conditioning token, or null
    const int32_t *order;        // a permutation of the rows that puts those with one logits row together, or null
    unsigned char *records;      // the truncating one-tile kernels: not a step, but these records of the rows (else null) ...
    RowRange range;              // ... in this range of them, where only the device knows it
};

struct IntervalArgs {
    const void *logits;
    int64_t rows;
    int64_t ld;
    int32_t V;
    as_dtype dtype;
    const int32_t *tokens;
    int64_t tok_stride;          // token of row r at tokens[r * tok_stride]
    float k;                     // log2(e)/temp
    const float *thr;            // per-row keep threshold on raw logits, or null
    const uint8_t *finished_in;
    int32_t eos_id;
    uint8_t *finished_out;
    double *lo;                  // [rows] in/out
    double *width;               // [rows] in/out
    const int32_t *row_ids;
};

// The positions of one window of an encode: columns t0 .. t0+Tw of R sequences; position p is column t0 + p % Tw of
// sequence p / Tw.
struct Positions {
    const int32_t *tokens;       // [R, T]
    const int32_t *prompts;      // [R / N]
    int64_t R;
    int32_t N, T, V, eos_id, t0, Tw;
    as_dtype dtype;
    int32_t *cond;               // [positions] the token each conditions on, -1 behind an EOS (claimed rows only)
    int32_t *slot;               // [positions] its logits row
    int32_t *order;              // [positions] the positions by logits row; -1 behind an EOS
    int32_t *token;              // [rows] token of each logits row
    int32_t *ends;               // [rows] where the row's positions end in `order`
    uint8_t *idle;               // [rows] 1 where no position reads the row
    uint8_t *ended;              // [R] sequences that have ended before the window
    int32_t *count;              // logits rows in use (claimed rows only) ...
    int32_t *chunk_rows;         // ... and in each chunk of `chunk` of them, or null
    int64_t chunk;
    double *f_lo, *p;            // [Tw, R] each position's shares
};

struct ChunkArgs {               // a chunk of an encode's logits rows: s0 .. s0+rows
    Positions w;
    const void *logits;          // [rows, ld]
    int64_t s0, rows, ld;
    int32_t V;
    float k;                     // log2(e)/temp
    const float *thr;            // [rows] keep thresholds, or null
    const float *sums;           // [rows, kRowSums]
};

struct RowSumsArgs {
    const void *logits;          // [rows, ld]
    int64_t ld;
    int32_t V;
    as_dtype dtype;
    float k;
    const float *thr;            // [rows] or null
    float *sums;                 // [rows, kRowSums]
    RowRange range;              // which of them, where only the device knows it
};

struct SelectArgs {              // a sampling step from the sums of rows that codes share
    StepArgs step;               // (row_ids is not used)
    const int32_t *prev;         // [rows] conditioning token ...
    const int32_t *slot;         // [V] ... whose logits row is this
    const float *sums;           // [.., kRowSums]
    int32_t *count;              // rows claimed so far: carried on to the next step, count[1] = count[0]
};

// What a decode from a table of every token's logits row reads of a row before its logits, kTableRecord apart.
struct RowRecord {               // sums of step_tile_kernel's chunks (as_tile.hpp)
    struct {
        double before, upto;     // the mass before each chunk, and with it, relative to R (the last no number: the row's plain form)
    } chunk[64];
    float ref[4], R;             // the waves' references, the largest of them
    float thr;                   // keep threshold
};
struct CandRecord {              // the candidates of topk_tile_kernel
    struct {
        double before;           // the mass before it in vocabulary order ...
        float w;                 // ... its own (0: not kept), and its token
        int32_t token;
    } cand[64];
    double S;                    // the mass of all; no number: the row's plain form
};
struct PlainRecord {             // the sums of generic_step_row (as_row.hpp), in a record of either kind that is marked so
    double run[64];              // the mass before every fourth thread's elements
    double S, run_last;          // of all; before the last thread's that have any ...
    float ref, thr;              // what they are relative to; keep threshold
    int32_t last;                // ... and that thread
};
static_assert(sizeof(RowRecord) <= kTableRecord && sizeof(CandRecord) <= kTableRecord && kTableRecord % 16 == 0, "records fit");
static_assert(sizeof(PlainRecord) <= 1000, "a plain record leaves the marks alone: RowRecord's last sum, CandRecord's S");

struct WalkArgs {                // the steps of a decode from such a table
    const void *logits;          // [V, ld]
    const unsigned char *records;
    int64_t ld;
    int32_t V;
    as_dtype dtype;
    float k;                     // log2(e)/temp
    int64_t rows;
    int32_t T, eos_id;
    const float *uniforms;       // [T, rows] the codes, or null: carried in `codes`
    float *codes;                // [rows], as are prev and finished: read first, written last
    int32_t *prev;
    uint8_t *finished;
    int32_t *tokens;             // [rows, T]
    // rows made on demand, else null:
    const int32_t *slot;         // [V] a token's row, or -1 where it is not there
    int32_t *wanted;             // [V] set for a token that a code waits for
    int32_t *at;                 // [rows] steps done
    int32_t *round;              // this round's numbers (Demand) ...
    int32_t every;               // ... to which one code in every + 1 adds (a power of two)
};
struct Demand {                  // rows made on demand: which, for whom
    int32_t *slot, *wanted, *at, *token;         // (token: of each row)
    // of round i, kNumbers apart: rows made before it, whether a code waits after it, and of a share of the codes the tokens that
    // had a row and those that had none (the first of a code's round aside, which has one)
    enum { kMade, kWaits, kMet, kMissed, kNumbers };
    int32_t *round;
};
constexpr int32_t kRounds = 6;   // rounds of a decode before all rows that are still missing are made
enum TableForm { kTablePlain, kTableNucleus, kTableTopK, kTableRows };    // what a step works from; kTableRows: the logits alone

struct SmallArgs {               // a whole decode of a model that fits LDS
    const void *E, *Ut;          // [V, d] each
    int32_t V, d;
    float alpha, k, temp;
    const int32_t *prompts;
    const float *u;              // shifts of the lattice, or null ...
    const float *uniforms;       // ... and then the codes [T, rows]
    int64_t rows;
    int32_t N, T, eos_id;
    int32_t *tokens;             // [rows, T]
    float *codes_out;            // [rows] or null
};

struct FusedArgs {
    const float2 *part;          // [rows, ldp]: (sum, reference) per group of 32 logits
    const int32_t *row_ids;      // row r's masses are row row_ids[r] of part, or null
    int64_t ldp;                 // multiple of 16
    int32_t ngroups;             // ceil(V / 32)
    int64_t rows;
    int32_t V;
    int32_t d;
    const uint16_t *E;           // [V, d] bf16
    const uint16_t *Ut;          // [V, d] bf16
    float alpha;                 // scale/sqrt(d) * log2(e)/temp
    const float *codes;
    float *codes_out;
    int32_t *tokens_out;
    int64_t tok_stride;
    const uint8_t *finished_in;
    int32_t eos_id;
    uint8_t *finished_out;
    const int32_t *prev;         // conditioning token of each row (may alias prev_out)
    int32_t *prev_out;
};

as_status launch_step(as_ctx *ctx, const StepArgs &a);
as_status launch_fused_sample(as_ctx *ctx, const FusedArgs &a);
as_status launch_bigram_partials(as_ctx *ctx, const as_model *m, const int32_t *prev, int64_t rows, float temp,
                                 float2 *part, int64_t ldp, RowRange range = RowRange{});
bool fused_path_applies(const as_ctx *ctx, const as_model *m);
as_status launch_interval(as_ctx *ctx, const IntervalArgs &a);
as_status launch_positions(as_ctx *ctx, const Positions &w, bool claimed);
as_status launch_positions_order(as_ctx *ctx, const Positions &w, int64_t max_rows);
as_status launch_interval_chunk(as_ctx *ctx, const ChunkArgs &a, bool by_sums);
as_status launch_fold(as_ctx *ctx, const Positions &w, double *lo, double *width);
as_status launch_row_sums(as_ctx *ctx, int kid, const RowSumsArgs &a, int64_t rows);
bool launch_topk_step(as_ctx *ctx, const StepArgs &a, int32_t top_k, float top_p, as_status *st);
as_status launch_wide(as_ctx *ctx, const StepArgs &a, int32_t top_k, float top_p, float *thr_out);
as_status launch_threshold(as_ctx *ctx, const void *logits, int64_t rows, int64_t ld,
                           const uint8_t *finished_in, const int32_t *row_ids,
                           float temp, int32_t top_k, float top_p, float *thr_out);
// prev_out: the prompts, clamped to the vocabulary; table_out: 0 .. V-1; wanted_out: [V], set for the prompts
as_status launch_lattice(as_ctx *ctx, const float *u, int32_t B, int32_t N, float *codes_out,
                         const int32_t *prompts, int32_t *prev_out, uint8_t *finished_out,
                         int32_t *row_ids_out = nullptr, int32_t *table_out = nullptr, int32_t *wanted_out = nullptr);
as_status launch_estimate(as_ctx *ctx, const int32_t *tokens, int32_t B, int32_t N, int32_t T, const float *score,
                          int32_t eos_id, double *est_out);
as_status launch_transpose(const void *U, void *Ut, int32_t d, int32_t V, as_dtype wdtype);
// range: which rows of prev and logits_out, at most `rows`, read on the device (persistent kernel only)
as_status launch_bigram_logits(as_ctx *ctx, const as_model *m, const int32_t *prev,
                               int64_t rows, void *logits_out, int64_t ld, RowRange range = RowRange{});

// Rows of a decode that condition on the same token have the same logits: one row of them is computed for each
// token in use, and the rows are told which.  Where a decode comes back to most of its tokens, the rows are kept from
// step to step and only those of new tokens are computed.  The tables live in the context's decode state.
struct RowShare {
    int32_t *mark = nullptr;     // [V] last step that used the token (kept rows: 0 where the token has one)
    int32_t *slot = nullptr;     // [V] its logits row in that step
    int32_t *token = nullptr;    // [logits rows] token of each logits row
    int32_t *count = nullptr;    // [T + 1] logits rows of each step (kept rows: up to and including it)
    int32_t *fill = nullptr;     // [logits rows] rows of each logits row, then where the next of them goes in `order`
    int32_t *order = nullptr;    // [R] the rows sorted by logits row
    int32_t kept = 0;            // the number of rows that are kept, or 0
};
bool mfma_applies(const as_model *m);
bool small_decode_applies(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T, float temp);
as_status launch_small_decode(as_ctx *ctx, const as_model *m, SmallArgs s);
bool sharing_pays(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T);
bool rows_on_device(const as_ctx *ctx, const as_model *m);
as_status launch_share_clear(as_ctx *ctx, const RowShare &s, int32_t T);
as_status launch_share(as_ctx *ctx, const RowShare &s, int32_t step, const int32_t *prev, int64_t rows,
                       int32_t *row_ids, bool sorted);
// kept rows: those of new tokens among prev[0 .. rows)
as_status launch_claim(as_ctx *ctx, const RowShare &s, int32_t step, const int32_t *prev, int64_t rows);
as_status launch_share_map(as_ctx *ctx, const RowShare &s, int32_t step, const int32_t *prev, int64_t rows,
                           int32_t *row_ids, bool sorted);
bool keeping_pays(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T, bool by_sums);
bool step_by_sums(const as_ctx *ctx, float temp);
// a table of every token's logits row, or of those that codes come to: whether it pays, its records, the steps from them
enum TableChoice { kNoTable, kTableAll, kTableDemand };
TableChoice table_pays(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T, TableForm form, bool keep, bool by_sums);
TableForm table_form(const as_ctx *ctx, int64_t rows, float temp, int32_t top_k, float top_p);
as_status launch_table_records(as_ctx *ctx, TableForm form, const void *logits, int64_t ld, float temp, int32_t top_k, float top_p,
                               unsigned char *records, int64_t rows, RowRange range);
as_status launch_row_records(as_ctx *ctx, const void *logits, int64_t ld, float temp, unsigned char *records, int64_t rows,
                             RowRange range);
as_status launch_demand_clear(as_ctx *ctx, const Demand &d, int64_t rows);
as_status launch_demand_claim(as_ctx *ctx, const Demand &d, int32_t i, int32_t T, int32_t each, bool last);
as_status launch_walk(as_ctx *ctx, TableForm form, const WalkArgs &a);
as_status launch_row_select(as_ctx *ctx, const SelectArgs &a);
// the same for the positions of an encode (prev < 0: none): rows claimed, counted and scanned, the order left to the caller
as_status launch_claim_positions(as_ctx *ctx, const RowShare &s, const int32_t *prev, int64_t rows, int32_t *row_ids);

// ------------------------------------------------------------ wave primitives
// Data-parallel-primitive (DPP) cross-lane moves.  bound_ctrl is off, so a lane
// whose source is outside its row (or that is masked out) receives `old`.

constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;

// A conditioning token as a row index of the embedding: tokens the library emits are in [0, V); one handed in
// from outside that is not (a prompt) is clamped rather than followed out of the table.
__device__ __forceinline__ int32_t clamp_token(int32_t t, int32_t V) { return t < 0 ? 0 : (t > V - 1 ? V - 1 : t); }

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp_i32(int old, int src)
{
    return __builtin_amdgcn_update_dpp(old, src, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_f32(float old, float src)
{
    return __builtin_bit_cast(
        float, dpp_i32<CTRL, ROW_MASK>(__builtin_bit_cast(int, old), __builtin_bit_cast(int, src)));
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp_f64(double old, double src)
{
    long long o = __builtin_bit_cast(long long, old), s = __builtin_bit_cast(long long, src);
    int lo = dpp_i32<CTRL, ROW_MASK>((int)o, (int)s);
    int hi = dpp_i32<CTRL, ROW_MASK>((int)(o >> 32), (int)(s >> 32));
    long long r = ((long long)hi << 32) | (unsigned int)lo;
    return __builtin_bit_cast(double, r);
}

// Inclusive prefix sum over the 64 lanes of a wave, lane order.
__device__ __forceinline__ float wave_scan_add(float x)
{
    x += dpp_f32<kRowShr1>(0.f, x);
    x += dpp_f32<kRowShr2>(0.f, x);
    x += dpp_f32<kRowShr4>(0.f, x);
    x += dpp_f32<kRowShr8>(0.f, x);
    x += dpp_f32<kRowBcast15, 0xa>(0.f, x);
    x += dpp_f32<kRowBcast31, 0xc>(0.f, x);
    return x;
}
__device__ __forceinline__ double wave_scan_add(double x)
{
    x += dpp_f64<kRowShr1>(0.0, x);
    x += dpp_f64<kRowShr2>(0.0, x);
    x += dpp_f64<kRowShr4>(0.0, x);
    x += dpp_f64<kRowShr8>(0.0, x);
    x += dpp_f64<kRowBcast15, 0xa>(0.0, x);
    x += dpp_f64<kRowBcast31, 0xc>(0.0, x);
    return x;
}

__device__ __forceinline__ float read_lane(float x, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double read_lane(double x, int lane)
{
    long long v = __builtin_bit_cast(long long, x);
    int lo = __builtin_amdgcn_readlane((int)v, lane);
    int hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
    long long r = ((long long)hi << 32) | (unsigned int)lo;
    return __builtin_bit_cast(double, r);
}

// Sum / max over the wave, result in every lane (wave-uniform).
// Written as six fused DPP instructions: destination and both sources are the
// same register, so a lane without a valid source (or masked off by row_mask)
// simply keeps its value, which is the identity for both operations.  A VALU
// write needs two wait states before a DPP read of the same register.
__device__ __forceinline__ float wave_sum(float x)
{
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 0"
        : "+v"(x));
    return read_lane(x, 63);
}
__device__ __forceinline__ double wave_sum(double x) { return read_lane(wave_scan_add(x), 63); }

__device__ __forceinline__ float wave_max(float x)
{
    asm volatile(
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 0"
        : "+v"(x));
    return read_lane(x, 63);
}

__device__ __forceinline__ int lane_id() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

}  // namespace as
