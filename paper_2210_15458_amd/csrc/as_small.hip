// A whole decode in one launch, for models that fit a compute unit's LDS: rows never interact (Remark after Prop. 1),
// so a block takes one row through all of its steps (Algorithm 1, Sec. 4.1) with nothing to wait for but itself.
//
// What bounds such a decode is launches: two kernels of 3 to 4 us a step whose work is a few hundred instructions.
// The block keeps the output matrix (K along the rows, so that neighbouring threads read neighbouring words), the
// conditioning token's embedding and the row of logits in LDS.  Each logit is the chain of the fp32 kernel
// (as_model.hip), the step is the single-tile kernel's (as_tile.hpp): the same bits as the loop of launches.
// V = 16, d = 8, 64 rows, 8 steps: 64 us as launches, 18.8 as one.
#include <type_traits>

#include "as_common.hpp"
#include "as_row.hpp"
#include "as_tile.hpp"

namespace as {
namespace {

constexpr int kSmallWeights = 8192;      // V * d: 32 KB of LDS, three blocks on a compute unit
constexpr int kSmallVocab = 1024, kSmallRank = 128;

__device__ __forceinline__ float model_value(float x) { return x; }
__device__ __forceinline__ float model_value(uint16_t h) { return bits_f32((uint32_t)h << 16); }
__device__ __forceinline__ float stored(float x, float) { return x; }
__device__ __forceinline__ uint16_t stored(float x, uint16_t)
{
    uint32_t b = __builtin_bit_cast(uint32_t, x);
    b += 0x7fffu + ((b >> 16) & 1u);     // round to nearest even, as the logits kernels do
    return (uint16_t)(b >> 16);
}

template <class WT, int DT>
__global__ __launch_bounds__(256, 3) void decode_small_kernel(SmallArgs s)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int ITERS = kTileIters, G = kTileGroup, NG = ITERS / G;
    __shared__ float weights[kSmallWeights];                 // [d][V]
    __shared__ __attribute__((aligned(16))) T row[kSmallVocab];
    __shared__ float embed[kSmallRank];
    __shared__ TileSums ts;
    __shared__ GenericScratch gen;
    // what one step leaves for the next; the step's last lane writes it
    __shared__ int32_t token;
    __shared__ float code;
    __shared__ uint8_t finished;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.x;
    const int32_t V = s.V, d = s.d;
    const WT *const E = reinterpret_cast<const WT *>(s.E), *const Ut = reinterpret_cast<const WT *>(s.Ut);
    for (int32_t i = tid; i < V * d; i += 256) weights[(i % d) * V + i / d] = model_value(Ut[i]);
    if (tid == 0) {
        const int32_t b = (int32_t)(r / s.N), i = (int32_t)(r % s.N);
        token = s.prompts[b];
        code = s.u ? fminf((float)(((double)i + (double)s.u[b]) / (double)s.N), 0x1.fffffep-1f) : 0.f;
        finished = 0;
    }
    StepArgs a{};
    a.logits = row; a.rows = 1; a.ld = V; a.V = V; a.dtype = (as_dtype)DT;
    a.codes = &code; a.temp = s.temp; a.k = s.k;
    a.tok_stride = 1; a.codes_out = &code; a.eos_id = s.eos_id;
    a.finished_out = s.eos_id >= 0 ? &finished : nullptr; a.prev_out = &token;
    const float k = s.k;
    const int32_t nvec = V / EPV, nchunks = (nvec + 63) / 64;
    const int32_t v0 = wave * ITERS * 64;
    int32_t mych = (nvec - v0 - lane + 63) >> 6;
    mych = mych < 0 ? 0 : (mych > ITERS ? ITERS : mych);
    f32x4 *const my_sums = reinterpret_cast<f32x4 *>(ts.chunk_sum + wave * ITERS);
    __syncthreads();
    for (int32_t t = 0; t < s.T; ++t) {
        if (finished != 0) {                                 // uniform: the rest is padding (Sec. 3.3)
            for (int32_t j = t + tid; j < s.T; j += 256) s.tokens[r * s.T + j] = s.eos_id;
            break;
        }
        const int32_t prev = clamp_token(token, V);
        for (int32_t i = tid; i < d; i += 256) embed[i] = model_value(E[(int64_t)prev * d + i]);
        if (s.uniforms && tid == 0) code = s.uniforms[(int64_t)t * s.rows + r];
        __syncthreads();
        for (int32_t v = tid; v < V; v += 256) {
            float acc = 0.f;
#pragma unroll 8
            for (int32_t i = 0; i < d; ++i) acc = fmaf(embed[i], weights[i * V + v], acc);
            row[v] = stored(acc * s.alpha, T{});
        }
        __syncthreads();
        // the row as the single-tile kernel has it: wave 0 holds all of it (at most 1024 logits)
        const float c = code;
        u32x4 raw[ITERS];
        float rw = kRefFloor;
#pragma unroll
        for (int j = 0; j < ITERS; ++j) raw[j] = u32x4{0u, 0u, 0u, 0u};
        if (wave == 0) {
            const int32_t last = mych > 0 ? (mych - 1) * 64 + lane : 0;
#pragma unroll
            for (int j = 0; j < ITERS; ++j)
                if (j < nchunks) {
                    const int32_t i = j * 64 + lane;
                    raw[j] = reinterpret_cast<const u32x4 *>(row)[i < last ? i : last];
                }
            rw = tile_reference<DT, false, true>(raw[0], k, 0.f, mych);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                float sum[G] = {0.f, 0.f, 0.f, 0.f};
                if (g * G < nchunks) {                       // (a chunk past the row's end sums to zero)
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        sum[j] = tile_lane_sum<DT, false>(raw[g * G + j], k, -rw, 0.f);
                        sum[j] = g * G + j < mych ? sum[j] : 0.f;
                    }
                    wave_sum4_in_lane63(sum[0], sum[1], sum[2], sum[3]);
                }
                if (lane == 63) my_sums[g] = f32x4{sum[0], sum[1], sum[2], sum[3]};
            }
        } else if (lane < NG) {
            my_sums[lane] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (lane == 0) ts.share_ref[wave] = rw;
        __syncthreads();
        // (row r of the call is row 0 of what this block owns; its token goes to the caller's array)
        a.tokens_out = s.tokens + r * s.T + t;
        tile_select<DT, false>(a, 0, c, 0.f, raw, rw, mych, true, v0, lane, wave, ts, gen);
        __syncthreads();
    }
    if (s.codes_out && tid == 0) s.codes_out[r] = code;
}

// The same for rows of one chunk (64 vectors): a wave per row, which needs no barrier.  A lane holds its vector's logits
// in registers from the chain to the search; output matrix and embeddings sit in LDS, ranks and rows padded with zeros
// (which leave a chain as it is).  The row's first chunk is all of it, so the chunk that holds the code is known, and no
// weight exceeds 1.  The bits are those of the launches that such a decode takes otherwise: rows of whole vectors have
// the wave's reference of step_tile_kernel; ragged rows and low temperatures (LANE_REF) step_kernel's reference per lane.
// V = 16, d = 8, 64 rows, 8 steps: 18.3 us as a block per row, 8.3 so (0.2 us a step); 2000 rows 71 (as launches), 9.5.
template <class WT, int DT, bool LANE_REF>
__global__ __launch_bounds__(64) void decode_wave_kernel(SmallArgs s)
{
    constexpr int EPV = Elem<DT>::kPerVec;
    extern __shared__ __attribute__((aligned(16))) float wave_lds[];
    __shared__ int32_t token;
    __shared__ float code;
    __shared__ uint8_t finished;

    // What a decode of a few steps costs is its start, a chain of loads: the prompt's and the weights' are on their way together, the
    // lattice's division runs under them, and an element's place is counted on instead of divided for (us, one after another /
    // so: 64 rows of 16, d = 8, T = 8 8.9 / 8.4, 2000 10.2 / 9.5, 64 of 64, d = 128 49.5 / 37.4, 64 of 256, d = 16, T = 16 29.2 / 23.4).
    const int lane = threadIdx.x;
    const int64_t r = blockIdx.x;
    const int32_t V = s.V, d = s.d, dpad = (d + 3) & ~3, Vpad = (V + EPV - 1) / EPV * EPV;
    float *const weights = wave_lds;                         // [dpad][Vpad]
    float *const embed = wave_lds + dpad * Vpad;             // [V][dpad]
    const WT *const E = reinterpret_cast<const WT *>(s.E), *const Ut = reinterpret_cast<const WT *>(s.Ut);
    const uint32_t of = blockIdx.x / (uint32_t)s.N;          // (rows fit a grid)
    const int32_t prompt = s.prompts[of];
    const float shift = s.u ? s.u[of] : 0.f;
    // (eight elements of each a lane at a time, requested together)
    constexpr int kAhead = 8;
    const int32_t n = V * d;
    WT u[kAhead], e0[kAhead];
    auto request = [&](int32_t i0) __attribute__((always_inline)) {
        if (i0 - lane + 64 * kAhead <= n) {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                u[q] = Ut[i0 + q * 64];
                e0[q] = E[i0 + q * 64];
            }
        } else {
#pragma unroll
            for (int q = 0; q < kAhead; ++q) {
                if (i0 - lane + q * 64 >= n) break;          // (small models: no loads for nothing)
                const int32_t i = i0 + q * 64 < n ? i0 + q * 64 : n - 1;
                u[q] = Ut[i];
                e0[q] = E[i];
            }
        }
    };
    request(lane);
    __builtin_amdgcn_sched_barrier(0);
    if (Vpad != V || dpad != d) {
        for (int32_t i = lane; i < dpad * Vpad; i += 64)
            if (i >= d * Vpad || i % Vpad >= V) weights[i] = 0.f;
        for (int32_t i = lane; i < V * (dpad - d); i += 64) embed[i / (dpad - d) * dpad + d + i % (dpad - d)] = 0.f;
    }
    if (lane == 0) {
        const uint32_t at = blockIdx.x - of * (uint32_t)s.N;
        token = prompt;
        code = s.u ? fminf((float)(((double)at + (double)shift) / (double)s.N), 0x1.fffffep-1f) : 0.f;
        finished = 0;
    }
    // (an element's place moves on by as much each time)
    const int32_t dv = 64 / d, dk = 64 - dv * d;
    int32_t v = lane / d, kk = lane - v * d;
    for (int32_t i0 = lane; i0 - lane < n; i0 += 64 * kAhead) {
        if (i0 != lane) request(i0);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            if (i0 - lane + q * 64 >= n) break;
            if (i0 + q * 64 < n) {
                weights[kk * Vpad + v] = model_value(u[q]);
                embed[v * dpad + kk] = model_value(e0[q]);
            }
            v += dv;
            kk += dk;
            if (kk >= d) {
                kk -= d;
                ++v;
            }
        }
    }
    StepArgs a{};
    a.rows = 1; a.ld = V; a.V = V; a.dtype = (as_dtype)DT;
    a.codes = &code; a.temp = s.temp; a.k = s.k;
    a.tok_stride = 1; a.codes_out = &code; a.eos_id = s.eos_id;
    a.finished_out = s.eos_id >= 0 ? &finished : nullptr; a.prev_out = &token;
    const float k = s.k;
    const bool live = lane < Vpad / EPV;
    const float *const mine = weights + (live ? lane : 0) * EPV;
    float next = s.uniforms ? s.uniforms[r] : 0.f;
    __syncthreads();
    for (int32_t t = 0; t < s.T; ++t) {
        if (finished != 0) {                                 // the rest is padding (Sec. 3.3)
            for (int32_t j = t + lane; j < s.T; j += 64) s.tokens[r * s.T + j] = s.eos_id;
            break;
        }
        const float c = s.uniforms ? next : code;
        if (s.uniforms && t + 1 < s.T) next = s.uniforms[(int64_t)(t + 1) * s.rows + r];
        const float *const e = embed + clamp_token(token, V) * dpad;
        float x[EPV];
#pragma unroll
        for (int i = 0; i < EPV; ++i) x[i] = 0.f;
#pragma unroll 4
        for (int32_t k0 = 0; k0 < dpad; k0 += 4) {
            const f32x4 ev = *reinterpret_cast<const f32x4 *>(e + k0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float *const w = mine + (k0 + q) * Vpad;
#pragma unroll
                for (int i = 0; i < EPV; ++i) x[i] = fmaf(ev[q], w[i], x[i]);
            }
        }
        if constexpr (LANE_REF) {
#pragma unroll
            for (int i = 0; i < EPV; ++i) {
                const float y = x[i] * s.alpha;              // past the row's end: no logit
                x[i] = lane * EPV + i < V ? y : -__builtin_inff();
            }
        } else {
#pragma unroll
            for (int i = 0; i < EPV; ++i) x[i] *= s.alpha;
        }
        u32x4 raw;
        if constexpr (DT == AS_BF16) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                raw[i] = (uint32_t)stored(x[2 * i], uint16_t{}) | (uint32_t)stored(x[2 * i + 1], uint16_t{}) << 16;
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) raw[i] = __builtin_bit_cast(uint32_t, x[i]);
        }
        float rw;
        int shf = 0;
        if constexpr (LANE_REF) {
            unpack<DT>(raw, x);
            rw = fmaxf(ceilf(vec_max<EPV>(x) * k), kRefFloor);
            rw = live ? rw : kRefFloor;
            shf = shift_of(rw, wave_max(rw));
        } else {
            rw = tile_reference<DT, false, true>(raw, k, 0.f, live ? 1 : 0);
        }
        float cl = tile_lane_sum<DT, false>(raw, k, -rw, 0.f);
        cl = live ? cl : 0.f;
        const double S = (double)wave_sum(LANE_REF ? ldexpf(cl, shf) : cl);
        a.tokens_out = s.tokens + r * s.T + t;
        tile_finish<DT, false>(a, 0, 0.f, raw, cl, rw, shf, (double)c * S, 0.0, S, 0, lane);
        __syncthreads();
    }
    if (s.codes_out && lane == 0) s.codes_out[r] = code;
}

}  // namespace

static size_t wave_decode_lds(const as_ctx *ctx, const as_model *m)
{
    const size_t epv = ctx->dtype == AS_BF16 ? 8 : 4, dpad = ((size_t)m->d + 3) / 4 * 4;
    return dpad * (((size_t)m->V + epv - 1) / epv * epv + (size_t)m->V) * sizeof(float);
}

// A wave per row: rows of one chunk, weights of which two blocks at least fit a compute unit's LDS, at most a few dozen rounds
// of blocks, and more than one step (which the first two launches otherwise take no longer for than the wave for its
// weights).  us a decode, a block per row or launches / a wave per row, fp32: 64 rows of 16, d = 8, T = 8 18.9 / 9.4, T = 64
// 47 / 21; 30 of 256, d = 8 20.0 / 12.8; 64 of 16, d = 128 32.3 / 29.8; 8000 of 16, d = 8 141 / 37; 16000 of 128, d = 16 289 /
// 125.  With bf16 logits half as many lanes form the chains: 64 of 16, d = 100 33 / 36.
static bool wave_decode_applies(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T)
{
    const bool half = ctx->dtype == AS_BF16;
    if (m->V > 64 * (half ? 8 : 4) || m->d > (half ? 64 : kSmallRank) || (T < 2 && (int64_t)m->V * m->d > 2048)) return false;
    const size_t lds = wave_decode_lds(ctx, m);
    const int64_t fit = lds > 0 ? (int64_t)(160 * 1024 / (lds + 64)) : 0;
    return fit >= 2 && rows <= 12 * (fit < 16 ? fit : 16) * (int64_t)ctx->num_cus;
}

// Models that the fp32 kernel computes (its chain is what these kernels repeat): a wave per row where that applies, or a
// block per row for rows that the single-tile step takes whole, weights that fit the LDS, and as many rows as the chip
// holds at once: a step then takes 2.2 us (V = 16, d = 8) to 5.5 us (V = 64, d = 128: few threads, long chains) where two
// launches take 7 to 10; a second round of blocks or a rank of 512 (16 us a step) would lose that.
bool small_decode_applies(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T, float temp)
{
    const int epv = ctx->dtype == AS_BF16 ? 8 : 4;
    if (mfma_applies(m) || ctx->step_shape != 0) return false;
    if (wave_decode_applies(ctx, m, rows, T)) return true;
    return m->V <= kSmallVocab && m->d <= kSmallRank && (int64_t)m->V * m->d <= kSmallWeights && m->V % epv == 0 &&
           rows <= 3 * (int64_t)ctx->num_cus && 1.44269504088896340736f / temp <= kTileMaxScale;
}

template <class WT, int DT>
static void launch_small(as_ctx *ctx, const as_model *m, const SmallArgs &s)
{
    const dim3 grid((unsigned)s.rows);
    if (!wave_decode_applies(ctx, m, s.rows, s.T)) {
        launch(ctx, kKernelStep, decode_small_kernel<WT, DT>, grid, dim3(256), 0, s);
        return;
    }
    const size_t lds = wave_decode_lds(ctx, m);
    if (m->V % Elem<DT>::kPerVec == 0 && s.k <= kTileMaxScale)
        launch(ctx, kKernelStep, decode_wave_kernel<WT, DT, false>, grid, dim3(64), lds, s);
    else
        launch(ctx, kKernelStep, decode_wave_kernel<WT, DT, true>, grid, dim3(64), lds, s);
}

as_status launch_small_decode(as_ctx *ctx, const as_model *m, SmallArgs s)
{
    s.E = m->E; s.Ut = m->Ut; s.V = m->V; s.d = m->d;
    s.alpha = (float)((double)m->scale / sqrt((double)m->d));
    s.k = 1.44269504088896340736f / s.temp;
    if (m->wdtype == AS_BF16) {
        if (ctx->dtype == AS_BF16) launch_small<uint16_t, AS_BF16>(ctx, m, s);
        else launch_small<uint16_t, AS_F32>(ctx, m, s);
    } else {
        if (ctx->dtype == AS_BF16) launch_small<float, AS_BF16>(ctx, m, s);
        else launch_small<float, AS_F32>(ctx, m, s);
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
