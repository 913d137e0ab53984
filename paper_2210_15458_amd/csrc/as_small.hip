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

}  // namespace

// Models that the fp32 kernel computes (its chain is what this kernel repeats), rows that the single-tile step takes
// whole, weights that fit the LDS, and as many rows as the chip holds at once: a step then takes 2.2 us (V = 16, d = 8)
// to 5.5 us (V = 64, d = 128: few threads, long chains) where two launches take 7 to 10; a second round of blocks or a
// rank of 512 (16 us a step) would lose that.
bool small_decode_applies(const as_ctx *ctx, const as_model *m, int64_t rows, float temp)
{
    const int epv = ctx->dtype == AS_BF16 ? 8 : 4;
    return !mfma_applies(m) && ctx->step_shape == 0 && m->V <= kSmallVocab && m->d <= kSmallRank &&
           (int64_t)m->V * m->d <= kSmallWeights && m->V % epv == 0 && rows <= 3 * (int64_t)ctx->num_cus &&
           1.44269504088896340736f / temp <= kTileMaxScale;
}

as_status launch_small_decode(as_ctx *ctx, const as_model *m, SmallArgs s)
{
    s.E = m->E; s.Ut = m->Ut; s.V = m->V; s.d = m->d;
    s.alpha = (float)((double)m->scale / sqrt((double)m->d));
    s.k = 1.44269504088896340736f / s.temp;
    const dim3 grid((unsigned)s.rows), block(256);
    if (m->wdtype == AS_BF16) {
        if (ctx->dtype == AS_BF16) launch(ctx, kKernelStep, decode_small_kernel<uint16_t, AS_BF16>, grid, block, 0, s);
        else launch(ctx, kKernelStep, decode_small_kernel<uint16_t, AS_F32>, grid, block, 0, s);
    } else {
        if (ctx->dtype == AS_BF16) launch(ctx, kKernelStep, decode_small_kernel<float, AS_BF16>, grid, block, 0, s);
        else launch(ctx, kKernelStep, decode_small_kernel<float, AS_F32>, grid, block, 0, s);
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
