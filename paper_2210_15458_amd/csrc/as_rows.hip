// The sums of logits rows that several codes or positions share: once per row here, then a wave per code or position
// works from them (as_interval.hip) and reads one KiB of the row instead of all of it.
#include "as_common.hpp"
#include "as_row.hpp"
#include "as_tile.hpp"

namespace as {
namespace {

// Rows of whole, aligned vectors that fit one tile: the 64 chunk sums and 4 references of step_tile_kernel (as_tile.hpp;
// the same loads, the same arithmetic, so the same bits), 272 bytes a row, and nothing behind them: no barrier, no
// search.  Bound by the row's transfer, or where the rows are still in the caches by the vector instructions per
// logit: 4096 x 32128 bf16 41 us, 6.5 TB/s.  A block per row.
template <int DT, bool HAS_THR, bool NT>
__global__ __launch_bounds__(256, 4) void row_sums_kernel(RowSumsArgs a)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int ITERS = kTileIters;
    constexpr int kShare = ITERS * 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x;
    if (a.rows_dev != nullptr && r >= *a.rows_dev) return;
    const int32_t nvec = a.V / EPV;
    const int32_t v0 = wave * kShare;
    f32x4 *const my_sums = reinterpret_cast<f32x4 *>(a.sums + r * kRowSums + wave * ITERS);
    if (v0 >= nvec) {                                        // past the row's end
        if (lane < ITERS / 4) my_sums[lane] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (lane == 0) a.sums[r * kRowSums + kTileWaves * ITERS + wave] = kRefFloor;
        return;
    }
    float thr = -__builtin_inff();
    if constexpr (HAS_THR) thr = a.thr[r];
    const unsigned char *const base =
        reinterpret_cast<const unsigned char *>(reinterpret_cast<const T *>(a.logits) + r * a.ld) + (size_t)v0 * 16u;
    int32_t mych = (nvec - v0 - lane + 63) >> 6;
    mych = mych < 0 ? 0 : (mych > ITERS ? ITERS : mych);
    const uint32_t off0 = (uint32_t)lane * 16u;
    const uint32_t off_last = mych > 0 ? off0 + (uint32_t)(mych - 1) * 1024u : 0u;
    u32x4 raw[ITERS];
#pragma unroll
    for (int j = 0; j < ITERS; ++j) {
        uint32_t off = off0 + (uint32_t)j * 1024u;
        off = off < off_last ? off : off_last;
        if constexpr (NT) raw[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(base + off));
        else raw[j] = *reinterpret_cast<const u32x4 *>(base + off);
    }
    __builtin_amdgcn_sched_barrier(0);
    float rw;
    if (v0 + kShare <= nvec) {
        rw = tile_reference<DT, HAS_THR, false>(raw[0], a.k, thr, mych);
        tile_chunk_sums<DT, HAS_THR, false>(raw, a.k, rw, thr, mych, lane, my_sums);
    } else {
        rw = tile_reference<DT, HAS_THR, true>(raw[0], a.k, thr, mych);
        tile_chunk_sums<DT, HAS_THR, true>(raw, a.k, rw, thr, mych, lane, my_sums);
    }
    if (lane == 0) a.sums[r * kRowSums + kTileWaves * ITERS + wave] = rw;
}

}  // namespace

static_assert(kRowSums == kTileWaves * kTileIters + kTileWaves, "the chunk sums and the waves' references");

as_status launch_row_sums(as_ctx *ctx, const RowSumsArgs &a, int64_t rows)
{
    if (rows == 0) return AS_OK;
    const dim3 grid((unsigned)rows), block(256);
    const bool nt = stream_rows(rows, a.ld, a.dtype == AS_BF16 ? 2 : 4);
#define AS_ROW_SUMS(DT_)                                                                                       \
    do {                                                                                                       \
        if (a.thr && nt) launch(ctx, kKernelInterval, row_sums_kernel<DT_, true, true>, grid, block, 0, a);    \
        else if (a.thr) launch(ctx, kKernelInterval, row_sums_kernel<DT_, true, false>, grid, block, 0, a);    \
        else if (nt) launch(ctx, kKernelInterval, row_sums_kernel<DT_, false, true>, grid, block, 0, a);       \
        else launch(ctx, kKernelInterval, row_sums_kernel<DT_, false, false>, grid, block, 0, a);              \
    } while (0)
    if (a.dtype == AS_BF16) AS_ROW_SUMS(AS_BF16);
    else AS_ROW_SUMS(AS_F32);
#undef AS_ROW_SUMS
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
