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
    const int64_t first = a.range.begin ? *a.range.begin : 0, end = a.range.end ? *a.range.end : first + gridDim.x;
    const int32_t nvec = a.V / EPV;
    const int32_t v0 = wave * kShare;
    // (as many blocks as rows, or as the chip holds a few times where only the device knows how many there are)
    for (int64_t r = first + blockIdx.x; r < end; r += gridDim.x) {
        f32x4 *const my_sums = reinterpret_cast<f32x4 *>(a.sums + r * kRowSums + wave * ITERS);
        if (v0 >= nvec) {                                        // past the row's end
            if (lane < ITERS / 4) my_sums[lane] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (lane == 0) a.sums[r * kRowSums + kTileWaves * ITERS + wave] = kRefFloor;
            continue;
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
}

// The sampling step of step_tile_kernel from those sums, bit for bit: a wave per code reads its row's sums, scans them,
// and reads the one KiB of logits that holds the code.  Bound by its ~400 vector instructions a code: 65536 codes 51 us
// (step_tile_kernel over the same rows, read in the order of the rows, 440).
template <int DT>
__global__ __launch_bounds__(256) void row_select_kernel(SelectArgs q)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int NW = kTileWaves, ITERS = kTileIters;
    __shared__ GenericScratch gen;
    __shared__ bool slow[NW];
    __shared__ int32_t slow_row[NW];
    const StepArgs &a = q.step;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x == 0) q.count[1] = q.count[0];
    const int64_t r = (int64_t)blockIdx.x * NW + wave;
    const int32_t nvec = a.V / EPV;
    const float k = a.k;
    bool beyond = false;
    int32_t row = 0;
    if (r < a.rows) {
        if (a.finished_in != nullptr && a.finished_in[r] != 0) {
            if (lane == 0) write_finished(a, r);
        } else {
            const float code = a.codes[r];
            row = q.slot[clamp_token(q.prev[r], a.V)];
            const float *const sums = q.sums + (int64_t)row * kRowSums;
            const float csum = sums[lane], my_ref = sums[NW * ITERS + lane / ITERS];
            float R = my_ref;
            R = fmaxf(fmaxf(read_lane(R, 0), read_lane(R, 16)), fmaxf(read_lane(R, 32), read_lane(R, 48)));
            const double cv = (double)ldexpf(csum, shift_of(my_ref, R));
            const double cincl = wave_scan_add(cv);
            const double S = read_lane(cincl, 63);
            if (!(S < (double)__builtin_inff())) {
                beyond = true;               // weights beyond fp32, or NaN in the data: the plain routine, below
            } else {
                const double tau = (double)code * S;
                const unsigned long long chit = __ballot(cincl > tau);
                const unsigned long long cnz = __ballot(cv > 0.0);
                const int ch = chit ? (__ffsll((long long)chit) - 1) : (cnz ? (63 - __clzll((long long)cnz)) : 0);
                const double run = read_lane(cincl - cv, ch);
                const float rw = read_lane(my_ref, ch);
                const bool inside = ch * 64 + lane < nvec;
                const u32x4 *const vecs = reinterpret_cast<const u32x4 *>(reinterpret_cast<const T *>(a.logits) + row * a.ld);
                const u32x4 hv = vecs[inside ? ch * 64 + lane : 0];
                float cl = tile_lane_sum<DT, false>(hv, k, -rw, 0.f);
                cl = inside ? cl : 0.f;
                tile_finish<DT, false>(a, r, 0.f, hv, cl, rw, shift_of(rw, R), tau, run, S, ch * 64, lane);
            }
        }
    }
    if (!__syncthreads_or(beyond)) return;
    if (lane == 0) {
        slow[wave] = beyond;
        slow_row[wave] = row;
    }
    __syncthreads();
    for (int w = 0; w < NW; ++w) {
        if (!slow[w]) continue;              // block-uniform
        StepArgs one = a;                    // row r of the call on the logits row of its token
        one.logits = reinterpret_cast<const T *>(a.logits) + ((int64_t)slow_row[w] - ((int64_t)blockIdx.x * NW + w)) * a.ld;
        one.row_ids = nullptr;
        generic_step_row<T>(one, (int64_t)blockIdx.x * NW + w, -__builtin_inff(), gen);
        __syncthreads();
    }
}

// The same sums as a RowRecord: what a decode from a table of every token's logits row needs of a row, a block per row.
template <int DT, bool NT>
__global__ __launch_bounds__(256, 4) void row_records_kernel(const void *logits, int64_t ld, int32_t V, float k,
                                                             unsigned char *records, RowRange range)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int ITERS = kTileIters;
    constexpr int kShare = ITERS * 64;
    __shared__ TileSums ts;
    __shared__ GenericScratch gen;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t r = blockIdx.x + (range.begin ? *range.begin : 0);
    if (range.end && r >= *range.end) return;
    const T *const row = reinterpret_cast<const T *>(logits) + r * ld;
    const int32_t nvec = V / EPV, v0 = wave * kShare;
    f32x4 *const my_sums = reinterpret_cast<f32x4 *>(ts.chunk_sum + wave * ITERS);
    if (v0 >= nvec) {                                            // past the row's end
        if (lane < ITERS / 4) my_sums[lane] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (lane == 0) ts.share_ref[wave] = kRefFloor;
    } else {
        const unsigned char *const base = reinterpret_cast<const unsigned char *>(row) + (size_t)v0 * 16u;
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
            rw = tile_reference<DT, false, false>(raw[0], k, 0.f, mych);
            tile_chunk_sums<DT, false, false>(raw, k, rw, 0.f, mych, lane, my_sums);
        } else {
            rw = tile_reference<DT, false, true>(raw[0], k, 0.f, mych);
            tile_chunk_sums<DT, false, true>(raw, k, rw, 0.f, mych, lane, my_sums);
        }
        if (lane == 0) ts.share_ref[wave] = rw;
    }
    __syncthreads();
    write_row_record(ts, row, V, k, -__builtin_inff(), gen, reinterpret_cast<RowRecord *>(records + r * kTableRecord), lane, wave);
}

// The steps of a decode from a table of every token's logits row, a wave per code through all of them: no row waits
// for another, so there is nothing between a code's steps but its own chain of loads.  A step reads the record of the
// token before (and, for a plain or nucleus step, the KiB of logits that holds the code) and gives what step_tile_kernel,
// nucleus_tile_kernel or topk_tile_kernel would, bit for bit.
//
// DEMAND: only the rows that codes have come to are there.  A code goes on until it meets a token without a row, asks for it
// and leaves its state for the next round.
template <int DT, TableForm FORM, bool DEMAND = false>
__global__ __launch_bounds__(256) void walk_kernel(WalkArgs a)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec, ITERS = kTileIters;
    constexpr bool HAS_THR = FORM == kTableNucleus;
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (DEMAND && blockIdx.x == 0 && threadIdx.x == 0)
        a.round[2 * Demand::kNumbers + Demand::kMade] = a.round[Demand::kNumbers + Demand::kMade];     // (for the next to add to)
    if (r >= a.rows) return;
    const int32_t t0 = DEMAND ? __builtin_amdgcn_readfirstlane(a.at[r]) : 0;
    if (DEMAND && t0 >= a.T) return;
    const int32_t nvec = a.V / EPV;
    const float k = a.k;
    int32_t tok = __builtin_amdgcn_readfirstlane(clamp_token(a.prev[r], a.V));
    float code = a.uniforms ? 0.f : a.codes[r];
    bool ended = a.eos_id >= 0 && __builtin_amdgcn_readfirstlane((int)a.finished[r]) != 0;
    const float *const uniforms = a.uniforms ? a.uniforms + r : nullptr;
    float u_next = uniforms ? uniforms[(int64_t)t0 * a.rows] : 0.f;
    int32_t held = 0;                                            // the tokens of up to 64 steps, a lane each
    int32_t t = t0, live = 0;
    for (; t < a.T; ++t) {
        int32_t place = tok;
        if constexpr (DEMAND) {
            if (!ended) place = __builtin_amdgcn_readfirstlane(a.slot[tok]);
            if (place < 0) break;
            live += ended ? 0 : 1;
        }
        if (uniforms) {
            code = u_next;
            u_next = uniforms[(int64_t)(t + 1 < a.T ? t + 1 : t) * a.rows];
        }
        if (ended) {
            tok = a.eos_id;
        } else {
            const unsigned char *const at = a.records + (int64_t)place * kTableRecord;
            const T *const row = reinterpret_cast<const T *>(a.logits) + (int64_t)place * a.ld;
            if constexpr (FORM == kTableTopK) {
                const CandRecord *const rec = reinterpret_cast<const CandRecord *>(at);
                const double S = rec->S, before = rec->cand[lane].before;
                const float w = rec->cand[lane].w;
                const int32_t mine = rec->cand[lane].token;
                if (!(S < (double)__builtin_inff())) {
                    float c_next;
                    tok = generic_pick_row(row, a.V, k, code, reinterpret_cast<const PlainRecord *>(at), c_next);
                    code = c_next;
                } else {
                    const double tau = (double)code * S;
                    const bool has_weight = w > 0.f;
                    unsigned long long sel = __ballot(has_weight && before <= tau && tau < before + (double)w);
                    if (sel == 0ull) {
                        // the code at the very top by rounding: the last kept token of the vocabulary
                        int32_t best = has_weight ? mine : -1;
#pragma unroll
                        for (int d = 32; d >= 1; d >>= 1) {
                            const int32_t o = __shfl_xor(best, d, 64);
                            best = o > best ? o : best;
                        }
                        sel = __ballot(has_weight && mine == best);
                    }
                    const int l = sel ? (int)__builtin_ctzll(sel) : 0;
                    code = sel ? read_lane(rescale_code(tau, before, (double)w), l) : 0.f;
                    tok = sel ? __builtin_amdgcn_readlane(mine, l) : 0;
                }
            } else {
                const RowRecord *const rec = reinterpret_cast<const RowRecord *>(at);
                const double before = rec->chunk[lane].before, upto = rec->chunk[lane].upto;
                // (ref[0..3], R, thr)
                const float meta = reinterpret_cast<const float *>(rec->ref)[lane < 6 ? lane : 5];
                const double S = read_lane(upto, 63);
                const float thr = HAS_THR ? read_lane(meta, 5) : -__builtin_inff();
                if (!(S < (double)__builtin_inff())) {
                    float c_next;
                    tok = generic_pick_row(row, a.V, k, code, reinterpret_cast<const PlainRecord *>(at), c_next);
                    code = c_next;
                } else {
                    const double tau = (double)code * S;
                    const unsigned long long chit = __ballot(upto > tau);
                    const unsigned long long cnz = __ballot(upto > before);
                    const int ch = chit ? (__ffsll((long long)chit) - 1) : (cnz ? (63 - __clzll((long long)cnz)) : 0);
                    const double run = read_lane(before, ch);
                    const float rw = read_lane(meta, ch / ITERS), R = read_lane(meta, 4);
                    const bool inside = ch * 64 + lane < nvec;
                    const u32x4 hv = reinterpret_cast<const u32x4 *>(row)[inside ? ch * 64 + lane : 0];
                    float e[EPV];
                    tile_weights<DT, HAS_THR>(hv, k, -rw, thr, e);
                    float cl = vec_sum<EPV>(e);
                    cl = inside ? cl : 0.f;
                    const int shf = shift_of(rw, R);
                    double acc, start, ev;
                    const int l = tile_lane(cl, shf, tau, run, acc);
                    const int ih = tile_element(e, shf, tau, acc, lane == l, start, ev);
                    code = read_lane(rescale_code(tau, start, ev), l);
                    tok = (ch * 64 + l) * EPV + __builtin_amdgcn_readlane(ih, l);
                    tok = tok > a.V - 1 ? a.V - 1 : tok;
                }
            }
            tok = __builtin_amdgcn_readfirstlane(tok);
            ended = a.eos_id >= 0 && tok == a.eos_id;
        }
        const int at = (t - t0) & 63;
        held = lane == at ? tok : held;
        if ((at == 63 || t + 1 == a.T) && lane <= at) a.tokens[r * a.T + t - at + lane] = held;
    }
    if constexpr (DEMAND) {
        const int n = (t - t0) & 63;
        if (t < a.T && lane < n) a.tokens[r * a.T + t - n + lane] = held;
        if (lane == 0) {
            a.at[r] = t;
            if (t < a.T) {
                // (looked at first, and few add: 65536 codes at one address, or at some, took 45 to 70 us a round)
                if (a.wanted[tok] == 0) a.wanted[tok] = 1;
                if (a.round[Demand::kWaits] == 0) a.round[Demand::kWaits] = 1;
            }
            if ((r & a.every) == 0) {
                if (live > 1) atomicAdd(&a.round[Demand::kMet], live - 1);
                if (t < a.T) atomicAdd(&a.round[Demand::kMissed], 1);
            }
        }
    }
    if (lane == 0) {
        if (!uniforms) a.codes[r] = code;
        a.prev[r] = tok;
        if (a.eos_id >= 0) a.finished[r] = ended ? 1 : 0;
    }
}

__global__ __launch_bounds__(256) void demand_clear_kernel(Demand d, int32_t V, int64_t rows)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < V) {
        d.slot[i] = -1;
        d.wanted[i] = 0;
    }
    if (i < rows) d.at[i] = 0;
    if (i < (kRounds + 2) * Demand::kNumbers) d.round[i] = 0;
}

// Rows for the tokens that codes wait for and that have none: one addition to the round's counter per block.  Which row a token
// gets differs from run to run; what is in it does not.  For all tokens without one in a last round that codes still wait for,
// and as soon as tokens seem to come evenly (asked once a 32nd of them have a row, of 64 codes): where the share that has one, of
// those that codes meet, is hardly above the share of all, and the codes that wait have steps enough left to come to what is
// missing, more rounds would make nearly all of them by and by.  (Tokens that are few are met again and again: 65536 codes, 3000
// tokens, after a round with 2900 rows 0.97 of those met against 0.09.)
__global__ __launch_bounds__(1024) void demand_claim_kernel(Demand d, int32_t i, int32_t T, int32_t each, bool last, int32_t V)
{
    __shared__ int32_t wave_n[16], block_at;
    const int64_t v = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    bool all = false;
    if (i >= 2) {
        const int32_t *const before = d.round + (i - 1) * Demand::kNumbers;
        const float met = (float)before[Demand::kMet], missed = (float)before[Demand::kMissed], n = met + missed;
        const float made = (float)d.round[i * Demand::kNumbers + Demand::kMade];
        const bool evenly = n >= 16.f && made * 32.f >= (float)V && met < n * (1.4f * made / (float)V + 0.02f) &&
                            missed * (float)each * (float)(T - i) * missed >= ((float)V - made) * n;
        all = before[Demand::kWaits] != 0 && (last || evenly);
    }
    const bool mine = v < V && d.slot[v] < 0 && (all || d.wanted[v] != 0);
    const unsigned long long m = __ballot(mine);
    if (lane == 0) wave_n[wave] = __builtin_popcountll(m);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t n = 0;
        for (int w = 0; w < 16; ++w) {
            const int32_t c = wave_n[w];
            wave_n[w] = n;
            n += c;
        }
        block_at = n ? atomicAdd(&d.round[(i + 1) * Demand::kNumbers + Demand::kMade], n) : 0;
    }
    __syncthreads();
    if (!mine) return;
    const int32_t at = block_at + wave_n[wave] + __builtin_popcountll(m & ((1ull << lane) - 1ull));
    d.slot[v] = at;
    d.token[at] = (int32_t)v;
}

}  // namespace

static_assert(kRowSums == kTileWaves * kTileIters + kTileWaves, "the chunk sums and the waves' references");
static_assert(kTileVecs == kTileWaves * kTileIters * 64, "the vectors of a tile");

as_status launch_row_sums(as_ctx *ctx, int kid, const RowSumsArgs &a, int64_t rows)
{
    if (rows == 0) return AS_OK;
    const int64_t most = 16 * (int64_t)ctx->num_cus;
    const dim3 grid((unsigned)(a.range.end && rows > most ? most : rows)), block(256);
    const bool nt = stream_rows(rows, a.ld, a.dtype == AS_BF16 ? 2 : 4);
#define AS_ROW_SUMS(DT_)                                                                                       \
    do {                                                                                                       \
        if (a.thr && nt) launch(ctx, kid, row_sums_kernel<DT_, true, true>, grid, block, 0, a);    \
        else if (a.thr) launch(ctx, kid, row_sums_kernel<DT_, true, false>, grid, block, 0, a);    \
        else if (nt) launch(ctx, kid, row_sums_kernel<DT_, false, true>, grid, block, 0, a);       \
        else launch(ctx, kid, row_sums_kernel<DT_, false, false>, grid, block, 0, a);              \
    } while (0)
    if (a.dtype == AS_BF16) AS_ROW_SUMS(AS_BF16);
    else AS_ROW_SUMS(AS_F32);
#undef AS_ROW_SUMS
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

// rows that step_tile_kernel would take
bool step_by_sums(const as_ctx *ctx, float temp)
{
    return one_tile_row(ctx->V, ctx->dtype == AS_BF16 ? 2 : 4) && ctx->step_shape == 0 &&
           1.44269504088896340736f / temp <= kTileMaxScale;
}

as_status launch_row_records(as_ctx *ctx, const void *logits, int64_t ld, float temp, unsigned char *records, int64_t rows,
                             RowRange range)
{
    const float k = 1.44269504088896340736f / temp;
    const dim3 grid((unsigned)rows), block(256);
    const bool nt = stream_rows(rows, ld, ctx->dtype == AS_BF16 ? 2 : 4);
    auto go = [&](auto kernel) { launch(ctx, kKernelThreshold, kernel, grid, block, 0, logits, ld, ctx->V, k, records, range); };
    if (ctx->dtype == AS_BF16) nt ? go(row_records_kernel<AS_BF16, true>) : go(row_records_kernel<AS_BF16, false>);
    else nt ? go(row_records_kernel<AS_F32, true>) : go(row_records_kernel<AS_F32, false>);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_walk(as_ctx *ctx, TableForm form, const WalkArgs &a)
{
    auto go = [&](auto kernel) { launch(ctx, kKernelStep, kernel, dim3((unsigned)((a.rows + 3) / 4)), dim3(256), 0, a); };
    auto either = [&](auto all, auto demand) { a.slot ? go(demand) : go(all); };
    if (form == kTableTopK) either(walk_kernel<AS_BF16, kTableTopK>, walk_kernel<AS_BF16, kTableTopK, true>);
    else if (form == kTableNucleus) either(walk_kernel<AS_BF16, kTableNucleus>, walk_kernel<AS_BF16, kTableNucleus, true>);
    else if (a.dtype == AS_BF16) either(walk_kernel<AS_BF16, kTablePlain>, walk_kernel<AS_BF16, kTablePlain, true>);
    else either(walk_kernel<AS_F32, kTablePlain>, walk_kernel<AS_F32, kTablePlain, true>);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_demand_clear(as_ctx *ctx, const Demand &d, int64_t rows)
{
    const int64_t n = larger(larger(ctx->V, rows), (kRounds + 2) * Demand::kNumbers);
    hipLaunchKernelGGL(demand_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, d, ctx->V, rows);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_demand_claim(as_ctx *ctx, const Demand &d, int32_t i, int32_t T, int32_t each, bool last)
{
    hipLaunchKernelGGL(demand_claim_kernel, dim3((unsigned)(((int64_t)ctx->V + 1023) / 1024)), dim3(1024), 0, ctx->stream, d, i, T,
                       each, last, ctx->V);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_row_select(as_ctx *ctx, const SelectArgs &a)
{
    if (a.step.rows == 0) return AS_OK;
    const dim3 grid((unsigned)((a.step.rows + kTileWaves - 1) / kTileWaves)), block(256);
    if (a.step.dtype == AS_BF16) launch(ctx, kKernelStep, row_select_kernel<AS_BF16>, grid, block, 0, a);
    else launch(ctx, kKernelStep, row_select_kernel<AS_F32>, grid, block, 0, a);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
