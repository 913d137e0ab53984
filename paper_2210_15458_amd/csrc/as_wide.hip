// Top-k and the nucleus (the logit modifiers of Sec. 2) together with the sampling step (Algorithm 1, Sec. 4.1)
// in one launch, for rows of any length, alignment and storage type: what the single-tile bf16 kernels do not
// take.  One work-group of 64 to 1024 threads per row (launch_type; 64, a wave, for very many rows of up to 16 KB), the row in its
// registers (up to 16 pieces of 16 bytes a thread: 256 KB with 1024 threads); a longer row goes through the registers a tile at a time and every pass but
// the first starts with the tile that is still there.
//
// What bounds it: a row of V = 50257 fp32 logits is 200 KB, one work-group fills a compute unit's registers with
// it, so nothing hides the work that follows the last load, and that is vector issue (13 slots a logit to count it,
// about 17 for its weight and integer mass) and the latency of some 25 block-wide steps.  Hence a histogram filled
// while the row lands, one more pass, and no visit of memory after the first but for the code's own chunk.
//
//   top-k by a table  (k up to table_most: 40, 48, 64, 96 or 128 by the form, the row's length and whether a nucleus follows)
//                     The k-th largest of 256 group maxima bounds the k-th largest logit from below; the few
//                     pieces that hold logits at or above it go to a table of their wave's, from which those logits become
//                     candidates (value, index), and everything that follows - the exact k-th with its ties, the nucleus
//                     over the survivors, the code's bucket - is ranks and scans over these, by one wave where 64 hold them.
//   nucleus, bf16     a counter a value while the row lands, look-ups in a table of the kept values' weights after it (see below)
//   nucleus           (fp32 rows, thresholds alone, bf16 rows that counters do not suit) 32-bit tallies in kBins bins over kOctaves factors of two (1024 to 4096 over 64; a wave has 512 over 32); the
//                     bin in which the nucleus closes; the chunk sums of everything above a window around it, the
//                     window's logits as a list that is closed by integer masses (see below).
//   larger k          counts in as many bins over 64 factors of two, the logits of the closing bin as a list; a nucleus after it
//                     by fixed-point masses.
// Then the chunk of the code (64 pieces, vocabulary order), its lane, its logit.  Sums that decide anything are taken
// in an order, or in integers, that does not depend on which lane comes first.
//
// One launch against threshold kernel and sampling kernel before: 1 row of 50257 bf16, p = 0.95 13.0 us (45; 20.8 by tallies),
// 512 rows of 50257 fp32, p = 0.92 39.7 us (76; the 103 MB alone take 19 at 5.5 TB/s), 230 rows of 256000 bf16, k = 50 then
// p = 0.95 33.7 us (171; 41.0 with candidates one by one and tiles in turn; 21).
#include <type_traits>

#include "as_common.hpp"
#include "as_pairs.hpp"
#include "as_row.hpp"
#include "as_tile.hpp"

namespace as {
namespace {

typedef unsigned long long u64;

constexpr int kWideTopK = 128;           // largest k of the candidate table
constexpr int kFewTopK = 56;             // ... whose candidates one wave finishes, if there are no more than 64 (ties)
constexpr int kWaveTopK = 40;            // ... where a wave has the row (64 candidates)

// The largest k that a form takes by the candidate table; above it, by counts.  A table of n candidates costs what their
// slots and places do, counts cost a pass over the row: on short rows, with no nucleus behind them, counts are ahead sooner
// (us, table / counts: 4 rows of 1501 bf16, k = 64 10.4 / 7.8, k = 100 13.0 / 7.9; 1000 of 4001 14.3 / 13.4, 17.7 / 13.3, k = 40
// 9.8 / 13.2; 1000 of 8001 k = 64 15.7 / 15.8, k = 100 19.2 / 15.9; 4 of 16001 k = 100 14.5 / 11.3, 300 17.3 / 14.6, 1000 23.1 / 23.8; with
// p = 0.9 1000 of 4001 k = 100 18.1 / 19.1.  fp32, whose pieces are half as many logits, is behind sooner: 4 of 4001 k = 56 8.2 / 7.5,
// 1000 of 3001 k = 60 13.6 / 11.8).
template <int NT, int NP> __host__ __device__ constexpr int32_t table_most(int32_t pieces, bool has_p)
{
    if (NT == 64) return kWaveTopK;
    if (NP > 4 || has_p) return kWideTopK;
    return NT > 256 ? 96 : pieces <= 512 ? 48 : 64;
}

// order-preserving key of a logit (-0 and +0 are one value: one key), and back
__device__ __forceinline__ uint32_t order_key(float f)
{
    uint32_t b = __builtin_bit_cast(uint32_t, f);
    b = (b << 1) ? b : 0u;
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float from_order_key(uint32_t k)
{
    return __builtin_bit_cast(float, (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k);
}

// The mass by which a nucleus is closed: 31 fractional bits of a weight e <= 1 against the row's own reference, what the
// other threshold kernels have (as_threshold.hip; its one-tile nucleus of bf16 rows has sums of fp32 weights), so that the kept set
// does not depend on the kernel.  Sums of them stay below 2^53 for any row.
__device__ __forceinline__ uint32_t mass_of(float e) { return (uint32_t)fmaf(e, 2147483648.f, 0.5f); }
// ... and the one by which a listed logit joins its chunk's weight: 40 fractional bits (24 significant bits: exact for every
// weight above 2^-17)
__device__ __forceinline__ u64 fixed_weight(float e)
{
    const float a = e * 256.f;
    const uint32_t hi = (uint32_t)a;
    const uint32_t lo = (uint32_t)((a - (float)hi) * 4294967296.f);
    return ((u64)hi << 32) | lo;
}

// NT = 64: a wave a row, for very many short ones.  A bin is as wide as in SHORT, over half the octaves (counts: as many octaves,
// twice the width), and a window takes fewer neighbours, so that it mostly closes within the 64 threads.  The list is what the
// waves of a unit leave room for: LDS is given out 1280 bytes at a time, 7680 for five waves a SIMD (16 bytes more of it cost
// all rows 5 to 10 %), 10240 for four.  With 128 entries flat rows were selected all over: 8000 rows of 8000 bf16, p = 0.9, of
// a standard deviation of 1 at a temperature of 0.9 249 us, 98 so, 114 in blocks; of 0.3 363, 122, 134.
// SHORT: the forms for many short rows, where as many blocks as the unit's waves allow hide each other's block-wide
// steps: half the LDS, 16 bins an octave where a nucleus's window is named (a bin's mass to a few parts in 10^4; the masses that
// close it are the same).
template <int NT, bool MULTI, bool SHORT> struct WideShared {
    static constexpr int kWaves = NT / 64;
    static constexpr bool kWave = NT == 64;                  // a wave a row
    static constexpr int kBins = NT == 1024 ? 4096 : kWave ? 512 : SHORT ? 1024 : 2048;
    static constexpr int kOctaves = kWave ? 32 : 64;         // factors of two that the bins take ...
    static constexpr int kTopOctaves = kOctaves / 4;         // ... and of them above the reference
    static constexpr int kPerOctave = kBins / kOctaves;
    static constexpr int kList = NT == 1024 ? 2048 : kWave ? (SHORT ? 240 : 480) : SHORT ? 512 : 1024;
    static constexpr float kBeside = kWave ? 12.f : 32.f;    // logits of a nucleus's window on either side of its bin
    static constexpr int kValues = kWave ? 960 : kBins < 2048 ? kBins : 2048;     // bf16 values with a counter of their own ...
    static constexpr int kHigher = kValues / 4;              // ... of which above the first pieces' largest (128 to a factor of two)
    // (a row of 2^21 fp32 logits: 8193; with 512 threads, where two blocks are to share a unit's LDS, rows of fewer)
    static constexpr int kChunks = !MULTI ? 16 * kWaves + 1 : NT == 1024 ? 8704 : 2304;
    union {
        u64 bins[kBins];
        uint32_t tally[(kBins > kValues ? kBins : kValues) + 64];    // (and a word per lane for what is not counted)
        double cw[2][NT];                                    // candidate weights: after top-k, after the nucleus
        struct {
            u32x4 piece[kWaves][64];                         // pieces with candidates, a table of each wave's
            int32_t first[kWaves][64];                       // the vocabulary index of each one's first logit, or its chunk
        } hot;
    };
    float chunk[kChunks];                                    // weight of every chunk of 64 pieces, vocabulary order ...
    static constexpr int kExtra = MULTI ? 2304 : kChunks;    // (longer rows do without the quick way)
    u64 extra[kExtra];                                       // ... and what the closing bin adds to it, fixed point
    __attribute__((aligned(16))) uint32_t key[kList + 4];    // a list: keys (selection) or values (candidates) ...
    union {
        uint32_t q[kList];                                   // ... with their integer weights
        __attribute__((aligned(16))) uint32_t idx[kList];    // ... or vocabulary indices
    };
    uint16_t at[kList];                                      // the chunk of a list entry
    uint32_t sorted[NT];                                     // a list in another order
    u64 sink[64];                                            // where a weight of zero is added
    u64 wave_q[kWaves];
    double wave_d[kWaves], wave_e[kWaves];
    float wave_f[kWaves];
    uint32_t wave_lo[kWaves], wave_hi[kWaves];
    u64 before;
    double run;
    int32_t pick, again;
    uint32_t n, sel;
    uint32_t stay;                                           // of n candidates, those that stay (n itself is still being read)
};

static_assert(sizeof(WideShared<64, false, true>) <= 7680 && sizeof(WideShared<64, false, false>) <= 10240, "five and four waves a SIMD");

// What the waves of a block have left in LDS, one value each, is taken in by one lane per wave (W <= 16): the row
// sits in most of the registers, a value per wave in every lane would not fit beside it.
__device__ __forceinline__ u64 read_lane(u64 x, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), lane);
    return ((u64)hi << 32) | lo;
}
// What a wave has written to LDS before is there for all its lanes after (it serves a wave in order).
__device__ __forceinline__ void wave_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int N> __device__ __forceinline__ u64 lane_scan(u64 x)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < N; d <<= 1) {
        const u64 y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}
// Exclusive prefix of one integer per thread, thread order, and the block's total.
template <int NT> __device__ __forceinline__ u64 wide_scan(u64 x, u64 *wave_tot, u64 &total)
{
    constexpr int W = NT / 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u64 incl = lane_scan<64>(x);
    __syncthreads();
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    const u64 t = lane < W ? wave_tot[lane] : 0ull;
    const u64 s = lane_scan<W>(t);
    total = read_lane(s, W - 1);
    return read_lane(s, wave) - read_lane(t, wave) + incl - x;
}
// Sum over the waves of a value that each has left; `base`: of those before this one.
template <int NT> __device__ __forceinline__ double wide_total(const double *wave_d, double &base)
{
    constexpr int W = NT / 64;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double t = lane < W ? wave_d[lane] : 0.0;
    const double s = wave_scan_add(t);
    base = as::read_lane(s, wave) - as::read_lane(t, wave);
    return as::read_lane(s, 63);
}
template <int NT> __device__ __forceinline__ float wide_max(float m, float *wave_f)
{
    const int lane = threadIdx.x & 63;
    m = wave_max(m);
    __syncthreads();
    if (lane == 0) wave_f[threadIdx.x >> 6] = m;
    __syncthreads();
    return wave_max(lane < NT / 64 ? wave_f[lane] : -__builtin_inff());
}

// TOPK: top_k is on (and the nucleus if top_p is below 1); otherwise the nucleus alone.  NP: pieces a thread holds.
// MULTI: the row is longer than that.  Without tokens_out only the keep threshold is written, to thr_out.
template <int DT, int NT, int NP, bool MULTI, bool TOPK, int WAVES>
__global__ __launch_bounds__(NT, WAVES) void wide_step_kernel(StepArgs a, int32_t top_k, float top_p, float *thr_out)
{
    using T = typename Elem<DT>::T;
    using Sh = WideShared<NT, MULTI, (WAVES > 4)>;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int W = NT / 64;
    constexpr uint32_t kNegInf = DT == AS_BF16 ? 0xff80ff80u : 0xff800000u;
    __shared__ Sh sh;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t r = blockIdx.x;
    if (a.finished_in != nullptr && a.finished_in[r] != 0) {
        if (tid == 0 && a.tokens_out) write_finished(a, r);
        return;
    }
    const int64_t src = a.row_ids ? (int64_t)a.row_ids[r] : r;
    const T *row = reinterpret_cast<const T *>(a.logits) + src * a.ld;
    const int32_t V = a.V;
    const float k = a.k;
    // The row as the 16-byte pieces it touches: `shift` elements of piece 0 lie before it; `nwhole` pieces end
    // inside it, and a last one may hold `tail` elements of it.
    const int32_t shift = (int32_t)((reinterpret_cast<uintptr_t>(row) & 15u) / sizeof(T));
    const u32x4 *const pieces = reinterpret_cast<const u32x4 *>(row - shift);
    const int32_t vend = V + shift;
    const int32_t nwhole = vend / EPV, tail = vend % EPV;
    const int32_t last = nwhole > 0 ? nwhole - 1 : 0;
    const int32_t ntiles = MULTI ? (nwhole + NT * NP - 1) / (NT * NP) : 1;
    const int32_t nfull = (nwhole + 63) / 64;                // chunks of 64 whole pieces

    // elements [first, live) of a piece are the row's; the others become -inf, which has no weight
    auto cut = [&](u32x4 v, int32_t first, int32_t live) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            if (e >= first && e < live) continue;
            if constexpr (DT == AS_BF16)
                v[e >> 1] = (e & 1) ? ((v[e >> 1] & 0xffffu) | 0xff800000u) : ((v[e >> 1] & 0xffff0000u) | 0xff80u);
            else v[e] = kNegInf;
        }
        return v;
    };
    const u32x4 nothing = u32x4{kNegInf, kNegInf, kNegInf, kNegInf};
    // piece i of the row wherever it lies (-inf past the end)
    auto piece_at = [&](int32_t i) __attribute__((always_inline)) {
        const int32_t at = i <= nwhole - (tail == 0 ? 1 : 0) ? i : 0;
        u32x4 v = pieces[at];
        if (i == 0 && shift != 0) v = cut(v, shift, EPV);
        if (i == nwhole) v = cut(v, i == 0 ? shift : 0, tail);
        return i < nwhole || (i == nwhole && tail != 0) ? v : nothing;
    };

    u32x4 raw[NP], rest = nothing;
    int32_t cur = 0;                                         // the tile in the registers
    auto load = [&](int32_t t) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int32_t i = (t * NP + p) * NT + tid;
            raw[p] = pieces[i < last ? i : last];
        }
        cur = t;
    };
    auto land = [&](int p) __attribute__((always_inline)) {
        const bool in = (cur * NP + p) * NT + tid < nwhole;
#pragma unroll
        for (int i = 0; i < 4; ++i) raw[p][i] = in ? raw[p][i] : kNegInf;
        if (p == 0 && shift != 0 && tid == 0 && cur == 0 && nwhole > 0) raw[0] = cut(raw[0], shift, EPV);
    };
    // whether the row reaches a tile's p-th piece of any thread: a row pays for the pieces it has, not for all that the
    // form can hold (block-uniform; the first is always taken in)
    auto present = [&](int p, int32_t t) __attribute__((always_inline)) { return p == 0 || (t * NP + p) * NT < nwhole; };
    load(0);
    if (tail != 0 && tid == 0) rest = piece_at(nwhole);
    __builtin_amdgcn_sched_barrier(0);

    // f(piece, p, tile) over the row's whole pieces, after4(p, tile) after every four of them (p: the first of the four).
    // FIRST: the resident tile has only been requested.
    auto nothing_more = [](int, int32_t) {};
    auto sweep = [&](auto first_c, auto f, auto after4) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first_c)::value;
        if constexpr (!MULTI) {
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                if constexpr (FIRST) land(p);
                if (present(p, 0)) {
                    u32x4 v = raw[p];
                    asm volatile("" : "+v"(v));              // (a copy: nothing derived in one pass is kept for another)
                    f(v, p, 0);
                }
                __builtin_amdgcn_sched_barrier(0);           // (a piece at a time: interleaved, several do not fit)
                if ((p & 3) == 3 && present(p - 3, 0)) after4(p - 3, 0);
            }
        } else {
            const int32_t begin = cur, step = cur == 0 ? 1 : -1;
            for (int32_t n = 0; n < ntiles; ++n) {
                const int32_t t = begin + n * step;
                if (n != 0) {
                    load(t);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    if (FIRST || n != 0) land(p);
                    if (present(p, t)) {
                        u32x4 v = raw[p];
                        asm volatile("" : "+v"(v));
                        f(v, p, t);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if ((p & 3) == 3 && present(p - 3, t)) after4(p - 3, t);
                }
            }
        }
    };
    typedef std::integral_constant<bool, true> Yes;
    typedef std::integral_constant<bool, false> No;
    auto values = [&](const u32x4 &v, float *x) __attribute__((always_inline)) { unpack<DT>(v, x); };

    auto safe_row = [&]() __attribute__((always_inline)) {   // no logit with weight: any row in range
        if (tid == 0) {
            RowOut o;
            o.token = 0;
            o.c_next = 0.f;
            o.prob = 0.f;
            o.f_lo = 0.f;
            write_row(a, r, o);
        }
    };

    // The candidates (n <= NT) that are among the k highest, with all whose upper 16 bits are the k-th's, to the front of the table, by
    // one wave: it finds those as it found the bound, which becomes that.  (bf16 has no other bits; in fp32 a few more stay.)
    auto shrink = [&](uint32_t n) __attribute__((always_inline)) {
        constexpr int kLow = 16;
        constexpr int M = NT / 64;
        uint32_t c[M];
        uint32_t lo = (uint32_t)sh.before >> kLow, hi = 0u;
#pragma unroll
        for (int i = 0; i < M; ++i) {
            c[i] = 0u;
            if ((uint32_t)(i * 64) < n) {
                const bool in = (uint32_t)(i * 64 + lane) < n;
                c[i] = in ? order_key(__builtin_bit_cast(float, sh.key[i * 64 + lane])) >> kLow : 0u;
                hi = max(hi, c[i]);
            }
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
        hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
        lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2u + 1u;
            int cnt = 0;
#pragma unroll
            for (int i = 0; i < M; ++i)
                if ((uint32_t)(i * 64) < n) cnt += __builtin_popcountll(__ballot(c[i] >= mid));
            if (cnt >= top_k) lo = mid;
            else hi = mid - 1u;
        }
        uint32_t at = 0;
#pragma unroll
        for (int i = 0; i < M; ++i)
            if ((uint32_t)(i * 64) < n) {
                // (a place is never behind where its candidate is)
                const uint32_t x = sh.key[i * 64 + lane], id = sh.idx[i * 64 + lane];
                const u64 in = __ballot(c[i] >= lo);
                wave_lds();
                if (c[i] >= lo) {
                    const uint32_t place = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
                    sh.key[place] = x;
                    sh.idx[place] = id;
                }
                at += (uint32_t)__builtin_popcountll(in);
            }
        if (lane == 0) {
            sh.stay = at;
            sh.before = (u64)lo << kLow;
        }
    };

    // The bound alone, and nothing of the table in registers, which hold two tiles of the row then.
    auto raise = [&](uint32_t n) __attribute__((always_inline)) {
        uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.before), hi = 0xff800000u;           // (+infinity's)
        while (lo < hi) {
            const uint32_t mid = lo + (hi - lo) / 2u + 1u;
            int cnt = 0;
#pragma unroll 2
            for (uint32_t i = 0; i < n; i += 64)
                cnt += __builtin_popcountll(__ballot(i + lane < n && order_key(__builtin_bit_cast(float, sh.key[i + lane])) >= mid));
            if (cnt >= top_k) lo = mid;
            else hi = mid - 1u;
        }
        if (lane == 0) sh.before = lo;
    };

    // The step from n <= 64 candidates, a lane each in sh.key and sh.idx, by one wave; `more`: others than the k highest among them.
    auto finish_few = [&](uint32_t n, bool more) __attribute__((always_inline)) {
        const uint32_t n4 = (n + 3u) & ~3u;
        const bool have = (uint32_t)lane < n;
        const float x = have ? __builtin_bit_cast(float, sh.key[lane]) : -__builtin_inff();
        const uint32_t idx = have ? sh.idx[lane] : 0xffffffffu;
        wave_lds();
        if (!have && (uint32_t)lane < n4) {
            sh.key[lane] = 0xff800000u;
            sh.idx[lane] = 0xffffffffu;
        }
        wave_lds();
        const bool by_mass = top_p > 0.f && top_p < 1.f;
        bool kept = have;
        uint32_t place = 0;
        if (more || by_mass) {
            // its place by value; among the k highest (all that are tied with the k-th) if fewer than k lie above
            uint32_t above = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < n4; j += 4) {
                const f32x4 o = *reinterpret_cast<const f32x4 *>(&sh.key[j]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    above += o[i] > x ? 1u : 0u;
                    place += o[i] == x && j + i < (uint32_t)lane ? 1u : 0u;
                }
            }
            place += above;
            kept = have && above < (uint32_t)top_k;
        }
        const float few_ref = fmaxf(ceilf(wave_max(x) * k), kRefFloor);
        float w = kept ? fast_exp2(fmaf(x, k, -few_ref)) : 0.f;
        if (by_mass) {
            // the value at which the running mass, from the highest down, reaches top_p of the survivors'
            if (have) {
                sh.cw[0][place] = (double)mass_of(w);
                sh.sorted[place] = __builtin_bit_cast(uint32_t, x);
            }
            wave_lds();
            const double v = have ? sh.cw[0][lane] : 0.0;
            const float by_place = have ? __builtin_bit_cast(float, sh.sorted[lane]) : 0.f;
            wave_lds();
            const double incl = wave_scan_add(v);
            const double goal = (double)top_p * as::read_lane(incl, 63);
            const u64 closes = __ballot(have && !(incl - v >= goal) && incl >= goal);
            const float low = closes ? as::read_lane(by_place, (int)__builtin_ctzll(closes)) : -__builtin_inff();
            kept = kept && x >= low;
            w = kept ? w : 0.f;
        }
        if (a.tokens_out == nullptr) {
            const float low = -wave_max(kept ? -x : -__builtin_inff());
            if (lane == 0) thr_out[r] = low;
            return;
        }
        // the kept ones in vocabulary order; the bucket is the last one that has weight and whose mass before it does not exceed c*S
        if (have && !(w > 0.f)) sh.idx[lane] = 0xffffffffu;
        sh.cw[1][lane] = 0.0;
        wave_lds();
        if (w > 0.f) {
            uint32_t place = 0;
#pragma unroll 4
            for (uint32_t j = 0; j < n4; j += 4) {
                const u32x4 o = *reinterpret_cast<const u32x4 *>(&sh.idx[j]);
#pragma unroll
                for (int i = 0; i < 4; ++i) place += o[i] < idx ? 1u : 0u;
            }
            sh.cw[1][place] = (double)w;
            sh.sorted[place] = idx;
        }
        wave_lds();
        const double v = sh.cw[1][lane];
        const double incl = wave_scan_add(v);
        const double S = as::read_lane(incl, 63);
        const double tau = (double)a.codes[r] * S, mine = incl - v;
        const u64 cand = __ballot(v > 0.0 && mine <= tau);
        if (cand == 0ull) {
            safe_row();
        } else if (lane == 63 - (int)__builtin_clzll(cand)) {
            const uint32_t token = sh.sorted[lane];
            RowOut o;
            o.token = (int32_t)(token < (uint32_t)V ? token : (uint32_t)(V - 1));
            o.c_next = rescale_code(tau, mine, v);
            o.prob = (float)(v / S);
            o.f_lo = (float)(mine / S);
            write_row(a, r, o);
        }
    };

    // The step from a single candidate, k = 1 as a rule: nothing to be placed or added up.  (us, by the block / as one of few / so: 1100
    // rows of 20011 bf16 16.0 / 16.8 / 16.1, of 10007 fp32 13.9 / 14.8 / 13.9, 100 of 4001 bf16 6.1 / 6.0 / 5.7, 300 of 50257 fp32 23.7 /
    // 22.4 / 21.4.)
    auto finish_one = [&]() __attribute__((always_inline)) {
        const float x = __builtin_bit_cast(float, sh.key[0]);
        const double v = (double)fast_exp2(fmaf(x, k, -fmaxf(ceilf(x * k), kRefFloor))), tau = (double)a.codes[r] * v;
        if (!(v > 0.0 && tau >= 0.0)) {
            safe_row();
        } else if (lane == 0) {
            const uint32_t token = sh.idx[0];
            RowOut o;
            o.token = (int32_t)(token < (uint32_t)V ? token : (uint32_t)(V - 1));
            o.c_next = rescale_code(tau, 0.0, v);
            o.prob = 1.f;
            o.f_lo = 0.f;
            write_row(a, r, o);
        }
    };

    // ------------------------------------------------------------------ top-k by a table of candidates
    if constexpr (TOPK) {
        const bool by_table = top_k <= table_most<NT, NP>(V / EPV, top_p > 0.f && top_p < 1.f);
        // Rows of several tiles by the table: the pieces of the tile after the next are requested as those of this one are looked at,
        // so that loads are on their way throughout.  (us, tiles of 16 pieces in turn, whose row spilled / so: 256 rows of 256000
        // bf16 k = 50, p = 0.95 45 / 36, k = 128 62 / 45, k = 1 37 / 29.5, 1000 k = 40 144 / 117, 128 of 256000 fp32 47 / 36; a
        // candidate one by one, each waiting for its place, where waves now keep pieces: 38.)
        constexpr bool STREAM = MULTI && NP == 8;
        u32x4 nxt[STREAM ? NP : 1];
        auto request = [&](u32x4 &v, int p, int32_t t) __attribute__((always_inline)) {
            const int32_t i = (t * NP + p) * NT + tid;
            v = pieces[i < last ? i : last];
        };
        if constexpr (STREAM) {
            if (by_table) {
#pragma unroll
                for (int p = 0; p < NP; ++p) request(nxt[p], p, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // the largest of the logits of 256 groups: of one, two or four lanes, or (a wave a row) of every fourth of a lane's pieces
        constexpr int kOwn = Sh::kWave ? 4 : 1;
        float gm[kOwn];
#pragma unroll
        for (int i = 0; i < kOwn; ++i) gm[i] = -__builtin_inff();
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            land(p);
            float x[EPV];
            values(raw[p], x);
            if constexpr (Sh::kWave) {
                // (of short rows a half of a piece each, so that they fill as many groups as they can)
                const bool halves = p < 2 && nwhole <= 128;
                float lo = x[0], hi = x[EPV / 2];
#pragma unroll
                for (int e = 1; e < EPV / 2; ++e) {
                    lo = fmaxf(lo, x[e]);
                    hi = fmaxf(hi, x[EPV / 2 + e]);
                }
                if (halves) {
                    gm[2 * p & 3] = fmaxf(gm[2 * p & 3], lo);
                    gm[(2 * p + 1) & 3] = fmaxf(gm[(2 * p + 1) & 3], hi);
                } else {
                    gm[p & 3] = max3(gm[p & 3], lo, hi);
                }
            } else {
                gm[0] = max3(gm[0], vec_max<EPV>(x), gm[0]);
            }
        }
        if (by_table) {
            if constexpr (STREAM) {                          // (the bound is of two tiles: half as many logits pass it)
#pragma unroll
                for (int p = 0; p < NP; ++p) {
                    const bool in = (NP + p) * NT + tid < nwhole;
                    float x[EPV];
#pragma unroll
                    for (int q = 0; q < 4; ++q) nxt[p][q] = in ? nxt[p][q] : kNegInf;
                    values(nxt[p], x);
                    gm[0] = max3(gm[0], vec_max<EPV>(x), gm[0]);
                }
            }
            if (tid == 0) {
                sh.n = 0;
                sh.sel = 0;
            }
            uint32_t g[4];
            if constexpr (!Sh::kWave) {
                constexpr int kPerGroup = NT / 256;
                float m = gm[0];
                if (kPerGroup >= 2) m = fmaxf(m, __shfl_xor(m, 1, 64));
                if (kPerGroup >= 4) m = fmaxf(m, __shfl_xor(m, 2, 64));
                if (tid % kPerGroup == 0) sh.key[tid / kPerGroup] = order_key(m);
                __syncthreads();
            }
            if (wave == 0) {
                // the largest key that at least k of the maxima reach, by bisection; a round is four ballots
#pragma unroll
                for (int i = 0; i < 4; ++i) g[i] = Sh::kWave ? order_key(gm[i % kOwn]) : sh.key[i * 64 + lane];
                uint32_t lo = min(min(g[0], g[1]), min(g[2], g[3])), hi = max(max(g[0], g[1]), max(g[2], g[3]));
#pragma unroll
                for (int d = 32; d >= 1; d >>= 1) {
                    lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
                    hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
                }
                lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
                hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi);
                while (lo < hi) {
                    const uint32_t mid = lo + (hi - lo) / 2u + 1u;
                    int cnt = 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) cnt += __builtin_popcountll(__ballot(g[i] >= mid));
                    if (cnt >= top_k) lo = mid;
                    else hi = mid - 1u;
                }
                if (lane == 0) sh.before = lo;
            }
            __syncthreads();
            float xb = from_order_key((uint32_t)sh.before);
            const bool bounded = xb > -__builtin_inff();
            // (positive bf16 in pairs, as they are stored: those above `below`, which is the value under the bound)
            bool in_pairs = DT == AS_BF16 && xb > 0.f;
            uint32_t below = ((__builtin_bit_cast(uint32_t, xb) >> 16) - 1u) * 0x10001u;
            int32_t held = 0;                                // pieces in the wave's table
            auto push = [&](const u32x4 &v, int32_t first) __attribute__((always_inline)) {
                bool hot;
                if (in_pairs) {
                    hot = pk_max_i16(pk_max_i16(pk_max_i16(v[0], v[1]), pk_max_i16(v[2], v[3])), below) != below;
                } else {
                    float x[EPV];
                    values(v, x);
                    hot = vec_max<EPV>(x) >= xb;
                }
                const u64 in = __ballot(hot);
                if (in == 0ull) return;
                const int32_t c = __builtin_popcountll(in);
                if (held + c <= 64) {
                    if (hot) {
                        const int32_t at = held + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
                        sh.hot.piece[wave][at] = v;
                        sh.hot.first[wave][at] = first - shift;
                    }
                    held += c;
                } else if (hot) {                            // (a wave whose table is full: one by one; small, it is there per piece)
#pragma unroll 1
                    for (int e = 0; e < EPV; ++e) {
                        const float xe = DT == AS_BF16 ? bits_f32(e & 1 ? v[e >> 1] & 0xffff0000u : v[e >> 1] << 16) : bits_f32(v[e]);
                        if (!(xe >= xb)) continue;
                        const uint32_t slot = atomicAdd(&sh.n, 1u);
                        if (slot < (uint32_t)NT) {
                            sh.key[slot] = __builtin_bit_cast(uint32_t, xe);
                            sh.idx[slot] = (uint32_t)(first + e - shift);
                        }
                    }
                }
            };
            // the wave's pieces taken apart, a lane each
            auto take_apart = [&]() __attribute__((always_inline)) {
                if (held == 0) return;
                wave_lds();
                float x[EPV];
                values(lane < held ? sh.hot.piece[wave][lane] : nothing, x);
                const int32_t first = sh.hot.first[wave][lane];
                uint32_t mine = 0;
#pragma unroll
                for (int e = 0; e < EPV; ++e) mine += (uint32_t)__builtin_popcountll(__ballot(x[e] >= xb));
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&sh.n, mine);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const u64 in = __ballot(x[e] >= xb);
                    const uint32_t slot = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
                    if (x[e] >= xb && slot < (uint32_t)NT) {
                        sh.key[slot] = __builtin_bit_cast(uint32_t, x[e]);
                        sh.idx[slot] = (uint32_t)(first + e);
                    }
                    at += (uint32_t)__builtin_popcountll(in);
                }
                held = 0;
            };
            if (bounded) {
                if constexpr (STREAM) {
                    auto take = [&](u32x4 &v, int p, int32_t t) __attribute__((always_inline)) {
                        const int32_t i = (t * NP + p) * NT + tid;
                        if (present(p, t)) {
                            if (t > 1) {
                                const bool in = i < nwhole;
#pragma unroll
                                for (int q = 0; q < 4; ++q) v[q] = in ? v[q] : kNegInf;
                            }
                            push(v, i * EPV);
                        }
                        request(v, p, t + 2);
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    for (int32_t t = 0; t < ntiles; t += 2) {
#pragma unroll
                        for (int p = 0; p < NP; ++p) take(raw[p], p, t);
#pragma unroll
                        for (int p = 0; p < NP; ++p) take(nxt[p], p, t + 1);
                        if (t + 2 < ntiles) {
                            // (Each tile brings as many as the first two did apiece: after 2, 4, 8 of them a better bound, from the table, if
                            // that is half full.  us, from a quarter / from a half: 16 rows of 190001 fp32 k = 100 43 / 28, 256 of 256000 k =
                            // 128 79 / 64.  Of bf16, twice as many logits a tile, not after 2: us, with / without that, 230 of 256000 k = 50, p
                            // = 0.95 34.7 / 33.7, k = 128 44.2 / 42.6, 1 row 20.2 / 19.1, rows in rising order 423 / 449; fp32 256 of 256000 k =
                            // 128 63.2 / 63.9.)
                            if ((DT == AS_BF16 && t == 0) || ((t + 2) & (t + 1)) != 0) continue;
                            take_apart();
                            __syncthreads();
                            const uint32_t n = sh.n;
                            __syncthreads();                 // (all have read it before a wave whose table fills adds to it)
                            if (n > (uint32_t)NT) break;
                            if (n > (uint32_t)NT / 2) {
                                if (wave == 0) raise(n);
                                __syncthreads();
                                xb = from_order_key((uint32_t)sh.before);
                                below = ((__builtin_bit_cast(uint32_t, xb) >> 16) - 1u) * 0x10001u;
                                in_pairs = DT == AS_BF16 && xb > 0.f;
                            }
                        }
                    }
                } else {
                    sweep(No{}, [&](const u32x4 &v, int p, int32_t t) __attribute__((always_inline)) {
                        push(v, ((t * NP + p) * NT + tid) * EPV);
                    }, nothing_more);
                }
                if (tail != 0 && wave == 0) push(rest, nwhole * EPV);
                take_apart();
            }
            __syncthreads();
            uint32_t n = sh.n;
            if constexpr (!Sh::kWave) {
                // One wave finishes where a lane each holds those that stay: the block takes eight more barriers and ranks all
                // candidates.  Of more than 64 it finds the k-th largest first, as it found the bound; where more than 64 stay, that
                // pays if most go (us, by the block / so: 1 row of 50257 bf16 k = 50, p = 0.95 11.9 / 10.0, 900 of 4001 k = 50, p = 0.8
                // 11.6 / 9.9, 2500 of 20003 k = 40 40.8 / 33.3, 300 of 50257 fp32 26.2 / 23.5; 16 of 9001 fp32 k = 64, of 75 candidates,
                // 11.1 / 13.8).
                if (bounded && n <= 64u) {
                    if (wave == 0) {
                        if (__builtin_expect(n == 1u && a.tokens_out != nullptr, 0)) finish_one();
                        else finish_few(n, true);
                    }
                    return;
                }
                if (bounded && n <= (uint32_t)NT && (top_k <= kFewTopK || n > 2u * (uint32_t)top_k)) {
                    if (wave == 0) {
                        shrink(n);
                        wave_lds();
                        if (sh.stay <= 64u) finish_few(sh.stay, DT != AS_BF16);
                    }
                    __syncthreads();
                    n = sh.stay;
                    if (n <= 64u) return;
                }
            }
            if (bounded && n <= (uint32_t)NT) {
                const uint32_t n4 = (n + 3u) & ~3u;
                if ((uint32_t)tid >= n && (uint32_t)tid < n4) {
                    sh.key[tid] = 0xff800000u;
                    sh.idx[tid] = 0xffffffffu;
                }
                const bool have = (uint32_t)tid < n;
                const float x = have ? __builtin_bit_cast(float, sh.key[tid]) : -__builtin_inff();
                const uint32_t idx = have ? sh.idx[tid] : 0xffffffffu;
                __syncthreads();
                // its place by value; among the k highest (all that are tied with the k-th) if fewer than k lie above
                uint32_t above = 0, place = 0;
                if (wave * 64 < (int)n) {
#pragma unroll 4
                    for (uint32_t j = 0; j < n4; j += 4) {
                        const f32x4 o = *reinterpret_cast<const f32x4 *>(&sh.key[j]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            above += o[i] > x ? 1u : 0u;
                            place += o[i] == x && j + i < (uint32_t)tid ? 1u : 0u;
                        }
                    }
                }
                place += above;
                bool kept = have && above < (uint32_t)top_k;
                const float ref = fmaxf(ceilf(wide_max<NT>(kept ? x : -__builtin_inff(), sh.wave_f) * k), kRefFloor);
                float w = kept ? fast_exp2(fmaf(x, k, -ref)) : 0.f;
                double before;
                if (top_p > 0.f && top_p < 1.f) {
                    // the value at which the running mass, from the highest down, reaches top_p of the survivors'
                    if (have) {
                        sh.cw[0][place] = (double)mass_of(w);
                        sh.sorted[place] = __builtin_bit_cast(uint32_t, x);
                    }
                    if (tid == 0) sh.run = -__builtin_inf();
                    __syncthreads();
                    const double v = have ? sh.cw[0][tid] : 0.0;
                    const double incl = wave_scan_add(v);
                    if (lane == 63) sh.wave_d[wave] = incl;
                    __syncthreads();
                    const double goal = (double)top_p * wide_total<NT>(sh.wave_d, before);
                    if (have && !(before + incl - v >= goal) && before + incl >= goal)
                        sh.run = (double)__builtin_bit_cast(float, sh.sorted[tid]);
                    __syncthreads();
                    kept = kept && (double)x >= sh.run;
                    w = kept ? w : 0.f;
                }
                if (a.tokens_out == nullptr) {
                    const float low = -wide_max<NT>(kept ? -x : -__builtin_inff(), sh.wave_f);
                    if (tid == 0) thr_out[r] = low;
                    return;
                }
                // the kept ones in vocabulary order; the bucket is the last one that has weight and whose mass before
                // it does not exceed c*S
                if (have && !(w > 0.f)) sh.idx[tid] = 0xffffffffu;
                if ((uint32_t)tid < n4) sh.cw[1][tid] = 0.0;
                __syncthreads();
                if (wave * 64 < (int)n && w > 0.f) {
                    place = 0;
#pragma unroll 4
                    for (uint32_t j = 0; j < n4; j += 4) {
                        const u32x4 o = *reinterpret_cast<const u32x4 *>(&sh.idx[j]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) place += o[i] < idx ? 1u : 0u;
                    }
                    sh.cw[1][place] = (double)w;
                    sh.sorted[place] = idx;
                }
                __syncthreads();
                const double v = (uint32_t)tid < n ? sh.cw[1][tid] : 0.0;
                const double incl = wave_scan_add(v);
                if (lane == 63) sh.wave_e[wave] = incl;
                __syncthreads();
                const double S = wide_total<NT>(sh.wave_e, before);
                const double tau = (double)a.codes[r] * S, mine = before + incl - v;
                const bool cand = v > 0.0 && mine <= tau;
                if (cand) atomicMax(&sh.sel, (uint32_t)tid + 1u);
                __syncthreads();
                const uint32_t sel = sh.sel;
                if (sel == 0u) safe_row();
                else if (cand && (uint32_t)tid + 1u == sel) {
                    const uint32_t token = sh.sorted[tid];
                    RowOut o;
                    o.token = (int32_t)(token < (uint32_t)V ? token : (uint32_t)(V - 1));
                    o.c_next = rescale_code(tau, mine, v);
                    o.prob = (float)(v / S);
                    o.f_lo = (float)(mine / S);
                    write_row(a, r, o);
                }
                return;
            }
            __syncthreads();
            if constexpr (!Sh::kWave) {
                // (the table has not taken them all: from the row's start, whose pieces are not kept beside the table)
                load(0);
#pragma unroll
                for (int p = 0; p < NP; ++p) land(p);
            }
        }
    }

    // ------------------------------------------------------------------ selection by integer weights
    float mx = -__builtin_inff();        // the row's largest logit, once a pass has seen all of it
    float ref, first_max;                // the first pieces' largest
    // Whether bf16 logits can be counted by value: those that are positive are expected to hold the nucleus.  Of the weights of
    // half the first pieces the others may be four fifths of what it leaves out (they miss the row's largest logits, so that
    // share is more likely too large than too small; a row that goes wrong is selected the other way, after one more pass).
    // Between rows that are counted late and those that are counted in vain (us, never counted / up to 0.4 / 0.8 / 1.2 / 2 of that:
    // 1000 rows of 9001 of a standard deviation of 1.5, p = 0.9 23.6 / 23.6 / 20.5 / 17.6 / 17.6; of 2, p = 0.98 24.3 / 24.3 / 26.7 / 30.1 /
    // 30.8; of 3 about -3, p = 0.9 24.1 / 22.9 / 18.3 / 17.3 / 17.4, p = 0.98 24.1 / 26.6 / 28.4 / 29.5 / 30.3; of 3, p = 0.5 to 0.98 24 / 17).
    constexpr bool COUNTED = DT == AS_BF16 && !TOPK;
    bool by_value = false;
    {
        if constexpr (!TOPK) land(0);
        float x[EPV];
        values(rest, x);
        float m = vec_max<EPV>(x);
        values(raw[0], x);
        m = fmaxf(m, vec_max<EPV>(x));
        float spare = 0.f;
        if constexpr (COUNTED) {
            m = wave_max(m);
            const float r0 = fmaxf(ceilf(m * k), kRefFloor), in = 0.8f * (1.f - top_p), out = in - 1.f;
#pragma unroll
            for (int i = 0; i < EPV; i += 2) spare = fmaf(fast_exp2(fmaf(x[i], k, -r0)), x[i] > 0.f ? in : out, spare);
            spare = wave_sum(spare);
            if (lane == 0 && !Sh::kWave) sh.wave_d[wave] = (double)spare;
        }
        first_max = COUNTED && Sh::kWave ? m : wide_max<NT>(m, sh.wave_f);
        ref = fmaxf(ceilf(first_max * k), kRefFloor);
        if constexpr (COUNTED) {
            if constexpr (!Sh::kWave) {
                const float r0 = fmaxf(ceilf((lane < W ? sh.wave_f[lane] : -__builtin_inff()) * k), kRefFloor);
                spare = wave_sum(lane < W ? (float)sh.wave_d[lane] * fast_exp2(r0 - ref) : 0.f);
            }
            by_value = a.tokens_out != nullptr && first_max > 0.f && spare >= 0.f;
        }
    }
    constexpr float kTwo23 = 8388608.f;
    constexpr float kScale = (float)Sh::kPerOctave;
    constexpr float kBinLo = kTwo23, kBinHi = kTwo23 + (float)(Sh::kBins - 1);
    constexpr float kBin0 = kTwo23 + (float)(Sh::kTopOctaves * Sh::kPerOctave);
    // coarse bin of an exponent argument relative to the reference, as a float whose low mantissa bits are the bin
    // (rounded to the nearest integer and clamped to the table; falls as the logit rises)
    auto bin_of = [&](float y) __attribute__((always_inline)) {
        return __builtin_amdgcn_fmed3f(fmaf(y, -kScale, kBin0), kBinLo, kBinHi);
    };
    typedef __attribute__((address_space(3))) u64 lds_u64;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    lds_u64 *const bins = (lds_u64 *)sh.bins;
    lds_u64 *const sink = (lds_u64 *)sh.sink + lane;
    auto add = [&](lds_u64 *at, u64 q) __attribute__((always_inline)) {
        __hip_atomic_fetch_add(at, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto clear_bins = [&]() __attribute__((always_inline)) {
        __syncthreads();
        for (int b = tid; b < Sh::kBins; b += NT) sh.bins[b] = 0;
        if (tid == 0) {
            sh.n = 0;
            sh.pick = -1;
        }
        __syncthreads();
    };
    // After the bins are filled: the first one, from the top, at which base + the running weight reaches the
    // goal.  Leaves it in sh.pick (-1: none does) and the weight above it, base included, in sh.before.
    auto reach = [&](u64 base, double &need, bool set_need, auto count_c) __attribute__((always_inline)) {
        constexpr bool COUNT = decltype(count_c)::value;     // counts, in 32 bits
        constexpr int kPer = Sh::kBins / NT;
        u64 h[kPer], local = 0, total;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            h[i] = COUNT ? (u64)sh.tally[tid * kPer + i] : sh.bins[tid * kPer + i];
            local += h[i];
        }
        const u64 excl = base + wide_scan<NT>(local, sh.wave_q, total);
        if (set_need) need = COUNT ? (double)top_k : (double)top_p * (double)total;
        if (!((double)excl >= need) && (double)(excl + local) >= need) {
            u64 acc = excl;
            bool open = true;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                if (open && (double)(acc + h[i]) >= need) {
                    sh.pick = tid * kPer + i;
                    sh.before = acc;
                    open = false;
                }
                acc += h[i];
            }
        }
        __syncthreads();
    };
    // The exact end of a selection: the list (n entries) holds the logits of the closing bin,
    // `base` is the weight above them; the key of the group of equal logits at which the running weight reaches
    // `need`, or 0 (no logit's key) if it does not get there.  all(put) puts every logit of the bin, for a list that did
    // not take them all.
    constexpr uint32_t kAll = 0xffffffffu;                   // (n for the whole row)
    auto close = [&](uint32_t n, u64 base, double need, auto all)
                     __attribute__((always_inline)) -> uint32_t {
        if (n <= (uint32_t)NT) {
            // every entry's place by key, the weights in that order, their running sums (integers below 2^53: exact)
            double *const sorted = sh.cw[0];
            uint32_t *const skey = sh.sorted;
            const uint32_t n4 = (n + 3u) & ~3u;
            if ((uint32_t)tid >= n && (uint32_t)tid < n4) sh.key[tid] = 0u;
            if (tid == 0) sh.sel = 0u;
            __syncthreads();
            if ((uint32_t)tid < n) {
                const uint32_t mine = sh.key[tid];
                uint32_t place = 0;
#pragma unroll 4
                for (uint32_t j = 0; j < n4; j += 4) {
                    const u32x4 o = *reinterpret_cast<const u32x4 *>(&sh.key[j]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) place += o[i] > mine || (o[i] == mine && j + i < (uint32_t)tid) ? 1u : 0u;
                }
                sorted[place] = (double)sh.q[tid];
                skey[place] = mine;
            }
            __syncthreads();
            const double v = (uint32_t)tid < n ? sorted[tid] : 0.0;
            const double incl = wave_scan_add(v);
            if (lane == 63) sh.wave_d[wave] = incl;
            __syncthreads();
            double first;
            wide_total<NT>(sh.wave_d, first);
            const double upto = (double)base + first + incl;
            if ((uint32_t)tid < n && !(upto - v >= need) && upto >= need) sh.sel = skey[tid];
            __syncthreads();
            return sh.sel;
        }
        // the range of their keys (a wave's: it has 512 bins, and a bin or a window is narrow: two rounds then, of the whole 32
        // bits four)
        uint32_t klo = 0u, khi = 0xffffffffu;
        if (Sh::kWave && n != kAll) {
            klo = 0xffffffffu;
            khi = 0u;
            auto span = [&](uint32_t key, u64) __attribute__((always_inline)) {
                klo = min(klo, key);
                khi = max(khi, key);
            };
            if (n <= (uint32_t)Sh::kList) {
                for (uint32_t i = tid; i < n; i += NT) span(sh.key[i], 0ull);
            } else {
                all(span);
            }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                klo = min(klo, (uint32_t)__shfl_xor((int)klo, d, 64));
                khi = max(khi, (uint32_t)__shfl_xor((int)khi, d, 64));
            }
            klo = (uint32_t)__builtin_amdgcn_readfirstlane((int)klo);
            khi = (uint32_t)__builtin_amdgcn_readfirstlane((int)khi);
            if (klo > khi) return 0u;
        }
        // it is cut into kBins intervals of 2^s keys, from the top, then the one that closes, until it is one key
        for (;;) {
            const uint32_t span = khi - klo;
            const int s = span >= (uint32_t)Sh::kBins ? 32 - __builtin_clz(span) - (31 - __builtin_clz((uint32_t)Sh::kBins)) : 0;
            clear_bins();
            auto put = [&](uint32_t key, u64 q) __attribute__((always_inline)) {
                if (key >= klo && key <= khi) add(bins + ((khi - key) >> s), q);
            };
            if (n <= (uint32_t)Sh::kList) {
                for (uint32_t i = tid; i < n; i += NT) put(sh.key[i], sh.q[i]);
            } else {
                all(put);
            }
            reach(base, need, false, No{});
            const int32_t at = sh.pick;
            if (at < 0) return 0u;
            base = sh.before;
            const uint32_t top = khi - ((uint32_t)at << s);
            const uint32_t low = (uint32_t)(1u << s) - 1u;
            klo = top - klo > low ? top - low : klo;
            khi = top;
            if (s == 0) break;
        }
        return khi;
    };

    // f(piece) over the row for the selection by integer weights: with top-k it is the way (k above table_most), from the
    // registers; after the quick way of the nucleus it is the rare case, and goes over memory (kept for it as
    // well, the row costs spilled registers on the way that is taken)
    auto every_piece = [&](auto f) __attribute__((always_inline)) {
        if constexpr (TOPK) {
            sweep(No{}, [&](const u32x4 &v, int, int32_t) __attribute__((always_inline)) { f(v); }, nothing_more);
            if (tail != 0 && wave == 0) f(rest);
        } else {
            for (int32_t i = tid; i <= nwhole; i += NT) f(piece_at(i));
        }
    };
    // the same many times over: from memory (the row's registers in a loop do not fit)
    auto every_piece_again = [&](auto f) __attribute__((always_inline)) {
        for (int32_t i = tid; i <= nwhole; i += NT) f(piece_at(i));
    };
    // One selection: the key of the group of equal logits at which the running weight, from the largest logit
    // down, reaches the goal.  COUNT: weights of 1 against top_k; otherwise masses of the logits >= floor_x
    // against top_p of their total (the reference is the row's own then).  False if no logit has weight.
    auto select = [&](auto count_c, float floor_x, float &thr) __attribute__((always_inline)) -> bool {
        constexpr bool COUNT = decltype(count_c)::value;
        // (counts always reach over 64 factors of two: a large k may lie deep)
        constexpr float kCountScale = (float)(Sh::kBins / 64), kCountBin0 = kTwo23 + (float)(Sh::kBins / 4);
        float nr = -ref;
        auto weight = [&](float x) __attribute__((always_inline)) -> u64 {
            if constexpr (COUNT) return 1ull;
            else return x >= floor_x ? (u64)mass_of(fast_exp2(fmaf(x, k, nr))) : 0ull;
        };
        auto fill = [&]() __attribute__((always_inline)) {
            float m = -__builtin_inff();
            auto one = [&](const u32x4 &v) __attribute__((always_inline)) {
                float x[EPV];
                values(v, x);
                m = max3(m, vec_max<EPV>(x), m);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    if constexpr (COUNT) {
                        // (what lies below the last bin, padding among it, goes to a word of the lane's own)
                        const float t = __builtin_amdgcn_fmed3f(fmaf(fmaf(x[e], k, nr), -kCountScale, kCountBin0), kBinLo,
                                                                kTwo23 + (float)(Sh::kBins + lane));
                        __hip_atomic_fetch_add((lds_u32 *)sh.tally + (__builtin_bit_cast(uint32_t, t) - 0x4B000000u), 1u,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    } else {
                        const uint32_t b = __builtin_bit_cast(uint32_t, bin_of(fmaf(x[e], k, nr))) & (uint32_t)(Sh::kBins - 1);
                        const u64 q = weight(x[e]);
                        add(q != 0 ? bins + b : sink, q);
                    }
                    if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            };
            every_piece(one);
            mx = wide_max<NT>(m, sh.wave_f);
        };
        clear_bins();
        fill();
        if constexpr (COUNT) {
            const float exact = fmaxf(ceilf(mx * k), kRefFloor);
            if (!(exact - ref <= 16.f)) {
                // a logit far above the first pieces' largest: once more against the row's own reference
                ref = exact;
                nr = -ref;
                clear_bins();
                fill();
            }
        }
        double need = 0.0;
        reach(0ull, need, true, count_c);
        const int32_t pick = sh.pick;
        if (pick < 0) {
            if constexpr (!COUNT) return false;
            // fewer than k logits within the bins: by key over the whole row
            const uint32_t key = close(kAll, 0ull, need, [&](auto put) __attribute__((always_inline)) {
                every_piece_again([&](const u32x4 &v) __attribute__((always_inline)) {
                    float x[EPV];
                    values(v, x);
                    for (int e = 0; e < EPV; ++e) put(order_key(x[e]), 1ull);
                });
            });
            thr = from_order_key(key);
            return key != 0u;
        }
        u64 base = sh.before;
        const float tpick = kTwo23 + (float)pick;
        auto member = [&](float x) __attribute__((always_inline)) {
            const float y = fmaf(x, k, nr);
            if constexpr (COUNT) return __builtin_amdgcn_fmed3f(fmaf(y, -kCountScale, kCountBin0), kBinLo, kBinHi) == tpick;
            else return bin_of(y) == tpick;
        };
        // f(key, weight) for the logits of that bin in one piece
        auto members = [&](const u32x4 &v, auto f) __attribute__((always_inline)) {
            float x[EPV];
            values(v, x);
            bool any = false;
#pragma unroll
            for (int e = 0; e < EPV; ++e) any |= member(x[e]);
            if (any) {
#pragma unroll
                for (int e = 0; e < EPV; ++e)
                    if (member(x[e])) {
                        const u64 q = weight(x[e]);
                        if (q) f(order_key(x[e]), q);
                    }
            }
        };
        every_piece([&](const u32x4 &v) __attribute__((always_inline)) {
            members(v, [&](uint32_t key, u64 q) __attribute__((always_inline)) {
                const uint32_t i = atomicAdd(&sh.n, 1u);
                if (i < (uint32_t)Sh::kList) {
                    sh.key[i] = key;
                    sh.q[i] = (uint32_t)q;
                }
            });
        });
        __syncthreads();
        const uint32_t n = sh.n;
        const uint32_t key = close(n, base, need, [&](auto put) __attribute__((always_inline)) {
            // more than the list takes
            every_piece_again([&](const u32x4 &v) __attribute__((always_inline)) { members(v, put); });
        });
        thr = from_order_key(key);
        return key != 0u;                                    // (0: the weights of a NaN row)
    };

    // four chunk sums of the wave, from its lanes' (0 for a piece that the row does not reach: chunks past the row's end
    // are written, and read by nobody)
    auto chunks_done = [&](float (&t)[4], int p, int32_t tile) __attribute__((always_inline)) {
        wave_sum4_in_lane63(t[0], t[1], t[2], t[3]);
        if (lane == 63) {
#pragma unroll
            for (int i = 0; i < 4; ++i) sh.chunk[(tile * NP + p + i) * W + wave] = t[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = 0.f;
    };

    float thr = -__builtin_inff();
    bool some = true, summed = false;    // summed: the chunk sums of the kept logits are in place, a part of them in `extra`
    bool in_chunks = false;              // ... or all of them in `chunk`
    if constexpr (TOPK) {
        some = select(Yes{}, 0.f, thr);
        if (some && top_p > 0.f && top_p < 1.f) {
            ref = fmaxf(ceilf(mx * k), kRefFloor);
            float inner = thr;
            some = select(No{}, thr, inner);
            thr = fmaxf(thr, inner);
        }
    } else {
        bool closed = false;
        if constexpr (COUNTED) {
            // bf16 logits by value.  One of 65536 values, so the mass of a group of equal logits is a count times a weight: while
            // the row lands every logit adds one to the counter of its value, in a window of kValues values around the first
            // pieces' largest, and its weight to the lane's total; what lies below the window or is not positive goes to a word of
            // the lane's own.  The counters, from the top, name the value at which the nucleus closes; they give way to a table of
            // the kept values' weights, and the chunk sums of the kept logits are look-ups: half the instructions of the
            // tallies and integer masses below, which is what bounds either (one row of 50257 takes 2400 a wave with those, 16 of
            // its 21 us).  us, tallies / counters: 1 row of 50257 20.8 / 13.1, of 256000 63 / 34, 200 of 33001 21.2 / 14.2, 2000 of
            // 20001 56 / 38, 2000 of 50257 112 / 77, 16000 of 8001 141 / 91, 14000 of 1501 54 / 43.  A logit above the window or a
            // nucleus that reaches below it: the other way.  The counters are weighed in the other way's integers; the total, a sum of
            // fp32 weights, is known to some 2e-6, and where that leaves open which group of equal logits closes (a row in 500 of
            // these), one more pass adds up the row's integers, so that the kept set is the other way's.  (A launch lasts as long as
            // its last such row, and the pass costs registers beside the row's: us, without / so, 200 rows of 33001 13.5 / 14.2, 2000 of
            // 32001 45.6 / 50.6, 2000 of 50257 72.5 / 77.3, 1100 of 12001 18.0 / 19.4, 16000 of 8001 even; with the whole other way for
            // such rows 17.5, 60.5, 91, 22.7, 105.)
            int32_t top = (int32_t)(__builtin_bit_cast(uint32_t, first_max) >> 16) + Sh::kHigher;
            top = top > 0x7f7f ? 0x7f7f : top;               // (the largest finite value)
            const int32_t bottom = top - (Sh::kValues - 1);
            if (by_value && bottom > 0) {
                lds_u32 *const tally = (lds_u32 *)sh.tally;
                __syncthreads();
                for (int b = tid; b < Sh::kValues + 64; b += NT) sh.tally[b] = 0u;
                constexpr int32_t kOpen = -2;
                if (tid == 0) sh.pick = sh.again = -1;
                __syncthreads();
                const float nr = -ref;
                double total = 0.0;
                uint32_t hi = 0x80008000u;                   // the largest of either half of a word, as the sign leaves them
                {
                    const uint32_t low2 = (uint32_t)bottom * 0x10001u, none = (uint32_t)(Sh::kValues + lane) * 0x10001u;
                    auto one = [&](const u32x4 &v) __attribute__((always_inline)) {
                        total += (double)tile_lane_sum<DT, false>(v, k, nr, 0.f);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            hi = pk_max_i16(hi, v[i]);
                            const uint32_t d = pk_min_u16(pk_sub_u16(v[i], low2), none);
                            __hip_atomic_fetch_add(tally + (d & 0xffffu), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                            __hip_atomic_fetch_add(tally + (d >> 16), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        }
                        asm volatile("" : "+v"(hi));
                    };
                    sweep(Yes{}, [&](const u32x4 &v, int, int32_t) __attribute__((always_inline)) { one(v); }, nothing_more);
                    if (tail != 0 && wave == 0) one(rest);
                }
                total = wave_sum(total);
                const float largest = wave_max((float)max((int32_t)hi >> 16, (int32_t)(hi << 16) >> 16));
                if (lane == 0) {
                    sh.wave_d[wave] = total;
                    sh.wave_f[wave] = largest;
                }
                __syncthreads();
                // running mass over the counters, from the top; a thread has kPer of them
                constexpr int kPer = Sh::kValues / NT;
                static_assert(kPer * NT == Sh::kValues, "a share of the counters for every thread");
                double local = 0.0, unused;
                total = wide_total<NT>(sh.wave_d, unused);
                // The row's largest value, as it is stored (a NaN's and infinity's are above the window).  From here on weights are
                // against it: the first pieces' largest may lie a hundred factors of two lower, where a chunk's sum leaves fp32 with
                // every lane's inside it.
                const int32_t stored = (int32_t)wave_max(lane < W ? sh.wave_f[lane] : 0.f);
                const bool inside = stored <= top;
                const float own = fmaxf(ceilf(bits_f32((uint32_t)stored << 16) * k), kRefFloor);
                // (Weights made anew where they are wanted again: kept, fifteen of them a lane spill a wave's row, and so does a branch
                // for the values above the largest, which no logit has and whose weights may be beyond fp32.)
                auto weight_of = [&](int32_t b) __attribute__((always_inline)) {
                    asm volatile("" : "+v"(b));
                    return fminf(fast_exp2(fmaf(bits_f32((uint32_t)(bottom + b) << 16), k, -own)), 1.f);
                };
                auto mass_at = [&](int32_t b) __attribute__((always_inline)) {
                    return (double)sh.tally[b] * (double)mass_of(weight_of(b));
                };
                const int32_t b0 = Sh::kValues - 1 - tid * kPer; // the thread's highest
#pragma unroll
                for (int i = 0; i < kPer; ++i) local += mass_at(b0 - i);
                const double incl = wave_scan_add(local);
                if (lane == 63) sh.wave_e[wave] = incl;
                __syncthreads();
                double lo;
                wide_total<NT>(sh.wave_e, lo);
                lo += incl - local;
                // In masses the total may be off, against the sum of the row's integers, by three roundings of a piece's sum and one of
                // a mass near 2^23, 2.5 2^-23 of it together, and by a half for every logit.  Where the reference was another, also by
                // two exponentials, 2^-23 each, and the rounding of their arguments: 2.8 2^-23 each where those are at most 16 (the
                // weights below 2^-16 are at most V 2^-16 together: 0.05 a logit), twice that up to 32, and so on.
                const double lower = (double)(own - ref);
                total = ldexp(total, (int)(ref - own) + 31);
                const double off = lower == 0.0 ? 3.2e-7 * total + 0.5 * (double)V
                                          : (1.3e-6 + 1e-7 * fmax(lower - 8.0, 0.0)) * total + 0.55 * (double)V;
                auto find = [&](double slack, int32_t *at) __attribute__((always_inline)) {
                    const double need = (double)top_p * total;
                    if (!(lo >= need) && lo + local >= need) {
                        double above = lo, upto = lo;        // (sums of integers below 2^53: exact)
                        int32_t found = -1;
#pragma unroll 1
                        for (int i = 0; i < kPer && found < 0; ++i) {
                            above = upto;
                            upto += mass_at(b0 - i);
                            if (upto >= need) found = b0 - i;
                        }
                        *at = above < need - slack && upto >= need + slack ? found : kOpen;
                    }
                    __syncthreads();
                    return *at;
                };
                const bool fits = inside && total < (double)__builtin_inff();
                int32_t pick = find((double)top_p * off, &sh.pick);
                if (pick == kOpen && fits) {
                    u64 all = 0;
                    auto one = [&](const u32x4 &v) __attribute__((always_inline)) {
                        float x[EPV];
                        values(v, x);
#pragma unroll
                        for (int i = 0; i < EPV; ++i) all += mass_of(fast_exp2(fmaf(x[i], k, -own)));
                        asm volatile("" : "+v"(all));
                    };
                    // (us, from memory / from the registers: 16000 rows of 8001 99 / 91, 2000 of 32001, whose registers are spilled, 50.6 / 53.4)
                    if constexpr (NT * NP <= 1024) {
                        sweep(No{}, [&](const u32x4 &v, int, int32_t) __attribute__((always_inline)) { one(v); }, nothing_more);
                        if (tail != 0 && wave == 0) one(rest);
                    } else {
                        every_piece(one);
                    }
                    const double all_wave = wave_sum((double)all);
                    if (lane == 0) sh.wave_d[wave] = all_wave;
                    __syncthreads();
                    total = wide_total<NT>(sh.wave_d, unused);
                    pick = find(0.0, &sh.again);
                }
                if (fits && pick >= 0) {
                    // The kept values' weights, from the threshold's on, and behind them 64 zeros, a word a lane, for all others.
                    float *const wtab = reinterpret_cast<float *>(sh.tally);
                    const int32_t kept = Sh::kValues - pick;
#pragma unroll
                    for (int i = 0; i < kPer; ++i)
                        if (b0 - i >= pick) wtab[b0 - i - pick] = weight_of(b0 - i);
                    if (wave == W - 1) wtab[kept + lane] = 0.f;
                    thr = bits_f32((uint32_t)(bottom + pick) << 16);
                    ref = own;
                    __syncthreads();
                    const uint32_t low2 = (uint32_t)(bottom + pick) * 0x10001u, none = (uint32_t)(kept + lane) * 0x10001u;
                    float t[4] = {0.f, 0.f, 0.f, 0.f};
                    sweep(No{}, [&](const u32x4 &v, int p, int32_t) __attribute__((always_inline)) {
                        float e[EPV];
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const uint32_t d = pk_min_u16(pk_sub_u16(v[i], low2), none);
                            e[2 * i] = wtab[d & 0xffffu];
                            e[2 * i + 1] = wtab[d >> 16];
                        }
                        t[p & 3] = vec_sum<EPV>(e);
                    }, [&](int p, int32_t tile) __attribute__((always_inline)) { chunks_done(t, p, tile); });
                    __syncthreads();
                    if (tid == 0) sh.chunk[nfull] = tail != 0 ? tile_lane_sum<DT, true>(rest, k, -own, thr) : 0.f;
                    closed = in_chunks = true;
                }
            }
        }
        if (!closed) {
        // The nucleus alone, the quick way.  While the row lands its logits are only counted, per bin, in 32 bits:
        // 2^s for each, corrected by where in the bin its weight lies (the weight over the bin's own, to 2^-s), so
        // a bin's tally times the weight at its centre is its mass to a few parts in 10^5.  That names the bin in
        // which the nucleus closes, give or take a neighbour.  One pass then adds up the masses of all logits and
        // of those above a window of bins around it, as integers, and the latter's weights per chunk, and lists the
        // logits of the window; the list is closed by the same integers, and what it keeps is added to its chunks.  If the
        // list overflows (heavy ties, flat rows), a wave closes the window from the row.  If the window was off (neighbouring
        // bins with more than kBeside logits stay out of it), or for a block, the general selection follows.
        // (Adding the masses themselves takes 64-bit LDS atomics, 45 cycles a wave, or float ones, 300.)
        const int s_bits = 31 - (32 - __builtin_clz((uint32_t)V));
        const float s_one = (float)(1u << s_bits);
        lds_u32 *const tally = (lds_u32 *)sh.tally;
        auto fill = [&](auto pass) __attribute__((always_inline)) {
            __syncthreads();
            for (int b = tid; b < Sh::kBins; b += NT) sh.tally[b] = 0u;
            if (tid == 0) {
                sh.n = 0;
                sh.pick = -1;
            }
            __syncthreads();
            // in bins: the bin's number, from kBin0 down, and what is left of the exponent inside the bin (-1/2 .. 1/2) as the
            // weight's part above 2^s
            const float slope = s_one * (0.6931471805599453f / kScale), half = s_one + 0.5f;
            const float kb = -kScale * k, bin0 = kBin0 + kScale * ref, ks = slope * kScale * k, zero = half - slope * kScale * ref;
            const float beyond = kTwo23 + (float)(Sh::kBins + lane);
            float m = -__builtin_inff();
            auto one = [&](const u32x4 &v) __attribute__((always_inline)) {
                float x[EPV];
                values(v, x);
                m = max3(m, vec_max<EPV>(x), m);
#pragma unroll
                for (int i = 0; i < EPV; ++i) {
                    const float t = __builtin_amdgcn_fmed3f(fmaf(x[i], kb, bin0), kBinLo, beyond);
                    uint32_t inc;                            // (none where it is negative: what is not counted)
                    asm("v_cvt_u32_f32 %0, %1" : "=v"(inc) : "v"(fmaf(t - kBin0, slope, fmaf(x[i], ks, zero))));
                    const uint32_t b = __builtin_bit_cast(uint32_t, t) - 0x4B000000u;
                    __hip_atomic_fetch_add(tally + b, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            };
            pass(one);
            if (tail != 0 && wave == 0) one(rest);
            mx = wide_max<NT>(m, sh.wave_f);
        };
        fill([&](auto one) __attribute__((always_inline)) {
            sweep(Yes{}, [&](const u32x4 &v, int, int32_t) __attribute__((always_inline)) { one(v); }, nothing_more);
        });
        const float exact = fmaxf(ceilf(mx * k), kRefFloor);
        if (!(exact - ref <= (float)Sh::kTopOctaves)) {
            // a logit far above the first pieces' largest: once more, from memory, against the row's own reference
            ref = exact;
            fill([&](auto one) __attribute__((always_inline)) {
                for (int32_t i = tid; i < nwhole; i += NT) one(piece_at(i));
            });
        }
        // The tallies are against the first pieces' reference; from here on it is the row's own, as the masses need it.
        const float lower = exact - ref;
        ref = exact;
        const float nr = -ref;
        {
            // running mass and running count over the bins
            constexpr int kPer = Sh::kBins / NT;
            const float down = 1.f / s_one;
            double m[kPer], local = 0.0;
            uint32_t cnt = 0;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int b = tid * kPer + i;
                const uint32_t h = sh.tally[b];
                m[i] = (double)((float)h * down * fast_exp2((float)(Sh::kTopOctaves * Sh::kPerOctave - b) / kScale));
                cnt += (h + (1u << s_bits) / 2u) >> s_bits;
                local += m[i];
            }
            const double incl = wave_scan_add(local);
            const float cincl = wave_scan_add((float)cnt);
            if (lane == 63) {
                sh.wave_d[wave] = incl;
                sh.wave_e[wave] = (double)cincl;
            }
            for (int c = tid; c < Sh::kExtra; c += NT) sh.extra[c] = 0ull;
            __syncthreads();
            double lo, clo;
            const double need = (double)top_p * wide_total<NT>(sh.wave_d, lo);
            wide_total<NT>(sh.wave_e, clo);
            lo += incl - local;
            clo += (double)(cincl - (float)cnt);
            if (!(lo >= need) && lo + local >= need) {
                double acc = lo;
                int32_t found = -1;
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    acc += m[i];
                    if (found < 0 && acc >= need) found = tid * kPer + i;
                }
                sh.pick = found >= 0 ? found : tid * kPer + kPer - 1;
                sh.sel = clo <= (double)Sh::kBeside ? 1u : 0u;              // few logits above: all of them go on the list
            }
            __syncthreads();
        }
        const int32_t pick = sh.pick;
        if (pick >= 0 && nfull < Sh::kExtra) {
            // the window: bins on either side of the picked one until they hold kBeside logits
            int32_t wlo, whi;
            {
                const int32_t b = pick - 32 + lane;
                const bool in = b >= 0 && b < Sh::kBins && lane != 32;
                const float c = in ? (float)((sh.tally[b >= 0 && b < Sh::kBins ? b : 0] + (1u << s_bits) / 2u) >> s_bits) : 0.f;
                const float incl = wave_scan_add(c);
                const float upto = as::read_lane(incl, 32);
                const u64 near_lo = __ballot(lane < 32 && upto - incl + c <= Sh::kBeside);
                const u64 far_hi = __ballot(lane > 32 && incl - upto > Sh::kBeside);
                wlo = pick - 32 + (near_lo ? (int32_t)__builtin_ctzll(near_lo) : 32);
                whi = pick - 32 + (far_hi ? (int32_t)__builtin_ctzll(far_hi) - 1 : 63);
                wlo = sh.sel != 0u || wlo < 0 ? 0 : wlo;
                whi = whi > Sh::kBins - 1 ? Sh::kBins - 1 : whi;
            }
            // (as exponent arguments; the bins' own rounding need not be met, every logit only has to fall on one side)
            const float yhi = wlo == 0 ? __builtin_inff()
                                       : ((float)(Sh::kTopOctaves * Sh::kPerOctave - wlo) + 0.5f) / kScale - lower;
            const float ylo = ((float)(Sh::kTopOctaves * Sh::kPerOctave - whi) - 0.5f) / kScale - lower;
            u64 all = 0, over = 0;                           // masses of the lane's logits; of those above the window
            // A logit of the window joins the list: from the pieces that a wave has kept, a lane each, at the pass's end, or, where
            // they are more than its table takes, one by one, each waiting for its place.  (us, one by one throughout / so: 512
            // rows of 50257 fp32 40.3 / 39.7, 3000 of 8001 43.2 / 41.0, 8000 of 1501 32.4 / 30.1; flat bf16 rows, which are not counted
            // by value, 2000 of 50257 149 / 138, 8000 of 8001 of a standard deviation of 1 104 / 98, of 0.3, whose lists none of this
            // makes fit, 118 / 122.  A row that has a unit to itself is better off one by one, with
            // a barrier and a pass over a table less: fp32, 1 of 5003 11.6 / 12.0, 250 12.6 / 12.9, 1 of 20011 14.7 / 15.0.)
            constexpr bool ONE_BY_ONE = NT == 1024 && !MULTI;
            if constexpr (!ONE_BY_ONE) __syncthreads();      // (the tallies give way to tables of pieces)
            int32_t held = 0;
            auto list = [&](float x, uint32_t q, uint32_t j, int32_t c) __attribute__((always_inline)) {
                if (j < (uint32_t)Sh::kList) {
                    sh.key[j] = order_key(x);
                    sh.q[j] = q;
                    sh.at[j] = (uint16_t)c;
                }
            };
            auto in_window = [&](float y) __attribute__((always_inline)) { return y >= ylo && y <= yhi; };
            // the lane's weight above the window
            auto part = [&](const u32x4 &v, int32_t c) __attribute__((always_inline)) {
                float x[EPV], sum[EPV / 4];
                bool any = false;
                values(v, x);
#pragma unroll
                for (int h = 0; h < EPV / 4; ++h) {          // (four at a time: eight do not fit the registers)
                    float y[4], e[4];
                    uint32_t q[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        y[i] = fmaf(x[4 * h + i], k, nr);
                        e[i] = fast_exp2(y[i]);
                        q[i] = mass_of(e[i]);
                        all += q[i];
                        any |= in_window(y[i]);
                    }
                    if constexpr (ONE_BY_ONE) {
                        if (any) {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (in_window(y[i])) list(x[4 * h + i], q[i], atomicAdd(&sh.n, 1u), c);
                        }
                        any = false;
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        e[i] = y[i] > yhi ? e[i] : 0.f;
                        over += y[i] > yhi ? q[i] : 0u;
                    }
                    sum[h] = (e[0] + e[1]) + (e[2] + e[3]);
                    asm volatile("" : "+v"(all), "+v"(over));    // (added up here, not as a tree over the row later)
                    __builtin_amdgcn_sched_barrier(0);
                }
                const u64 in = ONE_BY_ONE ? 0ull : __ballot(any);
                if (in != 0ull) {
                    const int32_t n = __builtin_popcountll(in);
                    if (held + n <= 64) {
                        if (any) {
                            const int32_t at = held + (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
                            sh.hot.piece[wave][at] = v;
                            sh.hot.first[wave][at] = c;
                        }
                        held += n;
                    } else if (any) {
#pragma unroll 1
                        for (int i = 0; i < EPV; ++i) {
                            const float xi = DT == AS_BF16 ? bits_f32(i & 1 ? v[i >> 1] & 0xffff0000u : v[i >> 1] << 16) : bits_f32(v[i]);
                            const float y = fmaf(xi, k, nr);
                            if (in_window(y)) list(xi, mass_of(fast_exp2(y)), atomicAdd(&sh.n, 1u), c);
                        }
                    }
                }
                if constexpr (EPV == 8) return sum[0] + sum[1];
                else return sum[0];
            };
            float t[4] = {0.f, 0.f, 0.f, 0.f};
            sweep(No{}, [&](const u32x4 &v, int p, int32_t tile) __attribute__((always_inline)) {
                t[p & 3] = part(v, (tile * NP + p) * W + wave);
            }, [&](int p, int32_t tile) __attribute__((always_inline)) { chunks_done(t, p, tile); });
            float tl = 0.f;
            if (tail != 0 && wave == 0) tl = part(rest, nfull);
            if (held != 0) {
                wave_lds();
                float x[EPV];
                values(lane < held ? sh.hot.piece[wave][lane] : nothing, x);
                const int32_t c = sh.hot.first[wave][lane];
                uint32_t mine = 0, at = 0;
#pragma unroll
                for (int i = 0; i < EPV; ++i) mine += (uint32_t)__builtin_popcountll(__ballot(in_window(fmaf(x[i], k, nr)) && lane < held));
                if (lane == 0) at = atomicAdd(&sh.n, mine);
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
                for (int i = 0; i < EPV; ++i) {
                    const float y = fmaf(x[i], k, nr);
                    const u64 in = __ballot(in_window(y) && lane < held);
                    const uint32_t j = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
                    if (in_window(y) && lane < held) list(x[i], mass_of(fast_exp2(y)), j, c);
                    at += (uint32_t)__builtin_popcountll(in);
                }
            }
            // (integers below 2^53: exact as doubles, in any order)
            const double all_wave = wave_sum((double)all), over_wave = wave_sum((double)over);
            if (lane == 63) {
                sh.wave_d[wave] = all_wave;
                sh.wave_e[wave] = over_wave;
            }
            __syncthreads();
            if (tid == 0) sh.chunk[nfull] = tl;              // (in the place of a chunk past the row's end)
            double unused;
            const double need = (double)top_p * wide_total<NT>(sh.wave_d, unused);
            const double above = wide_total<NT>(sh.wave_e, unused);
            const uint32_t n = sh.n;
            if ((Sh::kWave || n <= (uint32_t)Sh::kList) && above < need) {
                // (more than the list takes: the window's logits by their keys, and the chunk sums over again)
                const uint32_t key = close(n, (u64)above, need, [&](auto put) __attribute__((always_inline)) {
                    if constexpr (!Sh::kWave) return;
                    else every_piece_again([&](const u32x4 &v) __attribute__((always_inline)) {
                        float x[EPV];
                        values(v, x);
#pragma unroll
                        for (int e = 0; e < EPV; ++e) {
                            const float y = fmaf(x[e], k, nr);
                            if (y >= ylo && y <= yhi) put(order_key(x[e]), (u64)mass_of(fast_exp2(y)));
                        }
                    });
                });
                if (key != 0u) {
                    thr = from_order_key(key);
                    closed = true;
                    summed = n <= (uint32_t)Sh::kList;
                    if (summed)
                        for (uint32_t i = tid; i < n; i += NT)
                            if (sh.key[i] >= key)
                                add((lds_u64 *)sh.extra + sh.at[i],
                                    fixed_weight(fast_exp2(fmaf(from_order_key(sh.key[i]), k, nr))));
                }
            }
        }
        if (!closed) some = select(No{}, -__builtin_inff(), thr);
        }
    }
    if (a.tokens_out == nullptr) {
        if (tid == 0) thr_out[r] = some ? thr : -__builtin_inff();
        return;
    }
    if (!some) {
        safe_row();
        return;
    }

    // ------------------------------------------------------------------ the step over the kept logits
    const float nr = -ref;
    auto lane_sum = [&](const u32x4 &v) __attribute__((always_inline)) { return tile_lane_sum<DT, true>(v, k, nr, thr); };
    const int32_t nchunks = nfull + 1;                       // the last one: the piece that the row ends in
    if (!summed && !in_chunks) {
        __syncthreads();
        if constexpr (TOPK) {
            float t[4] = {0.f, 0.f, 0.f, 0.f};
            sweep(No{}, [&](const u32x4 &v, int p, int32_t) __attribute__((always_inline)) { t[p & 3] = lane_sum(v); },
                  [&](int p, int32_t tile) __attribute__((always_inline)) { chunks_done(t, p, tile); });
        } else {
            for (int32_t c = wave; c < nchunks - 1; c += W) {
                const int32_t i = c * 64 + lane;
                const float t = wave_sum(lane_sum(piece_at(i < nwhole ? i : nwhole + 1)));
                if (lane == 0) sh.chunk[c] = t;
            }
        }
        __syncthreads();
        if (tid == 0) sh.chunk[nchunks - 1] = tail != 0 ? lane_sum(rest) : 0.f;
    }
    __syncthreads();
    auto chunk_weight = [&](int32_t c) __attribute__((always_inline)) {
        return (double)sh.chunk[c] + (summed ? (double)sh.extra[c] * 0x1p-40 : 0.0);
    };
    const int32_t per = (nchunks + NT - 1) / NT;
    double mine = 0.0;
    for (int32_t i = 0; i < per; ++i) {
        const int32_t c = tid * per + i;
        if (c < nchunks) mine += chunk_weight(c);
    }
    const double incl_w = wave_scan_add(mine);
    if (lane == 63) sh.wave_d[wave] = incl_w;
    __syncthreads();
    double base;
    const double S = wide_total<NT>(sh.wave_d, base);
    const double tau = (double)a.codes[r] * S;
    // the first thread whose running sum passes c*S; past the end by rounding: the last that holds weight
    const u64 hit = __ballot(base + incl_w > tau), full = __ballot(mine > 0.0);
    if (lane == 0) {
        sh.wave_lo[wave] = hit ? (uint32_t)__builtin_ctzll(hit) : 64u;
        sh.wave_hi[wave] = full ? 63u - (uint32_t)__builtin_clzll(full) : 64u;
    }
    __syncthreads();
    int32_t owner = 0;
    {
        const uint32_t lo = lane < W ? sh.wave_lo[lane] : 64u, hi = lane < W ? sh.wave_hi[lane] : 64u;
        const u64 any = __ballot(lo < 64u), some = __ballot(hi < 64u);
        if (any) {
            const int w = (int)__builtin_ctzll(any);
            owner = w * 64 + __builtin_amdgcn_readlane((int)lo, w);
        } else if (some) {
            const int w = 63 - (int)__builtin_clzll(some);
            owner = w * 64 + __builtin_amdgcn_readlane((int)hi, w);
        }
    }
    if (tid == owner) {
        double acc = base + incl_w - mine, at = acc;
        int32_t found = -1, lastc = tid * per;
        for (int32_t i = 0; i < per; ++i) {
            const int32_t c = tid * per + i;
            if (c >= nchunks) break;
            const double v = chunk_weight(c);
            if (v > 0.0) {
                if (found < 0) { lastc = c; at = acc; }
                if (found < 0 && acc + v > tau) found = c;
            }
            acc += v;
        }
        sh.pick = found >= 0 ? found : lastc;
        sh.run = at;
    }
    __syncthreads();
    if (wave != 0) return;
    const int32_t ch = sh.pick < nchunks ? sh.pick : nchunks - 1;
    const double run = sh.run;
    // the chunk's pieces once more; lane, then logit
    const int32_t pi = ch < nchunks - 1 ? ch * 64 + lane : (lane == 0 ? nwhole : nwhole + 1);
    const u32x4 hv = piece_at(ch < nchunks - 1 && pi >= nwhole ? nwhole + 1 : pi);
    const double lv = (double)lane_sum(hv);
    const double incl = wave_scan_add(lv) + run;
    const u64 hit2 = __ballot(incl > tau), nz2 = __ballot(lv > 0.0);
    const int l2 = hit2 ? (int)__builtin_ctzll(hit2) : (nz2 ? 63 - (int)__builtin_clzll(nz2) : 0);
    if (lane != l2) return;
    float x[EPV];
    values(hv, x);
    double acc = incl - lv, before = acc, ev = 0.0, before_last = acc, ev_last = 0.0;
    int ih = -1, ilast = 0;
#pragma unroll
    for (int i = 0; i < EPV; ++i) {
        const double e = x[i] >= thr ? (double)fast_exp2(fmaf(x[i], k, nr)) : 0.0;
        if (e > 0.0) { ilast = i; before_last = acc; ev_last = e; }
        if (ih < 0 && acc + e > tau) { ih = i; before = acc; ev = e; }
        acc += e;
    }
    if (ih < 0) { ih = ilast; before = before_last; ev = ev_last; }
    int64_t token = (int64_t)pi * EPV + ih - shift;
    token = token < 0 ? 0 : (token > V - 1 ? V - 1 : token);
    RowOut o;
    o.token = (int32_t)token;
    o.c_next = rescale_code(tau, before, ev);
    o.prob = (float)(ev / S);
    o.f_lo = (float)(before / S);
    write_row(a, r, o);
}

template <int DT, int NT, int NP, bool MULTI, bool TOPK, int WAVES = 4>
void launch_form(as_ctx *ctx, int kid, const StepArgs &a, int32_t top_k, float top_p, float *thr_out)
{
    launch(ctx, kid, wide_step_kernel<DT, NT, NP, MULTI, TOPK, WAVES>, dim3((unsigned)a.rows), dim3(NT), 0, a, top_k, top_p, thr_out);
}

// Threads and pieces a thread by the row's pieces of 16 bytes and the number of rows.  With a row per compute unit or
// fewer, 1024 threads finish it soonest (one row of 50257 bf16: nucleus 13 us, top-k 40 9 us).  With more, smaller
// blocks that share a unit overlap each other's loads and tails: two blocks of 512 where two fit (nucleus, bf16: 300 rows
// of 33001 19 us, as blocks of 1024 24; 6439 of them 178, 284; 1000 of 65001 50, 66; fp32 2500 of 33001, which go
// tile by tile, 128, 204), and with many rows that 256 threads hold, those (nucleus, bf16, 6439 rows: of 9001 59
// us with 256 x 8, 95 with 512 x 4; of 20001 99 with 256 x 16, 130 with 512 x 8; top-k 40, 2500 of 20003 33, with 512
// threads 44).  With more than four short rows a unit the blocks are made to fit eight a unit (SHORT; six for k above 128 and
// for nuclei of two registers' pieces more): 12000 rows of 1281 to 8000 bf16, or half as many fp32, nuclei 1.17 to 1.22 times faster,
// top-k 1.38, k = 200 1.09; 600 of them no different.  With more rows still, a wave a row: nothing in it waits for
// another wave, and what a block does in some 25 steps of its waves overlaps over rows instead (us, blocks / waves: nuclei, 600
// rows of 1500 bf16 9.5 / 9.4, 1500 15.4 / 11.4, 14251 of 1923 86 / 46, 5252 of 3078 38 / 27, 1500 of 4001 17.1 / 15.4, 2600 of 8001 27.9 /
// 27.0, 4200 38.5 / 36.1; fp32 6000 of 4000 54 / 39, 1100 of 4001 18.7 / 20.2; k = 40 1500 of 3000 bf16 11.4 / 12.2, 2100 of 4001 15.5 / 14.9,
// 4200 of 8001 25.5 / 27.6, 9000 of 6001 44 / 39; k = 50, p = 0.73 4816 of 3315 28 / 38; counts, k = 1000, 4000 of 1500 31 / 18, 2100 of
// 4001 23.7 / 22.8, 9000 of 6001 83 / 72, 6000 of 4000 fp32 k = 200 40 / 35, but on flat or steep ones 38 / 45 and more).  Those rows
// have a standard deviation of 3 against the temperature; a wave has a shorter list, so flat rows decide whether its line holds:
// of 0.3 at a temperature of 0.9, nuclei p = 0.9 4000 of 1500 44 / 24, 6000 of 3000 72 / 44, 3000 of 4000 46 / 34, 8000 of 8000
// 134 / 122; k = 100 then p = 0.9 6000 of 1000 75 / 37, 6000 of 3000 62 / 62, which is behind only where the row is all but
// constant (0.05: 62 / 121).
template <int DT, bool TOPK>
void launch_type(as_ctx *ctx, int kid, const StepArgs &a, int32_t top_k, float top_p, float *thr_out)
{
    constexpr int EPV = Elem<DT>::kPerVec;
    const int64_t most = ((int64_t)a.V + EPV - 1) / EPV;     // whole pieces of a row, whatever its alignment
    const bool many = a.rows > (int64_t)ctx->num_cus, lots = a.rows > 2 * (int64_t)ctx->num_cus;
    const bool has_p = top_p > 0.f && top_p < 1.f;
    // (compute units' worth of rows beyond which a wave takes a row; counts on rows of more than 768 pieces or with a nucleus behind
    // them on more than 512, and a nucleus after the 64 best of a row of more than 256, never)
    const bool counts = TOPK && top_k > kWaveTopK;
    const bool table = counts && has_p && top_k <= 64 && most > 64 * 4;
    const int64_t never = 1LL << 40;
    const int64_t by_waves = DT == AS_BF16 && a.tokens_out ? 12 : 16;
    const int64_t waves = most <= 64 * 8 ? (table ? never : !TOPK ? 4 : counts ? 12 : 6) : !TOPK ? by_waves : !counts || (!has_p && most <= 64 * 12) ? 20 : never;
    if (most <= 64 * 16 && a.rows > waves * (int64_t)ctx->num_cus) {
        if (most <= 64 * 8) return launch_form<DT, 64, 8, false, TOPK, 5>(ctx, kid, a, top_k, top_p, thr_out);
        return launch_form<DT, 64, 16, false, TOPK, 4>(ctx, kid, a, top_k, top_p, thr_out);
    }
    if (most <= 256 * 4) {
        if (a.rows <= 4 * (int64_t)ctx->num_cus) return launch_form<DT, 256, 4, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
        if constexpr (TOPK) {
            if (top_k > table_most<256, 4>(a.V / EPV, has_p))
                return launch_form<DT, 256, 4, false, TOPK, 6>(ctx, kid, a, top_k, top_p, thr_out);
        }
        return launch_form<DT, 256, 4, false, TOPK, 8>(ctx, kid, a, top_k, top_p, thr_out);
    }
    if constexpr (!TOPK) {
        if (a.rows > 4 * (int64_t)ctx->num_cus && most <= 256 * 8)
            return launch_form<DT, 256, 8, false, TOPK, 6>(ctx, kid, a, top_k, top_p, thr_out);
        if (lots && most <= 256 * 8) return launch_form<DT, 256, 8, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    }
    if (lots && most <= 256 * 16 && (!TOPK || top_k <= kWideTopK))
        return launch_form<DT, 256, 16, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    if (many && most <= 512 * 4) return launch_form<DT, 512, 4, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    if (many && most <= 512 * 8) return launch_form<DT, 512, 8, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    if (many && most <= 512 * 16) return launch_form<DT, 512, 16, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    if constexpr (!TOPK) {
        // (with a tile of slack: the last one's chunks are written whole)
        if (many && most + 512 * 8 <= 64 * (int64_t)(WideShared<512, true, false>::kChunks - 1))
            return launch_form<DT, 512, 8, true, false>(ctx, kid, a, top_k, top_p, thr_out);
    }
    if (most <= 1024 * 4) return launch_form<DT, 1024, 4, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    if (most <= 1024 * 8) return launch_form<DT, 1024, 8, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    if constexpr (TOPK || DT == AS_F32) {
        if (most <= 1024 * 16) return launch_form<DT, 1024, 16, false, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
    }
    launch_form<DT, 1024, 8, true, TOPK>(ctx, kid, a, top_k, top_p, thr_out);
}

}  // namespace

// Truncation (top_k on: > 0, else 0; top_p on: in (0, 1), else 1) and the sampling step in one launch; without
// a.tokens_out the keep thresholds alone, to thr_out.
as_status launch_wide(as_ctx *ctx, const StepArgs &a, int32_t top_k, float top_p, float *thr_out)
{
    if (a.rows == 0) return AS_OK;
    const int kid = a.tokens_out ? kKernelStep : kKernelThreshold;
    if (a.dtype == AS_BF16) {
        if (top_k > 0) launch_type<AS_BF16, true>(ctx, kid, a, top_k, top_p, thr_out);
        else launch_type<AS_BF16, false>(ctx, kid, a, top_k, top_p, thr_out);
    } else {
        if (top_k > 0) launch_type<AS_F32, true>(ctx, kid, a, top_k, top_p, thr_out);
        else launch_type<AS_F32, false>(ctx, kid, a, top_k, top_p, thr_out);
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
