// Encode direction: the interval of a given token sequence (Sec. 4.1, the
// codebook recursion; Sec. 3.1 for one token's sub-interval).  Per step and row,
// with the row's kept, tempered softmax in vocabulary order,
//     lo    += width * F(token - 1)      (mass of the tokens before it)
//     width *= P(token)
// so that after the last step the codes in [lo, lo + width) are exactly the ones
// that decode to the sequence.  The per-row pass is the one of the sampling step
// with the search replaced by a lookup: weights exp2(x*k - ref) in fp32 against an
// integer reference ref >= max x*k, sums in fp64.  lo and width are fp64 state.
//
// A whole encode (as_encode) knows every token it conditions on before it starts, so its positions do not wait for
// each other: the logits of all positions are computed a chunk of rows at a time, one row per token in use where
// positions share tokens, each position's (F, P) is taken from its row, and one short recursion per sequence folds
// them (positions_kernel, row_sums_kernel, row_lookup_kernel / interval_items_kernel, fold_kernel).
#include <type_traits>

#include "as_common.hpp"
#include "as_row.hpp"
#include "as_tile.hpp"

namespace as {
namespace {

constexpr int kThreads = 256;


// g(v0, x, first, n) over the row's logits in runs: elements first..n-1 of x are logits v0+first..v0+n-1 of the
// row, each logit of the row exactly once per thread block.  The row is read as the whole 16-byte pieces it
// touches, four in flight per thread; only the pieces at the row's two ends have first > 0 or n < 8 (4).
template <class T, class G>
__device__ __forceinline__ void for_row(const T *row, int32_t V, G g)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int EPP = 16 / (int)sizeof(T);
    const int32_t shift = (int32_t)((reinterpret_cast<uintptr_t>(row) & 15u) / sizeof(T));
    const u32x4 *const pieces = reinterpret_cast<const u32x4 *>(row - shift);
    const int32_t vend = V + shift;
    const int32_t npieces = (vend + EPP - 1) / EPP;
    for (int32_t base = threadIdx.x; base < npieces; base += 4 * kThreads) {
        u32x4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t piece = base + u * kThreads;
            w[u] = piece < npieces ? __builtin_nontemporal_load(pieces + piece) : u32x4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int32_t piece = base + u * kThreads;
            if (piece >= npieces) break;
            float x[EPP];
#pragma unroll
            for (int e = 0; e < EPP; ++e) {
                if constexpr (sizeof(T) == 2) {
                    const uint32_t word = w[u][e >> 1];
                    x[e] = __builtin_bit_cast(float, (e & 1) ? (word & 0xffff0000u) : (word << 16));
                } else {
                    const uint32_t word = w[u][e];
                    x[e] = __builtin_bit_cast(float, word);
                }
            }
            const int32_t left = vend - piece * EPP;
            g(piece * EPP - shift, x, piece == 0 ? shift : 0, left < EPP ? left : EPP,
              std::integral_constant<int, EPP>{});
        }
    }
}

// three block-wide sums at once, each in a fixed order: lanes by the wave scan, then the waves in index order
__device__ __forceinline__ void block_sum3(double &a, double &b, double &c, double *scratch)
{
    a = wave_sum(a);
    b = wave_sum(b);
    c = wave_sum(c);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        scratch[wave] = a;
        scratch[kThreads / 64 + wave] = b;
        scratch[2 * (kThreads / 64) + wave] = c;
    }
    __syncthreads();
    a = b = c = 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) {
        a += scratch[w];
        b += scratch[kThreads / 64 + w];
        c += scratch[2 * (kThreads / 64) + w];
    }
}

// the mass before the token and its own, as shares of the row's total; a token outside the vocabulary or outside the
// kept set has probability zero
__device__ __forceinline__ void shares_of(double all, double before, double at, bool in_vocab, double &f_lo, double &p)
{
    f_lo = all > 0.0 ? before / all : 0.0;
    p = (all > 0.0 && in_vocab) ? at / all : 0.0;
}

// what they do to the interval
__device__ __forceinline__ void narrow(double &lo, double &w, double f_lo, double p)
{
    lo += w * f_lo;
    w = w * p;
}

// what a row's sums do to its interval (one thread)
__device__ __forceinline__ void narrow_interval(const IntervalArgs &a, int64_t r, int32_t tok, double all, double before,
                                                double at)
{
    double f_lo, p, lo = a.lo[r], w = a.width[r];
    shares_of(all, before, at, tok >= 0 && tok < a.V, f_lo, p);
    narrow(lo, w, f_lo, p);
    a.lo[r] = lo;
    a.width[r] = w;
    if (a.finished_out) a.finished_out[r] = (a.eos_id >= 0 && tok == a.eos_id) ? 1 : 0;
}

// One row by a block of 256 threads, any alignment, any V, one pass over memory: every thread keeps an integer
// reference that follows the largest logit it has seen (see below).  Every thread of the block must call it.
template <class T, class Done>
__device__ __forceinline__ void interval_row(const T *row, int32_t V, float k, const float *thr_at, int32_t tok,
                                             double *scratch, float *fscratch, Done done)
{
    const float thr = thr_at ? *thr_at : -__builtin_inff();

    auto each_run = [&](auto g) __attribute__((always_inline)) { for_row<T>(row, V, g); };

    // a run as the sums see it: what is cut off by the threshold or lies outside the row counts as -inf
    // (weight exactly 0); whole runs of an untruncated row, nearly all of them, pass through untouched
    const bool cut = thr_at != nullptr;
    auto kept = [&](const float *x, int first, int n, auto cap, float *y) __attribute__((always_inline)) {
        constexpr int E = decltype(cap)::value;
        if (!cut && first == 0 && n == E) {
#pragma unroll
            for (int e = 0; e < E; ++e) y[e] = x[e];
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) y[e] = (e >= first && e < n && x[e] >= thr) ? x[e] : -__builtin_inff();
        }
    };

    // per run: fp32 sum of its (at most 8) weights in order, then one fp64 add per total; only the one run
    // that holds the token looks at single weights
    double all = 0.0, before = 0.0, at = 0.0;
    auto add_run = [&](int32_t v0, const float *y, float nref, auto cap) __attribute__((always_inline)) {
        constexpr int E = decltype(cap)::value;
        float w[E];
        float s_all = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            w[e] = __builtin_amdgcn_exp2f(fmaf(y[e], k, nref));
            s_all += w[e];
        }
        const double d = (double)s_all;
        all += d;
        if (v0 + E <= tok) {
            before += d;
        } else if (v0 <= tok) {
            float s_before = 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                s_before += v0 + e < tok ? w[e] : 0.f;
                if (v0 + e == tok) at = (double)w[e];
            }
            before += (double)s_before;
        }
    };
    {
        // One pass over memory: every thread keeps an integer reference that follows the largest logit it has
        // seen; when it rises, what the thread has summed so far shrinks by an exact power of two.  At the end
        // the threads are brought to the block's reference the same way.
        float ref = -100000.f;
        auto rescale = [&](float to) __attribute__((always_inline)) {
            const int down = (int)fmaxf(ref - to, -2000.f);
            all = ldexp(all, down);
            before = ldexp(before, down);
            at = ldexp(at, down);
            ref = to;
        };
        each_run([&](int32_t v0, const float *x, int first, int n, auto cap) __attribute__((always_inline)) {
            constexpr int E = decltype(cap)::value;
            float y[E];
            kept(x, first, n, cap, y);
            float pm = y[0];
#pragma unroll
            for (int e = 1; e < E; ++e) pm = fmaxf(pm, y[e]);
            const float want = fmaxf(ceilf(pm * k), ref);
            if (want > ref) rescale(want);
            add_run(v0, y, -ref, cap);
        });
        float top = wave_max(ref);
        if ((threadIdx.x & 63) == 0) fscratch[threadIdx.x >> 6] = top;
        __syncthreads();
        top = fscratch[0];
#pragma unroll
        for (int w = 1; w < kThreads / 64; ++w) top = fmaxf(top, fscratch[w]);
        rescale(top);
    }
    block_sum3(all, before, at, scratch);
    if (threadIdx.x == 0) done(all, before, at);
}

// ... as as_interval_step has it: row r of the call narrows interval r
template <class T>
__device__ __forceinline__ void interval_row(const IntervalArgs &a, int64_t r, int32_t tok, double *scratch,
                                             float *fscratch)
{
    const int64_t src = a.row_ids ? (int64_t)a.row_ids[r] : r;
    interval_row<T>(reinterpret_cast<const T *>(a.logits) + src * a.ld, a.V, a.k, a.thr ? a.thr + r : nullptr, tok, scratch,
                    fscratch, [&](double all, double before, double at) { narrow_interval(a, r, tok, all, before, at); });
}

template <class T>
__global__ __launch_bounds__(kThreads) void interval_kernel(IntervalArgs a)
{
    __shared__ double scratch[3 * (kThreads / 64)];
    __shared__ float fscratch[kThreads / 64];
    const int64_t r = blockIdx.x;
    const int32_t tok = a.tokens[r * a.tok_stride];
    if (a.finished_in != nullptr && a.finished_in[r] != 0) {
        // past its EOS: the position is padding and does not narrow the interval
        if (threadIdx.x == 0) {
            if (a.finished_out) a.finished_out[r] = 1;
        }
        return;
    }
    interval_row<T>(a, r, tok, scratch, fscratch);
}

// The wave that holds the token's chunk: hv its lanes' vectors of the chunk, cl their sums (0 past the row's end), both
// relative to rw; S the row's total, chunk and run the chunk's share of it and what lies before the chunk.  Lane ln
// calls done(total, mass before the token, its own).
template <int DT, bool HAS_THR, class Done>
__device__ __forceinline__ void token_shares(const u32x4 &hv, float cl, float k, float rw, float thr, int shf, double S,
                                             double chunk, double run, int ln, int el, int lane, Done done)
{
    constexpr int EPV = Elem<DT>::kPerVec;
    const double lv = (double)ldexpf(cl, shf);
    const double scan2 = wave_scan_add(lv);
    const double before_lane = read_lane(scan2 - lv, ln) + run;
    // The total with this chunk and this lane taken the way `before` takes them (fp64 sums of the lane sums
    // and of the weights, where S has an fp32 wave sum and an fp32 lane sum): the mass before the token plus
    // its own can then not exceed the total by rounding, and nested intervals stay nested.
    const double S_rest = (S - chunk) + (read_lane(scan2, 63) - lv);
    if (lane != ln) return;
    float x[EPV];
    unpack<DT>(hv, x);
    double before = before_lane, at = 0.0, mine = 0.0;
#pragma unroll
    for (int i = 0; i < EPV; ++i) {
        float e = fast_exp2(fmaf(x[i], k, -rw));
        if constexpr (HAS_THR) e = (x[i] >= thr) ? e : 0.f;
        const double ed = (double)ldexpf(e, shf);
        mine += ed;
        before += i < el ? ed : 0.0;
        at = i == el ? ed : at;
    }
    done(S_rest + mine, before, at);
}

// Rows of whole, aligned vectors that fit one tile (the headline shape): the single-tile sampling kernel with
// the search replaced by a look-up.  Same loads, same chunk sums against one integer reference per wave, one
// barrier; then every wave scans the 64 chunk sums (fp64) for the total and the mass before the token's chunk,
// and the wave that holds the token's chunk adds the lanes before it and the elements before it.  Sums that
// leave fp32 against a first-chunk reference send the block to the one-pass routine above.
template <int DT, bool HAS_THR, bool NT>
__global__ __launch_bounds__(kThreads, 4) void interval_tile_kernel(IntervalArgs a)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int NW = kTileWaves, ITERS = kTileIters, G = kTileGroup, NG = ITERS / G;
    constexpr int kShare = ITERS * 64;
    __shared__ TileSums ts;
    __shared__ double scratch[3 * (kThreads / 64)];
    __shared__ float fscratch[kThreads / 64];

    const int64_t r = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t fin_word = 0u, fin_at = 0u;
    if (a.finished_in != nullptr) {
        const uint8_t *q = a.finished_in + r;
        fin_at = (uint32_t)(reinterpret_cast<uintptr_t>(q) & 3u);
        fin_word = *reinterpret_cast<const uint32_t *>(q - fin_at);
    }
    const int32_t tok = a.tokens[r * a.tok_stride];
    float thr = -__builtin_inff();
    if constexpr (HAS_THR) thr = a.thr[r];
    const int64_t src = a.row_ids ? (int64_t)a.row_ids[r] : r;
    const unsigned char *rowb =
        reinterpret_cast<const unsigned char *>(reinterpret_cast<const T *>(a.logits) + src * a.ld);
    const int32_t nvec = a.V / EPV;
    const float k = a.k;
    const int32_t v0 = wave * kShare;
    u32x4 raw[ITERS];
    float rw = kRefFloor;
    int32_t mych = (nvec - v0 - lane + 63) >> 6;
    mych = mych < 0 ? 0 : (mych > ITERS ? ITERS : mych);
    const bool live = v0 < nvec;
    const bool ragged = v0 + kShare > nvec;
    const unsigned char *base = rowb + (size_t)(live ? v0 : 0) * 16u;
    const uint32_t off0 = (uint32_t)lane * 16u;
    const uint32_t off_last = mych > 0 ? off0 + (uint32_t)(mych - 1) * 1024u : 0u;
    auto request_group = [&](int g) __attribute__((always_inline)) {
        // (ordinary loads where the tensor fits the caches, the non-temporal hint where it is streamed from HBM;
        // each load behind the two vector instructions of its own offset either way)
        if constexpr (NT) {
#pragma unroll
            for (int jj = 0; jj < G; ++jj) {
                uint32_t off = off0 + (uint32_t)(g * G + jj) * 1024u;
                off = off < off_last ? off : off_last;
                raw[g * G + jj] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(base + off));
            }
        } else {
#pragma unroll
            for (int jj = 0; jj < G; ++jj) {
                uint32_t off = off0 + (uint32_t)(g * G + jj) * 1024u;
                off = off < off_last ? off : off_last;
                raw[g * G + jj] = *reinterpret_cast<const u32x4 *>(base + off);
            }
        }
    };
    if (live) request_group(0);
    __builtin_amdgcn_sched_barrier(0);
    if (((fin_word >> (8u * fin_at)) & 0xffu) != 0u) {
        // past its EOS: the position is padding and does not narrow the interval
        if (threadIdx.x == 0) {
            if (a.finished_out) a.finished_out[r] = 1;
        }
        return;
    }
    f32x4 *const my_sums = reinterpret_cast<f32x4 *>(ts.chunk_sum + wave * ITERS);
    auto stream = [&](auto ragged_c) __attribute__((always_inline)) {
        constexpr bool RAGGED = decltype(ragged_c)::value;
#pragma unroll
        for (int g = 1; g < NG; ++g) request_group(g);
        __builtin_amdgcn_sched_barrier(0);
        rw = tile_reference<DT, HAS_THR, RAGGED>(raw[0], k, thr, mych);
        tile_chunk_sums<DT, HAS_THR, RAGGED>(raw, k, rw, thr, mych, lane, my_sums);
    };
    if (live) {
        if (!ragged) stream(std::false_type{});
        else stream(std::true_type{});
    } else {
#pragma unroll
        for (int j = 0; j < ITERS; ++j) raw[j] = u32x4{0u, 0u, 0u, 0u};
        if (lane < NG) my_sums[lane] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (lane == 0) ts.share_ref[wave] = rw;
    __syncthreads();

    float R = ts.share_ref[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) R = fmaxf(R, ts.share_ref[w]);
    const float my_ref = ts.share_ref[lane / ITERS];
    const double cv = (double)ldexpf(ts.chunk_sum[lane], shift_of(my_ref, R));
    const double cincl = wave_scan_add(cv);
    const double S = read_lane(cincl, 63);
    if (!(S < (double)__builtin_inff())) {
        interval_row<T>(a, r, tok, scratch, fscratch);
        return;
    }
    if (tok < 0 || tok >= a.V) {
        // outside the vocabulary: probability zero, everything (or nothing) before it
        if (threadIdx.x == 0) narrow_interval(a, r, tok, S, tok < 0 ? 0.0 : S, 0.0);
        return;
    }
    const int32_t vi = tok / EPV, el = tok % EPV;
    const int ch = vi >> 6, ln = vi & 63;
    if (wave != ch / ITERS) return;
    const double run = read_lane(cincl - cv, ch);
    const int shf = shift_of(rw, R);
    const int cj = ch % ITERS;
    u32x4 hv;
    with_uniform_index<0, ITERS>(cj, [&](auto c_c) __attribute__((always_inline)) {
        uint32_t w0 = raw[decltype(c_c)::value][0], w1 = raw[decltype(c_c)::value][1],
                 w2 = raw[decltype(c_c)::value][2], w3 = raw[decltype(c_c)::value][3];
        asm volatile("" : "+v"(w0), "+v"(w1), "+v"(w2), "+v"(w3));
        hv = u32x4{w0, w1, w2, w3};
    });
    float cl = tile_lane_sum<DT, HAS_THR>(hv, k, -rw, thr);
    if (ragged) cl = cj < mych ? cl : 0.f;
    token_shares<DT, HAS_THR>(hv, cl, k, rw, thr, shf, S, read_lane(cv, ch), run, ln, el, lane,
                              [&](double all, double before, double at) { narrow_interval(a, r, tok, all, before, at); });
}

// ------------------------------------------------------------ whole encodes

// The positions of one window of an encode (columns t0 .. t0+Tw of the sequences): which token each conditions on, and
// whether it lies behind its sequence's EOS.  A wave per sequence.  CLAIMED: the tokens go to `cond` (-1 behind an
// EOS) for the kernels that give each token in use a logits row.  Otherwise the rows are numbered here: one per prompt
// for the first step, where the N sequences of a prompt condition on the same token, one per position after it.
template <bool CLAIMED>
__global__ __launch_bounds__(256) void positions_kernel(Positions w)
{
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= w.R) return;
    bool ended = w.t0 > 0 && w.ended[r] != 0;
    const int32_t *const seq = w.tokens + r * w.T + w.t0;
    const bool prompts = w.t0 == 0 && w.N > 1;               // the first column's rows are the prompts'
    const int64_t first = prompts ? w.R / w.N : 0, per = prompts ? w.Tw - 1 : w.Tw;
    for (int32_t i0 = 0; i0 < w.Tw; i0 += 64) {
        const int32_t i = i0 + lane;
        const bool in = i < w.Tw;
        const int32_t tok = in ? seq[i] : -1;
        int32_t c = 0;
        if (in) {
            if (w.t0 + i == 0) {
                c = clamp_token(w.prompts[r / w.N], w.V);
            } else {
                c = seq[i - 1];
                c = (c >= 0 && c < w.V) ? c : 0;
            }
        }
        const unsigned long long eos = __ballot(in && w.eos_id >= 0 && tok == w.eos_id);
        const bool active = in && !ended && (eos & ((1ull << lane) - 1ull)) == 0ull;
        ended = ended || eos != 0ull;
        if (!in) continue;
        const int64_t p = r * w.Tw + i;
        if constexpr (CLAIMED) {
            w.cond[p] = active ? c : -1;
        } else {
            const bool of_prompt = prompts && i == 0;
            const int64_t slot = of_prompt ? r / w.N : first + r * per + i - (prompts ? 1 : 0);
            const int64_t at = of_prompt ? r : (prompts ? w.R : 0) + r * per + i - (prompts ? 1 : 0);
            w.slot[p] = (int32_t)slot;
            w.order[at] = active ? (int32_t)p : -1;
            if (!of_prompt || r % w.N == w.N - 1) {
                w.token[slot] = c;
                w.ends[slot] = (int32_t)(at + 1);
                w.idle[slot] = active || of_prompt ? 0 : 1;
            }
        }
    }
}

// the positions sorted by logits row, as share_order_kernel (those behind an EOS have none), and which rows are not in use
__global__ __launch_bounds__(256) void positions_order_kernel(Positions w, int64_t n, int64_t max_rows)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p < n && w.slot[p] >= 0) w.order[atomicAdd(&w.ends[w.slot[p]], 1)] = (int32_t)p;
    if (p < max_rows) w.idle[p] = p >= *w.count ? 1 : 0;
    if (p * w.chunk < max_rows) {
        const int64_t left = *w.count - p * w.chunk;
        w.chunk_rows[p] = (int32_t)(left < 0 ? 0 : (left > w.chunk ? w.chunk : left));
    }
}

// the positions whose rows a chunk holds: [begin, end) of w.order
__device__ __forceinline__ bool chunk_positions(const ChunkArgs &a, int32_t &begin, int32_t &end)
{
    const int64_t n = a.w.chunk_rows ? *a.w.count : a.s0 + a.rows;
    if (a.s0 >= n) return false;
    begin = a.s0 > 0 ? a.w.ends[a.s0 - 1] : 0;
    end = a.w.ends[(a.s0 + a.rows < n ? a.s0 + a.rows : n) - 1];
    return true;
}

// a position's shares, [Tw, R] each
__device__ __forceinline__ void write_shares(const ChunkArgs &a, int64_t p, int32_t tok, double all, double before, double at)
{
    double f_lo, pr;
    shares_of(all, before, at, tok >= 0 && tok < a.V, f_lo, pr);
    const int64_t o = p % a.w.Tw * a.w.R + p / a.w.Tw;
    a.w.f_lo[o] = f_lo;
    a.w.p[o] = pr;
}

// Rows whose chunk sums row_sums_kernel has left (rows of one tile): a wave per position reads them (272 bytes), scans
// them, and reads the one KiB of logits that holds its token.  The arithmetic of
// interval_tile_kernel, bit for bit.  Bound by its chain of four dependent loads: 11000 positions a launch 14 us.
template <int DT, bool HAS_THR>
__global__ __launch_bounds__(kThreads) void row_lookup_kernel(ChunkArgs a)
{
    using T = typename Elem<DT>::T;
    constexpr int EPV = Elem<DT>::kPerVec;
    constexpr int NW = kTileWaves, ITERS = kTileIters;
    __shared__ double scratch[3 * (kThreads / 64)];
    __shared__ float fscratch[kThreads / 64];
    __shared__ bool slow[kThreads / 64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t begin, end;
    if (!chunk_positions(a, begin, end)) return;
    const int32_t nvec = a.V / EPV;
    const float k = a.k;
    auto token_of = [&](int64_t p) { return a.w.tokens[p / a.w.Tw * a.w.T + a.w.t0 + p % a.w.Tw]; };
    for (int64_t j0 = begin + (int64_t)blockIdx.x * 4; j0 < end; j0 += (int64_t)gridDim.x * 4) {
        const int64_t p = j0 + wave < end ? (int64_t)a.w.order[j0 + wave] : -1;      // wave-uniform
        bool beyond = false;
        if (p >= 0) {
            const int64_t row = a.w.slot[p] - a.s0;
            const int32_t tok = token_of(p);
            const float *const sums = a.sums + row * kRowSums;
            const int32_t tc = clamp_token(tok, a.V);
            const int32_t vi = tc / EPV, el = tc % EPV;
            const int ch = vi >> 6, ln = vi & 63;
            const T *const lrow = reinterpret_cast<const T *>(a.logits) + row * a.ld;
            const bool inside = ch * 64 + lane < nvec;
            const u32x4 hv = reinterpret_cast<const u32x4 *>(lrow)[inside ? ch * 64 + lane : ch * 64];
            const float csum = sums[lane];
            float refs[NW];
#pragma unroll
            for (int w = 0; w < NW; ++w) refs[w] = sums[NW * ITERS + w];
            float thr = -__builtin_inff();
            if constexpr (HAS_THR) thr = a.thr[row];
            float R = refs[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) R = fmaxf(R, refs[w]);
            const float my_ref = sums[NW * ITERS + lane / ITERS];
            const double cv = (double)ldexpf(csum, shift_of(my_ref, R));
            const double cincl = wave_scan_add(cv);
            const double S = read_lane(cincl, 63);
            if (!(S < (double)__builtin_inff())) {
                beyond = true;                              // weights beyond fp32: the one-pass routine, below
            } else if (tok != tc) {
                // outside the vocabulary: probability zero, everything (or nothing) before it
                if (lane == 0) write_shares(a, p, tok, S, tok < 0 ? 0.0 : S, 0.0);
            } else {
                const double run = read_lane(cincl - cv, ch);
                const float rw = read_lane(my_ref, ch);
                const int shf = shift_of(rw, R);
                float cl = tile_lane_sum<DT, HAS_THR>(hv, k, -rw, thr);
                cl = inside ? cl : 0.f;
                token_shares<DT, HAS_THR>(hv, cl, k, rw, thr, shf, S, read_lane(cv, ch), run, ln, el, lane,
                                          [&](double all, double before, double at) {
                                              write_shares(a, p, tok, all, before, at);
                                          });
            }
        }
        if (!__syncthreads_or(beyond)) continue;             // (true or false, the same for the block)
        if (lane == 0) slow[wave] = beyond;
        __syncthreads();
        for (int w = 0; w < kThreads / 64; ++w) {
            if (!slow[w]) continue;                         // block-uniform
            const int64_t q = a.w.order[j0 + w], row = a.w.slot[q] - a.s0;
            const int32_t tok = token_of(q);
            interval_row<T>(reinterpret_cast<const T *>(a.logits) + row * a.ld, a.V, k, HAS_THR ? a.thr + row : nullptr, tok,
                            scratch, fscratch, [&](double all, double before, double at) {
                                write_shares(a, q, tok, all, before, at);
                            });
            __syncthreads();
        }
        __syncthreads();                                    // (before the next positions' flags)
    }
}

// other rows: a block per position, one pass over its row, as interval_kernel
template <class T>
__global__ __launch_bounds__(kThreads) void interval_items_kernel(ChunkArgs a)
{
    __shared__ double scratch[3 * (kThreads / 64)];
    __shared__ float fscratch[kThreads / 64];
    int32_t begin, end;
    if (!chunk_positions(a, begin, end)) return;
    for (int64_t j = begin + (int64_t)blockIdx.x; j < end; j += gridDim.x) {
        const int64_t p = a.w.order[j];
        if (p < 0) continue;
        const int64_t row = a.w.slot[p] - a.s0;
        const int32_t tok = a.w.tokens[p / a.w.Tw * a.w.T + a.w.t0 + p % a.w.Tw];
        interval_row<T>(reinterpret_cast<const T *>(a.logits) + row * a.ld, a.V, a.k, a.thr ? a.thr + row : nullptr, tok, scratch,
                        fscratch, [&](double all, double before, double at) { write_shares(a, p, tok, all, before, at); });
        __syncthreads();
    }
}

// The codebook recursion itself over one window: lo += width * F, width *= P, up to and including the sequence's EOS.
// A thread per sequence, eight positions' shares requested together (they do not depend on the recursion).
__global__ __launch_bounds__(64) void fold_kernel(Positions w, double *lo_out, double *width_out)
{
    constexpr int kAhead = 8;
    const int64_t r = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (r >= w.R) return;
    double lo = w.t0 > 0 ? lo_out[r] : 0.0, width = w.t0 > 0 ? width_out[r] : 1.0;
    bool ended = w.t0 > 0 && w.ended[r] != 0;
    for (int32_t i0 = 0; i0 < w.Tw && !ended; i0 += kAhead) {
        double f[kAhead], p[kAhead];
        int32_t tok[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const int32_t at = i0 + i < w.Tw ? i0 + i : w.Tw - 1;
            f[i] = w.f_lo[at * w.R + r];                     // (behind an EOS: not written, not used)
            p[i] = w.p[at * w.R + r];
            tok[i] = w.tokens[r * w.T + w.t0 + at];
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (ended || i0 + i >= w.Tw) continue;
            narrow(lo, width, f[i], p[i]);
            ended = w.eos_id >= 0 && tok[i] == w.eos_id;
        }
    }
    lo_out[r] = lo;
    width_out[r] = width;
    w.ended[r] = ended ? 1 : 0;
}

}  // namespace

as_status launch_interval(as_ctx *ctx, const IntervalArgs &args)
{
    if (args.rows == 0) return AS_OK;
    const IntervalArgs &a = args;
    const dim3 grid((unsigned)a.rows), block(kThreads);
    const size_t esz = a.dtype == AS_BF16 ? 2 : 4;
    const bool nt = stream_rows(a.rows, a.ld, esz);
    const int epv = (int)(16 / esz);
    const bool tile = a.V % epv == 0 && a.V / epv <= kTileWaves * kTileIters * 64 &&
                      reinterpret_cast<uintptr_t>(a.logits) % 16 == 0 && (a.ld * (int64_t)esz) % 16 == 0 &&
                      ctx->step_shape == 0 && a.k <= kTileMaxScale;
    if (tile) {
#define AS_INTERVAL_TILE(DT_)                                                                                   \
    do {                                                                                                        \
        if (a.thr && nt) launch(ctx, kKernelInterval, interval_tile_kernel<DT_, true, true>, grid, block, 0, a);   \
        else if (a.thr) launch(ctx, kKernelInterval, interval_tile_kernel<DT_, true, false>, grid, block, 0, a);   \
        else if (nt) launch(ctx, kKernelInterval, interval_tile_kernel<DT_, false, true>, grid, block, 0, a);      \
        else launch(ctx, kKernelInterval, interval_tile_kernel<DT_, false, false>, grid, block, 0, a);             \
    } while (0)
        if (a.dtype == AS_BF16) AS_INTERVAL_TILE(AS_BF16);
        else AS_INTERVAL_TILE(AS_F32);
#undef AS_INTERVAL_TILE
    } else if (a.dtype == AS_BF16) {
        launch(ctx, kKernelInterval, interval_kernel<uint16_t>, grid, block, 0, a);
    } else {
        launch(ctx, kKernelInterval, interval_kernel<float>, grid, block, 0, a);
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_positions(as_ctx *ctx, const Positions &w, bool claimed)
{
    const dim3 grid((unsigned)((w.R + 3) / 4));
    if (claimed) hipLaunchKernelGGL(positions_kernel<true>, grid, dim3(256), 0, ctx->stream, w);
    else hipLaunchKernelGGL(positions_kernel<false>, grid, dim3(256), 0, ctx->stream, w);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_positions_order(as_ctx *ctx, const Positions &w, int64_t max_rows)
{
    const int64_t n = w.R * w.Tw, most = n > max_rows ? n : max_rows;
    hipLaunchKernelGGL(positions_order_kernel, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, ctx->stream, w, n,
                       max_rows);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_interval_chunk(as_ctx *ctx, const ChunkArgs &a, bool by_sums)
{
    // (how many positions a chunk's rows have, the device knows: blocks for all of them, or as many as the chip holds)
    const int64_t n = a.w.R * a.w.Tw, fit = 8 * (int64_t)ctx->num_cus;
    const dim3 block(kThreads);
    if (by_sums) {
        const int64_t blocks = (n + 3) / 4 < fit ? (n + 3) / 4 : fit;
        const dim3 grid((unsigned)blocks);
        if (a.w.dtype == AS_BF16) {
            if (a.thr) launch(ctx, kKernelInterval, row_lookup_kernel<AS_BF16, true>, grid, block, 0, a);
            else launch(ctx, kKernelInterval, row_lookup_kernel<AS_BF16, false>, grid, block, 0, a);
        } else {
            if (a.thr) launch(ctx, kKernelInterval, row_lookup_kernel<AS_F32, true>, grid, block, 0, a);
            else launch(ctx, kKernelInterval, row_lookup_kernel<AS_F32, false>, grid, block, 0, a);
        }
    } else {
        const dim3 grid((unsigned)(n < fit ? n : fit));
        if (a.w.dtype == AS_BF16) launch(ctx, kKernelInterval, interval_items_kernel<uint16_t>, grid, block, 0, a);
        else launch(ctx, kKernelInterval, interval_items_kernel<float>, grid, block, 0, a);
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_fold(as_ctx *ctx, const Positions &w, double *lo, double *width)
{
    hipLaunchKernelGGL(fold_kernel, dim3((unsigned)((w.R + 63) / 64)), dim3(64), 0, ctx->stream, w, lo, width);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
