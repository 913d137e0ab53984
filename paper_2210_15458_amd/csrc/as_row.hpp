// What a sampling step writes per row, and the plain three-pass form of the step (Sec. 4.1, Algorithm 1 loop
// body: vocabulary-order cumulative sums, first bucket above the code, rescale), shared by the kernels that
// finish a row.
#ifndef AS_ROW_HPP
#define AS_ROW_HPP

#include "as_common.hpp"

namespace as {

constexpr float kRefFloor = -100000.f;  // reference when only -inf has been seen

// exp2 straight on the hardware instruction (no denormal fix-up: results below
// 2^-126 may flush to zero, which is far below anything that can matter here)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float widen_stored(float h) { return h; }
__device__ __forceinline__ float widen_stored(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// The row of this block.  ORDERED: the blocks of an XCD (work-groups go to the 8 of them round-robin) take one run of
// a.order, so that rows with one logits row are read through one L2 at about the same time; false past its end.  (A
// form of its own: with the choice made in the kernel every other launch waits for it, 64 rows of 32128 fp32 7.7 us
// instead of 7.2.)
template <bool ORDERED> __device__ __forceinline__ bool block_row(const StepArgs &a, int64_t &r)
{
    r = blockIdx.x;
    if constexpr (ORDERED) {
        const int64_t at = (int64_t)(blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        if (at >= a.rows) return false;
        r = a.order[at];
    }
    return true;
}

struct RowOut {
    int32_t token;
    float c_next, prob, f_lo;
};

__device__ __forceinline__ void write_row(const StepArgs &a, int64_t r, const RowOut &o)
{
    a.tokens_out[r * a.tok_stride] = o.token;
    a.codes_out[r] = o.c_next;
    if (a.finished_out) a.finished_out[r] = (a.eos_id >= 0 && o.token == a.eos_id) ? 1 : 0;
    if (a.prob_out) a.prob_out[r] = o.prob;
    if (a.flo_out) a.flo_out[r] = o.f_lo;
    if (a.prev_out) a.prev_out[r] = o.token;
}

// finished sequence: padding after EOS (Sec. 3.3); the code stops moving
__device__ __forceinline__ void write_finished(const StepArgs &a, int64_t r)
{
    a.tokens_out[r * a.tok_stride] = a.eos_id;
    a.codes_out[r] = a.codes[r];
    if (a.finished_out) a.finished_out[r] = 1;
    if (a.prob_out) a.prob_out[r] = 1.f;
    if (a.flo_out) a.flo_out[r] = 0.f;
    if (a.prev_out) a.prev_out[r] = a.eos_id;
}

// c' = (c*S - before)/e_v: the difference is taken in fp64, the quotient is an fp32 result anyway
__device__ __forceinline__ float rescale_code(double tau, double before, double ev)
{
    float cnf = (float)(tau - before) / (float)ev;
    cnf = fminf(cnf, 0x1.fffffep-1f);        // 1 - 2^-24
    if (!(cnf >= 0.f)) cnf = 0.f;
    return cnf;
}

struct GenericScratch {
    float red[4];
    double tot[256];
    int hit;
    double run;
};

// f(v, x) for the elements [lo, hi) in order.  WHOLE: rows of whole, aligned vectors, read by those: the threads' runs lie in
// lines of their own, and one element at a time a block fetches each of its lines dozens of times (a decode of 1024 codes x
// 64 of 32128 bf16 whose table is of plain rows 21.6 ms, 4.7 by vectors).
template <bool WHOLE, class T, class F>
__device__ __forceinline__ void each_element(const T *row, int32_t lo, int32_t hi, F f)
{
    if constexpr (WHOLE) {
        constexpr int EPV = 16 / (int)sizeof(T);
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        for (int32_t at = lo / EPV * EPV; at < hi; at += EPV) {
            const u32x4 q = *reinterpret_cast<const u32x4 *>(row + at);
#pragma unroll
            for (int e = 0; e < EPV; ++e) {
                const uint32_t word = q[EPV == 8 ? e / 2 : e];
                const float x = EPV == 8 ? widen_stored((uint16_t)(word >> 16 * (e % 2))) : __builtin_bit_cast(float, word);
                if (at + e >= lo && at + e < hi) f(at + e, x);
            }
        }
    } else {
        for (int32_t v = lo; v < hi; ++v) f(v, widen_stored(row[v]));
    }
}

// One row by a block of 256 threads, any alignment, any V: three plain passes (max, sums, search), each
// thread owning one contiguous run of elements so that thread order is vocabulary order.  Every thread of
// the block must call it (those past 256, which only blocks on rows of one tile have, own nothing); keeps x >= thr.
// The first two: the reference, and every thread's sum in sh.tot (behind a barrier).
template <bool WHOLE, class T>
__device__ __forceinline__ float generic_totals(const T *row, int32_t V, float k, float thr, GenericScratch &sh)
{
    const int tid = threadIdx.x;
    const int32_t len = (V + 255) / 256;
    const int32_t lo = tid * len, hi = (lo + len < V) ? lo + len : V;
    float m = -__builtin_inff();
    each_element<WHOLE>(row, lo, hi, [&](int32_t, float x) __attribute__((always_inline)) {
        if (x >= thr) m = fmaxf(m, x);
    });
    m = wave_max(m);
    if ((tid & 63) == 0 && tid < 256) sh.red[tid >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(sh.red[0], sh.red[1]), fmaxf(sh.red[2], sh.red[3]));
    const float ref = fmaxf(ceilf(m * k), kRefFloor);

    double tot = 0.0;
    each_element<WHOLE>(row, lo, hi, [&](int32_t, float x) __attribute__((always_inline)) {
        if (x >= thr) tot += (double)fast_exp2(fmaf(x, k, -ref));
    });
    if (tid < 256) sh.tot[tid] = tot;
    __syncthreads();
    return ref;
}

// The last: the element of [lo, hi) that holds tau, where `run` is the mass before lo; `before` the mass before it, `ev` its own.
template <bool WHOLE, class T>
__device__ __forceinline__ int32_t generic_element(const T *row, int32_t V, int32_t lo, int32_t hi, float k, float thr, float ref,
                                                   double tau, double run, double &before, double &ev)
{
    double acc = run, before_last = run, ev_last = 0.0;
    int32_t tok = -1, tok_last = lo < V ? lo : V - 1;
    before = run;
    ev = 0.0;
    each_element<WHOLE>(row, lo, hi, [&](int32_t v, float x) __attribute__((always_inline)) {
        const double e = (x >= thr) ? (double)fast_exp2(fmaf(x, k, -ref)) : 0.0;
        if (e > 0.0) { tok_last = v; before_last = acc; ev_last = e; }
        if (tok < 0 && acc + e > tau) { tok = v; before = acc; ev = e; }
        acc += e;
    });
    if (tok < 0) { tok = tok_last; before = before_last; ev = ev_last; }
    return tok;
}

template <class T>
__device__ __forceinline__ void generic_step_row(const StepArgs &a, int64_t r, float thr, GenericScratch &sh)
{
    const int tid = threadIdx.x;
    const int64_t src = a.row_ids ? (int64_t)a.row_ids[r] : r;
    const T *row = reinterpret_cast<const T *>(a.logits) + src * a.ld;
    const int32_t V = a.V;
    const int32_t len = (V + 255) / 256;
    const int32_t lo = tid * len, hi = (lo + len < V) ? lo + len : V;
    const float ref = generic_totals<false>(row, V, a.k, thr, sh);
    if (tid == 0) {
        double S = 0.0;
        for (int i = 0; i < 256; ++i) S += sh.tot[i];
        const double tau = (double)a.codes[r] * S;
        double run = 0.0, run_last = 0.0;
        int hit = -1, last_nz = 0;
        for (int i = 0; i < 256; ++i) {
            if (sh.tot[i] > 0.0) { last_nz = i; run_last = run; }
            if (run + sh.tot[i] > tau) { hit = i; break; }
            run += sh.tot[i];
        }
        if (hit < 0) { hit = last_nz; run = run_last; }
        sh.hit = hit;
        sh.run = run;
        sh.tot[0] = S;                     // thread 0's own total is not needed any more
    }
    __syncthreads();
    if (tid != sh.hit) return;
    const double S = sh.tot[0];
    const double tau = (double)a.codes[r] * S;
    double before, ev;
    const int32_t tok = generic_element<false>(row, V, lo, hi, a.k, thr, ref, tau, sh.run, before, ev);
    RowOut o;
    o.token = tok;
    o.c_next = rescale_code(tau, before, ev);
    o.prob = (float)(ev / S);
    o.f_lo = (float)(before / S);
    write_row(a, r, o);
}

// What steps to come need of a row of whole, aligned vectors that generic_step_row would take (a block; as generic_totals).  Its places are those of
// the record whose kernel gave the row up; the caller marks it as such.
template <class T>
__device__ __forceinline__ void write_plain_record(const T *row, int32_t V, float k, float thr, GenericScratch &sh, PlainRecord *rec)
{
    const float ref = generic_totals<true>(row, V, k, thr, sh);
    if (threadIdx.x != 0) return;
    double run = 0.0, run_last = 0.0;
    int last = 0;
    for (int i = 0; i < 256; ++i) {
        if (i % 4 == 0) rec->run[i / 4] = run;
        if (sh.tot[i] > 0.0) { last = i; run_last = run; }
        run += sh.tot[i];
    }
    rec->S = run;
    rec->run_last = run_last;
    rec->ref = ref;
    rec->thr = thr;
    rec->last = last;
}

// generic_step_row from that, by one wave, bit for bit: the four threads' runs of elements among which the code lies are summed
// again by as many lanes, then the one that holds it is searched; the token and the rescaled code, in every lane.
// (ms a decode of 16384 codes x 16 of 32128 bf16, p = 0.9, on logits with a Zipf bias, where the nucleus's kernel gives most rows
// up: from the block of each step's own kernel 89, with all 256 sums made anew by a wave 152, so 8.6.)
template <class T>
__device__ __forceinline__ int32_t generic_pick_row(const T *row, int32_t V, float k, float code, const PlainRecord *rec, float &c_next)
{
    const int lane = threadIdx.x & 63;
    const int32_t len = (V + 255) / 256;
    const double S = rec->S, mine = rec->run[lane], upto = lane < 63 ? rec->run[lane < 63 ? lane + 1 : 63] : S;
    const float ref = rec->ref, thr = rec->thr;
    const double tau = (double)code * S;
    const unsigned long long over = __ballot(upto > tau);
    int hit = rec->last;
    double run = rec->run_last;
    if (over) {
        const int j = __ffsll((long long)over) - 1;
        double tot = 0.0;
        if (lane < 4) {
            const int32_t lo = (4 * j + lane) * len, hi = (lo + len < V) ? lo + len : V;
            each_element<true>(row, lo, hi, [&](int32_t, float x) __attribute__((always_inline)) {
                if (x >= thr) tot += (double)fast_exp2(fmaf(x, k, -ref));
            });
        }
        run = read_lane(mine, j);
        hit = 4 * j + 3;
        for (int c = 0; c < 4; ++c) {
            const double t = read_lane(tot, c);
            if (run + t > tau) { hit = 4 * j + c; break; }
            if (c < 3) run += t;
        }
    }
    const int32_t lo = hit * len, hi = (lo + len < V) ? lo + len : V;
    double before, ev;
    const int32_t tok = generic_element<true>(row, V, lo, hi, k, thr, ref, tau, run, before, ev);
    c_next = rescale_code(tau, before, ev);
    return tok;
}

}  // namespace as
#endif
