// Lattice initialisation (Sec. 4.2, Definition "Arithmetic sampling") and the
// synthetic low-rank bigram model that stands in for P(X_t | X_<t) (Sec. 3.3):
// logits[r, v] = (scale/sqrt(d)) * sum_k E[prev[r], k] * U[k, v].
//
// The model keeps U transposed (Ut[V, d], K contiguous) so that both MFMA
// operands are read as 16-byte K-runs; the logits GEMM is then an "NT" product
// C[R, V] = gather(E, prev)[R, d] * Ut[V, d]^T on v_mfma_f32_32x32x16_bf16 with
// fp32 accumulation.  It is the only dense contraction on the path.
#include <type_traits>

#include "as_common.hpp"

namespace as {
namespace {

// ------------------------------------------------------------------ lattice

__global__ void lattice_kernel(const float *u, int32_t B, int32_t N, float *codes,
                               const int32_t *prompts, int32_t *prev, uint8_t *finished, int32_t *row_ids, int32_t V,
                               int32_t *table, int32_t *wanted)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (table && idx < V) table[idx] = (int32_t)idx;     // the rows of a table of all tokens
    if (idx >= (int64_t)B * N) return;
    const int32_t b = (int32_t)(idx / N), i = (int32_t)(idx % N);
    // c_i = (i + u)/N: spacing exactly 1/N around the circle, one shift per prompt
    const double c = codes ? ((double)i + (double)u[b]) / (double)N : 0.0;
    if (codes) codes[idx] = fminf((float)c, 0x1.fffffep-1f);
    if (prev) prev[idx] = clamp_token(prompts[b], V);
    if (wanted && i == 0) wanted[clamp_token(prompts[b], V)] = 1;
    if (finished) finished[idx] = 0;
    if (row_ids) row_ids[idx] = b;           // the first step's logits: one row per prompt
}

// ------------------------------------------------------------ shared logits rows

__global__ __launch_bounds__(256) void share_clear_kernel(RowShare s, int32_t V, int32_t T)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < V) s.mark[i] = -1;
    if (i < T) s.count[i] = 0;
}

// The first row to come with a token takes the next logits row for it: one addition to the step's counter per block
// (65536 of them on one address would take longer than the product they save).  Which row a token gets differs
// from run to run; what is in it does not.
// Kept rows (s.kept) are claimed once a decode: `mark` then says that the token has a row, and the counter goes on from
// the step before.  SKIP: a negative token is no token.
template <bool SKIP>
__global__ __launch_bounds__(1024) void share_claim_kernel(RowShare s, int32_t step, int32_t V, const int32_t *prev,
                                                           int64_t rows)
{
    __shared__ int32_t wave_n[16], block_at;
    const int64_t r = (int64_t)blockIdx.x * 1024 + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t stamp = s.kept ? 0 : step;
    bool mine = false;
    int32_t v = 0;
    if (r < rows && (!SKIP || prev[r] >= 0)) {
        v = clamp_token(prev[r], V);
        // (looked at first: the rows that have ended all come with one token)
        if (__hip_atomic_load(&s.mark[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != stamp)
            mine = atomicExch(&s.mark[v], stamp) != stamp;
    }
    // (kept rows: counted anew each step)
    if (s.fill != nullptr)
        for (int64_t i = r; i < s.kept; i += (int64_t)gridDim.x * 1024) s.fill[i] = 0;
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
        block_at = n ? atomicAdd(&s.count[step], n) : 0;
    }
    __syncthreads();
    if (mine) {
        const int32_t at = block_at + wave_n[wave] + __builtin_popcountll(m & ((1ull << lane) - 1ull));
        s.slot[v] = at;
        s.token[at] = v;
        if (!s.kept) s.fill[at] = 0;
    }
}

template <bool SORTED, bool SKIP>
__global__ __launch_bounds__(256) void share_map_kernel(RowShare s, int32_t step, int32_t V, const int32_t *prev,
                                                        int64_t rows, int32_t *row_ids)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (s.kept && r == 0) s.count[step + 1] = s.count[step];
    if (r >= rows) return;
    if (SKIP && prev[r] < 0) {
        row_ids[r] = -1;
        return;
    }
    const int32_t at = s.slot[clamp_token(prev[r], V)];
    row_ids[r] = at;
    if constexpr (SORTED) atomicAdd(&s.fill[at], 1);
}

// Counts per logits row to where its rows start.  One block; a wave takes one run of the table, 64 neighbouring words
// at a time and eight of those requested together (a run per thread, each word a line of its own: 40 us at 28000).
__global__ __launch_bounds__(1024) void share_scan_kernel(RowShare s, int32_t step)
{
    constexpr int kAhead = 8;
    __shared__ int32_t wave_tot[16];
    const int32_t n = s.count[step], per = (n + 1023) / 1024 * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t lo = wave * per < n ? wave * per : n, hi = lo + per < n ? lo + per : n;
    int32_t mine = 0;
    for (int32_t i = lo; i < hi; i += 64 * kAhead) {
#pragma unroll
        for (int j = 0; j < kAhead; ++j) mine += i + j * 64 + lane < hi ? s.fill[i + j * 64 + lane] : 0;
    }
    for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
    if (lane == 0) wave_tot[wave] = mine;
    __syncthreads();
    int32_t at = 0;
    for (int w = 0; w < wave; ++w) at += wave_tot[w];
    for (int32_t i = lo; i < hi; i += 64 * kAhead) {
        int32_t c[kAhead];
#pragma unroll
        for (int j = 0; j < kAhead; ++j) c[j] = i + j * 64 + lane < hi ? s.fill[i + j * 64 + lane] : 0;
#pragma unroll
        for (int j = 0; j < kAhead; ++j) {
            int32_t incl = c[j];
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int32_t y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            if (i + j * 64 + lane < hi) s.fill[i + j * 64 + lane] = at + incl - c[j];
            at += __shfl(incl, 63, 64);
        }
    }
}

__global__ __launch_bounds__(256) void share_order_kernel(RowShare s, int64_t rows, const int32_t *row_ids)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < rows) s.order[atomicAdd(&s.fill[row_ids[r]], 1)] = (int32_t)r;
}

// ---------------------------------------------------------------- transpose

template <class T>
__global__ __launch_bounds__(256) void transpose_kernel(const T *U, T *Ut, int32_t d, int32_t V)
{
    __shared__ T tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;      // 32 x 8
    const int64_t v0 = (int64_t)blockIdx.x * 32, k0 = (int64_t)blockIdx.y * 32;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t k = k0 + ty + i * 8, v = v0 + tx;
        if (k < d && v < V) tile[ty + i * 8][tx] = U[k * V + v];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t v = v0 + ty + i * 8, k = k0 + tx;
        if (k < d && v < V) Ut[v * d + k] = tile[tx][ty + i * 8];
    }
}

// -------------------------------------------------------------- logits GEMM

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void glb_void;

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t b = __builtin_bit_cast(uint32_t, f);
    b += 0x7fffu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

template <class OutT> __device__ __forceinline__ OutT to_out(float f);
template <> __device__ __forceinline__ float to_out<float>(float f) { return f; }
template <> __device__ __forceinline__ uint16_t to_out<uint16_t>(float f) { return f32_to_bf16_rne(f); }

// Two fp32 values to one packed pair of bf16 (round to nearest even), low half first.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    uint32_t r;
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(r) : "v"(lo), "v"(hi));
    return r;
}

// ---- persistent kernel --------------------------------------------------------
//
// Block tile 256 x 256, K step 64, 512 threads = 8 waves as 4 (M) x 2 (N), each wave 64 x 128 = 2 x 4 MFMA
// tiles of 32 x 32 (128 accumulator registers per lane).  One block per CU walks its tiles.
//
// Operands go global -> LDS directly (global_load_lds_dwordx4: lane l's 16 bytes land at base + 16*l), as whole
// 128-byte lines per tile row, into a ring of two 64 KB stages.  The load stream runs on across tile
// boundaries: the next tile's first two stages are requested before this tile's epilogue, and because a wave's
// vector-memory operations complete in issue order, those loads land before the epilogue's stores do.
// Fragment reads are hand-placed ds_read_b128, one between every two MFMAs, a K slice of 16 ahead.
// LDS rows are 128 B; 16-byte piece c of row r sits at piece c ^ ((r >> 1) & 7), which makes both the
// 16-row fragment reads and the contiguous loader writes bank-conflict free.
//
// The accumulators are kept transposed (vocabulary along the MFMA's rows): register v of lane l is
// vocabulary 8*(v/4) + 4*(l/32) + v%4 of the tile, batch row l%32, so a lane holds runs of 4 consecutive
// logits of one row.  The epilogue stages them through a private 4 KB of LDS per wave and writes whole
// 128-byte row pieces.
constexpr int PM = 256, PN = 256, PK = 64;
constexpr int kRingA = PM * PK * 2;                    // 32 KB of A rows per stage
constexpr int kRing = (PM + PN) * PK * 2;              // 64 KB per stage
constexpr int kWaveStage = 4096;                       // epilogue staging per wave: 32 rows x 128 B
constexpr int kPersistLds = 2 * kRing + 8 * kWaveStage;   // 160 KB: all of a CU's LDS

__device__ __forceinline__ bf16x8 lds_read16(uint32_t addr)
{
    bf16x8 r;
    asm volatile("ds_read_b128 %0, %1" : "=v"(r) : "v"(addr));
    return r;
}

// FUSED: instead of the logits, write per row and per group of 32 consecutive logits the pair
// (sum of exp2(y - ref), ref) with y = logit * log2(e)/temp and ref = ceil(max y) -- what the sampling
// step needs to find the group its code falls into (the logits never reach memory).  C then is that table,
// float2 [R, ldc], and alpha carries the extra factor log2(e)/temp.
template <class OutT, bool FUSED = false>
__global__ __launch_bounds__(512, 1) void bigram_gemm_persistent(const uint16_t *__restrict__ E,
                                                                 const uint16_t *__restrict__ Ut,
                                                                 const int32_t *__restrict__ prev, int64_t R,
                                                                 int32_t V, int32_t d, float alpha,
                                                                 OutT *__restrict__ C, int64_t ldc, int vec_store,
                                                                 int gm, RowRange range)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kPersistLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);       // uniform: LDS targets stay scalar
    const int wm = wave >> 1, wn = wave & 1;

    // Work-groups are handed to the 8 XCDs round-robin, so block b runs on XCD b & 7 and is worker b >> 3 of
    // the W workers there.  XCD x owns column tiles x, x+8, ...  A worker keeps one row tile as long as it can
    // (its gathered A rows stay the same from tile to tile) and the workers of an XCD sit on the same few
    // column tiles at the same time, so a Ut tile is fetched into that XCD's L2 once.  With more row tiles
    // than workers, the W workers of an XCD stand gm x W/gm over row and column tiles: what they have open
    // at one time, gm A tiles and W/gm Ut tiles, has to fit that XCD's L2 or every tile refetches both.
    if (range.end != nullptr) {
        const int64_t first = range.begin ? *range.begin : 0;
        R = *range.end - first;
        if (R <= 0) return;
        prev += first;
        C += first * ldc * (FUSED ? 2 : 1);
    }
    // Logits of twice the last-level cache and more are written past the caches: nothing of them is still there when they are read
    // (32128 rows of 32128, d = 512: 1017 us, 997 so, and the pass over them after it 375, 345; 263 MB, which are: an encode 1192,
    // 1202).  Whole lines only: 16160 x 80198, whose rows start inside a line, a decode 39.3 ms, 43.5.
    const bool past = R * ldc * (int64_t)sizeof(OutT) > (512LL << 20) && ldc * (int64_t)sizeof(OutT) % 128 == 0 &&
                      reinterpret_cast<uintptr_t>(C) % 128 == 0;
    const int64_t m_blocks = (R + PM - 1) / PM;
    const int64_t n_blocks = ((int64_t)V + PN - 1) / PN;
    const int W = (int)(gridDim.x >> 3);
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int64_t nbx = n_blocks > xcd ? (n_blocks - xcd + 7) / 8 : 0;
    const int64_t cg = m_blocks < W ? W / m_blocks : 0;
    auto item = [&](int64_t j, int64_t &bm, int64_t &bn) __attribute__((always_inline)) -> bool {
        if (nbx <= 0) return false;
        if (m_blocks >= W || (m_blocks >= gm && m_blocks % gm == 0)) {
            const int gn = W / gm, qm = q % gm, qn = q / gm;        // host: gm divides W
            if (nbx <= qn) return false;
            const int64_t mine = (nbx - qn + gn - 1) / gn;         // column tiles of this XCD that are this worker's
            bm = qm + gm * (j / mine);
            bn = xcd + 8 * (qn + gn * (j % mine));
            return bm < m_blocks;
        }
        if (q >= cg * m_blocks) return false;
        bm = q % m_blocks;
        const int64_t bnx = q / m_blocks + cg * j;
        bn = xcd + 8 * bnx;
        return bnx < nbx;
    };
    int64_t j = 0, bm, bn, bm_next = 0, bn_next = 0;
    if (!item(j, bm, bn)) return;

    // Loader: a stage is 64 chunks of 1 KB (8 tile rows x 128 B); chunk it*8 + wave, it 0..3, is A rows
    // it*64 + rowb, it 4..7 is B rows (it-4)*64 + rowb; a lane always moves logical piece pc of its row.
    // Every address is a uniform base plus a 32-bit offset per lane: the B offsets never change (Ut is padded
    // to whole column tiles, so no row needs a bound), the A offsets change with the row tile.
    const uint32_t rowbytes = (uint32_t)d * 2;
    const unsigned char *Eb = reinterpret_cast<const unsigned char *>(E);
    const unsigned char *Ub = reinterpret_cast<const unsigned char *>(Ut);
    const int rowb = wave * 8 + (lane >> 3);
    const uint32_t pcoff = (uint32_t)(((lane & 7) ^ ((rowb >> 1) & 7)) << 4);
    uint32_t aoff[4], boff[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) boff[it] = (uint32_t)(it * 64 + rowb) * rowbytes + pcoff;
    auto load_aoff = [&](int64_t m0) __attribute__((always_inline)) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            int64_t m = m0 + it * 64 + rowb;
            if (m > R - 1) m = R - 1;
            aoff[it] = (uint32_t)clamp_token(prev[m], V) * rowbytes + pcoff;
        }
    };
    // request chunk `it` of K stage `st` of the tile whose columns start at n0_ into ring slot buf_
    auto issue1 = [&](int64_t n0_, int st, int buf_, auto it_c) __attribute__((always_inline)) {
        constexpr int it = decltype(it_c)::value;
        unsigned char *dst = smem + buf_ * kRing + (it * 8 + wave) * 1024;
        if constexpr (it < 4) {
            __builtin_amdgcn_global_load_lds((glb_void *)(Eb + (int64_t)st * (PK * 2) + aoff[it]), (lds_void *)dst,
                                             16, 0, 0);
        } else {
            const unsigned char *base = Ub + n0_ * (int64_t)rowbytes + (int64_t)st * (PK * 2);
            __builtin_amdgcn_global_load_lds((glb_void *)(base + boff[it - 4]), (lds_void *)dst, 16, 0, 0);
        }
    };

    f32x16 acc[2][4];
    const int frow = lane & 31, fc = lane >> 5;
    uint32_t fa_addr[2], fb_addr[4];
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void *)smem;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = wm * 64 + i * 32 + frow;
        fa_addr[i] = lds_base + row * 128 + ((fc ^ ((row >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
        const int row = wn * 128 + jj * 32 + frow;
        fb_addr[jj] = lds_base + kRingA + row * 128 + ((fc ^ ((row >> 1) & 7)) << 4);
    }

    // The schedule below is spelled out instruction by instruction; the scheduling barriers keep it that way.
#define AS_SB() __builtin_amdgcn_sched_barrier(0)
#define AS_GL(n0_, st_, buf_, n_)                                                                            \
    do {                                                                                                     \
        issue1(n0_, st_, buf_, std::integral_constant<int, n_>{});                                           \
        AS_SB();                                                                                             \
    } while (0)
    // fragment of K slice kk (0..3) of the stage at ring offset so_: the slice is an XOR on the piece index
#define AS_RD_A(fr_, i_, so_, kk_)                                                                           \
    do {                                                                                                     \
        fr_[i_] = lds_read16((fa_addr[i_] + (so_)) ^ ((kk_) << 5));                                          \
        AS_SB();                                                                                             \
    } while (0)
#define AS_RD_B(fr_, j_, so_, kk_)                                                                           \
    do {                                                                                                     \
        fr_[j_] = lds_read16((fb_addr[j_] + (so_)) ^ ((kk_) << 5));                                          \
        AS_SB();                                                                                             \
    } while (0)
#define AS_MM(fa_, fb_, i_, j_)                                                                              \
    do {                                                                                                     \
        acc[i_][j_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb_[j_], fa_[i_], acc[i_][j_], 0, 0, 0);      \
        AS_SB();                                                                                             \
    } while (0)
    // the fragments are outputs of hand-written reads: tie the wait to them so no MFMA moves above it
#define AS_WAIT_FR(fa_, fb_)                                                                                 \
    do {                                                                                                     \
        asm volatile("s_waitcnt lgkmcnt(0)"                                                                  \
                     : "+v"(fa_[0]), "+v"(fa_[1]), "+v"(fb_[0]), "+v"(fb_[1]), "+v"(fb_[2]), "+v"(fb_[3]));  \
        AS_SB();                                                                                             \
    } while (0)
    // multiply the slice held in (ca, cb) while reading slice kk_ into (na, nb_)
#define AS_SLICE(ca, cb, na, nb_, so_, kk_)                                                                  \
    do {                                                                                                     \
        AS_RD_A(na, 0, so_, kk_); AS_MM(ca, cb, 0, 0); AS_RD_B(nb_, 0, so_, kk_); AS_MM(ca, cb, 0, 1);       \
        AS_RD_B(nb_, 1, so_, kk_); AS_MM(ca, cb, 0, 2); AS_RD_A(na, 1, so_, kk_); AS_MM(ca, cb, 0, 3);       \
        AS_RD_B(nb_, 2, so_, kk_); AS_MM(ca, cb, 1, 0); AS_RD_B(nb_, 3, so_, kk_); AS_MM(ca, cb, 1, 1);      \
        AS_MM(ca, cb, 1, 2); AS_MM(ca, cb, 1, 3);                                                            \
    } while (0)

    const int nstages = d / PK;                  // host guarantees nstages >= 2
    bf16x8 xa[2], xb[4], ya[2], yb[4];
    int gs = 0;                                  // running stage count: stage gs lives in ring slot gs & 1
    bool fresh = true;                           // this tile's first stages are not on their way yet
    int stores_behind = 0;                       // stores of the previous tile issued after this tile's stage 1
    for (;;) {
        const int64_t m0 = bm * PM, n0 = bn * PN;
        const bool has_next = item(j + 1, bm_next, bn_next);
        const bool carry = has_next && bm_next == bm;      // the next tile's loads may run ahead of this epilogue
        const int64_t n0n = bn_next * PN;
        if (fresh) {
            load_aoff(m0);
            const int b0 = gs & 1, b1 = b0 ^ 1;
            AS_GL(n0, 0, b0, 0); AS_GL(n0, 0, b0, 1); AS_GL(n0, 0, b0, 2); AS_GL(n0, 0, b0, 3);
            AS_GL(n0, 0, b0, 4); AS_GL(n0, 0, b0, 5); AS_GL(n0, 0, b0, 6); AS_GL(n0, 0, b0, 7);
            AS_GL(n0, 1, b1, 0); AS_GL(n0, 1, b1, 1); AS_GL(n0, 1, b1, 2); AS_GL(n0, 1, b1, 3);
            AS_GL(n0, 1, b1, 4); AS_GL(n0, 1, b1, 5); AS_GL(n0, 1, b1, 6); AS_GL(n0, 1, b1, 7);
            asm volatile("s_waitcnt vmcnt(8)" ::: "memory");      // stage 0 has landed, stage 1 may still fly
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const uint32_t so0 = b0 * kRing;
            AS_RD_A(xa, 0, so0, 0); AS_RD_A(xa, 1, so0, 0);
            AS_RD_B(xb, 0, so0, 0); AS_RD_B(xb, 1, so0, 0); AS_RD_B(xb, 2, so0, 0); AS_RD_B(xb, 3, so0, 0);
            stores_behind = 0;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][jj][v] = 0.f;
        for (int s = 0; s < nstages; ++s, ++gs) {
            const int cur = gs & 1, nb = cur ^ 1;
            const uint32_t so = cur * kRing, son = nb * kRing;
            // Stage s+2 is requested whole during the last slice of stage s, into the ring slot that stage s
            // has just left; past the end of this tile it is stage 0 or 1 of the next one.
            const bool in2 = s + 2 < nstages;
            const bool ld2 = in2 || carry;
            const int st2 = in2 ? s + 2 : s + 2 - nstages;
            const int64_t nn2 = in2 ? n0 : n0n;
            AS_WAIT_FR(xa, xb);
            AS_SLICE(xa, xb, ya, yb, so, 1);
            AS_WAIT_FR(ya, yb);
            AS_SLICE(ya, yb, xa, xb, so, 2);
            AS_WAIT_FR(xa, xb);
            AS_SLICE(xa, xb, ya, yb, so, 3);
            AS_WAIT_FR(ya, yb);
            // Every wave has read all of this stage and the next stage has landed.  Behind the next stage's
            // loads there may be the previous tile's stores: let those drain on (vmcnt counts in issue order).
            if (s == 0 && stores_behind == 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            else if (s == 0 && stores_behind == 32) asm volatile("s_waitcnt vmcnt(32)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            AS_SB();
            // last slice, with the first fragments of the next stage (read for nothing after the last stage
            // of the last tile) and, where there is a stage to request, its eight chunks; the MFMAs stay
            // outside the conditions (a second copy of them costs the accumulators a second set of registers)
            AS_RD_A(xa, 0, son, 0); AS_MM(ya, yb, 0, 0);
            AS_RD_B(xb, 0, son, 0); AS_MM(ya, yb, 0, 1);
            if (ld2) AS_GL(nn2, st2, cur, 0);
            AS_RD_B(xb, 1, son, 0); AS_MM(ya, yb, 0, 2);
            if (ld2) AS_GL(nn2, st2, cur, 1);
            AS_RD_A(xa, 1, son, 0); AS_MM(ya, yb, 0, 3);
            if (ld2) AS_GL(nn2, st2, cur, 2);
            AS_RD_B(xb, 2, son, 0); AS_MM(ya, yb, 1, 0);
            if (ld2) AS_GL(nn2, st2, cur, 3);
            AS_RD_B(xb, 3, son, 0); AS_MM(ya, yb, 1, 1);
            if (ld2) { AS_GL(nn2, st2, cur, 4); AS_GL(nn2, st2, cur, 5); }
            AS_MM(ya, yb, 1, 2);
            if (ld2) { AS_GL(nn2, st2, cur, 6); AS_GL(nn2, st2, cur, 7); }
            AS_MM(ya, yb, 1, 3);
        }

        // ---- epilogue: scale, round once to the storage type, transpose through this wave's 32 x 128 B of
        // staging (16-byte pieces permuted by the row's bits 1..3), write 128-byte row pieces.  The LDS
        // accesses are written by hand so that the compiler does not tie them to the loads in flight.
        if constexpr (FUSED) {
            // Lane l holds, for each 32-row group i and each 32-column MFMA tile j, 16 logits of batch row
            // l%32: columns 8q + 4*(l/32) + 0..3, q = 0..3; the other 16 of that row and tile sit in lane l^32.
            const int b = lane & 31, h = lane >> 5;
            float2 *P = reinterpret_cast<float2 *>(C);
            if (n0 + PN > V) {                    // last column tile: columns past V carry no mass
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int jx = 0; jx < 4; ++jx)
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int64_t n = n0 + wn * 128 + jx * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
                            if (n >= V) acc[i][jx][v] = -__builtin_inff();
                        }
            }
            // references of the 8 groups first (alpha > 0: the maximum commutes with the scaling), then the sums
            float ref[2][4];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int jx = 0; jx < 4; ++jx) {
                    float mx = acc[i][jx][0];
#pragma unroll
                    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[i][jx][v]);
                    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
                    ref[i][jx] = fmaxf(ceilf(mx * alpha), -100000.f);
                }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int jx = 0; jx < 4; ++jx) {
                    float sum = 0.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(fmaf(acc[i][jx][v], alpha, -ref[i][jx]));
                    sum += __shfl_xor(sum, 32, 64);
                    const int64_t ncol = n0 + wn * 128 + jx * 32;
                    const int64_t m = m0 + wm * 64 + i * 32 + b;
                    if (h == 0 && m < R && ncol < V) P[m * ldc + (ncol >> 5)] = float2{sum, ref[i][jx]};
                }
            stores_behind = -1;      // few small stores: the next tile's first barrier simply waits for them
        } else {
            constexpr int kPerPiece = 16 / (int)sizeof(OutT);     // outputs per 16-byte piece
            constexpr int kCols = 8 * kPerPiece;                  // tile columns per pass: 64 (bf16) or 32 (fp32)
            constexpr int kPasses = 128 / kCols;                  // per 32-row group of the wave tile
            const uint32_t stg = lds_base + 2 * kRing + wave * kWaveStage;
            const int b = lane & 31, h = lane >> 5;
            const bool interior = vec_store && m0 + PM <= R && n0 + PN <= V;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int ps = 0; ps < kPasses; ++ps) {
                    if constexpr (sizeof(OutT) == 2) {
#pragma unroll
                        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                            for (int qq = 0; qq < 4; ++qq) {
                                const int jx = ps * 2 + jj;
                                u32x2 w;
                                w[0] = pack_bf16(acc[i][jx][4 * qq + 0] * alpha, acc[i][jx][4 * qq + 1] * alpha);
                                w[1] = pack_bf16(acc[i][jx][4 * qq + 2] * alpha, acc[i][jx][4 * qq + 3] * alpha);
                                const int piece = (jj * 4 + qq) ^ ((b >> 1) & 7);
                                asm volatile("ds_write_b64 %0, %1" ::"v"(stg + b * 128 + piece * 16 + h * 8), "v"(w)
                                             : "memory");
                            }
                    } else {
#pragma unroll
                        for (int qq = 0; qq < 4; ++qq) {
                            u32x4 w;
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                w[e] = __builtin_bit_cast(uint32_t, acc[i][ps][4 * qq + e] * alpha);
                            const int piece = (qq * 2 + h) ^ ((b >> 1) & 7);
                            asm volatile("ds_write_b128 %0, %1" ::"v"(stg + b * 128 + piece * 16), "v"(w) : "memory");
                        }
                    }
                    u32x4 val[4];
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int idx = p * 64 + lane;
                        const int row = idx >> 3, piece = idx & 7;
                        asm volatile("ds_read_b128 %0, %1"
                                     : "=v"(val[p])
                                     : "v"(stg + row * 128 + ((piece ^ ((row >> 1) & 7)) << 4))
                                     : "memory");
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)"
                                 : "+v"(val[0]), "+v"(val[1]), "+v"(val[2]), "+v"(val[3])
                                 :
                                 : "memory");
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int idx = p * 64 + lane;
                        const int row = idx >> 3, piece = idx & 7;
                        const int64_t m = m0 + wm * 64 + i * 32 + row;
                        const int64_t n = n0 + wn * 128 + ps * kCols + piece * kPerPiece;
                        OutT *gp = C + m * ldc + n;
                        if (interior && past) {
                            __builtin_nontemporal_store(val[p], reinterpret_cast<u32x4 *>(gp));
                        } else if (interior) {
                            *reinterpret_cast<u32x4 *>(gp) = val[p];
                        } else if (m < R && n < V) {
                            if (vec_store && n + kPerPiece <= V) {
                                *reinterpret_cast<u32x4 *>(gp) = val[p];
                            } else {
#pragma unroll
                                for (int e = 0; e < kPerPiece; ++e) {
                                    if (n + e >= V) continue;
                                    // (copy the lane out first: a bit cast applied to a vector element
                                    // designator reads the vector's first element)
                                    const uint32_t bits = val[p][sizeof(OutT) == 2 ? e >> 1 : e];
                                    if constexpr (sizeof(OutT) == 2)
                                        gp[e] = (OutT)(bits >> ((e & 1) * 16));
                                    else
                                        gp[e] = __builtin_bit_cast(OutT, bits);
                                }
                            }
                        }
                    }
                }
            stores_behind = interior ? 8 * kPasses : -1;
        }
        if (!has_next) break;
        fresh = !carry;
        if (fresh) {
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
        ++j;
        bm = bm_next;
        bn = bn_next;
    }
#undef AS_SB
#undef AS_GL
#undef AS_RD_A
#undef AS_RD_B
#undef AS_MM
#undef AS_WAIT_FR
#undef AS_SLICE
}

// ---- tile kernel: any rank d that is a multiple of 64, any size ----------------------
//
// Block tile 128 x 256, K step 64; 4 waves as 2 (M) x 2 (N), each wave 64 x 128.  Operands are staged
// global -> registers -> LDS one K step ahead.  Used where the persistent kernel does not apply.
constexpr int BM = 128, BN = 256, BK = 64;
constexpr int kPieces = BK / 8;                       // 16-byte pieces per tile row
constexpr int kStageRows = 32;                        // C rows staged per epilogue pass

// Byte offset of 16-byte piece c of tile row `row`: pieces of a row are permuted by the row's bits 1..3 so
// that the 16 lanes served together by a fragment read touch all LDS banks once.
__device__ __forceinline__ int swz(int row, int c) { return row * (BK * 2) + ((c ^ ((row >> 1) & 7)) << 4); }

template <class OutT>
__global__ __launch_bounds__(256, 2) void bigram_gemm_bf16(const uint16_t *__restrict__ E,
                                                           const uint16_t *__restrict__ Ut,
                                                           const int32_t *__restrict__ prev, int64_t R,
                                                           int32_t V, int32_t d, float alpha,
                                                           OutT *__restrict__ C, int64_t ldc, int vec_store)
{
    constexpr int WNT = 4;
    constexpr int kBPieces = BN / 32;                  // 16-byte pieces of B per thread and K step
    constexpr int kABytes = BM * BK * 2, kBBytes = BN * BK * 2;
    constexpr int kStageStride = BN * (int)sizeof(OutT) + 16;          // bytes per staged C row
    constexpr int kStageBytes = kStageRows * kStageStride;
    constexpr int kLds = (kABytes + kBBytes) > kStageBytes ? (kABytes + kBBytes) : kStageBytes;
    __shared__ __attribute__((aligned(16))) unsigned char smem[kLds];
    unsigned char *sA = smem, *sB = smem + kABytes;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // Work-groups are handed to the 8 XCDs round-robin.  Give each XCD whole
    // column tiles and let it walk the row tiles of one column tile back to
    // back, so the Ut tile they share is fetched into that XCD's L2 once.
    const int64_t m_blocks = (R + BM - 1) / BM;
    const int64_t n_blocks = ((int64_t)V + BN - 1) / BN;
    const int64_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
    const int64_t bn = xcd + 8 * (slot / m_blocks), bm = slot % m_blocks;
    if (bn >= n_blocks) return;
    const int64_t m0 = bm * BM, n0 = bn * BN;

    // global -> register -> LDS: 4 pieces of A and 8 of B per thread and K step
    const int prow = tid >> 3, pc = tid & 7;
    const uint16_t *gA[4], *gB[kBPieces];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int64_t m = m0 + prow + i * 32;
        if (m > R - 1) m = R - 1;
        gA[i] = E + (int64_t)clamp_token(prev[m], V) * d + pc * 8;
    }
#pragma unroll
    for (int i = 0; i < kBPieces; ++i) {
        int64_t n = n0 + prow + i * 32;
        if (n > V - 1) n = V - 1;
        gB[i] = Ut + n * d + pc * 8;
    }

    f32x16 acc[2][WNT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < WNT; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    u32x4 ra[4], rb[kBPieces];
#pragma unroll
    for (int i = 0; i < 4; ++i) ra[i] = *reinterpret_cast<const u32x4 *>(gA[i]);
#pragma unroll
    for (int i = 0; i < kBPieces; ++i) rb[i] = *reinterpret_cast<const u32x4 *>(gB[i]);

    const int frow = lane & 31, fc = lane >> 5;
    for (int k0 = 0; k0 < d; k0 += BK) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4 *>(sA + swz(prow + i * 32, pc)) = ra[i];
#pragma unroll
        for (int i = 0; i < kBPieces; ++i) *reinterpret_cast<u32x4 *>(sB + swz(prow + i * 32, pc)) = rb[i];
        __syncthreads();
        if (k0 + BK < d) {
#pragma unroll
            for (int i = 0; i < 4; ++i) ra[i] = *reinterpret_cast<const u32x4 *>(gA[i] + k0 + BK);
#pragma unroll
            for (int i = 0; i < kBPieces; ++i) rb[i] = *reinterpret_cast<const u32x4 *>(gB[i] + k0 + BK);
        }
#pragma unroll
        for (int kk = 0; kk < kPieces; kk += 2) {
            bf16x8 fa[2], fb[WNT];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fa[i] = *reinterpret_cast<const bf16x8 *>(sA + swz(wm * 64 + i * 32 + frow, kk + fc));
#pragma unroll
            for (int j = 0; j < WNT; ++j)
                fb[j] = *reinterpret_cast<const bf16x8 *>(sB + swz(wn * (WNT * 32) + j * 32 + frow, kk + fc));
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < WNT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }

    // Epilogue: scale, round once to the storage type, stage 32 rows at a time in
    // LDS and write them out as whole 16-byte pieces along the row.
    // D layout of the 32x32 MFMA: register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32.
    constexpr int kOutPerPiece = 16 / (int)sizeof(OutT);
    constexpr int kPiecesPerRow = BN / kOutPerPiece;
    auto do_pass = [&](auto pass_c) {
        constexpr int pass = decltype(pass_c)::value;
        constexpr int i = pass & 1;
        __syncthreads();
        if (wm == pass / 2) {
#pragma unroll
            for (int j = 0; j < WNT; ++j) {
                const int col = wn * (WNT * 32) + j * 32 + (lane & 31);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                    *reinterpret_cast<OutT *>(smem + row * kStageStride + col * (int)sizeof(OutT)) =
                        to_out<OutT>(acc[i][j][v] * alpha);
                }
            }
        }
        __syncthreads();
        for (int p = tid; p < kStageRows * kPiecesPerRow; p += 256) {
            const int row = p / kPiecesPerRow, pcol = p % kPiecesPerRow;
            const int64_t m = m0 + pass * kStageRows + row;
            const int64_t n = n0 + (int64_t)pcol * kOutPerPiece;
            if (m >= R || n >= V) continue;
            const unsigned char *sp = smem + row * kStageStride + pcol * 16;
            OutT *gp = C + m * ldc + n;
            if (vec_store && n + kOutPerPiece <= V) {
                *reinterpret_cast<u32x4 *>(gp) = *reinterpret_cast<const u32x4 *>(sp);
            } else {
                const OutT *se = reinterpret_cast<const OutT *>(sp);
                for (int e = 0; e < kOutPerPiece; ++e)
                    if (n + e < V) gp[e] = se[e];
            }
        }
    };
    static_assert(BM / kStageRows == 4, "epilogue passes are spelled out");
    do_pass(std::integral_constant<int, 0>{});
    do_pass(std::integral_constant<int, 1>{});
    do_pass(std::integral_constant<int, 2>{});
    do_pass(std::integral_constant<int, 3>{});
}

// ---- thin kernel: few rows (a prompt's handful of codes, a first step's prompts), small products ---------------
//
// With few rows the product is a pass over Ut (33 MB at 32128 x 512), and on any small product the persistent kernel's
// 256 x 256 tiles leave most of the chip without one, each with 3 us of latency in front of its first product and
// rows of padding behind.  Here a block of four waves takes 128 columns and MT tiles of 32 rows (which of 1, 2 and 4:
// thin_tiles), so that V = 32128 is 251 blocks; K stages of 64 (one 128-byte line per row, loader and swizzle as in the persistent
// kernel) run through a ring of four, three stages requested ahead: 48 KB of Ut in flight per block, two blocks on a CU
// at MT = 1.  Same MFMA, K ascending, same epilogue arithmetic: a row's logits (and group masses) are the same
// bits whichever kernel makes them.
constexpr int TN = 128, kThinRing = 4;
template <int MT> constexpr int kThinStage = (TN + 32 * MT) * PK * 2;

// the fragments of two K slices in one go: all reads, one wait, in one piece of text, so that nothing can come between
// a read in flight and its register
template <int MT> struct ThinFrags {
    bf16x8 a[2], b[2][MT];
};
template <int MT>
__device__ __forceinline__ void thin_read(ThinFrags<MT> &f, uint32_t a0, uint32_t b0, uint32_t a1, uint32_t b1)
{
    if constexpr (MT == 1) {
        asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(f.a[0]), "=&v"(f.b[0][0]), "=&v"(f.a[1]), "=&v"(f.b[1][0])
                     : "v"(a0), "v"(b0), "v"(a1), "v"(b1)
                     : "memory");
    } else if constexpr (MT == 2) {
        asm volatile("ds_read_b128 %0, %6\n\tds_read_b128 %1, %7\n\tds_read_b128 %2, %7 offset:4096\n\t"
                     "ds_read_b128 %3, %8\n\tds_read_b128 %4, %9\n\tds_read_b128 %5, %9 offset:4096\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(f.a[0]), "=&v"(f.b[0][0]), "=&v"(f.b[0][1]), "=&v"(f.a[1]), "=&v"(f.b[1][0]), "=&v"(f.b[1][1])
                     : "v"(a0), "v"(b0), "v"(a1), "v"(b1)
                     : "memory");
    } else {
        static_assert(MT == 4, "one, two or four tiles of 32 rows");
        asm volatile("ds_read_b128 %0, %10\n\tds_read_b128 %1, %11\n\tds_read_b128 %2, %11 offset:4096\n\t"
                     "ds_read_b128 %3, %11 offset:8192\n\tds_read_b128 %4, %11 offset:12288\n\t"
                     "ds_read_b128 %5, %12\n\tds_read_b128 %6, %13\n\tds_read_b128 %7, %13 offset:4096\n\t"
                     "ds_read_b128 %8, %13 offset:8192\n\tds_read_b128 %9, %13 offset:12288\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(f.a[0]), "=&v"(f.b[0][0]), "=&v"(f.b[0][1]), "=&v"(f.b[0][2]), "=&v"(f.b[0][3]),
                       "=&v"(f.a[1]), "=&v"(f.b[1][0]), "=&v"(f.b[1][1]), "=&v"(f.b[1][2]), "=&v"(f.b[1][3])
                     : "v"(a0), "v"(b0), "v"(a1), "v"(b1)
                     : "memory");
    }
}

// FUSED: as in the persistent kernel, group masses instead of logits (C: float2 [R, ldc], alpha with log2(e)/temp).
// TILES: more row tiles than one (a form of its own: their numbers take 0.7 us to work out, of 5).
template <class OutT, int MT, bool FUSED, bool TILES>
__global__ __launch_bounds__(256) void bigram_gemm_thin(const uint16_t *__restrict__ E, const uint16_t *__restrict__ Ut,
                                                        const int32_t *__restrict__ prev, int32_t rows, int32_t V,
                                                        int32_t d, float alpha, OutT *__restrict__ C, int64_t ldc,
                                                        int vec_store)
{
    constexpr int kStage = kThinStage<MT>, kPerWave = 4 + MT;         // 1 KB requests of a wave per stage
    constexpr int kOutStride = TN * (int)sizeof(OutT) + 16;           // bytes of a staged row of C
    constexpr int kLds = kThinRing * kStage > 32 * MT * kOutStride ? kThinRing * kStage : 32 * MT * kOutStride;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int64_t n0 = (int64_t)blockIdx.x * TN;
    int32_t R = rows;
    if constexpr (TILES) {
        // blocks of one column tile follow each other eight apart, on one XCD: its Ut rows come through that L2 once
        const uint32_t mtiles = gridDim.y, bid = blockIdx.y * gridDim.x + blockIdx.x;
        const uint32_t group = bid / (8 * mtiles), in_group = bid % (8 * mtiles);
        const uint32_t width = gridDim.x - group * 8 < 8 ? gridDim.x - group * 8 : 8;
        n0 = (int64_t)(group * 8 + in_group % width) * TN;
        const int32_t m0 = (int32_t)(in_group / width) * 32 * MT;
        prev += m0;
        C += m0 * ldc * (FUSED ? 2 : 1);
        R = rows - m0;                                                // rows from the tile's first on
    }
    const uint32_t rowbytes = (uint32_t)d * 2;
    const unsigned char *Eb = reinterpret_cast<const unsigned char *>(E);
    const unsigned char *Ub = reinterpret_cast<const unsigned char *>(Ut) + n0 * (int64_t)rowbytes;

    // Loader: chunk c of a stage is 8 rows of 128 bytes; chunks 0..15 are Ut rows (padded to whole tiles of 256: no
    // bound), 16.. are E rows.  Wave w moves chunks w, w+4, ...  A lane moves piece (lane & 7) ^ swizzle of its row.
    const int rl = wave * 8 + (lane >> 3);                            // row within 32 of every chunk of this wave
    const uint32_t pcoff = (uint32_t)(((lane & 7) ^ ((rl >> 1) & 7)) << 4);
    int64_t off[kPerWave];
#pragma unroll
    for (int i = 0; i < 4; ++i) off[i] = (int64_t)(i * 32 + rl) * rowbytes + pcoff;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
        int32_t m = i * 32 + rl;
        m = m < R ? m : R - 1;
        off[4 + i] = (int64_t)clamp_token(prev[m], V) * rowbytes + pcoff;
    }
    auto request = [&](int st) __attribute__((always_inline)) {
        unsigned char *const slot = smem + (st & (kThinRing - 1)) * kStage + wave * 1024;
#pragma unroll
        for (int i = 0; i < kPerWave; ++i)
            __builtin_amdgcn_global_load_lds((glb_void *)((i < 4 ? Ub : Eb) + off[i] + (int64_t)st * (PK * 2)),
                                             (lds_void *)(slot + i * 4096), 16, 0, 0);
    };
    const uint32_t lds_base = (uint32_t)(uintptr_t)(lds_void *)smem;
    const int frow = lane & 31, fc = lane >> 5;
    const uint32_t fsw = (uint32_t)((fc ^ ((frow >> 1) & 7)) << 4);
    const uint32_t fa = lds_base + (uint32_t)(wave * 32 + frow) * 128 + fsw, fb = lds_base + TN * 128 + (uint32_t)frow * 128 + fsw;

    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    const int n = d / PK;
    for (int st = 0; st < kThinRing - 1 && st < n; ++st) request(st);
    for (int s = 0; s < n; ++s) {
        // stage s has landed; up to two more stay in flight behind it
        const int behind = n - 1 - s;
        if (behind >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kPerWave) : "memory");
        else if (behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPerWave) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // (every wave has left stage s - 1, whose slot this is)
        if (s + kThinRing - 1 < n) request(s + kThinRing - 1);
        const uint32_t so = (uint32_t)(s & (kThinRing - 1)) * kStage;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            ThinFrags<MT> f;
            thin_read<MT>(f, (fa + so) ^ (uint32_t)(h * 64), (fb + so) ^ (uint32_t)(h * 64),
                          (fa + so) ^ (uint32_t)(h * 64 + 32), (fb + so) ^ (uint32_t)(h * 64 + 32));
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int i = 0; i < MT; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[q], f.b[q][i], acc[i], 0, 0, 0);
        }
    }
    // register v of lane l is vocabulary 8*(v/4) + 4*(l/32) + v%4 of the wave's 32, batch row l%32 of the tile
    const int b = lane & 31, h = lane >> 5;
    if constexpr (FUSED) {
        float2 *P = reinterpret_cast<float2 *>(C);
        const int64_t ncol = n0 + wave * 32;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            if (ncol + 32 > V) {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (ncol + 8 * (v >> 2) + 4 * h + (v & 3) >= V) acc[i][v] = -__builtin_inff();
            }
            float mx = acc[i][0];
#pragma unroll
            for (int v = 1; v < 16; ++v) mx = fmaxf(mx, acc[i][v]);
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float ref = fmaxf(ceilf(mx * alpha), -100000.f);
            float sum = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(fmaf(acc[i][v], alpha, -ref));
            sum += __shfl_xor(sum, 32, 64);
            const int32_t m = i * 32 + b;
            if (h == 0 && m < R && ncol < V) P[m * ldc + (ncol >> 5)] = float2{sum, ref};
        }
    } else {
        __syncthreads();                                              // the ring gives way to the rows of C
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                unsigned char *at = smem + (i * 32 + b) * kOutStride + (wave * 32 + 8 * q + 4 * h) * (int)sizeof(OutT);
                if constexpr (sizeof(OutT) == 2) {
                    u32x2 w;
                    w[0] = pack_bf16(acc[i][4 * q + 0] * alpha, acc[i][4 * q + 1] * alpha);
                    w[1] = pack_bf16(acc[i][4 * q + 2] * alpha, acc[i][4 * q + 3] * alpha);
                    *reinterpret_cast<u32x2 *>(at) = w;
                } else {
                    u32x4 w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[e] = __builtin_bit_cast(uint32_t, acc[i][4 * q + e] * alpha);
                    *reinterpret_cast<u32x4 *>(at) = w;
                }
            }
        __syncthreads();
        constexpr int kPerPiece = 16 / (int)sizeof(OutT), kPieces = TN / kPerPiece;
        for (int p = tid; p < 32 * MT * kPieces; p += 256) {
            const int32_t m = p / kPieces;
            const int64_t col = n0 + (p % kPieces) * kPerPiece;
            if (m >= R || col >= V) continue;
            const unsigned char *sp = smem + m * kOutStride + (p % kPieces) * 16;
            OutT *gp = C + m * ldc + col;
            if (vec_store && col + kPerPiece <= V) {
                *reinterpret_cast<u32x4 *>(gp) = *reinterpret_cast<const u32x4 *>(sp);
            } else {
                const OutT *se = reinterpret_cast<const OutT *>(sp);
                for (int e = 0; e < kPerPiece; ++e)
                    if (col + e < V) gp[e] = se[e];
            }
        }
    }
}

// Which kernel a product of `rows` rows takes: MT of the thin one, or 0 for the 256 x 256 tiles of the persistent one, which
// leave most of the chip without a tile on small products and start 3 us later.  S K stages take, in us (fitted to the
// launches below), 0.4 + 0.22 S for each of the busiest compute unit's blocks at MT = 1 beside 2.6 for the launch (two
// stand there at a time, of the others one), 1.8 + 0.43 S a round at MT = 2, 3.0 + 0.63 S at MT = 4, and a round of the persistent kernel 1.05 S and up to
// 2.5 for the traffic of the others, beside 5.2.  Measured, d = 512, persistent / MT = 1 / 2 / 4: 257 x 3000 14.4 / 5.2 / 6.3 /
// 8.9; 1024 x 3000 15.7 / 10.1 / 11.5 / 9.5; 200 x 8000 14.9 / 7.1 / 6.8 / 9.1; 768 x 8000 16.4 / 16.5 / 16.1 / 16.6; 16 x 32128
// 16.5 / 5.2; 100 x 32128 16.1 / 12.2 / 11.8 / 9.9; 129 x 32128 16.3 / 14.4 / 16.2 / 17.6; 200 x 32128 17.3 / 18.8 / 21.0 / 17.7;
// 33 x 50000 17.6 / 12.4 / 12.1 / 16.7; d = 1024: 512 x 3000 23.1 / 9.9 / 9.7 / 13.6, 65 x 100000 49.0 / 41.9 / 58.6 / 53.4, 100 x
// 100000 50.1 / 54.4 / 61.8 / 55.7; d = 128: 512 x 2000 7.6 / 4.2 / 4.3 / 5.0.
// The same line where the persistent kernel cannot run and bigram_gemm_bf16 is the other one (us, here / there, as the line has
// it).  d = 64: 16 x 300 4.1 / 7.2, 8192 x 300 6.0 / 12.8, 1024 x 4000 5.3 / 8.8, 512 x 8000 5.3 / 9.7, 384 x 16000 7.8 / 9.5,
// 200 x 32128 9.3 / 10.0, 64 x 256000 17.8 / 20.7, and of 160 shapes only 4096 x 2000 (10.2 / 9.6) and 768 x 8000 (9.6 / 9.3)
// slower.  Operands of 4 GiB, 2^21 tokens, d = 1024: 1 row 711 / 822, 32 792 / 868, 64 988 / 923.
struct ProductTimes {            // us by these lines
    double thin[3], persistent;  // MT = 1, 2, 4
};
static ProductTimes product_times(const as_ctx *ctx, const as_model *m, int64_t rows)
{
    const double S = (double)m->d / PK, cus = ctx->num_cus > 0 ? ctx->num_cus : 1;
    const int64_t cols = (m->V + TN - 1) / TN;
    auto rounds_of = [&](int mt) { return ceil((double)((rows + 32 * mt - 1) / (32 * mt) * cols) / cus); };
    auto more = [&](int mt) { return rows > 32 * mt ? 0.7 : 0.0; };          // (what TILES costs)
    ProductTimes t;
    t.thin[0] = 2.6 + rounds_of(1) * (0.4 + 0.22 * S) + more(1);
    t.thin[1] = 0.6 + rounds_of(2) * (1.8 + 0.43 * S) + more(2);
    t.thin[2] = 0.5 + rounds_of(4) * (3.0 + 0.63 * S) + more(4);
    const double tiles = (double)((rows + PM - 1) / PM * (((int64_t)m->V + PN - 1) / PN)), rounds = ceil(tiles / cus);
    t.persistent = 5.2 + rounds * (1.05 * S + 2.5 * (tiles < cus ? tiles / cus : 1.0));
    return t;
}
static int thin_tiles(const as_ctx *ctx, const as_model *m, int64_t rows)
{
    if (ctx->gemm_shape != 0) return 0;
    const ProductTimes t = product_times(ctx, m, rows);
    const double t1 = t.thin[0], t2 = t.thin[1], t4 = t.thin[2];
    const double best = t1 < t2 ? (t1 < t4 ? t1 : t4) : (t2 < t4 ? t2 : t4);
    if (best > 0.95 * t.persistent || rows > 0x7fffffff - 256) return 0;
    return best == t1 ? 1 : best == t2 ? 2 : 4;
}

template <class OutT, bool FUSED>
void launch_thin(as_ctx *ctx, const as_model *m, const int32_t *prev, int64_t rows, OutT *out, int64_t ld, float alpha,
                 int vec_store, int mt)
{
    const uint16_t *Ep = (const uint16_t *)m->E, *Up = (const uint16_t *)m->Ut;
    const unsigned cols = (unsigned)((m->V + TN - 1) / TN);
    const dim3 grid(cols, (unsigned)((rows + 32 * mt - 1) / (32 * mt))), block(256);
#define AS_THIN(MT_)                                                                                                   \
    do {                                                                                                               \
        if (grid.y > 1)                                                                                                \
            launch(ctx, kKernelLogits, bigram_gemm_thin<OutT, MT_, FUSED, true>, grid, block, 0, Ep, Up, prev,         \
                   (int32_t)rows, m->V, m->d, alpha, out, ld, vec_store);                                              \
        else                                                                                                           \
            launch(ctx, kKernelLogits, bigram_gemm_thin<OutT, MT_, FUSED, false>, grid, block, 0, Ep, Up, prev,        \
                   (int32_t)rows, m->V, m->d, alpha, out, ld, vec_store);                                              \
    } while (0)
    if (mt == 1) AS_THIN(1);
    else if (mt == 2) AS_THIN(2);
    else AS_THIN(4);
#undef AS_THIN
}

// ---- chain kernel: what the bf16 MFMA kernels do not take (fp32 weights, or a rank d that is not a multiple of their K
// step), any size and alignment -----------------------------------------------------------------------------
//
// Every logit is one fp32 fused-multiply-add chain over k in ascending order, from zero, which keeps it the same whatever
// tile it is computed in.  v_mfma_f32_16x16x4_f32 adds its four products to the accumulator one after the other, each
// rounded (the chain bit for bit: tests/test_gpu_logits_shapes.py), at twice the rate of vector fused multiply-adds and
// with an operand register a lane for 16 x 16 x 4 products.  So operands hardly matter and a block is plain: 4 waves as
// GM x GN, a wave TM x TN tiles of 16 x 16, K steps of KS through one LDS buffer, the next step's elements in registers
// meanwhile.  MFMA s of a group of 16 k takes k = 4 s + q from the lanes of quarter q: LDS holds a row's group as four
// 16-byte pieces, piece q its k = q, q + 4, q + 8, q + 12, so that one read feeds four MFMAs; rows are padded by 16
// bytes (conflict-free for the reads' and the whole pieces' 16 lanes).
__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

// WHOLE: rows start on 16 bytes and the rank is a multiple of 16: a thread moves 16 consecutive k of a bf16 row at a time, or a
// 16-byte piece of an fp32 row (otherwise single elements, consecutive threads consecutive k).  With 16 k of an fp32 row a
// thread its loads are 64 bytes apart, and each of a wave's requests takes a quarter of 64 lines; pieces of whole lines cost four
// small LDS writes for one of 16 bytes and are ahead all the same (us, 16 k / pieces: 4100 x 4100 x 128 56.8 / 53.2, 4096 x 4096 x
// 256 90.0 / 85.2, 1024 x 32128 x 512 322 / 311, 256 x 4100 x 128 7.5 / 7.2).
template <class WT, class OutT, int GM, int GN, int TM, int TN, int KS, int AHEAD, bool WHOLE>
__global__ __launch_bounds__(256) void bigram_gemm_chain(const WT *__restrict__ E, const WT *__restrict__ Ut,
                                                         const int32_t *__restrict__ prev, int64_t R, int32_t V,
                                                         int32_t d, float alpha, OutT *__restrict__ C, int64_t ldc)
{
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    static_assert(GM * GN == 4, "four waves");
    constexpr int MT = GM * TM * 16, NT = GN * TN * 16, ROWS = MT + NT;
    constexpr int kGroups = KS / 16, kStride = KS * 4 + 16;
    // what a thread moves per K step: runs of 16 k, or elements
    constexpr int kRun = !WHOLE ? 1 : sizeof(WT) == 4 ? 4 : 16;
    constexpr int kUnits = ROWS * KS / kRun, kMine = (kUnits + 255) / 256;
    __shared__ __attribute__((aligned(16))) unsigned char smem[ROWS * kStride];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t m0 = (int64_t)blockIdx.x * MT, n0 = (int64_t)blockIdx.y * NT;

    const WT *src[kMine];                     // row starts; rows past the end repeat the last
    int row_of[kMine], k_of[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int u = tid + i * 256;
        constexpr int kPerRow = KS / kRun;
        row_of[i] = u / kPerRow;
        k_of[i] = u % kPerRow * kRun;
        if (kUnits % 256 != 0 && u >= kUnits) row_of[i] = ROWS - 1;
        if (row_of[i] < MT) {
            int64_t m = m0 + row_of[i];
            if (m > R - 1) m = R - 1;
            src[i] = E + (int64_t)clamp_token(prev[m], V) * d;
        } else {
            int64_t n = n0 + row_of[i] - MT;
            if (n > V - 1) n = V - 1;
            src[i] = Ut + n * d;
        }
    }
    WT raw[AHEAD][kMine][kRun];               // K steps requested ahead of the one worked on
    auto request = [&](int k0, auto slot_c) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            int k = k0 + k_of[i];
            k = k < d ? k : d - kRun;         // (past the rank: anything, replaced by zeros)
            if constexpr (WHOLE) {
                constexpr int kPieces = kRun * (int)sizeof(WT) / 16;
#pragma unroll
                for (int q = 0; q < kPieces; ++q)
                    reinterpret_cast<u32x4 *>(raw[slot][i])[q] = reinterpret_cast<const u32x4 *>(src[i] + k)[q];
            } else {
                raw[slot][i][0] = src[i][k];
            }
        }
    };
    auto land = [&](int k0, auto slot_c) __attribute__((always_inline)) {
        constexpr int slot = decltype(slot_c)::value;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            if (kUnits % 256 != 0 && tid + i * 256 >= kUnits) continue;
            const bool in = k0 + k_of[i] < d; // past the rank: zeros, which leave a chain as it is
            unsigned char *const at = smem + row_of[i] * kStride + (k_of[i] / 16) * 64;
            if constexpr (kRun == 4) {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float *>(at + q * 16 + (k_of[i] & 15)) = in ? widen(raw[slot][i][q]) : 0.f;
            } else if constexpr (WHOLE) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = in ? widen(raw[slot][i][4 * e + q]) : 0.f;
                    *reinterpret_cast<f32x4 *>(at + q * 16) = v;
                }
            } else {
                const int k = k_of[i] & 15;
                *reinterpret_cast<float *>(at + (k & 3) * 16 + (k >> 2) * 4) = in ? widen(raw[slot][i][0]) : 0.f;
            }
        }
    };

    const int wm = wave / GN, wn = wave % GN;
    const unsigned char *const fa = smem + (wm * TM * 16 + (lane & 15)) * kStride + (lane >> 4) * 16;
    const unsigned char *const fb = smem + (MT + wn * TN * 16 + (lane & 15)) * kStride + (lane >> 4) * 16;
    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](int k0, auto slot_c) __attribute__((always_inline)) {
        if (k0 != 0) __syncthreads();
        land(k0, slot_c);
        __syncthreads();
        if (k0 + AHEAD * KS < d) request(k0 + AHEAD * KS, slot_c);
        const int groups = d - k0 < KS ? (d - k0 + 15) / 16 : kGroups;
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            if (g >= groups) break;           // uniform
            f32x4 a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = *reinterpret_cast<const f32x4 *>(fa + i * 16 * kStride + g * 64);
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = *reinterpret_cast<const f32x4 *>(fb + j * 16 * kStride + g * 64);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
        }
    };
    request(0, std::integral_constant<int, 0>{});
    if constexpr (AHEAD == 2) {
        if (KS < d) request(KS, std::integral_constant<int, 1>{});
        for (int k0 = 0; k0 < d; k0 += 2 * KS) {
            step(k0, std::integral_constant<int, 0>{});
            if (k0 + KS < d) step(k0 + KS, std::integral_constant<int, 1>{});
        }
    } else {
        for (int k0 = 0; k0 < d; k0 += KS) step(k0, std::integral_constant<int, 0>{});
    }
    // register v of lane l is row 4 * (l / 16) + v, column l % 16 of its tile
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t m = m0 + (wm * TM + i) * 16 + 4 * (lane >> 4) + v;
            if (m >= R) continue;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t n = n0 + (wn * TN + j) * 16 + (lane & 15);
                if (n < V) C[m * ldc + n] = to_out<OutT>(acc[i][j][v] * alpha);
            }
        }
}

template <class WT, class OutT>
void launch_chain(as_ctx *ctx, const as_model *m, const int32_t *prev, int64_t rows, void *out, int64_t ld, float alpha)
{
    const bool whole = m->d % 16 == 0 && reinterpret_cast<uintptr_t>(m->E) % 16 == 0 && reinterpret_cast<uintptr_t>(m->Ut) % 16 == 0;
#define AS_CHAIN(GM_, GN_, TM_, TN_, KS_, AHEAD_)                                                                              \
    do {                                                                                                               \
        const dim3 grid((unsigned)((rows + GM_ * TM_ * 16 - 1) / (GM_ * TM_ * 16)),                                    \
                        (unsigned)((m->V + GN_ * TN_ * 16 - 1) / (GN_ * TN_ * 16)));                                   \
        if (whole)                                                                                                     \
            launch(ctx, kKernelLogits, bigram_gemm_chain<WT, OutT, GM_, GN_, TM_, TN_, KS_, AHEAD_, true>, grid, dim3(256), 0, \
                   (const WT *)m->E, (const WT *)m->Ut, prev, rows, m->V, m->d, alpha, (OutT *)out, ld);               \
        else                                                                                                           \
            launch(ctx, kKernelLogits, bigram_gemm_chain<WT, OutT, GM_, GN_, TM_, TN_, KS_, AHEAD_, false>, grid, dim3(256),   \
                   0, (const WT *)m->E, (const WT *)m->Ut, prev, rows, m->V, m->d, alpha, (OutT *)out, ld);            \
    } while (0)
    // us a launch, 16 x 64 / 32 x 64 / 64 x 128 / 128 x 128 tiles: 64 x 1000 x 100 4.3 / 5.1 / 9.2 / 14.3; 200 x 3000 x 144
    // 7.6 / 7.1 / 10.2 / 15.2; 256 x 4100 x 128 8.2 / 7.4 / 9.1 / 13.8; 512 x 5000 x 120 16.0 / 12.5 / 15.6 / 16.2; 300 x 9000 x
    // 72 16.8 / 12.0 / 12.5 / 13.4; 1024 x 4096 x 256 35.5 / 29.1 / 25.6 / 25.2; 1024 x 32128 x 512 450 / 326 / 321 / 310 to 346;
    // 4096 x 32128 x 520 (bf16) 2120 / 1642 / 1357 / 1307.  By the blocks of 32 x 64 and of 128 x 128 a compute unit:
    const int64_t fine = (rows + 31) / 32 * ((m->V + 63) / 64), coarse = (rows + 127) / 128 * ((m->V + 127) / 128);
    // (small ranks in K steps of their size: a step moves zeros past the rank)
    if (fine <= ctx->num_cus && m->d <= 16) AS_CHAIN(1, 4, 1, 1, 16, 1);
    else if (fine <= ctx->num_cus && m->d <= 32) AS_CHAIN(1, 4, 1, 1, 32, 1);
    else if (fine <= ctx->num_cus) AS_CHAIN(1, 4, 1, 1, 64, 1);
    else if (fine <= 6 * (int64_t)ctx->num_cus) AS_CHAIN(2, 2, 1, 2, 32, 2);
    else if (coarse < 16 * (int64_t)ctx->num_cus) AS_CHAIN(2, 2, 2, 4, 32, 1);
    else AS_CHAIN(2, 2, 4, 4, 32, 1);
#undef AS_CHAIN
}

// ------------------------------------------------------------------ estimator

// (1/N) sum_i s(x_i) per prompt (Sec. 4.2) for additive per-token scores: s(x) = sum of score[x_t] up to
// and including the first EOS.  One block per prompt, 2^width lanes (at most a wave) per sequence, its tokens side by side:
// bound by the two dependent loads of a round, of which a thread per sequence made T, one after another (64 x 16 x 128 tokens 36
// us, now 6).  A block has 1, 4 or 16 waves: no more than its sequences fill, nor than the chip holds twice over all prompts;
// otherwise many prompts of few sequences wait for idle waves to start and end (us, by prompts x sequences x tokens, 16 waves
// always / by size: 65536 x 1 x 1 116 / 16.6, 65536 x 4 x 8 117 / 16.5, 8192 x 300 x 1 17.8 / 5.9).  fp64 sums in a fixed order.
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void estimate_kernel(const int32_t *tokens, int32_t N, int32_t T, int32_t V,
                                                        const float *score, int32_t eos_id, double *est, int width)
{
    __shared__ double part[WAVES];
    const int64_t b = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int per = 64 >> width, sub = lane >> width, at = lane & ((1 << width) - 1);
    const unsigned long long before = ((1ull << at) - 1ull) << (sub << width);
    double acc = 0.0;
    for (int64_t i = (int64_t)wave * per + sub; i - sub < N; i += WAVES * per) {
        const int32_t *seq = tokens + (b * N + i) * T;
        for (int32_t t = at; t - at < T; t += 64) {              // (more than one round with the wave's whole width only)
            const bool in = i < N && t < T;
            const int32_t tok = in ? seq[t] : -1;
            const unsigned long long ends = __ballot(in && eos_id >= 0 && tok == eos_id);
            if (in && (ends & before) == 0ull && tok >= 0 && tok < V) acc += (double)score[tok];
            if (width == 6 && ends != 0ull) break;
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double all = 0.0;
        for (int w = 0; w < WAVES; ++w) all += part[w];
        est[b] = all / (double)N;
    }
}

}  // namespace

as_status launch_lattice(as_ctx *ctx, const float *u, int32_t B, int32_t N, float *codes_out,
                         const int32_t *prompts, int32_t *prev_out, uint8_t *finished_out, int32_t *row_ids_out,
                         int32_t *table_out, int32_t *wanted_out)
{
    const int64_t rows = (int64_t)B * N, n = table_out && ctx->V > rows ? ctx->V : rows;
    if (rows == 0) return AS_OK;
    hipLaunchKernelGGL(lattice_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, u, B, N,
                       codes_out, prompts, prev_out, finished_out, row_ids_out, ctx->V, table_out, wanted_out);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_estimate(as_ctx *ctx, const int32_t *tokens, int32_t B, int32_t N, int32_t T, const float *score,
                          int32_t eos_id, double *est_out)
{
    if (B == 0) return AS_OK;
    int width = 0;
    while (width < 6 && (1 << width) < T) ++width;
    const int64_t filled = ((int64_t)N + (64 >> width) - 1) / (64 >> width), room = 64LL * ctx->num_cus / B;
    auto go = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)B), dim3(64 * waves), 0, ctx->stream, tokens, N, T, ctx->V, score, eos_id, est_out,
                           width);
    };
    if (filled > 4 && room >= 16) go(estimate_kernel<16>, 16);
    else if (filled > 1 && room >= 4) go(estimate_kernel<4>, 4);
    else go(estimate_kernel<1>, 1);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_transpose(const void *U, void *Ut, int32_t d, int32_t V, as_dtype wdtype)
{
    const dim3 grid((unsigned)((V + 31) / 32), (unsigned)((d + 31) / 32));
    if (wdtype == AS_BF16)
        hipLaunchKernelGGL((transpose_kernel<uint16_t>), grid, dim3(256), 0, nullptr,
                           (const uint16_t *)U, (uint16_t *)Ut, d, V);
    else
        hipLaunchKernelGGL((transpose_kernel<float>), grid, dim3(256), 0, nullptr, (const float *)U,
                           (float *)Ut, d, V);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(nullptr, e, "transpose launch");
    e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) return hip_fail(nullptr, e, "transpose sync");
    return AS_OK;
}

// Workers of an XCD along the row tiles when there are more row tiles than workers (a divisor of their number)
static int persistent_gm(const as_ctx *ctx)
{
    const int W = ctx->num_cus / 8;
    if (ctx->gemm_gm > 0 && W % ctx->gemm_gm == 0) return ctx->gemm_gm;
    // 8 x W/8: with 256 KB per operand tile (d = 512) that is 2 MB of A and 1 MB of Ut open in a 4 MB L2;
    // measured at 65536 x 32128 x 512: 768 TFLOP/s with all workers along the rows, 992 with 8, 938 with 4
    return W % 8 == 0 ? 8 : W;
}

// Whether the MFMA kernels take the model (otherwise the chain kernel does).
bool mfma_applies(const as_model *m)
{
    return m->wdtype == AS_BF16 && m->d % BK == 0 && reinterpret_cast<uintptr_t>(m->E) % 16 == 0 &&
           reinterpret_cast<uintptr_t>(m->Ut) % 16 == 0;
}

// Tiles that the busiest worker of the persistent kernel computes, one after the other, for m row tiles (its mapping: with
// fewer row tiles than workers, and not a multiple of gm of them, some of the workers have none).
static int64_t tile_rounds(int64_t m, int64_t n_blocks, int W, int gm)
{
    const int64_t nbx = (n_blocks + 7) / 8;
    if (m >= W || (m >= gm && m % gm == 0)) return (m + gm - 1) / gm * ((nbx + W / gm - 1) / (W / gm));
    return (nbx + W / m - 1) / (W / m);
}

// Whether the logits kernel that takes the model can read the number of rows on the device (the persistent one).
bool rows_on_device(const as_ctx *ctx, const as_model *m)
{
    return ctx->gemm_shape != 1 && ctx->num_cus >= 8 && mfma_applies(m) && m->d >= 2 * PK &&
           (int64_t)m->V * m->d * 2 < (1LL << 32);
}

// Whether a decode of `rows` rows shares logits rows after its first step.  With tokens spread evenly over the vocabulary
// (the worst case) rows - V(1 - exp(-rows/V)) rows of product are saved; the sharing itself takes 6 to 12 us a step,
// 20 to 25 where the rows are sorted too, and is asked to save 20.  What the product then takes less lies between
// the work saved, at 1 PFLOP/s, and the tiles that the busiest worker is spared, 1.72 us a K step and 2.3 for the rest:
// the rows in use may fit the workers worse than all rows do.  Half of each is what was measured (us a step, every
// row its own / shared; V = 32128): d = 512, 6144 rows 238 / 262, 6700 303 / 255 (24 row tiles fit, 27 do not), 8192
// 313 / 335, 9000 364 / 343, 12288 473 / 393, 65536 2680 / 1260; d = 1024, 6144 rows 376 / 421, 6700 478 / 373, 8192
// 497 / 487.  V = 4096, d = 512: 4096 rows 49 / 44, 8192 80 / 57.
bool sharing_pays(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T)
{
    if (T < 2 || !rows_on_device(ctx, m)) return false;
    const double tokens = (double)m->V * (1.0 - exp(-(double)rows / (double)m->V));
    const int W = ctx->num_cus / 8, gm = persistent_gm(ctx);
    const int64_t n_blocks = ((int64_t)m->V + PN - 1) / PN;
    const int64_t spared = tile_rounds((rows + PM - 1) / PM, n_blocks, W, gm) -
                           tile_rounds(((int64_t)tokens + PM) / PM, n_blocks, W, gm);
    const double work = ((double)rows - tokens) * (double)m->V * (double)m->d * 2.0 / 1e15;
    const double tiles = (double)spared * ((double)m->d / PK * 1.72e-6 + 2.3e-6);
    return 0.5 * (work + tiles) > 20e-6;
}

// Whether a decode keeps logits rows from step to step.  With tokens spread evenly over the vocabulary (the worst case)
// U = V(1 - exp(-rows (T - 1)/V)) rows are computed after the first step; what that spares is rows of product, at 1 PFLOP/s, and, where the
// steps work from sums (by_sums), a pass over a logits row (5 TB/s, at least 4 ns) per row of codes less one per logits
// row computed and 0.5 ns a code (against a row per token in each step where the decode would share those).  It costs
// the claims and a launch more, up to 22 us while steps still meet new tokens (about 6 V/rows of them) and 4 after.  us a step, without / with, bf16, V = 32128, d = 512: 8192 rows T = 4 285 / 212,
// T = 16 325 / 117; 65536 rows T = 16 1275 / 153.  V = 8000, d = 512:
// 2048 rows T = 4 31.4 / 38.2, T = 16 33.6 / 31.6; 4096 rows T = 4 51.6 / 44.9.  V = 2000, d = 128: 1024 rows T = 64 15.1 /
// 15.5, 2048 20.9 / 13.8.  Not by sums, V = 5001, d = 512: 2048 rows T = 16 39.0 / 42.1, T = 64 37.5 / 31.6; 8192 rows
// T = 4 91.7 / 86.5.  Group masses, V = 32128: 16384 rows T = 16 485 / 182; V = 4096: 1024 rows
// T = 64 23.8 / 24.2.
// (How large its table may be: kept_rows_most.)
bool keeping_pays(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T, bool by_sums)
{
    if (T < 3 || !rows_on_device(ctx, m) || ctx->kept_rows == 1 || ctx->kept_rows == 3) return false;
    if (ctx->kept_rows == 2) return true;
    const double V = (double)m->V, R = (double)rows;
    const double steps = T - 1;
    const double computed = V * (1.0 - exp(-R * steps / V)) / steps;           // logits rows a step
    const double without = sharing_pays(ctx, m, rows, T) ? V * (1.0 - exp(-R / V)) : R;
    double spared = (without - computed) * V * (double)m->d * 2.0 / 1e15;
    if (by_sums) {
        const double pass = V * (ctx->dtype == AS_BF16 ? 2.0 : 4.0) / 5e12;
        spared += R * ((pass > 4e-9 ? pass : 4e-9) - 0.5e-9) - computed * pass;
    }
    const double meeting = 6.0 * V / (R * steps);
    return spared > 4e-6 + 18e-6 * (meeting < 1.0 ? meeting : 1.0);
}

// What a product of `rows` rows takes, in us
static double product_us(const as_ctx *ctx, const as_model *m, double rows)
{
    if (!mfma_applies(m)) return 3.5 + rows * (double)m->V * (2.0 * (double)m->d / 1e8 + (ctx->dtype == AS_BF16 ? 2.0 : 4.0) / 5e6);
    const ProductTimes t = product_times(ctx, m, (int64_t)rows + 1);
    const double thin = t.thin[0] < t.thin[1] ? (t.thin[0] < t.thin[2] ? t.thin[0] : t.thin[2])
                                              : (t.thin[1] < t.thin[2] ? t.thin[1] : t.thin[2]);
    // (the line for small products is low where every compute unit has several tiles)
    const int64_t row_tiles = ((int64_t)rows + PM) / PM, n_blocks = ((int64_t)m->V + PN - 1) / PN;
    const int W = ctx->num_cus / 8;
    const double large = W > 0 && row_tiles * n_blocks > ctx->num_cus ?
        4.0 + (double)tile_rounds(row_tiles, n_blocks, W, persistent_gm(ctx)) * (1.72 * (double)m->d / PK + 2.3) : t.persistent;
    return (thin < large ? thin : large) + (ctx->dtype == AS_BF16 ? 0.0 : rows * (double)m->V * 2.0 / 5e6);
}

// Whether a decode makes the logits rows of all tokens first, against a row per code, token in use or new token (`keep`) in
// each step.  Then it has one large product, one pass over its rows, and steps of 2 us (1 from candidates; 0.4 ns a code where
// those are many) that share a launch; where the steps' kernels have to read the rows (kTableRows) it spares the products alone.
// us a decode, every step its own rows / kept / table: 1024 codes x 64 of 32128 x 512 3124 / - / 1486, 16 x 64 638 / - / 1550;
// k = 40, 1024 x 128 6548 / - / 1504; 65536 x 16 20260 / 2465 / 1808; 3605 x 126 of 1600 x 1024 5281 / 2052 / 267; 406 x 59 of
// 504 x 128 538 / - / 77; 270 x 117 of 3424 x 832 1401 / - / 193; 1 x 73 of 657 x 19 fp32, k = 100 1056 / - / 838 (rows); 2004 x
// 49 of 9640 x 768, k = 100 4178 / - / 2265 (rows); against the table: 5579 x 5 of 14277 x 192, fp32 logits 567 / 491 / 535, 12 x
// 115 of 18904 x 896, fp32 (rows) 1431 / - / 1695; 2732 x 4 of 8744 x 576, k = 40 (rows) 280 / - / 308.
//
// All that is by tokens that come evenly, which is the table's best case: it has a row for each whatever comes.  Rows of one's
// own cost what they cost by any tokens (ended codes included: their rows are computed too), but kept rows are fewer where
// tokens are few.  So against those a table of all has to win by the least that they can take (on 300 tokens, measured / by the
// line below: 65536 codes x 16 914 / 829, 65536 x 6 475 / 336, 16384 x 16 464 / 357, 8192 x 64 1005 / 995, 4096 x 16 274 / 239,
// 5997 x 6 169 / 122); else rows are made on demand, for the tokens that codes come to, where steps work from
// records.  us a decode of 32128 x 512, kept / table / on demand, on even tokens: 65536 x 16 2495 / 1729 / 1998, 8192 x 64 3318 / 1580 /
// 1692, k = 40 16384 x 16 4007 / 1395 / 1571; with a Zipf bias 2501 / 1679 / 2006, 3089 / 1528 / 2127, 3010 / 1363 / 1622; on 300 tokens
// 923 / 1658 / 515, 1008 / 1508 / 325, 2324 / 1347 / 225.  Behind kept rows where a low rank makes their products cheap and tokens are
// neither even nor few: 9524 x 11 of 28256 x 128 878 / 765 / 863, Zipf 643 / 759 / 868, on 200 263 / 755 / 184.
TableChoice table_pays(const as_ctx *ctx, const as_model *m, int64_t rows, int32_t T, TableForm form, bool keep, bool by_sums)
{
    if (ctx->kept_rows == 3) return kTableAll;
    if (ctx->kept_rows == 5) return form == kTableRows || !rows_on_device(ctx, m) ? kNoTable : kTableDemand;
    if (ctx->kept_rows != 0) return kNoTable;
    const double V = (double)m->V, R = (double)rows, row_us = V * (ctx->dtype == AS_BF16 ? 2.0 : 4.0) / 6e6;
    const double kept = V * (1.0 - exp(-R * (T - 1) / V)) / (T - 1);
    const double own = keep ? kept : sharing_pays(ctx, m, rows, T) ? V * (1.0 - exp(-R / V)) : R;      // rows a step
    const double sampling = 3.5 + R * row_us;
    // (the first step's product has a row per prompt; half a us lies between launches)
    const double without = 5.0 + (T - 1) * product_us(ctx, m, own) +
                           T * (1.0 + (keep ? 12.0 : 0.0) + (keep && by_sums ? 4.0 + R * 0.0007 + own * row_us : sampling));
    // (rows of a table beyond the caches are read from memory, those of a step's own product where it left them)
    const double row_bytes = V * (ctx->dtype == AS_BF16 ? 2.0 : 4.0);
    const double cold = !keep && V * row_bytes > 256e6 && own * row_bytes < 256e6 ? 1.25 : 1.0;
    const double step = form == kTableRows ? sampling * cold + 0.5 : 2.0 + R * 0.0004;
    const double table = product_us(ctx, m, V) + (form == kTableRows ? 0.0 : 4.0 + V * row_us);
    // (kept rows that have no records are read in an order of the rows, where that pays)
    if (table + T * step >= (!keep ? 0.95 : form == kTableRows ? 0.85 : 0.9) * without) return kNoTable;
    const double least = 40.0 + T * (10.0 + R * 0.0006);
    if (!keep || table + (form == kTableRows ? 0.0 : T * step) < least) return kTableAll;
    return form == kTableRows ? kNoTable : kTableDemand;
}

as_status launch_share_clear(as_ctx *ctx, const RowShare &s, int32_t T)
{
    const int64_t n = ctx->V > T ? ctx->V : T;
    hipLaunchKernelGGL(share_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, ctx->stream, s, ctx->V, T);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_claim(as_ctx *ctx, const RowShare &s, int32_t step, const int32_t *prev, int64_t rows)
{
    hipLaunchKernelGGL(share_claim_kernel<false>, dim3((unsigned)((rows + 1023) / 1024)), dim3(1024), 0, ctx->stream, s, step,
                       ctx->V, prev, rows);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_share_map(as_ctx *ctx, const RowShare &s, int32_t step, const int32_t *prev, int64_t rows,
                           int32_t *row_ids, bool sorted)
{
    const dim3 blocks((unsigned)((rows + 255) / 256));
    if (!sorted) {
        hipLaunchKernelGGL((share_map_kernel<false, false>), blocks, dim3(256), 0, ctx->stream, s, step, ctx->V, prev, rows,
                           row_ids);
    } else {
        hipLaunchKernelGGL((share_map_kernel<true, false>), blocks, dim3(256), 0, ctx->stream, s, step, ctx->V, prev, rows,
                           row_ids);
        AS_HIP_TRY(ctx, hipGetLastError());
        hipLaunchKernelGGL(share_scan_kernel, dim3(1), dim3(1024), 0, ctx->stream, s, step);
        AS_HIP_TRY(ctx, hipGetLastError());
        hipLaunchKernelGGL(share_order_kernel, blocks, dim3(256), 0, ctx->stream, s, rows, row_ids);
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_share(as_ctx *ctx, const RowShare &s, int32_t step, const int32_t *prev, int64_t rows,
                       int32_t *row_ids, bool sorted)
{
    const as_status st = launch_claim(ctx, s, step, prev, rows);
    return st != AS_OK ? st : launch_share_map(ctx, s, step, prev, rows, row_ids, sorted);
}

as_status launch_claim_positions(as_ctx *ctx, const RowShare &s, const int32_t *prev, int64_t rows, int32_t *row_ids)
{
    as_status st = launch_share_clear(ctx, s, 1);
    if (st != AS_OK) return st;
    hipLaunchKernelGGL(share_claim_kernel<true>, dim3((unsigned)((rows + 1023) / 1024)), dim3(1024), 0, ctx->stream, s, 0,
                       ctx->V, prev, rows);
    AS_HIP_TRY(ctx, hipGetLastError());
    hipLaunchKernelGGL((share_map_kernel<true, true>), dim3((unsigned)((rows + 255) / 256)), dim3(256), 0, ctx->stream, s, 0,
                       ctx->V, prev, rows, row_ids);
    AS_HIP_TRY(ctx, hipGetLastError());
    hipLaunchKernelGGL(share_scan_kernel, dim3(1), dim3(1024), 0, ctx->stream, s, 0);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

as_status launch_bigram_logits(as_ctx *ctx, const as_model *m, const int32_t *prev, int64_t rows,
                               void *logits_out, int64_t ld, RowRange range)
{
    if (rows == 0) return AS_OK;
    const float alpha = (float)((double)m->scale / sqrt((double)m->d));
    if (mfma_applies(m)) {
        const size_t osz = ctx->dtype == AS_BF16 ? 2 : 4;
        const int vec_store = (reinterpret_cast<uintptr_t>(logits_out) % 16 == 0) && ((ld * osz) % 16 == 0);
        const uint16_t *Ep = (const uint16_t *)m->E, *Up = (const uint16_t *)m->Ut;
        // the persistent kernel addresses operand rows with 32-bit byte offsets and wants two K stages
        const bool persistent = ctx->gemm_shape != 1 && m->d >= 2 * PK && (int64_t)m->V * m->d * 2 < (1LL << 32) &&
                                ctx->num_cus >= 8;
        if (const int mt = range.end == nullptr ? thin_tiles(ctx, m, rows) : 0) {
            if (ctx->dtype == AS_BF16)
                launch_thin<uint16_t, false>(ctx, m, prev, rows, (uint16_t *)logits_out, ld, alpha, vec_store, mt);
            else
                launch_thin<float, false>(ctx, m, prev, rows, (float *)logits_out, ld, alpha, vec_store, mt);
        } else if (persistent) {
            const dim3 grid((unsigned)(8 * (ctx->num_cus / 8))), block(512);
            if (ctx->dtype == AS_BF16)
                launch(ctx, kKernelLogits, bigram_gemm_persistent<uint16_t>, grid, block, 0, Ep, Up, prev, rows,
                       m->V, m->d, alpha, (uint16_t *)logits_out, ld, vec_store, persistent_gm(ctx), range);
            else
                launch(ctx, kKernelLogits, bigram_gemm_persistent<float>, grid, block, 0, Ep, Up, prev, rows, m->V,
                       m->d, alpha, (float *)logits_out, ld, vec_store, persistent_gm(ctx), range);
        } else {
            // grid: 8 XCD lanes x ceil(column tiles / 8) x row tiles (see the kernel's tile mapping)
            const int64_t m_blocks = (rows + BM - 1) / BM, n_blocks = ((int64_t)m->V + BN - 1) / BN;
            const int64_t blocks = 8 * ((n_blocks + 7) / 8) * m_blocks;
            if (blocks > 0x7fffffffLL) return fail(ctx, AS_ERR_UNSUPPORTED, "logits GEMM grid too large");
            const dim3 grid((unsigned)blocks), block(256);
            if (ctx->dtype == AS_BF16)
                launch(ctx, kKernelLogits, bigram_gemm_bf16<uint16_t>, grid, block, 0, Ep, Up, prev, rows, m->V,
                       m->d, alpha, (uint16_t *)logits_out, ld, vec_store);
            else
                launch(ctx, kKernelLogits, bigram_gemm_bf16<float>, grid, block, 0, Ep, Up, prev, rows, m->V, m->d,
                       alpha, (float *)logits_out, ld, vec_store);
        }
    } else {
        if (m->wdtype == AS_BF16) {
            if (ctx->dtype == AS_BF16) launch_chain<uint16_t, uint16_t>(ctx, m, prev, rows, logits_out, ld, alpha);
            else launch_chain<uint16_t, float>(ctx, m, prev, rows, logits_out, ld, alpha);
        } else {
            if (ctx->dtype == AS_BF16) launch_chain<float, uint16_t>(ctx, m, prev, rows, logits_out, ld, alpha);
            else launch_chain<float, float>(ctx, m, prev, rows, logits_out, ld, alpha);
        }
    }
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

// The fused decode needs the persistent kernel (bf16 weights, rank a multiple of 64 and at least 128,
// operands within 4 GB, 16-byte aligned).
bool fused_path_applies(const as_ctx *ctx, const as_model *m)
{
    return m->wdtype == AS_BF16 && m->d % PK == 0 && m->d >= 2 * PK && (int64_t)m->V * m->d * 2 < (1LL << 32) &&
           reinterpret_cast<uintptr_t>(m->E) % 16 == 0 && reinterpret_cast<uintptr_t>(m->Ut) % 16 == 0 &&
           ctx->num_cus >= 8;
}

as_status launch_bigram_partials(as_ctx *ctx, const as_model *m, const int32_t *prev, int64_t rows, float temp,
                                 float2 *part, int64_t ldp, RowRange range)
{
    if (rows == 0) return AS_OK;
    const float alpha = (float)((double)m->scale / sqrt((double)m->d) * 1.44269504088896340736 / (double)temp);
    if (const int mt = range.end == nullptr ? thin_tiles(ctx, m, rows) : 0) {
        launch_thin<float, true>(ctx, m, prev, rows, reinterpret_cast<float *>(part), ldp, alpha, 0, mt);
        AS_HIP_TRY(ctx, hipGetLastError());
        return AS_OK;
    }
    const dim3 grid((unsigned)(8 * (ctx->num_cus / 8))), block(512);
    launch(ctx, kKernelLogits, bigram_gemm_persistent<float, true>, grid, block, 0, (const uint16_t *)m->E,
           (const uint16_t *)m->Ut, prev, rows, m->V, m->d, alpha, reinterpret_cast<float *>(part), ldp, 0,
           persistent_gm(ctx), range);
    AS_HIP_TRY(ctx, hipGetLastError());
    return AS_OK;
}

}  // namespace as
