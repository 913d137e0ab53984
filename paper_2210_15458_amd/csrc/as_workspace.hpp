// How much of a context's workspace a call takes: plain arithmetic on sizes, with nothing of HIP in it (the tests compile
// this file for the host and go through its ranges).
//
// A call reserves by its rows and steps, the vocabulary and the storage type alone, whatever its temperature, truncation
// and model, and never less for more rows or more steps.  So a call of the same or a smaller size than an earlier one
// finds its workspace in whichever form it takes: it allocates nothing, can be captured, and leaves alone the buffers
// that a graph captured earlier works on.
#ifndef AS_WORKSPACE_HPP
#define AS_WORKSPACE_HPP

#include <stddef.h>
#include <stdint.h>

namespace as {

constexpr int kRowSums = 68;                 // floats that row_sums_kernel leaves per row: 64 chunk sums, 4 references
constexpr int64_t kKeptBytes = 4LL << 30;    // largest table of kept rows that has more rows than a step
constexpr int64_t kTileVecs = 4096;          // 16-byte vectors of a row of one tile

inline int64_t larger(int64_t a, int64_t b) { return a > b ? a : b; }
inline int64_t smaller(int64_t a, int64_t b) { return a < b ? a : b; }

// a row of logits (starting on 16 bytes), a row of group masses (float2, 16 at a time)
inline int64_t logits_row_bytes(int64_t V, int64_t esz) { return (V + 7) / 8 * 8 * esz; }
inline int64_t mass_row_bytes(int64_t V) { return ((V + 31) / 32 + 15) / 16 * 16 * 8; }

// rows of whole vectors that fit one tile: their sums can be made once and kept
inline bool one_tile_row(int64_t V, int64_t esz) { return V * esz % 16 == 0 && V * esz / 16 <= kTileVecs; }

// The rows that a decode's table of kept logits rows can come to, or 0 where none is kept: steps enough to come back to a
// token, at most four times the rows of one step, and a table of more rows than those within kKeptBytes.  The bound by the
// vocabulary alone holds for any number of steps (kept_rows_most); a larger vocabulary meets it over three or four steps
// only (kept_rows_few), so that a decode of those would take more than a longer one: it may grow the workspace only where
// no earlier call was of its size or larger (RowsSeen).
inline int64_t kept_rows_most(int64_t V, int64_t rows, int64_t T, int64_t row_bytes)
{
    if (T < 3 || V > 4 * rows || (V > rows && V * row_bytes > kKeptBytes)) return 0;
    return smaller(V, rows * T);
}
inline int64_t kept_rows_few(int64_t V, int64_t rows, int64_t T, int64_t row_bytes)
{
    return T >= 3 && T <= 4 && V > 4 * rows && rows * T * row_bytes <= kKeptBytes ? rows * T : 0;
}

// The rows of a table of every token's logits row, made before the first step, or 0 where no decode of the size wants one:
// a row for each of V tokens against T steps of `rows` rows and of the launches that a table spares, which cost what
// 6e6 / V rows cost (6 us at a rank of 512), within kKeptBytes.  A call is not to take memory out of proportion to what it
// works on: a table beyond kTableBytes has at most 128 times the decode's own rows.  (16 codes over many steps of 32128, which
// are out by that, would have 2 GB for 1 MB, and be faster from 260 steps on: 512 steps 2.1 ms, 5.1 a row per code.)  The
// rank is not known here; of sizes spread over 500 to 64000 tokens, 1 to 2000 codes, 4 to 512 steps and ranks of 128 to
// 1024, 3 % reserve a table that is then not made, 112 MiB of it on average.  (Whether one is made: table_pays.)
constexpr int64_t kTableRecord = 1056;       // bytes that a step reads of a row before its logits: RowRecord, CandRecord
constexpr int64_t kTableBytes = 512LL << 20;
inline int64_t table_rows(int64_t V, int64_t rows, int64_t T, int64_t row_bytes)
{
    if (T < 4 || V * row_bytes > kKeptBytes || (V > 128 * rows && V * row_bytes > kTableBytes)) return 0;
    return (double)T * ((double)rows + 6e6 / (double)V) >= 1.25 * (double)V ? V : 0;
}

// Most rows of the calls made so far that had three steps and more, four and more.
struct RowsSeen {
    int64_t three = 0, four = 0;
    bool covers(int64_t rows, int64_t T) const { return rows <= (T >= 4 ? four : three); }      // for T of three or four
    void add(int64_t rows, int64_t T)
    {
        if (T >= 3) three = larger(three, rows);
        if (T >= 4) four = larger(four, rows);
    }
};

// Rows of an encode's logits computed at a time.  The product wants many (us an encode by rows a chunk 256 / 512 / 1024 /
// 2048 / 3072 / 4096 / 8192: 65536 positions of 32128 bf16, d = 512 3013 / 1942 / 1564 / 1344 / 1366 / 1268 / 1228; 38985
// of 153375, d = 896 17213 / 12969 / 12043 / 11419 / 12370 / 11364 / 11350; 15457 of 4597, d = 960 701 / 407 / 258 / 199 /
// 208 / 182 / 177), in whole sets of 8 row tiles (3072 is not); whether they stay in the caches hardly matters, so
// memory draws the line.
inline int64_t encode_chunk(int64_t row_bytes)
{
    if (8192 * row_bytes <= 256LL << 20) return 8192;
    if (4096 * row_bytes <= 256LL << 20) return 4096;
    if (2048 * row_bytes <= 768LL << 20) return 2048;
    return 1024 * row_bytes <= 1024LL << 20 ? 1024 : 256;
}

// Its positions are taken a window of columns at a time, which bounds the tables: at most so many, or one column.
constexpr int64_t kEncodePositions = 1LL << 19;
inline int64_t encode_window(int64_t rows, int64_t T) { return larger(1, smaller(T, kEncodePositions / rows)); }
inline int64_t encode_positions_most(int64_t rows, int64_t T)
{
    return smaller(rows * larger(T, 1), larger(rows, kEncodePositions));
}

// The tables of a window: offsets in bytes, and what they take.  `positions` in it, `most_rows` logits rows for them,
// `chunk` of these at a time; cond, mark and claim only where tokens share logits rows (`claimed`), sums only for rows that
// have them.
struct EncodeTables {
    size_t f_lo, p, sums, thr, slot, order, token, ends, idle, ended, cond, mark, claim, count, chunks, bytes;
};
inline EncodeTables encode_tables(int64_t V, int64_t esz, int64_t rows, int64_t positions, int64_t most_rows, int64_t chunk,
                                  bool claimed)
{
    EncodeTables t;
    size_t end = 0;
    auto part = [&](int64_t n) { const size_t at = end; end += (size_t)((n + 15) / 16 * 16); return at; };
    t.f_lo = part(positions * 8); t.p = part(positions * 8);
    t.sums = part(one_tile_row(V, esz) ? chunk * kRowSums * 4 : 0); t.thr = part(chunk * 4);
    t.slot = part(positions * 4); t.order = part(positions * 4);
    t.token = part(most_rows * 4); t.ends = part(most_rows * 4); t.idle = part(most_rows); t.ended = part(rows);
    t.cond = part(claimed ? positions * 4 : 0); t.mark = part(claimed ? V * 4 : 0); t.claim = part(claimed ? V * 4 : 0);
    t.count = part(4); t.chunks = part((most_rows + chunk - 1) / chunk * 4);
    t.bytes = end;
    return t;
}

// What a decode reserves: logits (or group masses), a row of them per row, which every form can do with, or a table
// that is preferred where it can be had (of kept rows, or of every token's); and the state: codes, tokens, flags, the
// tables of shared rows in any form, and the sums of kept rows, or with the records of a table of every token's rows, which is
// done without where they cannot be had.  A decode of logits leaves room for one of group masses of its size, and for an
// encode of its size a column and kPlainChunk rows at a time.
constexpr int64_t kPlainChunk = 1024;
struct DecodeSizes {
    size_t needed, kept, preferred;          // bytes of logits
    size_t state, state_preferred;
};
// The state of a decode from a table: codes, prev twice (or the steps done), the table's tokens, flags; with records, those,
// and what rows on demand take: a row and a mark per token, and the rounds' numbers.
inline size_t table_state(int64_t V, int64_t rows, bool with_records)
{
    return (size_t)((with_records ? V * kTableRecord + (2 * V + 48) * 4 : 0) + (3 * rows + V) * 4 + rows);
}
inline DecodeSizes decode_sizes(int64_t V, int64_t esz, int64_t rows, int64_t T, bool masses)
{
    const int64_t lb = logits_row_bytes(V, esz), mb = mass_row_bytes(V);
    const int64_t kept = masses ? 0 : kept_rows_most(V, rows, T, lb), kept_masses = kept_rows_most(V, rows, T, mb);
    DecodeSizes z;
    z.needed = (size_t)(rows * larger(masses ? 0 : lb, mb));
    const int64_t table = masses ? 0 : table_rows(V, rows, T, lb), table_masses = table_rows(V, rows, T, mb);
    z.kept = (size_t)larger((int64_t)z.needed, larger(kept * lb, kept_masses * mb));
    z.preferred = (size_t)larger((int64_t)z.kept, larger(table * lb, table_masses * mb));
    const int64_t sums = one_tile_row(V, esz) && T >= 3 ? smaller(V, rows * (V > 4 * rows ? smaller(T, 4) : T)) * kRowSums : 0;
    // (codes, prev, order, token of rows that are not kept; mark, slot, fill, or token of rows that are)
    const size_t steps = (size_t)((sums + 4 * rows + 4 * V + T + 1) * 4 + rows);
    const size_t column = encode_tables(V, esz, rows, rows, rows, smaller(rows, kPlainChunk), false).bytes;
    z.state = steps > column ? steps : column;
    const size_t whole = table > 0 ? table_state(V, rows, one_tile_row(V, esz)) : 0;
    z.state_preferred = whole > z.state ? whole : z.state;
    return z;
}

// What an encode asks for, in a workspace of its own: the logits of a chunk, and the tables of a window in any form (37
// bytes a position, 276 a logits row of the chunk, 8 a token of the vocabulary, 1 a sequence).
struct EncodeSizes {
    size_t logits, state;                    // bytes
};
inline EncodeSizes encode_sizes(int64_t V, int64_t esz, int64_t rows, int64_t T)
{
    const int64_t most = encode_positions_most(rows, T), chunk = smaller(encode_chunk(logits_row_bytes(V, esz)), most);
    return EncodeSizes{(size_t)(T > 0 ? chunk * logits_row_bytes(V, esz) : 0),
                       encode_tables(V, esz, rows, most, most, chunk, true).bytes};
}

}  // namespace as
#endif
