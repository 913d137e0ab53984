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
// token, a vocabulary of at most four times the rows of one step, and a table of more rows than those within kKeptBytes.
// (By the vocabulary, not by the rows that the decode's steps can come to: a larger one would be within the bound for
// three or four steps and beyond it for more, so that a shorter decode took more than a longer one.)
inline int64_t kept_rows_most(int64_t V, int64_t rows, int64_t T, int64_t row_bytes)
{
    if (T < 3 || V > 4 * rows || (V > rows && V * row_bytes > kKeptBytes)) return 0;
    return smaller(V, rows * T);
}

// What a decode reserves: logits (or group masses), a row of them per row, which every form can do with, or a table
// that is preferred where it can be had; and the state: codes, tokens, flags, the tables of shared rows in any form, and
// the sums of kept rows.  A decode of logits leaves room for one of group masses of its size.
struct DecodeSizes {
    size_t needed, preferred, state;         // bytes
};
inline DecodeSizes decode_sizes(int64_t V, int64_t esz, int64_t rows, int64_t T, bool masses)
{
    const int64_t lb = logits_row_bytes(V, esz), mb = mass_row_bytes(V);
    const int64_t kept = masses ? 0 : kept_rows_most(V, rows, T, lb), kept_masses = kept_rows_most(V, rows, T, mb);
    DecodeSizes z;
    z.needed = (size_t)(rows * larger(masses ? 0 : lb, mb));
    z.preferred = (size_t)larger((int64_t)z.needed, larger(kept * lb, kept_masses * mb));
    const int64_t sums = one_tile_row(V, esz) ? kept * kRowSums : 0;
    // (codes, prev, order, token of rows that are not kept; mark, slot, fill, or token of rows that are)
    z.state = (size_t)((sums + 4 * rows + 4 * V + T + 1) * 4 + rows);
    return z;
}

}  // namespace as
#endif
