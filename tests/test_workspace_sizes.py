"""The arithmetic by which calls reserve workspace (csrc/as_workspace.hpp, compiled here for the host): never less for more
rows or steps, and enough for every form that a call can take."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "as_workspace.hpp"
using namespace as;
extern "C" {
void sizes(int64_t V, int64_t esz, int64_t rows, int64_t T, int masses, int64_t *out)
{
    const DecodeSizes z = decode_sizes(V, esz, rows, T, masses != 0);
    out[0] = (int64_t)z.needed; out[1] = (int64_t)z.kept; out[2] = (int64_t)z.preferred; out[3] = (int64_t)z.state;
    out[4] = (int64_t)z.state_preferred;
}
int64_t table(int64_t V, int64_t rows, int64_t T, int64_t row_bytes) { return table_rows(V, rows, T, row_bytes); }
int64_t record() { return kTableRecord; }
void encode(int64_t V, int64_t esz, int64_t rows, int64_t T, int64_t *out)
{
    const EncodeSizes z = encode_sizes(V, esz, rows, T);
    out[0] = (int64_t)z.logits; out[1] = (int64_t)z.state;
}
int64_t tables(int64_t V, int64_t esz, int64_t rows, int64_t positions, int64_t most_rows, int64_t chunk, int claimed)
{
    return (int64_t)encode_tables(V, esz, rows, positions, most_rows, chunk, claimed != 0).bytes;
}
int64_t chunk(int64_t rb) { return encode_chunk(rb); }
int64_t window(int64_t rows, int64_t T) { return encode_window(rows, T); }
int64_t kept(int64_t V, int64_t rows, int64_t T, int64_t row_bytes) { return kept_rows_most(V, rows, T, row_bytes); }
int64_t few(int64_t V, int64_t rows, int64_t T, int64_t row_bytes) { return kept_rows_few(V, rows, T, row_bytes); }
static RowsSeen seen;
void forget() { seen = RowsSeen{}; }
void add(int64_t rows, int64_t T) { seen.add(rows, T); }
int covers(int64_t rows, int64_t T) { return seen.covers(rows, T); }
int64_t row_bytes(int64_t V, int64_t esz, int masses) { return masses ? mass_row_bytes(V) : logits_row_bytes(V, esz); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("sizes")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared", "-I",
                    os.path.join(ROOT, "paper_2210_15458_amd", "csrc"), str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    L = ctypes.CDLL(str(d / "shim.so"))
    i64 = ctypes.c_int64
    L.sizes.argtypes = [i64, i64, i64, i64, ctypes.c_int, ctypes.POINTER(i64)]
    L.encode.argtypes = [i64, i64, i64, i64, ctypes.POINTER(i64)]
    L.tables.argtypes, L.tables.restype = [i64] * 6 + [ctypes.c_int], i64
    L.chunk.argtypes, L.chunk.restype = [i64], i64
    L.window.argtypes, L.window.restype = [i64] * 2, i64
    L.kept.argtypes, L.kept.restype = [i64] * 4, i64
    L.few.argtypes, L.few.restype = [i64] * 4, i64
    L.table.argtypes, L.table.restype = [i64] * 4, i64
    L.record.restype = i64
    L.add.argtypes, L.add.restype = [i64] * 2, None
    L.covers.argtypes = [i64] * 2
    L.row_bytes.argtypes, L.row_bytes.restype = [i64, i64, ctypes.c_int], i64
    return L


def _sizes(lib, V, esz, rows, T, masses=False):
    out = (ctypes.c_int64 * 5)()
    lib.sizes(V, esz, rows, T, int(masses), out)
    return dict(zip(("needed", "kept", "preferred", "state", "state_preferred"), out))


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _pairs(n=20000):
    """A size, and one of no more rows and no more steps (often of the same), over all vocabularies."""
    rng = random.Random(5)
    for _ in range(n):
        V, esz = _log(rng, 1, 1 << 21), rng.choice([2, 4])
        rows, T = _log(rng, 1, rng.choice([64, 4096, 1 << 20])), rng.choice([0, 1, 2, 3, 4, 5, 6, 16, 64, 1000])
        if rng.random() < 0.5:                               # near the lines that the vocabulary draws
            rows = max(1, round(V * rng.choice([0.125, 0.25, 0.3, 0.5, 1.0, 2.0])) + rng.randint(-3, 3))
        yield (V, esz, rows, T), (V, esz, rows if rng.random() < 0.4 else rng.randint(1, rows),
                                  T if rng.random() < 0.3 else rng.randint(0, T))


def test_a_smaller_decode_finds_the_workspace_of_a_larger_one(lib):
    for large, small in _pairs():
        a, b = _sizes(lib, *large), _sizes(lib, *small)
        assert all(b[k] <= a[k] for k in a), (large, small)
        # group masses after logits of the same size
        c = _sizes(lib, *small, masses=True)
        assert all(c[k] <= a[k] for k in a), (large, small)


def test_what_a_decode_reserves_holds_every_form_of_it(lib):
    rng = random.Random(6)
    kept_at_all = tables = 0
    for (V, esz, R, T), _ in _pairs():
        N = rng.choice([1, 2, 3, R])
        B = max(1, R // N)
        R = B * N
        for masses in (False, True):
            z, rb = _sizes(lib, V, esz, R, T, masses), lib.row_bytes(V, esz, int(masses))
            assert z["needed"] >= R * rb and z["preferred"] >= z["needed"]
            forms = [2 * R, 2 * R + R + R + 2 * V + V + T + 1]                # own rows; rows shared in a step
            most, few = lib.kept(V, R, T, rb), lib.few(V, R, T, rb)
            assert most == 0 or few == 0
            if most or few:
                K = min(V, R * (T - 1) + B)
                kept_at_all += 1
                assert K <= max(most, few) and (K <= R or K * rb <= 4 << 30) and K <= 4 * R
                assert few or z["preferred"] >= K * rb
                by_sums = 68 * K if not masses and V * esz % 16 == 0 and V * esz <= 65536 else 0
                forms += [2 * R + R + K + 2 * V + K + T + 1 + by_sums]
            assert z["state"] >= max(forms) * 4 + R, (V, esz, R, T, masses)
            # a table of every token's rows: records where rows are of one tile, codes, prev twice, the tokens, flags; or rows
            # on demand: records, codes, prev, steps, tokens, rows, marks, 48 numbers, flags.  No state that a decode has to have holds its records
            assert z["preferred"] >= z["kept"] >= z["needed"] and z["state_preferred"] >= z["state"]
            if not lib.table(V, R, T, rb):
                assert z["preferred"] <= max(z["kept"], V * lib.row_bytes(V, esz, 1) if lib.table(V, R, T, lib.row_bytes(V, esz, 1)) else 0)
            else:
                tables += 1
                records = V * lib.record() if not masses and V * esz % 16 == 0 and V * esz <= 65536 else 0
                assert V * rb <= 4 << 30 and z["preferred"] >= V * rb and (V <= 128 * R or V * rb <= 512 << 20)
                # what the header says
                assert T >= 4 and T * (R + 6e6 / V) >= 1.25 * V and records + (3 * R + 3 * V) * 4 + R <= 1068 * V + 13 * R
                assert z["state_preferred"] >= records + (3 * R + (3 * V + 48 if records else V)) * 4 + R
            assert z["state"] <= max((68 * min(V, 4 * R) + 4 * R + 4 * V + T + 1) * 4 + R, lib.tables(V, esz, R, R, R, min(R, 1024), 0))
            # ... and an encode of its size, a column at a time
            assert z["state"] >= lib.tables(V, esz, R, R, R, min(R, 1024), 0)
    assert kept_at_all > 1000 and tables > 1000


def test_sizes_that_a_shorter_decode_once_took_more_for(lib):
    # 65536 codes of 32128 keep 32128 rows over 16 steps and have a row each over 2; 8000 codes
    for V, esz, rows, long, short in ((32128, 2, 65536, 16, 2), (32128, 2, 8000, 16, 4), (2000, 2, 8192, 8, 8)):
        assert _sizes(lib, V, esz, rows, short)["preferred"] <= _sizes(lib, V, esz, rows, long)["preferred"]
    assert _sizes(lib, 32128, 2, 65536, 16)["needed"] == 65536 * 64256
    assert _sizes(lib, 32128, 2, 8000, 4)["preferred"] == 8000 * 64256       # (V > 4 x 8000)


def test_few_codes_take_no_table_out_of_proportion(lib):
    for steps in (64, 256, 1024, 1 << 20):
        for rows in (1, 16, 250):
            z = _sizes(lib, 32128, 2, rows, steps)                           # (a table: 2 GB and 34 MB)
            assert z["preferred"] == rows * 64256 or z["preferred"] <= 512 << 20, (rows, steps)
            assert z["state_preferred"] == z["state"] <= 8 << 20
    assert _sizes(lib, 32128, 2, 1024, 64)["preferred"] == 32128 * 64256     # (31 times the codes)
    assert _sizes(lib, 16000, 2, 1, 64)["preferred"] == 16000 * 32000        # (488 MiB)


def test_a_table_over_few_steps_is_made_by_first_calls_only(lib):
    rng = random.Random(7)
    for _ in range(200):
        lib.forget()
        calls = []
        for _ in range(30):
            rows, T = rng.randint(1, 40), rng.choice([0, 1, 2, 3, 4, 5, 9])
            if T in (3, 4):
                assert bool(lib.covers(rows, T)) == any(r >= rows and t >= T for r, t in calls)
            lib.add(rows, T)
            calls.append((rows, T))


def _encode(lib, V, esz, rows, T):
    out = (ctypes.c_int64 * 2)()
    lib.encode(V, esz, rows, T, out)
    return dict(zip(("logits", "state"), out))


def test_a_smaller_encode_finds_the_workspace_of_a_larger_one(lib):
    for large, small in _pairs():
        a, b = _encode(lib, *large), _encode(lib, *small)
        assert all(b[k] <= a[k] for k in a), (large, small)
    # 100 sequences of 2000 tokens: fewer columns take a row per position instead of one per token; a window of two columns
    for V, long, short in ((2000, (100, 300), (100, 200)), (1000, (300000, 8), (200000, 8))):
        a, b = _encode(lib, V, 2, *long), _encode(lib, V, 2, *short)
        assert all(b[k] <= a[k] for k in a)


def test_what_an_encode_reserves_holds_every_form_of_it(lib):
    for (V, esz, rows, T), _ in _pairs(4000):
        if T == 0:
            continue
        z, rb = _encode(lib, V, esz, rows, T), lib.row_bytes(V, esz, 0)
        window = lib.window(rows, T)
        assert 1 <= window <= T
        positions = rows * window
        for claimed, most in ((0, positions), (1, min(V, positions))):
            chunk = min(lib.chunk(rb), most)
            assert z["logits"] >= chunk * rb
            assert z["state"] >= lib.tables(V, esz, rows, positions, most, chunk, claimed)
        # what the header says
        chunk = min(lib.chunk(rb), positions)
        assert z["state"] <= 37 * rows * T + 276 * chunk + 8 * V + rows + 4 * (rows * T // chunk + 1) + 15 * 16
        assert rows > 1 << 19 or z["state"] <= (37 << 19) + 276 * 8192 + 8 * V + rows + (4 << 19) // chunk + 4 + 15 * 16
