"""Top-k by the wide kernel's table of candidates: rows of several tiles (as many pieces as two, three and more take, with a tail),
candidates that one wave finishes and that it does not (ties, flat rows), all of them in one wave's pieces."""
import numpy as np
import pytest

from paper_2210_15458_amd import synth

pytestmark = pytest.mark.gpu
ANY = {"thr_path": 3}
CODES = np.array([0.0, 0.2, 0.41, 0.5, 0.77, 0.99, 1 - 2.0 ** -24], np.float32)


def _rows(V):
    rng = np.random.default_rng(V)
    x = np.stack([rng.standard_normal(V) * 3.0, rng.standard_normal(V) * 0.05, np.sort(rng.standard_normal(V) * 2.0),
                  np.sort(rng.standard_normal(V) * 2.0)[::-1], rng.standard_normal(V) - 40.0, np.full(V, 1.5),
                  rng.standard_normal(V)]).astype(np.float32)
    x[6, V // 3:V // 3 + min(600, V // 2)] += 30.0           # every candidate among neighbours
    return x


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pieces,more", [(0, 3), (3, 1), (1024, 2), (4096, 1), (16384, 1), (24576, 0), (24577, 3), (57344, 1), (65537, 2)])
def test_candidate_table(pieces, more, dtype):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    V = pieces * (8 if dtype == "bf16" else 4) + more
    x = _rows(V)
    stored = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    for top_k, top_p in ((1, 1.0), (1, 0.3), (5, 0.9), (48, 1.0), (56, 0.95), (57, 0.9), (128, 0.8)):
        if top_k >= V:
            continue
        label = f"V={V} {dtype} k={top_k} p={top_p}"
        print("case", label, flush=True)
        gpu = run_gpu_step(stored, CODES, V, temp=0.9, top_k=top_k, top_p=top_p, tuning=ANY)
        ref = oracle_step(stored, CODES, V, temp=0.9, top_k=top_k, top_p=top_p)
        print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=CODES), flush=True)


# Where more than 64 stay whatever one wave leaves out, each wave goes by the number that all of them counted: k on either side of
# the line between the two ways, candidates on either side of twice as many, in blocks of 256, 512 and 1024.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pieces,rows", [(1000, 256), (2040, 600), (4000, 300), (4000, 7), (8000, 300), (12000, 7)])
def test_candidates_that_stay(pieces, rows, dtype):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    V = pieces * (8 if dtype == "bf16" else 4) + 1
    rng = np.random.default_rng(pieces)
    x = (rng.standard_normal((5, V)) * 2.0).astype(np.float32)
    for r, n in enumerate((100, 115, 130, 200, 250)):        # (so many above the rest, among them ties)
        x[r, rng.permutation(V)[:n]] = np.round(20.0 + rng.standard_normal(n) * 2.0, 1)
    stored = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    rid = (np.arange(rows) % len(x)).astype(np.int32)
    codes = synth.uniform_codes(rows, seed=pieces)
    for top_k, top_p in ((56, 0.95), (57, 0.95), (65, 1.0), (80, 0.9), (128, 1.0)):
        label = f"V={V} R={rows} {dtype} k={top_k} p={top_p}"
        print("case", label, flush=True)
        gpu = run_gpu_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid, tuning=ANY)
        ref = oracle_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid.astype(np.int64))
        print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


def _filling(V, per):
    """Rows of several tiles in which single waves meet more pieces with candidates than their tables take, between the places where
    the block counts what it has: neighbouring logits (a wave's own pieces) in every tile, as many as bring the table to a half, to its
    end and past it; a row that keeps rising; one whose last tile alone holds them."""
    rng = np.random.default_rng(V)
    tile = 8192 * per
    x = (rng.standard_normal((6, V)) * 2.0).astype(np.float32)
    for r, run in enumerate((90, 260, 700)):
        for at in range(3 * 64 * per, V - run, tile):
            x[r, at:at + run] += 25.0 + rng.standard_normal(run).astype(np.float32)
    x[3] = np.sort(x[3])
    x[4] += np.arange(V) // tile * 6.0
    x[5, V - 3000:] += 20.0
    return x


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("tiles", [3, 4, 5, 8, 9])
def test_tables_that_fill_between_tiles(tiles, dtype):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    per = 8 if dtype == "bf16" else 4
    V = tiles * 8192 * per - 5
    x = _filling(V, per)
    stored = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    rows = 300 if tiles == 3 else 12
    rid = (np.arange(rows) % len(x)).astype(np.int32)
    codes = synth.uniform_codes(rows, seed=tiles)
    for top_k, top_p in ((1, 1.0), (40, 0.9), (64, 1.0), (100, 1.0), (128, 0.9)):
        label = f"V={V} {dtype} k={top_k} p={top_p}"
        print("case", label, flush=True)
        gpu = run_gpu_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid, tuning=ANY)
        ref = oracle_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid.astype(np.int64))
        print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


# Rows that break the contract among ordinary ones, in each form of the kernel (a wave a row, 256, 512 and 1024 threads, several
# tiles): outputs stay in their range, and the other rows get what they get without these beside them.  A row without a finite
# logit gets the first token.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pieces,rows", [(500, 3200), (1000, 5200), (1000, 9), (2040, 600), (4000, 600), (4000, 300), (8000, 300),
                                         (12000, 9), (20000, 300), (20000, 9)])
def test_rows_of_nan_and_infinities(pieces, rows, dtype):
    from gpu_util import run_gpu_step
    V = pieces * (8 if dtype == "bf16" else 4) + 1
    rng = np.random.default_rng(pieces)
    nan, inf = np.float32(np.nan), np.float32(np.inf)
    x = (rng.standard_normal((9, V)) * 2.0 + 3.0).astype(np.float32)
    good = [1, 4, 8]
    x[0] = nan
    x[2, rng.integers(0, V, V // 50)] = nan
    x[3, V // 2] = inf                                       # (past the first pieces)
    x[5] = -inf
    x[6, ::2] = inf
    x[6, 1::2] = -nan
    x[7] = -inf
    x[7, V - 1] = -nan
    stored = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    rid = (np.arange(rows) % len(x)).astype(np.int32)
    codes = synth.uniform_codes(rows, seed=pieces)
    mine = np.isin(rid, good)
    for top_k, top_p in ((0, 0.9), (0, 0.999), (40, 1.0), (50, 0.9), (128, 1.0), (1000, 0.9)):
        print(f"case V={V} R={rows} {dtype} k={top_k} p={top_p}", flush=True)
        out = run_gpu_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid, tuning=ANY)
        tok, c = out["token"], out["c_next"]
        assert ((tok >= 0) & (tok < V)).all()
        assert np.isfinite(c).all() and (c >= 0.0).all() and (c <= np.float32(1.0) - np.float32(2.0 ** -24)).all()
        assert (tok[rid == 5] == 0).all()
        other = run_gpu_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=np.where(mine, rid, 8).astype(np.int32), tuning=ANY)
        for key in ("token", "c_next", "p"):
            assert np.array_equal(out[key][mine], other[key][mine]), key
