"""The truncated sampling step for rows of any length and alignment (one launch, 256 to 1024 threads a row): each
form of the kernel at the ends of its range, against the oracle with the acceptance rules of the step tests."""
import numpy as np
import pytest

from paper_2210_15458_amd import synth
from test_gpu_step import _check

pytestmark = pytest.mark.gpu
ANY = {"thr_path": 3}

# (V, rows): pieces of 16 bytes just inside and just past a form, in bf16 (8 logits a piece); with few rows and with
# more rows than compute units
FEW = [(1, 3), (5, 3), (8191, 5), (8193, 5), (32768, 4), (32769, 4), (65536, 3), (65537, 3), (131073, 3), (262145, 2)]
MANY = [(8193, 300), (16385, 300), (16385, 520), (32769, 300)]
MODES = [(0, 0.9), (1, 1.0), (40, 1.0), (128, 0.9), (129, 1.0), (300, 0.8)]


@pytest.mark.parametrize("V,rows", FEW + MANY)
def test_forms_bf16(V, rows):
    for top_k, top_p in MODES[:3] if rows >= 300 else MODES:
        if top_k < V:
            _check(V, rows, "bf16", temp=0.9, top_k=top_k, top_p=top_p, seed=V, tuning=ANY)


@pytest.mark.parametrize("V,rows", [(max(1, v // 2), r) for v, r in FEW] + [(v // 2, r) for v, r in MANY])
def test_forms_f32(V, rows):
    for top_k, top_p in MODES[:3] if rows >= 300 else MODES:
        if top_k < V:
            _check(V, rows, "f32", temp=0.9, top_k=top_k, top_p=top_p, seed=V + 1, tuning=ANY)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("sigma,temp", [(0.01, 1.0), (0.5, 1.0), (30.0, 0.3)])
def test_flat_and_peaked_rows(sigma, temp, dtype):
    # ties and near-ties by the thousand, and rows whose logits lie far beyond the histogram
    for V in (3001, 40001, 140001):
        for top_k, top_p in ((0, 0.95), (50, 0.9), (200, 1.0)):
            _check(V, 4, dtype, temp=temp, sigma=sigma, top_k=top_k, top_p=top_p, seed=21, tuning=ANY)


def test_special_rows():
    from gpu_util import compare_step, oracle_step, run_gpu_step
    from paper_2210_15458_amd import synth
    V = 9001
    x = synth.gaussian_logits(6, V, seed=31, dtype="f32").copy()
    x[0, :] = -np.inf; x[0, 4321] = 0.5              # one-hot: fewer kept than k
    x[1, :] = 0.0                                    # uniform: every logit tied
    x[2, ::2] = -np.inf
    x[3, :] = -80.0; x[3, V - 1] = 80.0              # the row's largest logit far above the first pieces'
    x[4, 5000:] += 40.0
    x[5, :] = -0.0; x[5, ::3] = 0.0                  # one value in two spellings
    codes = np.array([0.4, 0.7, 1 - 2.0 ** -24, 0.3, 0.0, 0.999], np.float32)
    for top_k, top_p in ((0, 0.9), (7, 1.0), (40, 0.9), (200, 0.9), (8000, 1.0)):
        for dtype in ("f32", "bf16"):
            stored = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
            gpu = run_gpu_step(stored, codes, V, top_k=top_k, top_p=top_p, tuning=ANY)
            ref = oracle_step(stored, codes, V, top_k=top_k, top_p=top_p)
            compare_step(gpu, ref, V, f"special {dtype} k={top_k} p={top_p}", trunc=True, codes=codes)


# The forms that are taken with more rows than compute units, by the pieces of 16 bytes of a row: 256 threads x 8 and
# x 16, 512 x 4, x 8 and x 16, 512 and 1024 tile by tile (143296 pieces: the longest row that 512 threads take)
LOTS_OF_ROWS = [(1025, 520), (2048, 520), (2049, 520), (4096, 520), (1025, 300), (2048, 300), (2049, 300), (4096, 300),
                (4097, 300), (8192, 300), (8193, 300), (20000, 300)]


def _check_shared(V, rows, dtype, top_k, top_p, tuning):
    """_check with a few rows of logits for many codes."""
    from gpu_util import compare_step, oracle_step, run_gpu_step
    held = 3
    stored = synth.gaussian_logits(held, V, seed=V, dtype=dtype)
    rid = (np.arange(rows) % held).astype(np.int32)
    codes = synth.uniform_codes(rows, seed=rows)
    label = f"V={V} R={rows} {dtype} k={top_k} p={top_p}"
    print("case", label, flush=True)
    gpu = run_gpu_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid, tuning=tuning)
    ref = oracle_step(stored, codes, V, temp=0.9, top_k=top_k, top_p=top_p, row_ids=rid.astype(np.int64))
    print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("pieces,rows", LOTS_OF_ROWS)
def test_forms_for_many_rows(pieces, rows, dtype):
    V = pieces * (8 if dtype == "bf16" else 4)
    for top_k, top_p in ((0, 0.9), (40, 1.0), (128, 0.9), (300, 0.8)):
        _check_shared(V, rows, dtype, top_k, top_p, ANY)
    _check_shared(V - 1, rows, dtype, 0, 0.9, None)       # (rows that start off 16 bytes; the library's own choice)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("more", [0, 1])
def test_longest_rows_of_512_threads(more, dtype):
    _check_shared(143296 * (8 if dtype == "bf16" else 4) + more, 260, dtype, 0, 0.9, None)


@pytest.mark.parametrize("V,dtype", [(65537, "bf16"), (100000, "bf16"), (32769, "f32"), (50257, "f32")])
def test_streamed_kernel(V, dtype):
    # what is left to it: k above 128 on rows of more than 128 KB, more rows than compute units
    for top_k, top_p in ((129, 1.0), (300, 0.8), (5000, 0.95)):
        _check_shared(V, 300, dtype, top_k, top_p, None)


# the forms for many short rows (more than four a compute unit: less LDS and fewer registers a block), at their ends
@pytest.mark.parametrize("V,dtype", [(9, "bf16"), (1281, "bf16"), (8185, "bf16"), (8199, "bf16"), (16370, "bf16"), (5, "f32"),
                                     (4090, "f32"), (4103, "f32"), (8180, "f32")])
@pytest.mark.parametrize("sigma", [0.05, 3.0])
def test_many_short_rows(V, dtype, sigma):
    for top_k, top_p in MODES:
        if top_k < V:
            _check(V, 1030, dtype, temp=0.9, sigma=sigma, top_k=top_k, top_p=top_p, seed=V, tuning=ANY)


# the one-tile top-k kernel's line: ranks it takes and the next, on rows of one to four waves' worth of logits
@pytest.mark.parametrize("V,k", [(400, 30), (400, 31), (8000, 33), (8000, 34), (9600, 37), (9600, 38), (16384, 41), (16384, 42),
                                 (32128, 47), (32128, 48)])
def test_one_tile_top_k_at_its_line(V, k):
    for top_p in (1.0, 0.9):
        _check(V, 70, "bf16", temp=0.9, top_k=k, top_p=top_p, seed=V + k)


# the forms of a wave a row (as many rows as make them worth it), at their ends: 512 and 1024 pieces of 16 bytes
@pytest.mark.parametrize("V,rows,dtype", [(3, 3100, "bf16"), (700, 3100, "bf16"), (4089, 3100, "bf16"), (4096, 3100, "bf16"),
                                          (4097, 5200, "bf16"), (8186, 5200, "bf16"), (2, 3100, "f32"), (2047, 3100, "f32"),
                                          (2050, 5200, "f32"), (4093, 5200, "f32")])
@pytest.mark.parametrize("sigma,temp", [(0.05, 1.0), (3.0, 0.9), (9.0, 0.4)])
def test_a_wave_a_row(V, rows, dtype, sigma, temp):
    # k at the ends of its candidate table and of the counts; flat rows overflow both lists
    from gpu_util import compare_step, oracle_step, run_gpu_step
    held = 37                                             # rows of logits for many codes
    stored = synth.gaussian_logits(held, V, sigma=sigma, seed=V + rows, dtype=dtype)
    rid = (np.arange(rows) % held).astype(np.int32)
    codes = synth.uniform_codes(rows, seed=rows + V)
    for top_k, top_p in ((0, 0.9), (1, 1.0), (40, 0.8), (41, 1.0), (41, 0.9), (128, 1.0), (600, 1.0), (600, 0.7)):
        if top_k >= V:
            continue
        label = f"V={V} R={rows} {dtype} sigma={sigma} k={top_k} p={top_p}"
        print("case", label, flush=True)
        gpu = run_gpu_step(stored, codes, V, temp=temp, top_k=top_k, top_p=top_p, row_ids=rid, tuning=ANY)
        ref = oracle_step(stored, codes, V, temp=temp, top_k=top_k, top_p=top_p, row_ids=rid.astype(np.int64))
        print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


# rows of up to 128 pieces, whose candidates are bounded by halves of them, and the first above; windows and bins with more logits
# than a wave's list
@pytest.mark.parametrize("V,rows,dtype,sigma", [(1016, 3100, "bf16", 3.0), (1024, 3100, "bf16", 0.3), (1033, 3100, "bf16", 3.0),
                                                (505, 3100, "f32", 3.0), (512, 3100, "f32", 0.3), (520, 3100, "f32", 3.0),
                                                (4090, 3100, "bf16", 0.3), (8186, 5200, "bf16", 0.3), (4093, 5200, "f32", 0.2)])
def test_a_wave_on_flat_and_on_short_rows(V, rows, dtype, sigma):
    test_a_wave_a_row(V, rows, dtype, sigma, 0.9)


# short rows, few of them: the largest k of the candidate table and the first that is counted, on either side of the lengths at
# which that line moves
@pytest.mark.parametrize("V,dtype,ks", [(4103, "bf16", (48, 49)), (4104, "bf16", (64, 65)), (2051, "f32", (48, 49)),
                                        (2052, "f32", (64, 65)), (8200, "bf16", (96, 97)), (16383, "f32", (96, 97))])
def test_candidates_or_counts(V, dtype, ks):
    for k in ks:
        _check(V, 6, dtype, temp=0.9, top_k=k, seed=V + k, tuning=ANY)
