"""The truncated sampling step for rows of any length and alignment (one launch, 256 to 1024 threads a row): each
form of the kernel at the ends of its range, against the oracle with the acceptance rules of the step tests."""
import numpy as np
import pytest

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
