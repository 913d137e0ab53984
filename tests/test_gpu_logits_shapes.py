"""GPU parity of the logits kernels at the edges of their tiles: against fp64, and a row's logits must not depend on
which other rows are computed with it (every kernel that can take a row runs the same products in the same order)."""
import math

import numpy as np
import pytest

from paper_2210_15458_amd import synth

pytestmark = pytest.mark.gpu

# (V, d, weights, logits, R): the fp32 kernel around tiles of 64 (one short, exact, one over, in each
# direction) and K steps of 32 and 64, many rows
_VEC = [(63, 7, "f32", "f32", 1), (64, 32, "f32", "f32", 64), (65, 33, "f32", "bf16", 65), (1001, 130, "f32", "f32", 3),
        (700, 72, "bf16", "f32", 100), (333, 257, "bf16", "bf16", 129), (16500, 40, "f32", "f32", 520),
        (8200, 31, "f32", "bf16", 1030)]

# the MFMA kernels: the one for few rows at its tiles of 32 rows and 128 columns, one K stage to five (its ring holds
# four), and one row more than it takes
_THIN = [(127, 64, "bf16", "bf16", 1), (129, 64, "bf16", "f32", 32), (128, 128, "bf16", "bf16", 33),
         (1000, 192, "bf16", "f32", 64), (257, 256, "bf16", "bf16", 65), (4099, 320, "bf16", "bf16", 128),
         (300, 64, "bf16", "f32", 129), (300, 576, "bf16", "bf16", 17)]


def _logits(model, prev, V, ldt, rows):
    import torch
    from paper_2210_15458_amd import binding as B
    from gpu_util import from_dev_logits
    ctx = B.Ctx(rows, V, torch.float32 if ldt == "f32" else torch.bfloat16)
    ld = (V + 7) // 8 * 8 + 8
    out = torch.full((rows, ld), 7.0, dtype=ctx.torch_dtype, device="cuda")
    B.as_bigram_logits(ctx, model, torch.from_numpy(prev).cuda(), out)
    torch.cuda.synchronize()
    ctx.close()
    got = from_dev_logits(out)
    got = got if ldt == "f32" else synth.bf16_bits_to_f32(got)
    assert np.all(got[:, V:] == 7.0)                    # padding columns untouched
    return got[:, :V]


@pytest.mark.parametrize("V,d,wdt,ldt,R", _VEC + _THIN)
def test_logits_tile_edges(V, d, wdt, ldt, R):
    import torch
    from paper_2210_15458_amd import binding as B
    from gpu_util import to_dev_logits
    E, U = synth.bigram_weights(V, d, seed=V + d, dtype=wdt)
    model = B.Model(to_dev_logits(E), to_dev_logits(U), scale=3.0)
    prev = np.random.default_rng(R).integers(0, V, R).astype(np.int32)
    got = _logits(model, prev, V, ldt, R)
    Ew = (synth.bf16_bits_to_f32(E) if wdt == "bf16" else E).astype(np.float64)[prev]
    Uw = (synth.bf16_bits_to_f32(U) if wdt == "bf16" else U).astype(np.float64)
    ref = (Ew @ Uw) * (3.0 / math.sqrt(d))
    # fp32 accumulation of d terms (each sum rounds by at most half an ulp of the sum of magnitudes), then one
    # rounding to the storage type
    tol = 4 * d * 2.0 ** -24 * (np.abs(Ew) @ np.abs(Uw)) * (3.0 / math.sqrt(d)) + 1e-30
    if ldt == "bf16":
        tol = tol + np.abs(ref) * 2.0 ** -8
    err = np.abs(got - ref)
    assert np.all(err <= tol), float((err / tol).max())
    for r in {0, R // 2, R - 1}:
        assert np.array_equal(_logits(model, prev[r:r + 1], V, ldt, 1)[0], got[r])
    model.close()


@pytest.mark.parametrize("V,d,R", [(127, 128, 1), (1000, 192, 33), (4099, 320, 65), (33001, 128, 64)])
def test_group_masses_of_few_rows(V, d, R):
    # the few-rows kernel against the persistent one: the same bits
    import torch
    from paper_2210_15458_amd import binding as B
    from gpu_util import to_dev_logits
    E, U = synth.bigram_weights(V, d, seed=V + d, dtype="bf16")
    model = B.Model(to_dev_logits(E), to_dev_logits(U), scale=3.0)
    prev = torch.from_numpy(np.random.default_rng(R).integers(0, V, R).astype(np.int32)).cuda()
    ldp = (-(-V // 32) + 15) // 16 * 16
    res = []
    for shape in (0, 2):
        ctx = B.Ctx(R, V, torch.bfloat16)
        ctx.set_tuning("gemm_shape", shape)
        mass = torch.zeros((R, ldp, 2), dtype=torch.float32, device="cuda")
        B.as_bigram_group_mass(ctx, model, prev, 0.8, mass)
        torch.cuda.synchronize()
        res.append(mass.cpu().numpy())
        ctx.close()
    model.close()
    assert np.array_equal(res[0], res[1])


# ranks and sizes where a product was once one thread per logit; single elements, ranks off every K step
_SMALL = [(1024, 12, "f32", "bf16", 64), (1024, 26, "f32", "f32", 65), (1024, 27, "f32", "f32", 64),
          (128, 38, "f32", "bf16", 512), (128, 32, "f32", "f32", 3), (8200, 11, "f32", "f32", 33), (1, 1, "f32", "f32", 1),
          (563, 33, "bf16", "f32", 116), (2003, 56, "bf16", "bf16", 40), (700, 57, "bf16", "f32", 9)]


@pytest.mark.parametrize("V,d,wdt,ldt,R", _SMALL)
def test_small_products(V, d, wdt, ldt, R):
    test_logits_tile_edges(V, d, wdt, ldt, R)


# both sides of each line between the fp32 kernel's tilings (256 compute units): K steps of 16, 32 and 64 by the rank up to
# 256 blocks of 32 x 64, two waves of rows up to six times as many, the largest tiles from 16 times as many of 128 x 128
_LINES = [(1024, 16, "f32", 512), (1024, 17, "f32", 512), (1024, 32, "f32", 512), (1024, 33, "f32", 512), (1025, 16, "f32", 512),
          (1024, 33, "bf16", 513), (6144, 40, "f32", 512), (6145, 40, "f32", 512), (6144, 40, "bf16", 513),
          (32641, 24, "f32", 2048), (32640, 24, "f32", 2048), (32768, 24, "bf16", 2049)]


@pytest.mark.parametrize("V,d,wdt,R", _LINES)
def test_fp32_logits_at_the_lines_between_tilings(V, d, wdt, R):
    test_fp32_logits_are_one_chain_over_k(V, d, wdt, R)


# the fp32 kernel's four tilings (16 x 64, 32 x 64, 64 x 128, 128 x 128 by the number of blocks), whole rows (ranks of a
# multiple of 16) and single elements, a last group of k short
_CHAIN = [(300, 9, "f32", 40), (300, 16, "bf16", 40), (300, 17, "f32", 40), (300, 32, "f32", 40), (1000, 100, "f32", 17), (1000, 16, "f32", 64), (4100, 128, "f32", 129), (4100, 75, "f32", 200), (4100, 48, "bf16", 1000),
          (4100, 31, "f32", 1001), (16500, 32, "f32", 4100), (16500, 19, "bf16", 4100)]


@pytest.mark.parametrize("V,d,wdt,R", _CHAIN)
def test_fp32_logits_are_one_chain_over_k(V, d, wdt, R):
    """Each logit is fma(a_k, b_k, sum) for k = 0, 1, ... from zero, bit for bit: libm's fmaf on the CPU."""
    import ctypes
    import torch
    from paper_2210_15458_amd import binding as B
    from gpu_util import to_dev_logits
    fmaf = ctypes.CDLL("libm.so.6").fmaf
    fmaf.restype, fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    E, U = synth.bigram_weights(V, d, seed=V + d, dtype=wdt)
    model = B.Model(to_dev_logits(E), to_dev_logits(U), scale=math.sqrt(d))      # (alpha = 1: the chain itself)
    rng = np.random.default_rng(d)
    prev = rng.integers(0, V, R).astype(np.int32)
    got = _logits(model, prev, V, "f32", R)
    Ew = synth.bf16_bits_to_f32(E) if wdt == "bf16" else E
    Uw = synth.bf16_bits_to_f32(U) if wdt == "bf16" else U
    at = [(0, 0), (R - 1, V - 1), (0, V - 1), (R - 1, 0)] + list(zip(rng.integers(0, R, 200), rng.integers(0, V, 200)))
    for r, v in at:
        acc = 0.0
        for a, b in zip(Ew[prev[r]].tolist(), Uw[:, v].tolist()):
            acc = fmaf(a, b, acc)
        assert got[r, v] == np.float32(acc), (r, v)
    model.close()


# several row tiles of the few-rows kernel (of 32, 64 and 128 rows), the last of them short, column tiles not a multiple of 8
_ROW_TILES = [(1000, 512, "bf16", 33), (3000, 512, "bf16", 257), (3000, 512, "f32", 500), (3000, 512, "bf16", 1001),
              (2100, 128, "f32", 1025), (1030, 1024, "bf16", 130)]


@pytest.mark.parametrize("V,d,ldt,R", _ROW_TILES)
def test_row_tiles_of_small_products(V, d, ldt, R):
    test_logits_tile_edges(V, d, "bf16", ldt, R)


@pytest.mark.parametrize("V,d,R", [(3000, 512, 257), (3000, 512, 1001), (1030, 128, 65)])
def test_row_tiles_of_group_masses(V, d, R):
    test_group_masses_of_few_rows(V, d, R)


@pytest.mark.parametrize("V,d,wdt,R", [(300, 17, "f32", 40), (300, 48, "f32", 40), (1000, 100, "f32", 17), (4100, 75, "f32", 200),
                                       (4100, 48, "bf16", 1000), (4100, 31, "f32", 1001), (16500, 19, "bf16", 4100)])
def test_fp32_chain_of_values_at_the_ends_of_the_range(V, d, wdt, R):
    """The same with subnormal factors, products and sums, sums beyond fp32, infinities and NaN: the bits of libm's fmaf
    (a NaN is a NaN).  One class of values a row, so that one does not hide another."""
    import ctypes
    from paper_2210_15458_amd import binding as B
    from gpu_util import to_dev_logits
    fmaf = ctypes.CDLL("libm.so.6").fmaf
    fmaf.restype, fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    rng = np.random.default_rng(V + d)
    kind = np.arange(V) % 5
    E = rng.standard_normal((V, d)).astype(np.float32)
    E[kind == 0] *= np.float32(2.0 ** -130)                       # subnormal factors, subnormal sums
    E[kind == 1] *= np.float32(2.0 ** -75)                        # with the columns' 2^-70: products below the normal range
    E[kind == 2] *= np.float32(2.0 ** 120)                        # with the columns' 2^10: sums beyond fp32, inf - inf
    E[kind == 3, d // 2] = np.inf                                 # with a zero in the column: NaN
    E[kind == 4, d - 1] = np.nan
    U = rng.standard_normal((d, V)).astype(np.float32)
    U[:, 1::4] *= np.float32(2.0 ** -70)
    U[:, 2::4] *= np.float32(2.0 ** 10)
    U[d // 2, 3::4] = 0.0
    if wdt == "bf16":                                             # (cut, not rounded: the same classes; a cut NaN stays one)
        E, U = ((x.view(np.uint32) >> 16).astype(np.uint16) for x in (E, U))
        Ew, Uw = synth.bf16_bits_to_f32(E), synth.bf16_bits_to_f32(U)
    else:
        Ew, Uw = E, U
    model = B.Model(to_dev_logits(E), to_dev_logits(U), scale=math.sqrt(d))      # (alpha = 1: the chain itself)
    prev = rng.integers(0, V, R).astype(np.int32)
    got = _logits(model, prev, V, "f32", R)
    seen = {"subnormal": 0, "inf": 0, "nan": 0, "normal": 0}
    for r, v in zip(rng.integers(0, R, 400), rng.integers(0, V, 400)):
        acc = 0.0
        for a, b in zip(Ew[prev[r]].tolist(), Uw[:, v].tolist()):
            acc = fmaf(a, b, acc)
        want = np.float32(acc)
        seen["nan" if np.isnan(want) else "inf" if np.isinf(want) else
             "subnormal" if 0 < abs(want) < 2.0 ** -126 else "normal"] += 1
        assert np.isnan(got[r, v]) if np.isnan(want) else got[r, v] == want, (r, v, kind[prev[r]], got[r, v], want)
    assert min(seen.values()) > 0, seen
    model.close()
