"""The nucleus of bf16 rows of any shape, whose logits the wide kernel counts by value: rows on which that holds and rows on
which it does not (a logit above the counters, a nucleus that reaches below them or below zero), each form of the kernel."""
import numpy as np
import pytest

from paper_2210_15458_amd import synth

pytestmark = pytest.mark.gpu
ANY = {"thr_path": 3}
CODES = np.array([0.0, 0.03, 0.2, 0.41, 0.5, 0.77, 0.9, 0.99, 1 - 2.0 ** -24], np.float32)


def _rows(V):
    rng = np.random.default_rng(V)
    n = lambda s: rng.standard_normal(V) * s
    x = np.stack([n(3.0), n(2.0) + 20.0, n(1.0), n(0.3), n(2.5) - 30.0,       # (one that is negative throughout)
                  np.full(V, 4.0), n(3.0), n(3.0), np.where(rng.random(V) < 0.3, -np.inf, n(2.0))]).astype(np.float32)
    x[6, V // 2] = 4000.0                                    # above every counter
    x[7, V - 1] = 40.0                                       # the row's last, far above the first ones
    return synth.f32_to_bf16_bits(x)


# a wave a row, 256, 512 and 1024 threads, one tile and several; rows that start off 16 bytes and end inside a piece
@pytest.mark.parametrize("V,rows", [(5, 9), (1023, 9), (4095, 3200), (4097, 9), (8191, 3200), (8193, 600), (16380, 600), (16385, 300),
                                    (32769, 9), (50257, 300), (65537, 9), (70001, 300), (140001, 9)])
def test_counted_rows(V, rows):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    stored = _rows(V)
    rid = (np.arange(rows) % len(stored)).astype(np.int32)
    codes = CODES if rows == len(CODES) else synth.uniform_codes(rows, seed=V)
    for temp, top_p in ((1.0, 0.9), (0.7, 0.5), (0.4, 0.98), (1.3, 0.97)):
        label = f"V={V} R={rows} temp={temp} p={top_p}"
        print("case", label, flush=True)
        gpu = run_gpu_step(stored, codes, V, temp=temp, top_p=top_p, row_ids=rid, tuning=ANY)
        ref = oracle_step(stored, codes, V, temp=temp, top_p=top_p, row_ids=rid.astype(np.int64))
        print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


# rows of one tile of whole pieces, which have a kernel of their own: on either side of the groups of pieces that a wave's share has
@pytest.mark.parametrize("V", [8, 2040, 2048, 2056, 8192, 8200, 10240, 10248, 30720, 30728, 32768])
def test_one_tile_by_the_groups_of_a_share(V):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    stored = synth.gaussian_logits(9, V, seed=V, dtype="bf16")
    for top_p in (0.5, 0.95):
        gpu = run_gpu_step(stored, CODES, V, temp=0.9, top_p=top_p)
        ref = oracle_step(stored, CODES, V, temp=0.9, top_p=top_p)
        print(f"V={V} p={top_p}", compare_step(gpu, ref, V, f"V={V} p={top_p}", trunc=True, codes=CODES), flush=True)


# Weights against the first pieces' largest logit, 118 to 127 factors of two below many tied ones: a piece's eight add up, a
# chunk's 512 pass what fp32 holds.  (a wave a row; 256 threads with counters of 1024 and of 2048 values; 512; 1024; several tiles)
@pytest.mark.parametrize("V,rows", [(4095, 3200), (8191, 3200), (8193, 1100), (16380, 600), (16380, 300), (33001, 300), (50257, 3),
                                    (140001, 3)])
def test_largest_far_above_the_first_pieces(V, rows):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    x = np.full((7, V), 10.0, np.float32)
    at = (V // 2 + 511) // 512 * 512
    for r, (value, n) in enumerate(((14.125, 100), (14.25, 100), (14.375, 100), (14.25, 512), (14.375, 1500), (14.375, 1))):
        x[r, at:at + n] = value
    x[6, V // 2:] = 14.25
    stored = synth.f32_to_bf16_bits(x)
    rid = (np.arange(rows) % len(x)).astype(np.int32)
    codes = synth.uniform_codes(rows, seed=V)
    codes[:3] = 0.0, 0.5, 0.999
    for temp, top_p in ((0.05, 0.9), (0.05, 0.5), (0.0487, 0.97)):
        label = f"V={V} R={rows} temp={temp} p={top_p}"
        print("case", label, flush=True)
        gpu = run_gpu_step(stored, codes, V, temp=temp, top_p=top_p, row_ids=rid, tuning=ANY)
        ref = oracle_step(stored, codes, V, temp=temp, top_p=top_p, row_ids=rid.astype(np.int64))
        print("   ", compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


def test_half_a_row_far_above_the_other():
    from gpu_util import compare_step, oracle_step, run_gpu_step
    V = 50257
    x = np.full((3, V), 10.0, np.float32)
    x[:, 25000:50000] = 95.0                                 # (not the row's tail, which is looked at with the first pieces)
    stored, codes = synth.f32_to_bf16_bits(x), np.array([0.0, 0.5, 0.99], np.float32)
    gpu = run_gpu_step(stored, codes, V, temp=1.0, top_p=0.9)
    print(compare_step(gpu, oracle_step(stored, codes, V, temp=1.0, top_p=0.9), V, "95 above 10", trunc=True, codes=codes))


# At shares next to a group's end the counted way keeps what the integer masses keep: a step's probability and the width that its
# token has as an interval are quotients by the kept weight, equal to the rounding of its fp32 sums (below 1e-6), where a group more
# or less, a thousandth of the weight here, is another set.  So each token sampled is one that the encode direction keeps.
@pytest.mark.parametrize("V,rows", [(2047, 1600), (4095, 3200), (8191, 3200), (8193, 1100), (16380, 600), (33001, 300), (50257, 60), (70001, 260), (140001, 20)])
def test_shares_next_to_a_groups_end(V, rows):
    import torch
    from gpu_util import to_dev_logits
    from paper_2210_15458_amd import binding as B
    rng = np.random.default_rng(V)
    one = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits((rng.standard_normal(V) * 1.5 + 3.0).astype(np.float32)))
    x = np.stack([rng.permutation(one) for _ in range(rows)])    # (one set of values, summed in many orders)
    logits = to_dev_logits(synth.f32_to_bf16_bits(x))
    values, counts = np.unique(one, return_counts=True)
    share = np.cumsum(counts[::-1] * np.exp(values[::-1].astype(np.float64)))
    share /= share[-1]
    near = share[(share > 0.3) & (share < 0.95)].astype(np.float32)
    codes = torch.from_numpy(synth.uniform_codes(rows, seed=V)).cuda()
    token = torch.zeros(rows, dtype=torch.int32, device="cuda")
    prob, c_out = torch.zeros(rows, device="cuda"), torch.zeros(rows, device="cuda")
    lo, width = (torch.zeros(rows, dtype=torch.float64, device="cuda") for _ in range(2))
    ctx = B.Ctx(rows, V, logits.dtype)
    ctx.set_tuning("thr_path", 3)
    differ = 0
    for p in rng.choice(near, min(20, len(near)), replace=False):
        for share_of in (np.nextafter(p, np.float32(0)), p, np.nextafter(p, np.float32(1))):
            lo.zero_()
            width.fill_(1.0)
            B.as_step_ex(ctx, logits, codes, 1.0, 0, float(share_of), token, c_out, prob_out=prob)
            B.as_interval_step(ctx, logits, token, 1.0, 0, float(share_of), lo, width)
            differ += int(((prob.double() - width).abs() > 1e-5 * prob).sum())
    print(f"V={V} rows={rows}: {differ} steps differ", flush=True)
    ctx.close()
    assert differ == 0
