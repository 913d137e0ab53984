"""The nucleus in the kernel for rows of any shape, on rows built against what its quick way takes for granted: where the
approximate tallies say the nucleus closes, how far the row's largest logit lies above its first ones."""
import numpy as np
import pytest

from paper_2210_15458_amd import synth

pytestmark = pytest.mark.gpu
ANY = {"thr_path": 3}
LOG2E = 1.4426950408889634


def _against_oracle(x, dtype, codes, top_p, label):
    from gpu_util import compare_step, oracle_step, run_gpu_step
    V = x.shape[1]
    stored = synth.f32_to_bf16_bits(x) if dtype == "bf16" else x
    gpu = run_gpu_step(stored, codes, V, top_p=top_p, tuning=ANY)
    ref = oracle_step(stored, codes, V, top_p=top_p)
    print(label, compare_step(gpu, ref, V, label, trunc=True, codes=codes), flush=True)


def _past_a_full_window(V, per_octave, closing):
    """A row whose closing bin, by the tallies, ends just before its nucleus does, and the nucleus's share p.

    A tally takes a weight for linear within its bin, which is exact at the bin's centre and too little elsewhere.  Here
    everything down to the closing bin sits at centres and what lies below at the bins' ends: by the tallies the
    total is too small by up to (ln2 / per_octave / 2)^2 / 2 of it, and the goal with it.  The bins on either side of
    the closing one hold too many logits to be looked at along with it.
    """
    y = np.full(V, -4.0 - 6.499 / per_octave)
    at = 0
    for n, v in ((100, -3.0), (40, -4.0 + 1.0 / per_octave), (closing, -4.0), (40, -4.0 - 1.0 / per_octave)):
        y[at:at + n] = v
        at += n
    w = np.exp2(y)
    upto, total = w[:140 + closing].sum(), w.sum()
    low = (np.log(2.0) / per_octave * 0.499) ** 2 / 2 * w[at:].sum()
    p = np.float32(upto / (total - low / 2))
    assert upto / total < p < upto / (total - low)
    # (the first logits of the row among them: the reference is the row's own)
    return (y / LOG2E).astype(np.float32), float(p)


@pytest.mark.parametrize("V,per_octave,closing", [(4096, 32, 200), (4096, 32, 300), (4096, 32, 900),
                                                  (12288, 64, 800), (12288, 64, 1500), (12288, 64, 2000)])
def test_goal_just_past_the_closing_bin(V, per_octave, closing):
    x, p = _past_a_full_window(V, per_octave, closing)
    codes = np.array([0.1, 0.5, 0.9, 0.999, 1 - 2.0 ** -24], np.float32)
    rows = np.stack([np.roll(x, s) for s in (0, 17, 64, 1, 333)])
    _against_oracle(rows, "f32", codes, p, f"V={V} closing={closing} p={p}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("gap", [8.5, 9.1, 9.8, 10.4, 11.0])
def test_largest_logits_past_the_first_ones(gap, dtype):
    # 2^12 to 2^16 times the weight of the row's first logits, from a few of these to more than any table takes, in one run
    V = 50257
    counts = (1, 300, 512, 1000, 1500, 2000, 5000)
    x = np.zeros((len(counts), V), np.float32)
    for r, n in enumerate(counts):
        x[r, 10240:10240 + n] = gap
    x[:, 20000:20003] = gap - 1.0
    codes = np.array([0.5, 0.9, 0.3, 0.95, 0.05, 0.7, 0.999], np.float32)
    for top_p in (0.3, 0.9):
        _against_oracle(x, dtype, codes, top_p, f"gap={gap} {dtype} p={top_p}")


# (V, rows): the forms with 256, 512 and 1024 threads, one tile and several, and rows that start off 16 bytes; by the
# library's own choice also the kernels that hold a row or stream it (32128 aligned, odd ones up to 33001)
SAME = [(4096, 8), (4099, 8), (9001, 600), (20003, 300), (32128, 8), (32128, 300), (33001, 520), (40000, 6), (140001, 3),
        (70001, 260)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,rows", SAME)
def test_same_threshold_as_the_radix_select(V, rows, dtype):
    """The nucleus closes where the fixed-point masses of the general selection say so, whatever the kernel: at shares p
    that are next to a group's end on purpose, the kept sets are equal (an interval's width is a quotient by the
    kept weight: the same bits or another set)."""
    import torch
    from gpu_util import to_dev_logits
    from paper_2210_15458_amd import binding as B
    rng = np.random.default_rng(V)
    one = synth.gaussian_logits(1, V, sigma=0.7, seed=V, dtype=dtype)[0]
    x = np.stack([rng.permutation(one) for _ in range(rows)])   # (one set of values, summed in many orders)
    value = synth.bf16_bits_to_f32(one) if dtype == "bf16" else one
    logits = to_dev_logits(x)
    tokens = torch.from_numpy((synth.bf16_bits_to_f32(x) if dtype == "bf16" else x).argmax(axis=1).astype(np.int32)).cuda()
    ctx = B.Ctx(rows, V, logits.dtype)

    def widths(path, top_k, top_p):
        ctx.set_tuning("thr_path", path)
        lo = torch.zeros(rows, dtype=torch.float64, device="cuda")
        width = torch.ones(rows, dtype=torch.float64, device="cuda")
        B.as_interval_step(ctx, logits, tokens, 0.9, top_k, top_p, lo, width)
        return width

    # groups of equal logits, from the largest down, and the running share of the weight
    values, counts = np.unique(value, return_counts=True)
    weight = counts[::-1] * np.exp(values[::-1].astype(np.float64) / 0.9)
    differ = 0
    for top_k in (0, 100, 300):
        kept = weight if top_k == 0 else weight[:np.searchsorted(np.cumsum(counts[::-1]), top_k) + 1]
        share = np.cumsum(kept) / kept.sum()
        tries = 4 if rows * V > 5e6 else 100 if top_k == 0 else 20
        for p in rng.choice(share[:-1], min(tries, len(share) - 1), replace=False).astype(np.float32):
            want = widths(1, top_k, float(p))
            for path in (3, 0):
                differ += int((widths(path, top_k, float(p)) != want).sum())
    print(f"V={V} rows={rows} {dtype}: {differ} rows differ", flush=True)
    assert differ == 0
    ctx.close()
