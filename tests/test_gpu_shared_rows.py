"""Decodes that compute one logits row for all rows with the same conditioning token (the first step's prompts; later
steps of wide lattices over small vocabularies) against the loop of exported calls, which computes every row: the
same bits."""
import numpy as np
import pytest
import torch

from paper_2210_15458_amd import binding as B
from paper_2210_15458_amd import synth

pytestmark = pytest.mark.gpu

# (V, d, prompts, codes, steps, logits): many rows per token in every step; the same with a ragged vocabulary and fp32
# logits; shared in the first step only, with few prompts (the logits kernel for few rows) and with one code each; rows
# beyond the caches, which are also sorted by logits row
CASES = [(2000, 1024, 4, 2048, 4, "bf16"), (1501, 1024, 1, 9000, 3, "f32"), (5000, 128, 3, 50, 3, "bf16"),
         (5000, 128, 70, 1, 3, "bf16"), (1501, 1024, 2, 12000, 3, "f32")]
EOS, TEMP = 1, 1.1


def _setup(V, d, Bn, N, ldt):
    from gpu_util import to_dev_logits
    E, U = synth.bigram_weights(V, d, seed=V, dtype="bf16")
    U = synth.bf16_bits_to_f32(U).copy()
    U[:, EOS] += 0.15                                   # rows end at different steps
    model = B.Model(to_dev_logits(E), to_dev_logits(synth.f32_to_bf16_bits(U)), scale=3.0)
    ctx = B.Ctx(Bn * N, V, torch.float32 if ldt == "f32" else torch.bfloat16)
    prompts = torch.from_numpy(synth.prompts(Bn, V, seed=1)).cuda()
    u = torch.from_numpy(synth.shifts(Bn, seed=2)).cuda()
    return model, ctx, prompts, u


@pytest.mark.parametrize("V,d,Bn,N,T,ldt", CASES)
@pytest.mark.parametrize("top_k,top_p", [(0, 1.0), (40, 0.9), (0, 0.9)])
def test_decode_and_encode(V, d, Bn, N, T, ldt, top_k, top_p):
    model, ctx, prompts, u = _setup(V, d, Bn, N, ldt)
    R = Bn * N
    out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
    last = torch.empty(R, dtype=torch.float32, device="cuda")
    for _ in range(2):                                  # twice: the tables are left from the call before
        B.as_decode(ctx, model, prompts, N, T, u, TEMP, top_k, top_p, EOS, out, codes_out=last)
    lo, width = (torch.empty(R, dtype=torch.float64, device="cuda") for _ in range(2))
    B.as_encode(ctx, model, prompts, N, T, out, TEMP, top_k, top_p, EOS, lo, width)

    logits = torch.empty((R, (V + 7) // 8 * 8), dtype=ctx.torch_dtype, device="cuda")
    codes = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_lattice(ctx, u, N, codes)
    prev = prompts.repeat_interleave(N).contiguous()
    fin = torch.zeros(R, dtype=torch.uint8, device="cuda")
    efin = torch.zeros(R, dtype=torch.uint8, device="cuda")
    elo = torch.zeros(R, dtype=torch.float64, device="cuda")
    ewidth = torch.ones(R, dtype=torch.float64, device="cuda")
    for t in range(T):
        B.as_bigram_logits(ctx, model, prev, logits)
        tok = torch.empty(R, dtype=torch.int32, device="cuda")
        B.as_step_ex(ctx, logits, codes, TEMP, top_k, top_p, tok, codes, finished_in=fin, eos_id=EOS, finished_out=fin)
        assert torch.equal(tok, out.view(R, T)[:, t]), f"step {t}"
        B.as_interval_step(ctx, logits, tok, TEMP, top_k, top_p, elo, ewidth, finished_in=efin, eos_id=EOS,
                           finished_out=efin)
        prev = tok
    assert torch.equal(codes, last)
    assert torch.equal(elo, lo) and torch.equal(ewidth, width)
    assert 0 < int(fin.sum()) < R or R < 200
    ctx.close()
    model.close()


@pytest.mark.parametrize("V,d,Bn,N,T,ldt", CASES)
def test_fused_decode(V, d, Bn, N, T, ldt):
    model, ctx, prompts, u = _setup(V, d, Bn, N, ldt)
    R = Bn * N
    out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
    B.as_decode_fused(ctx, model, prompts, N, T, u, TEMP, EOS, out)
    ldp = (-(-V // 32) + 15) // 16 * 16
    mass = torch.zeros((R, ldp, 2), dtype=torch.float32, device="cuda")
    codes = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_lattice(ctx, u, N, codes)
    prev = prompts.repeat_interleave(N).contiguous()
    fin = torch.zeros(R, dtype=torch.uint8, device="cuda")
    for t in range(T):
        B.as_bigram_group_mass(ctx, model, prev, TEMP, mass)
        tok = torch.empty(R, dtype=torch.int32, device="cuda")
        B.as_step_fused(ctx, model, mass, prev, codes, TEMP, tok, codes, finished_in=fin, eos_id=EOS, finished_out=fin)
        assert torch.equal(tok, out.view(R, T)[:, t]), f"step {t}"
        prev = tok
    ctx.close()
    model.close()
