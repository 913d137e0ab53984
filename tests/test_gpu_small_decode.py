"""The whole decode in one launch (models that fit LDS) against the loop of exported calls: the same bits."""
import numpy as np
import pytest
import torch

from paper_2210_15458_amd import binding as B
from paper_2210_15458_amd import synth

pytestmark = pytest.mark.gpu

# (V, d, weights, logits, prompts, codes, steps): the smallest, one vector a lane short of, at and over a chunk of 64
# vectors, the largest vocabulary and rank it takes, many steps, as many rows as it takes, a rank
# beyond it
CASES = [(4, 1, "f32", "f32", 1, 3, 2), (16, 8, "f32", "f32", 1, 64, 8), (252, 9, "f32", "f32", 2, 5, 3),
         (256, 32, "f32", "f32", 3, 7, 4), (260, 31, "f32", "f32", 1, 33, 40), (1024, 8, "f32", "bf16", 4, 16, 5),
         (64, 128, "f32", "bf16", 1, 4, 3), (512, 15, "bf16", "bf16", 2, 9, 4), (520, 9, "bf16", "f32", 2, 9, 4),
         (64, 24, "f32", "f32", 12, 64, 6), (16, 129, "f32", "f32", 1, 4, 3)]


@pytest.mark.parametrize("V,d,wdt,ldt,Bn,N,T", CASES)
@pytest.mark.parametrize("eos", [1, -1])
def test_small_decode_equals_the_loop(V, d, wdt, ldt, Bn, N, T, eos):
    from gpu_util import to_dev_logits
    E, U = synth.bigram_weights(V, d, seed=V + d, dtype=wdt)
    model = B.Model(to_dev_logits(E), to_dev_logits(U), scale=3.0)
    R = Bn * N
    ctx = B.Ctx(R, V, torch.float32 if ldt == "f32" else torch.bfloat16)
    prompts = torch.from_numpy(synth.prompts(Bn, V, seed=1)).cuda()
    u = torch.from_numpy(synth.shifts(Bn, seed=2)).cuda()
    uniforms = torch.from_numpy(np.random.default_rng(3).random((T, R)).astype(np.float32)).cuda()
    out, anc = (torch.empty((Bn, N, T), dtype=torch.int32, device="cuda") for _ in range(2))
    last = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_decode(ctx, model, prompts, N, T, u, 0.9, 0, 1.0, eos, out, codes_out=last)
    B.as_decode_ancestral(ctx, model, prompts, N, T, uniforms, 0.9, 0, 1.0, eos, anc)

    logits = torch.empty((R, (V + 7) // 8 * 8), dtype=ctx.torch_dtype, device="cuda")
    for ancestral, got in ((False, out), (True, anc)):
        codes = torch.empty(R, dtype=torch.float32, device="cuda")
        B.as_lattice(ctx, u, N, codes)
        prev = prompts.repeat_interleave(N).contiguous()
        fin = torch.zeros(R, dtype=torch.uint8, device="cuda")
        state = dict(finished_in=fin, eos_id=eos, finished_out=fin) if eos >= 0 else {}
        for t in range(T):
            B.as_bigram_logits(ctx, model, prev, logits)
            tok = torch.empty(R, dtype=torch.int32, device="cuda")
            B.as_step_ex(ctx, logits, uniforms[t].contiguous() if ancestral else codes, 0.9, 0, 1.0, tok, codes, **state)
            assert torch.equal(tok, got.view(R, T)[:, t]), f"ancestral {ancestral} step {t}"
            prev = tok
        if not ancestral:
            assert torch.equal(codes, last)
    ctx.close()
    model.close()


# a wave per row: ragged vocabularies up to a chunk of 64 vectors and one past it, low temperatures (step_kernel's
# references), ranks and weights at its limits, more rows than the chip holds at once
WAVE = [(5, 3, "f32", "f32", 1, 3, 3, 0.9), (39, 10, "f32", "f32", 3, 36, 5, 0.9), (255, 33, "f32", "f32", 2, 7, 4, 0.7),
        (257, 8, "f32", "f32", 2, 5, 3, 0.9), (101, 128, "f32", "bf16", 1, 9, 4, 0.9), (101, 64, "f32", "bf16", 1, 9, 4, 0.9),
        (511, 17, "bf16", "bf16", 2, 9, 4, 0.9), (513, 3, "f32", "bf16", 2, 9, 4, 0.9), (64, 12, "f32", "f32", 2, 9, 6, 0.2),
        (61, 12, "f32", "bf16", 2, 9, 6, 0.2), (16, 8, "f32", "f32", 3, 1500, 4, 0.9), (230, 40, "f32", "f32", 1, 700, 3, 0.9),
        (1, 1, "f32", "f32", 1, 2, 2, 1.0)]


@pytest.mark.parametrize("V,d,wdt,ldt,Bn,N,T,temp", WAVE)
def test_decode_by_waves_equals_the_loop(V, d, wdt, ldt, Bn, N, T, temp):
    from gpu_util import to_dev_logits
    E, U = synth.bigram_weights(V, d, seed=V + d, dtype=wdt)
    model = B.Model(to_dev_logits(E), to_dev_logits(U), scale=3.0)
    R, eos = Bn * N, 1 if V > 1 else -1
    ctx = B.Ctx(R, V, torch.float32 if ldt == "f32" else torch.bfloat16)
    prompts = torch.from_numpy(synth.prompts(Bn, V, seed=1)).cuda()
    prompts[-1] = V + 3                                                       # outside: clamped
    u = torch.from_numpy(synth.shifts(Bn, seed=2)).cuda()
    out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
    last = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_decode(ctx, model, prompts, N, T, u, temp, 0, 1.0, eos, out, codes_out=last)
    logits = torch.empty((R, (V + 7) // 8 * 8), dtype=ctx.torch_dtype, device="cuda")
    codes = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_lattice(ctx, u, N, codes)
    prev = prompts.repeat_interleave(N).contiguous()
    fin = torch.zeros(R, dtype=torch.uint8, device="cuda")
    state = dict(finished_in=fin, eos_id=eos, finished_out=fin) if eos >= 0 else {}
    for t in range(T):
        B.as_bigram_logits(ctx, model, prev, logits)
        tok = torch.empty(R, dtype=torch.int32, device="cuda")
        B.as_step_ex(ctx, logits, codes, temp, 0, 1.0, tok, codes, **state)
        assert torch.equal(tok, out.view(R, T)[:, t]), f"step {t}"
        prev = tok
    assert torch.equal(codes, last)
    ctx.close()
    model.close()
