"""as_encode, which takes all positions of a call at once, against the loop of exported calls, which takes them step by
step: the same bits.  Shapes at the edges of what it chooses by: logits rows given to tokens or to positions, several
chunks of rows and windows of columns, rows of one tile and others, sequences that end and do not, rows beyond fp32."""
import pytest
import torch

from paper_2210_15458_amd import binding as B

pytestmark = pytest.mark.gpu

EOS = 1
DT = {"bf16": torch.bfloat16, "f32": torch.float32}

# V, d, prompts, codes, steps, temperature, top_k, top_p, weights, logits, scale
CASES = [
    (2000, 128, 3, 40, 70, 0.9, 0, 1.0, "bf16", "bf16", 3.0),       # a row per token; a second run of 64 columns
    (2000, 128, 3, 40, 70, 0.9, 20, 0.9, "bf16", "bf16", 3.0),
    (2000, 128, 1, 3000, 9, 1.0, 0, 1.0, "bf16", "f32", 3.0),       # many positions on a prompt's row
    (30000, 128, 4, 700, 4, 1.0, 0, 0.9, "bf16", "bf16", 3.0),      # several chunks of rows, the last one short
    (1000, 128, 7, 10001, 9, 1.0, 0, 1.0, "bf16", "bf16", 3.0),     # two windows of columns
    (40, 24, 3, 20001, 10, 1.0, 0, 1.0, "f32", "f32", 3.0),         # ... with a row per position, fp32 model
    (5001, 192, 2, 33, 65, 1.0, 0, 1.0, "bf16", "bf16", 3.0),       # ragged vocabulary: the one-pass kernel
    (33000, 128, 2, 9, 5, 0.8, 30, 1.0, "bf16", "bf16", 3.0),       # rows of more than one tile
    (8200, 128, 5, 1, 3, 0.3, 0, 1.0, "bf16", "f32", 3.0),          # low temperature
    (16384, 128, 2, 6, 4, 1.0, 0, 1.0, "bf16", "f32", 300.0),       # weights beyond fp32 against a first chunk
    (24, 8, 1, 1, 1, 1.0, 0, 1.0, "f32", "bf16", 3.0),
    (24, 8, 2, 3, 1, 1.0, 5, 1.0, "f32", "f32", 3.0),
]


@pytest.mark.parametrize("V,d,Bn,N,T,temp,top_k,top_p,wdt,ldt,scale", CASES)
@pytest.mark.parametrize("eos", [EOS, -1])
def test_encode_equals_the_loop_of_exported_calls(V, d, Bn, N, T, temp, top_k, top_p, wdt, ldt, scale, eos):
    g = torch.Generator(device="cuda").manual_seed(V + T)
    E = torch.randn(V, d, device="cuda", generator=g).to(DT[wdt])
    U = torch.randn(d, V, device="cuda", generator=g).to(DT[wdt])
    model = B.Model(E, U, scale=scale)
    R = Bn * N
    ctx = B.Ctx(R, V, DT[ldt])
    prompts = torch.randint(0, V, (Bn,), device="cuda", generator=g, dtype=torch.int32)
    prompts[-1] = V + 5                                             # outside: clamped
    # half of the tokens from a few, so that positions share rows; ends at any column; some outside the vocabulary
    tokens = torch.randint(0, V, (R, T), device="cuda", generator=g, dtype=torch.int32)
    few = torch.rand(R, T, device="cuda", generator=g) < 0.5
    tokens[few] = tokens[few] % 37
    stray = torch.rand(R, T, device="cuda", generator=g)
    tokens[stray < 0.01] = V + 2
    tokens[stray > 0.99] = -3
    tokens = tokens.contiguous()
    lo, width = (torch.full((R,), 7.0, dtype=torch.float64, device="cuda") for _ in range(2))
    for _ in range(2):                                              # twice: the tables are left from the call before
        B.as_encode(ctx, model, prompts, N, T, tokens.view(Bn, N, T), temp, top_k, top_p, eos, lo, width)

    logits = torch.empty((R, (V + 7) // 8 * 8), dtype=DT[ldt], device="cuda")
    prev = prompts.repeat_interleave(N).contiguous()
    fin = torch.zeros(R, dtype=torch.uint8, device="cuda")
    elo = torch.zeros(R, dtype=torch.float64, device="cuda")
    ewidth = torch.ones(R, dtype=torch.float64, device="cuda")
    for t in range(T):
        B.as_bigram_logits(ctx, model, prev, logits)
        tok = tokens[:, t].contiguous()
        B.as_interval_step(ctx, logits, tok, temp, top_k, top_p, elo, ewidth, finished_in=fin if eos >= 0 else None,
                           eos_id=eos, finished_out=fin if eos >= 0 else None)
        prev = torch.where((tok >= 0) & (tok < V), tok, torch.zeros_like(tok))
    assert torch.equal(elo, lo) and torch.equal(ewidth, width)
    assert (eos >= 0 and T > 1) == bool(fin.any()) or R * T < 500
    ctx.close()
    model.close()


def test_encode_of_no_columns_is_the_whole_interval():
    E = torch.randn(16, 8, device="cuda")
    model = B.Model(E, torch.randn(8, 16, device="cuda"), scale=3.0)
    ctx = B.Ctx(6, 16, torch.float32)
    lo, width = (torch.full((6,), 7.0, dtype=torch.float64, device="cuda") for _ in range(2))
    B.as_encode(ctx, model, torch.zeros(2, dtype=torch.int32, device="cuda"), 3, 0,
                torch.empty((2, 3, 0), dtype=torch.int32, device="cuda"), 1.0, 0, 1.0, EOS, lo, width)
    assert bool((lo == 0).all()) and bool((width == 1).all())
    ctx.close()
    model.close()
