"""Decodes that keep a logits row per token from step to step, against the loop of exported calls: the same bits.  Sampled
from the rows' sums (untruncated rows of one tile) and not; a table of more rows than the decode has; weights beyond
fp32 against a first chunk; rows that end; replayed from a graph."""
import pytest
import torch

import bench
from paper_2210_15458_amd import binding as B

pytestmark = pytest.mark.gpu

EOS, TEMP = 1, 1.1
DT = {"bf16": torch.bfloat16, "f32": torch.float32}

# V, d, prompts, codes, steps, top_k, top_p, logits, scale
CASES = [
    (3000, 128, 3, 1000, 18, 0, 1.0, "bf16", 3.0),
    (8000, 512, 2, 2100, 6, 0, 1.0, "bf16", 3.0),         # more kept rows than rows
    (2000, 128, 1, 4097, 10, 0, 1.0, "f32", 300.0),       # sums beyond fp32
    (3000, 1024, 4, 2000, 6, 20, 0.9, "bf16", 3.0),       # truncated: its own kernels, from the kept rows
    (9001, 512, 2, 6000, 5, 0, 1.0, "bf16", 3.0),         # ragged rows, 108 MB of them
    (9001, 512, 2, 6000, 5, 0, 1.0, "f32", 3.0),          # ... beyond the caches: read in the order of the rows
]


def _setup(V, d, Bn, N, ldt, scale):
    g = torch.Generator(device="cuda").manual_seed(V)
    E = torch.randn(V, d, device="cuda", generator=g).bfloat16()
    U = torch.randn(d, V, device="cuda", generator=g)
    U[:, EOS] += 0.15                                     # rows end at different steps
    model = B.Model(E, U.bfloat16(), scale=scale)
    prompts = torch.randint(0, V, (Bn,), device="cuda", generator=g, dtype=torch.int32)
    prompts[-1] = V + 9                                   # outside: clamped
    return model, B.Ctx(Bn * N, V, DT[ldt]), prompts, torch.rand(Bn, device="cuda", generator=g)


@pytest.mark.parametrize("V,d,Bn,N,T,top_k,top_p,ldt,scale", CASES)
def test_kept_rows_equal_the_loop_of_exported_calls(V, d, Bn, N, T, top_k, top_p, ldt, scale):
    model, ctx, prompts, u = _setup(V, d, Bn, N, ldt, scale)
    R = Bn * N
    assert bench.rows_kept(V, d, R, Bn, T, "bf16", (V + 7) // 8 * 8 * (2 if ldt == "bf16" else 4),
                           bench.step_by_sums(V, ldt, top_k, top_p, TEMP))
    ctx.set_tuning("kept_rows", 2)                        # (here whatever the rule comes to be)
    out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
    last = torch.empty(R, dtype=torch.float32, device="cuda")
    for _ in range(2):                                    # twice: the tables are left from the call before
        B.as_decode(ctx, model, prompts, N, T, u, TEMP, top_k, top_p, EOS, out, codes_out=last)
    ctx.profile(True)
    B.as_decode(ctx, model, prompts, N, T, u, TEMP, top_k, top_p, EOS, out, codes_out=last)
    steps = ctx.profile_read(0)[1]
    ctx.profile(False)
    assert steps == (2 if bench.step_by_sums(V, ldt, top_k, top_p, TEMP) else 1) * T
    logits = torch.empty((R, (V + 7) // 8 * 8), dtype=DT[ldt], device="cuda")
    codes = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_lattice(ctx, u, N, codes)
    prev = prompts.repeat_interleave(N).contiguous()
    fin = torch.zeros(R, dtype=torch.uint8, device="cuda")
    for t in range(T):
        B.as_bigram_logits(ctx, model, prev, logits)
        tok = torch.empty(R, dtype=torch.int32, device="cuda")
        B.as_step_ex(ctx, logits, codes, TEMP, top_k, top_p, tok, codes, finished_in=fin, eos_id=EOS, finished_out=fin)
        assert torch.equal(tok, out.view(R, T)[:, t]), f"step {t}"
        prev = tok
    assert torch.equal(codes, last)
    ctx.close()
    model.close()


def test_kept_rows_replay_from_a_graph():
    V, d, Bn, N, T = 3000, 128, 3, 1000, 18
    model, ctx, prompts, u = _setup(V, d, Bn, N, "bf16", 3.0)
    stream = torch.cuda.Stream()
    ctx.close()
    with torch.cuda.stream(stream):
        ctx = B.Ctx(Bn * N, V, torch.bfloat16)
        ctx.set_tuning("kept_rows", 2)
        out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
        eager = torch.empty_like(out)
        B.as_decode(ctx, model, prompts, N, T, u, TEMP, 0, 1.0, EOS, out)       # (makes the workspace)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        B.as_decode(ctx, model, prompts, N, T, u, TEMP, 0, 1.0, EOS, out)
    for i in range(4):
        with torch.cuda.stream(stream):
            u.uniform_(0.0, 0.99)
            out.fill_(-1)
            graph.replay()
            got = out.clone()
            B.as_decode(ctx, model, prompts, N, T, u, TEMP, 0, 1.0, EOS, eager)
        stream.synchronize()
        assert torch.equal(got, eager), f"replay {i}"
    ctx.close()
    model.close()


def _step_launches(ctx, model, prompts, N, T, u, out):
    ctx.profile(True)
    B.as_decode(ctx, model, prompts, N, T, u, TEMP, 0, 1.0, EOS, out)
    n = ctx.profile_read(0)[1]
    ctx.profile(False)
    return n


# on either side of the rule: by rows, by steps, by the vocabulary that the workspace has room for
@pytest.mark.parametrize("V,d,R,T,kept", [(2000, 128, 2048, 64, True), (2000, 128, 1024, 64, False), (8000, 512, 4096, 4, True),
                                          (8000, 512, 2048, 16, False), (32128, 512, 8192, 5, True), (32128, 512, 8000, 5, False),
                                          (32128, 512, 8000, 4, True), (3000, 64, 8192, 16, False)])
def test_which_decodes_keep_rows(V, d, R, T, kept):
    """Steps from sums are two launches: the library's choice where it makes no table of all tokens' rows, the knob's, and what
    the benchmark takes the choice to be."""
    model, ctx, prompts, u = _setup(V, d, 1, R, "bf16", 3.0)
    ctx.set_tuning("kept_rows", 4)
    prompts[0] = 7
    out = torch.empty((1, R, T), dtype=torch.int32, device="cuda")
    assert _step_launches(ctx, model, prompts, R, T, u, out) == (2 * T if kept else T)
    assert bench.rows_kept(V, d, R, 1, T, "bf16", V * 2, True) == kept
    want = out.clone()
    ctx.set_tuning("kept_rows", 1)
    assert _step_launches(ctx, model, prompts, R, T, u, out) == T
    assert torch.equal(out, want)
    ctx.close()
    model.close()
