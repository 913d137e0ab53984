"""Decodes that make the logits rows of all tokens before the first step, against the loop of exported calls: the same bits.
Every form that its steps take (sums, candidates, the rows themselves); rows that a one-tile kernel gives up (equal logits,
weights beyond fp32); rows that end; more steps than a wave holds tokens; replayed from a graph; without the memory."""
import pytest
import torch

from paper_2210_15458_amd import binding as B

pytestmark = pytest.mark.gpu

TEMP = 1.1
DT = {"bf16": torch.bfloat16, "f32": torch.float32}

# V, d, prompts, codes, steps, top_k, top_p, weights, logits, temp, scale
CASES = [
    (8200, 128, 3, 20, 70, 0, 1.0, "bf16", "bf16", TEMP, 3.0),       # a share of the row past its end; 70 steps
    (600, 64, 1, 37, 20, 0, 1.0, "bf16", "bf16", TEMP, 300.0),       # sums beyond fp32: the plain form of the row
    (4100, 40, 2, 30, 12, 0, 1.0, "f32", "f32", 0.8, 3.0),
    (2000, 128, 1, 41, 64, 0, 1.0, "bf16", "f32", 0.36, 3.0),
    (16000, 128, 2, 100, 65, 40, 1.0, "bf16", "bf16", TEMP, 3.0),    # candidates
    (16000, 128, 1, 130, 64, 20, 0.9, "bf16", "bf16", 0.3, 3.0),
    (20000, 192, 2, 130, 64, 0, 0.9, "bf16", "bf16", TEMP, 3.0),     # the nucleus alone
    (4096, 128, 2, 13, 30, 0, 0.5, "bf16", "bf16", TEMP, 30.0),
    (2001, 128, 2, 100, 16, 0, 1.0, "bf16", "bf16", TEMP, 3.0),      # ragged rows, a low temperature, k the wide kernel's
    (2000, 128, 2, 100, 16, 0, 1.0, "bf16", "bf16", 0.2, 3.0),
    (3000, 128, 1, 70, 20, 100, 0.9, "bf16", "f32", TEMP, 3.0),
    # rows in their plain form: sums beyond fp32, runs of 256ths that end inside a vector; candidates and nuclei of rows that are
    # all but equal
    (8200, 128, 2, 40, 20, 0, 1.0, "bf16", "bf16", 0.4, 200.0),
    (4100, 128, 2, 40, 20, 0, 1.0, "bf16", "f32", 0.4, 200.0),
    (8200, 128, 2, 40, 20, 20, 1.0, "bf16", "bf16", 0.4, 0.001),
    (8200, 128, 2, 40, 20, 0, 0.9, "bf16", "bf16", 0.4, 0.02),
    (9000, 128, 2, 40, 20, 0, 0.9, "bf16", "bf16", 0.4, 200.0),
]


def _setup(V, d, Bn, N, wdt, ldt, scale):
    g = torch.Generator(device="cuda").manual_seed(V)
    E = torch.randn(V, d, device="cuda", generator=g)
    E[::5] = 0.0                                          # rows of equal logits
    U = torch.randn(d, V, device="cuda", generator=g)
    model = B.Model(E.to(DT[wdt]), U.to(DT[wdt]), scale=scale)
    prompts = torch.randint(0, V, (Bn,), device="cuda", generator=g, dtype=torch.int32)
    prompts[-1] = V + 9                                   # outside: clamped
    return model, B.Ctx(Bn * N, V, DT[ldt]), prompts, torch.rand(Bn, device="cuda", generator=g), g


def _loop(ctx, model, prompts, N, T, codes, uniforms, temp, top_k, top_p, eos, ldt):
    """The exported calls, a step at a time: tokens [R, T] and the last codes."""
    R, V = prompts.numel() * N, model.V
    logits = torch.empty((R, (V + 7) // 8 * 8), dtype=DT[ldt], device="cuda")
    prev, fin = prompts.repeat_interleave(N).contiguous(), torch.zeros(R, dtype=torch.uint8, device="cuda")
    out = torch.empty((R, T), dtype=torch.int32, device="cuda")
    for t in range(T):
        B.as_bigram_logits(ctx, model, prev, logits)
        tok = torch.empty(R, dtype=torch.int32, device="cuda")
        code = uniforms[t].contiguous() if uniforms is not None else codes
        B.as_step_ex(ctx, logits, code, temp, top_k, top_p, tok, codes, finished_in=fin, eos_id=eos, finished_out=fin)
        out[:, t] = tok
        prev = tok
    return out, codes


# on either side of the rule: by codes, by steps, by the rank
@pytest.mark.parametrize("V,d,R,T,top_k,table", [(32128, 512, 1024, 64, 0, True), (32128, 512, 512, 24, 0, False),
                                                 (32128, 512, 1024, 128, 40, True), (32128, 512, 64, 64, 0, False),
                                                 (4096, 128, 256, 32, 0, True), (8000, 512, 4096, 16, 0, True),
                                                 (8000, 512, 16, 4, 0, False), (16000, 128, 64, 64, 0, True), (16000, 1024, 16, 64, 0, False)])
def test_which_decodes_make_a_table(V, d, R, T, top_k, table):
    """The library's own choice, as it runs: a product and a walk for a table, a product a step otherwise."""
    model, ctx, prompts, u, _ = _setup(V, d, 1, R, "bf16", "bf16", 3.0)
    prompts[0] = 7
    out = torch.empty((1, R, T), dtype=torch.int32, device="cuda")
    ctx.profile(True)
    B.as_decode(ctx, model, prompts, R, T, u, 1.0, top_k, 1.0, 1, out)
    assert (ctx.profile_read(1)[1] == 1 and ctx.profile_read(0)[1] == 1) == table
    ctx.profile(False)
    want = out.clone()
    B.as_decode(ctx, model, prompts, R, T, u, 1.0, top_k, 1.0, 1, out)
    assert torch.equal(out, want)
    ctx.close()
    model.close()


def _logits_launches(ctx, call):
    ctx.profile(True)
    call()
    n = ctx.profile_read(1)[1]
    ctx.profile(False)
    return n


@pytest.mark.parametrize("V,d,Bn,N,T,top_k,top_p,wdt,ldt,temp,scale", CASES)
def test_decode_from_a_table_equals_the_loop_of_exported_calls(V, d, Bn, N, T, top_k, top_p, wdt, ldt, temp, scale):
    _compare(V, d, Bn, N, T, top_k, top_p, wdt, ldt, temp, scale, 3, 1)


# bf16 weights, ranks of whole K steps, rows of one tile; rounds that are enough (as many as steps), and those after which
# all rows are made
@pytest.mark.parametrize("V,d,Bn,N,T,top_k,top_p,wdt,ldt,temp,scale",
                         [c for c in CASES if c[7] == "bf16" and c[1] >= 128 and c[0] % 8 == 0 and c[9] > 0.37 and c[5] < 48] +
                         [(4096, 128, 2, 150, 5, 0, 1.0, "bf16", "bf16", TEMP, 3.0), (4096, 128, 1, 900, 7, 0, 0.9, "bf16", "bf16", TEMP, 3.0),
                          (8192, 128, 3, 60, 130, 0, 1.0, "bf16", "f32", TEMP, 3.0)])
def test_rows_on_demand_equal_the_loop_of_exported_calls(V, d, Bn, N, T, top_k, top_p, wdt, ldt, temp, scale):
    _compare(V, d, Bn, N, T, top_k, top_p, wdt, ldt, temp, scale, 5, min(T, 7))


def _compare(V, d, Bn, N, T, top_k, top_p, wdt, ldt, temp, scale, knob, launches):
    model, ctx, prompts, u, g = _setup(V, d, Bn, N, wdt, ldt, scale)
    R = Bn * N
    ctx.set_tuning("kept_rows", knob)                     # (whatever the rule comes to be)
    out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
    last = torch.empty(R, dtype=torch.float32, device="cuda")

    def decode():
        B.as_decode(ctx, model, prompts, N, T, u, temp, top_k, top_p, eos, out, codes_out=last)

    eos = -1
    decode()
    eos = int(out.view(R, T)[:, T // 3].mode().values)    # a token that some codes end with, at different steps
    decode()                                              # (on the tables that the call before has left)
    codes = torch.empty(R, dtype=torch.float32, device="cuda")
    B.as_lattice(ctx, u, N, codes)
    want, want_codes = _loop(ctx, model, prompts, N, T, codes, None, temp, top_k, top_p, eos, ldt)
    assert torch.equal(out.view(R, T), want) and torch.equal(last, want_codes)
    assert (want == eos).any()
    out.fill_(-1)
    assert _logits_launches(ctx, decode) == launches      # (that was what ran)
    assert torch.equal(out.view(R, T), want) and torch.equal(last, want_codes)

    uniforms = torch.rand(T, R, device="cuda", generator=g).clamp_max_(1.0 - 2.0 ** -24)
    B.as_decode_ancestral(ctx, model, prompts, N, T, uniforms, temp, top_k, top_p, eos, out)
    want, _ = _loop(ctx, model, prompts, N, T, codes, uniforms, temp, top_k, top_p, eos, ldt)
    assert torch.equal(out.view(R, T), want)
    ctx.close()
    model.close()


@pytest.mark.parametrize("hot", [0, 100, 2000])
def test_rows_are_made_for_the_tokens_that_come(hot):
    """Wide decodes on all tokens, and on a few that hold nearly all the mass: as the rule has it, against a row a token and
    step; the same tokens."""
    V, d, R, T = 32128, 512, 16384, 16
    g = torch.Generator(device="cuda").manual_seed(hot)
    E, U = torch.randn(V, d, device="cuda", generator=g), torch.randn(d, V, device="cuda", generator=g)
    if hot:
        E[:, 0] = 4.0
        bias = torch.full((V,), -20.0, device="cuda")
        bias[torch.randperm(V, device="cuda", generator=g)[:hot]] = 0.0
        U[0] = bias / (3.0 / d ** 0.5 * 4.0)
    model, ctx = B.Model(E.bfloat16(), U.bfloat16(), scale=3.0), B.Ctx(R, V, torch.bfloat16)
    prompts, u = torch.tensor([5], dtype=torch.int32, device="cuda"), torch.rand(1, device="cuda", generator=g)
    outs = []
    for knob in (0, 1):
        ctx.set_tuning("kept_rows", knob)
        out = torch.empty((1, R, T), dtype=torch.int32, device="cuda")
        n = _logits_launches(ctx, lambda: B.as_decode(ctx, model, prompts, R, T, u, 1.0, 0, 1.0, -1, out))
        assert n == (7 if knob == 0 else T)
        outs.append(out)
    assert torch.equal(*outs)
    if hot:
        assert torch.unique(outs[0]).numel() < 1.2 * hot + 50
    ctx.close()
    model.close()


def test_fused_decode_from_a_table():
    V, d, Bn, N, T = 6007, 128, 2, 100, 20
    model, ctx, prompts, u, _ = _setup(V, d, Bn, N, "bf16", "bf16", 3.0)
    outs = []
    for knob in (3, 1):
        ctx.set_tuning("kept_rows", knob)
        out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
        n = _logits_launches(ctx, lambda: B.as_decode_fused(ctx, model, prompts, N, T, u, TEMP, 1, out))
        assert n == (1 if knob == 3 else T)
        outs.append(out)
    assert torch.equal(*outs)
    ctx.close()
    model.close()


@pytest.mark.parametrize("knob", [3, 5])
@pytest.mark.parametrize("top_k,ldt", [(0, "bf16"), (10, "bf16"), (0, "f32")])
def test_decode_from_a_table_replays_from_a_graph(top_k, ldt, knob):
    V, d, Bn, N, T = 16000, 128, 2, 100, 66
    model, ctx, prompts, u, _ = _setup(V, d, Bn, N, "bf16", ldt, 3.0)
    ctx.close()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx = B.Ctx(Bn * N, V, DT[ldt])
        ctx.set_tuning("kept_rows", knob)
        out = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
        eager = torch.empty_like(out)
        B.as_decode(ctx, model, prompts, N, T, u, TEMP, top_k, 1.0, 1, out)       # (makes the workspace)
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        B.as_decode(ctx, model, prompts, N, T, u, TEMP, top_k, 1.0, 1, out)
    for i in range(4):
        with torch.cuda.stream(stream):
            u.uniform_(0.0, 0.99)
            out.fill_(-1)
            graph.replay()
            got = out.clone()
            B.as_decode(ctx, model, prompts, N, T, u, TEMP, top_k, 1.0, 1, eager)
        stream.synchronize()
        assert torch.equal(got, eager), f"replay {i}"
    # the table is a choice: without its memory the decode takes a row per code
    other = B.Ctx(Bn * N, V, DT[ldt])
    other.set_tuning("workspace_mib", 100)
    B.as_decode(other, model, prompts, N, T, u, TEMP, top_k, 1.0, 1, out)
    torch.cuda.synchronize()
    assert torch.equal(out, eager) and B.lib().as_last_error(other._h) == b""
    other.close()
    ctx.close()
    model.close()


@pytest.mark.parametrize("top_k", [0, 10])
def test_decode_without_the_memory_for_the_records(top_k):
    """They are 17 MB, a row per code 2 and the rest of the state a third of one: a cap between them takes the table away,
    not the decode."""
    V, d, N, T = 16000, 128, 64, 64
    model, ctx, prompts, u, _ = _setup(V, d, 2, N // 2, "bf16", "bf16", 3.0)
    ctx.set_tuning("kept_rows", 3)
    out = torch.empty((2, N // 2, T), dtype=torch.int32, device="cuda")
    assert _logits_launches(ctx, lambda: B.as_decode(ctx, model, prompts, N // 2, T, u, TEMP, top_k, 1.0, 1, out)) == 1
    small = B.Ctx(N, V, torch.bfloat16)
    small.set_tuning("workspace_mib", 10)
    got = torch.empty_like(out)
    for _ in range(2):
        B.as_decode(small, model, prompts, N // 2, T, u, TEMP, top_k, 1.0, 1, got)
        torch.cuda.synchronize()
        assert torch.equal(got, out) and B.lib().as_last_error(small._h) == b""
    small.close()
    ctx.close()
    model.close()
