"""The work that the arithmetic-sampling library is timed on, through its public entry points.

Six kinds of call, as a user's program makes them:
  decode      whole decode of N lattice codes per prompt under the bigram model (as_decode)
  fused       the same without the logits round trip (as_decode_fused)
  estimate    lattice decode, then the estimator over its tokens (as_decode, as_estimate_mean)
  ancestral   decode from the caller's own uniforms (as_decode_ancestral)
  encode      code intervals of given sequences (as_encode)
  step        one sampling step on logits the caller brings, as a serving loop calls it (as_step_ex)

listed() are the benchmark's configurations and the ordinary calls around them; draw() gives more of the same
ranges.  prepare() makes inputs on the GPU from the seed alone; run() is one pass; work() is what a pass
cannot do without; tolerance() how far another correct implementation may be.
"""
import math

import torch

from paper_2210_15458_amd import binding as B

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
SCALE = 3.0      # the bigram model's logit scale: each logit close to N(0, 9)
EOS = 1


def _decode(name, kind, V, d, prompts, codes, steps, temp, top_k=0, top_p=1.0, weights="bf16", logits="bf16"):
    case = {"kind": kind, "V": V, "d": d, "prompts": prompts, "codes": codes, "steps": steps, "temp": temp,
            "top_k": top_k, "top_p": top_p, "weights": weights, "logits": logits}
    return dict(case, name=name) if name else case


def _step(name, rows, V, temp, top_k, top_p, logits, pad=0, finished=0.0):
    case = {"kind": "step", "rows": rows, "V": V, "temp": temp, "top_k": top_k, "top_p": top_p, "logits": logits,
            "pad": pad, "finished": finished}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest decode: a toy model in fp32, 64 codes of one prompt, eight steps; nothing but launches
        _decode("tiny_decode", "decode", 16, 8, 1, 64, 8, 1.0, weights="f32", logits="f32"),
        # one user's prompt, sixteen diverse continuations: the interactive use of arithmetic sampling
        _decode("prompt_decode", "decode", 32128, 512, 1, 16, 64, 0.7),
        # the headline workload: a batch of prompts, 64 codes each
        _decode("batch_decode", "decode", 32128, 512, 16, 64, 64, 0.7),
        # a very wide lattice on one prompt: the largest call
        _decode("wide_decode", "decode", 32128, 512, 1, 65536, 16, 1.0),
        # many prompts, few codes, top-k, and the lattice estimator over the result
        _decode("topk_estimate", "estimate", 32128, 512, 64, 16, 128, 1.0, top_k=40),
        # a large vocabulary, decoded without writing the logits
        _decode("large_vocab_fused", "fused", 256000, 1024, 8, 128, 32, 1.0),
        # a small fp32 model sampled ancestrally (the comparison method), fp32 logits
        _decode("f32_ancestral", "ancestral", 4100, 128, 8, 32, 32, 0.8, weights="f32", logits="f32"),
        # the encode direction: the intervals of a batch of sequences
        _decode("batch_encode", "encode", 32128, 512, 16, 64, 64, 0.7),
        # one serving step with the nucleus on a full batch of bf16 logits
        _step("step_nucleus", 1024, 32128, 1.0, 0, 0.9, "bf16"),
        # a large vocabulary with top-k and nucleus together, some sequences of the batch already ended
        _step("step_large_vocab", 256, 256000, 0.8, 50, 0.95, "bf16", finished=0.1),
        # fp32 logits whose rows start off 16 bytes (a contiguous tensor of odd width), nucleus
        _step("step_f32_odd", 512, 50257, 0.7, 0, 0.92, "f32"),
        # the smallest serving call: one row
        _step("step_one_row", 1, 50257, 0.8, 0, 0.95, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _modifiers(rng):
    """top_k, top_p: each alone, both, or neither."""
    pick = rng.random()
    top_k = rng.choice([1, 5, 20, 40, 50, 64, 100, 200, 1000]) if pick < 0.5 else 0
    top_p = round(rng.uniform(0.5, 0.98), 3) if 0.3 < pick < 0.8 else 1.0
    return top_k, top_p


def draw(rng):
    pick = rng.random()
    temp = round(rng.uniform(0.4, 1.3), 3)
    if pick < 0.40:
        V = _log_int(rng, 1000, 256000)
        rows = _log_int(rng, 1, max(1, min(16384, 520_000_000 // V)))
        top_k, top_p = _modifiers(rng)
        if top_k >= V:
            top_k = 40
        if top_k == 0 and top_p == 1.0:
            top_p = 0.9
        return _step(None, rows, V, temp, top_k, top_p, rng.choice(["bf16", "bf16", "f32"]),
                     pad=rng.choice([0, 0, 8 - V % 8]), finished=rng.choice([0.0, 0.0, 0.25]))
    if pick < 0.48:      # small fp32 models
        V = _log_int(rng, 16, 6000)
        d = _log_int(rng, 8, 160)
        prompts = _log_int(rng, 1, 8)
        codes = _log_int(rng, 1, max(1, min(64, 120_000_000 // (V * d * prompts))))
        return _decode(None, rng.choice(["decode", "ancestral", "encode"]), V, d, prompts, codes,
                       _log_int(rng, 2, 24), temp, weights="f32", logits="f32")
    kind = rng.choice(["decode", "decode", "decode", "fused", "estimate", "ancestral", "encode", "encode"])
    V = _log_int(rng, 2000, 256000)
    d = 64 * rng.randint(2, 16)
    steps = _log_int(rng, 2, 64)
    # total work at most the wide lattice's: rows x steps x V x d, and a logits tensor of at most 4 GB
    most = min(65536, int(1.7e13 / (float(V) * d * steps)), 2_000_000_000 // V)
    if kind == "encode":
        most = min(most, 2048)           # (its sequences are sampled in prepare)
    rows = _log_int(rng, 1, max(1, most))
    prompts = _log_int(rng, 1, min(rows, 64))
    codes = max(1, rows // prompts)
    logits = "bf16" if kind == "fused" else rng.choice(["bf16", "bf16", "bf16", "f32"])
    top_k, top_p = (0, 1.0)
    if kind == "ancestral" and rng.random() < 0.7:
        top_k, top_p = _modifiers(rng)
    elif kind == "encode" and rng.random() < 0.6:
        top_k = rng.choice([10, 40, 100])
    elif kind == "estimate" and V <= 32768:
        top_k = rng.choice([10, 40])
    return _decode(None, kind, V, d, prompts, codes, steps, temp, top_k, top_p, "bf16", logits)


def _sequences(case, E, U, prompts, g):
    """Token sequences [B, N, T] sampled from the model (EOS sticky): what as_encode is given."""
    V, d, N, T = case["V"], case["d"], case["codes"], case["steps"]
    R = prompts.numel() * N
    Uf = U.float()
    prev = prompts.long().repeat_interleave(N)
    out = torch.empty((R, T), dtype=torch.int32, device="cuda")
    ended = torch.zeros(R, dtype=torch.bool, device="cuda")
    for t in range(T):
        x = (E[prev].float() @ Uf) * (SCALE / math.sqrt(d))
        if case["top_k"]:
            # well inside the top k: the k-th place can differ by how the logits are rounded
            keep = max(1, case["top_k"] // 2)
            x = x.masked_fill(x < x.topk(keep, dim=1).values[:, -1:], -math.inf)
        noise = torch.empty_like(x).exponential_(generator=g).clamp_min_(1e-30)
        nxt = (x / case["temp"] - noise.log_()).argmax(dim=1)
        nxt = torch.where(ended, torch.full_like(nxt, EOS), nxt)
        ended |= nxt == EOS
        out[:, t] = nxt.int()
        prev = nxt
    return out.view(prompts.numel(), N, T).contiguous()


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    V = case["V"]
    ldt = DTYPES[case["logits"]]
    s = {"case": case}

    def codes_in(*shape):
        return torch.rand(*shape, device="cuda", generator=g).clamp_max_(1.0 - 2.0 ** -24)

    if case["kind"] == "step":
        rows, ld = case["rows"], V + case["pad"]
        # next-token logits, some rows flatter and some more confident than others
        x = torch.randn(rows, ld, device="cuda", generator=g)
        x *= torch.empty(rows, 1, device="cuda").uniform_(2.0, 4.0, generator=g)
        s["logits"] = x.to(ldt)
        s["u"] = codes_in(rows)
        s["ctx"] = B.Ctx(rows, V, ldt)
        s["tokens"] = torch.empty(rows, dtype=torch.int32, device="cuda")
        s["codes"] = torch.empty(rows, dtype=torch.float32, device="cuda")
        s["fin"] = None
        if case["finished"] > 0:
            s["fin"] = (torch.rand(rows, device="cuda", generator=g) < case["finished"]).to(torch.uint8)
            s["fin_out"] = torch.empty_like(s["fin"])
        return s

    wdt = DTYPES[case["weights"]]
    Bn, N, T, d = case["prompts"], case["codes"], case["steps"], case["d"]
    s["E"] = torch.randn(V, d, device="cuda", generator=g).to(wdt)
    U = torch.randn(d, V, device="cuda", generator=g).to(wdt)
    s["model"] = B.Model(s["E"], U, scale=SCALE)
    s["prompts"] = torch.randint(0, V, (Bn,), device="cuda", generator=g, dtype=torch.int32)
    s["u"] = codes_in(Bn)
    s["ctx"] = B.Ctx(Bn * N, V, ldt)
    if case["kind"] == "encode":
        s["tokens"] = _sequences(case, s["E"], U, s["prompts"], g)
        s["lo"] = torch.empty(Bn * N, dtype=torch.float64, device="cuda")
        s["width"] = torch.empty(Bn * N, dtype=torch.float64, device="cuda")
        return s
    s["tokens"] = torch.empty((Bn, N, T), dtype=torch.int32, device="cuda")
    if case["kind"] == "ancestral":
        s["uniforms"] = codes_in(T, Bn * N)
    if case["kind"] == "estimate":
        s["score"] = torch.randn(V, device="cuda", generator=g)
        s["est"] = torch.empty(Bn, dtype=torch.float64, device="cuda")
    return s


def run(s):
    c = s["case"]
    kind, temp, top_k, top_p = c["kind"], c["temp"], c["top_k"], c["top_p"]
    if kind == "step":
        if s["fin"] is None:
            B.as_step(s["ctx"], s["logits"], s["u"], temp, top_k, top_p, s["tokens"], s["codes"])
            return s["tokens"], s["codes"]
        B.as_step_ex(s["ctx"], s["logits"], s["u"], temp, top_k, top_p, s["tokens"], s["codes"],
                     finished_in=s["fin"], eos_id=EOS, finished_out=s["fin_out"])
        return s["tokens"], s["codes"], s["fin_out"]
    N, T = c["codes"], c["steps"]
    if kind == "encode":
        B.as_encode(s["ctx"], s["model"], s["prompts"], N, T, s["tokens"], temp, top_k, top_p, EOS, s["lo"], s["width"])
        return s["lo"], s["width"]
    if kind == "fused":
        B.as_decode_fused(s["ctx"], s["model"], s["prompts"], N, T, s["u"], temp, EOS, s["tokens"])
    elif kind == "ancestral":
        B.as_decode_ancestral(s["ctx"], s["model"], s["prompts"], N, T, s["uniforms"], temp, top_k, top_p, EOS,
                              s["tokens"])
    else:
        B.as_decode(s["ctx"], s["model"], s["prompts"], N, T, s["u"], temp, top_k, top_p, EOS, s["tokens"])
        if kind == "estimate":
            B.as_estimate_mean(s["ctx"], s["tokens"], s["score"], EOS, s["est"])
            return s["tokens"], s["est"]
    return s["tokens"]


def work(case):
    V = case["V"]
    esz = 2 if case["logits"] == "bf16" else 4
    if case["kind"] == "step":
        rows = case["rows"]
        live = rows * (1.0 - case["finished"])
        # the logits of the rows still running, codes in and out, tokens; per logit a multiply-add, an exponential
        # and an addition
        return {"bytes": live * V * esz + rows * 12.0, "flops": live * V * 4.0}
    wsz = 2 if case["weights"] == "bf16" else 4
    R, T, d = case["prompts"] * case["codes"], case["steps"], case["d"]
    # Per step: the output matrix once, the embedding rows in use, the sampling state and the tokens (no logits:
    # they need not reach memory); the logits product of every row that conditions on a token of its own (at
    # most V of them; in the first step the prompts), and the sampling arithmetic per row and token.
    own = [min(R, V, case["prompts"] if t == 0 else R) for t in range(T)]
    flops = sum(2.0 * o * V * d + 4.0 * R * V for o in own)
    byts = sum(float(V) * d * wsz + o * d * wsz for o in own) + T * R * 12.0
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["kind"] == "step":
        # one token in a few hundred thousand may fall to the other side of an interval end (sums of fp32 weights
        # in another order); the next code is a difference of such sums divided by the token's probability
        return {"rel": 0.02, "max": 0.9, "differ": 0.004}
    if case["kind"] == "encode":
        # fp64 intervals of products of fp32-accurate probabilities, one factor a step
        return {"rel": 1e-4, "max": 1e-3}
    # tokens; a row whose code once falls to the other side of an interval end differs from there on
    return {"rel": 0.01, "max": 0.5, "differ": 0.01}
