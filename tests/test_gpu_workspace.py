"""What a call may do to the context's workspace: a call of the same or a smaller size than an earlier one allocates nothing,
can be captured, and leaves alone the buffers that a graph captured before it works on, whatever form it takes; what
cannot be had is done without."""
import pytest
import torch

from paper_2210_15458_amd import binding as B

pytestmark = pytest.mark.gpu

EOS, TEMP = 1, 1.1


class Job:
    """A model, a context on a stream of its own, and decodes and encodes on it."""

    def __init__(self, V, d, rows, ldt=torch.bfloat16, wdt=torch.bfloat16):
        g = torch.Generator(device="cuda").manual_seed(V)
        self.V = V
        self.model = B.Model(torch.randn(V, d, device="cuda", generator=g).to(wdt),
                             torch.randn(d, V, device="cuda", generator=g).to(wdt), scale=3.0)
        self.prompts = torch.randint(0, V, (1,), device="cuda", generator=g, dtype=torch.int32)
        self.u = torch.rand(1, device="cuda", generator=g)
        self.stream = torch.cuda.Stream()
        torch.cuda.synchronize()
        self.tokens = torch.randint(0, V, (min(rows, 256), 300), device="cuda", generator=g, dtype=torch.int32)
        self.columns = {}
        self.rows, self.ldt = rows, ldt
        self.ctx = self.context()

    def context(self):
        with torch.cuda.stream(self.stream):
            return B.Ctx(self.rows, self.V, self.ldt)

    def decode(self, N, T, temp=TEMP, top_k=0, ctx=None, out=None):
        with torch.cuda.stream(self.stream):
            out = torch.empty((1, N, T), dtype=torch.int32, device="cuda") if out is None else out
            B.as_decode(ctx or self.ctx, self.model, self.prompts, N, T, self.u, temp, top_k, 1.0, EOS, out)
        return self.done(out)

    def encode(self, N, T, temp=TEMP, top_k=0, ctx=None, out=None):
        """Of tokens that are the same for every call: the first columns of the first sequences."""
        if T not in self.columns:
            self.columns[T] = self.tokens[:, :T].contiguous()
            torch.cuda.synchronize()
        with torch.cuda.stream(self.stream):
            out = tuple(torch.empty(N, dtype=torch.float64, device="cuda") for _ in range(2)) if out is None else out
            B.as_encode(ctx or self.ctx, self.model, self.prompts, N, T, self.columns[T][:N], temp, top_k, 1.0, -1, *out)
        return self.done(out)

    def done(self, out):
        if not torch.cuda.is_current_stream_capturing():
            self.stream.synchronize()
        return out

    def captured(self, call, out):
        """The graph of a call; raises if the call allocates (it would wait for the stream, which a capture refuses)."""
        graph = torch.cuda.CUDAGraph()
        self.stream.synchronize()
        with torch.cuda.graph(graph, stream=self.stream):
            call(out)
        return graph

    def replay(self, graph, out):
        with torch.cuda.stream(self.stream):
            for o in out if isinstance(out, tuple) else (out,):
                o.fill_(-1)
            graph.replay()
        self.stream.synchronize()
        return out

    def close(self):
        self.ctx.close()
        self.model.close()


def test_a_kept_table_that_is_refused_is_not_asked_for_again():
    V, d, N, T = 8000, 512, 4200, 6                       # kept rows: 128 MB, against 67 of a row per code
    job = Job(V, d, N)
    want = job.decode(N, T)
    small = job.context()
    small.set_tuning("workspace_mib", 100)
    assert torch.equal(job.decode(N, T, ctx=small), want)
    assert B.lib().as_last_error(small._h) == b""         # the call succeeded: nothing to report
    # the second call finds its workspace: it neither waits nor moves it
    out = torch.empty_like(want)
    graph = job.captured(lambda o: job.decode(N, T, ctx=small, out=o), out)
    assert torch.equal(job.replay(graph, out), want)
    assert torch.equal(job.decode(N, T, ctx=small), want) and torch.equal(job.replay(graph, out), want)
    other = job.context()
    other.set_tuning("workspace_mib", 10)
    with pytest.raises(B.ArithSamplingError, match="workspace"):
        job.decode(N, T, ctx=other)
    other.close()
    small.close()
    job.close()


def test_kept_rows_where_a_table_of_every_token_is_refused():
    """8000 rows are 128 MB, the 7600 that four steps of 1900 codes can come to 122; a cap between them."""
    V, d, N, T = 8000, 512, 1900, 4
    job = Job(V, d, N)
    want = job.decode(N, T)
    small = job.context()
    small.set_tuning("workspace_mib", 118)
    small.set_tuning("kept_rows", 2)
    small.profile(True)
    assert torch.equal(job.decode(N, T, ctx=small), want)
    assert small.profile_read(0)[1] == 2 * T              # (from sums: two launches a step)
    small.close()
    job.close()


def _same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


# steps, temperature, top-k and rows of calls no larger than a decode of 20000 codes x 8 steps that keeps 8000 rows
OTHERS = [(2, TEMP, 0, 20000), (8, TEMP, 40, 20000), (8, 0.2, 0, 20000), (8, TEMP, 0, 7000), (1, TEMP, 0, 1), (4, TEMP, 3, 2001)]


def test_decodes_no_larger_than_an_earlier_one_leave_its_workspace_alone():
    V, d, N, T = 8000, 512, 20000, 8                      # a row per code: 320 MB
    job = Job(V, d, N)
    own = job.context()                                   # for what the other calls give on a workspace of their own
    want = job.decode(N, T)
    out = torch.empty_like(want)
    others = [(o, job.decode(o[3], o[0], o[1], o[2], ctx=own)) for o in OTHERS]
    outs = [torch.empty_like(w) for _, w in others]
    graph = job.captured(lambda o: job.decode(N, T, out=o), out)
    before = _free()
    for (o, w), buf in zip(others, outs):
        assert torch.equal(job.decode(o[3], o[0], o[1], o[2], out=buf), w), o
        assert abs(_free() - before) < 32 << 20, o        # (the runtime's own, not the workspace)
    assert torch.equal(job.replay(graph, out), want)
    # and each of them can be captured on a context that has seen the largest alone
    own.close()
    own = job.context()
    assert torch.equal(job.decode(N, T, ctx=own, out=out), want)
    for (o, w), buf in zip(others, outs):
        g = job.captured(lambda b, o=o: job.decode(o[3], o[0], o[1], o[2], ctx=own, out=b), buf)
        for _ in range(3):
            assert torch.equal(job.replay(g, buf), w), o
            assert torch.equal(job.decode(N, T, ctx=own, out=out), want)
    own.close()
    job.close()


# columns, temperature, top-k and sequences of calls no larger than an encode of 100 x 300: without shared rows, sums or
# truncation, or with them
ENCODES = [(100, TEMP, 0, 100), (300, 0.2, 0, 100), (300, TEMP, 30, 100), (300, TEMP, 0, 60), (20, TEMP, 5, 37), (1, TEMP, 0, 1)]


def test_encodes_no_larger_than_an_earlier_one_leave_its_workspace_alone():
    V, d, N, T = 2000, 128, 100, 300                      # a row per token: 16 MB; a row per position of 100 columns: 64
    job = Job(V, d, N, ldt=torch.float32)
    own = job.context()
    want = job.encode(N, T)
    out = tuple(torch.empty_like(w) for w in want)
    others = [(o, job.encode(o[3], o[0], o[1], o[2], ctx=own)) for o in ENCODES]
    outs = [tuple(torch.empty_like(x) for x in w) for _, w in others]
    graph = job.captured(lambda o: job.encode(N, T, out=o), out)
    before = _free()
    for (o, w), buf in zip(others, outs):
        assert _same(job.encode(o[3], o[0], o[1], o[2], out=buf), w), o
        assert abs(_free() - before) < 16 << 20, o
    assert _same(job.replay(graph, out), want)
    own.close()
    own = job.context()
    assert _same(job.encode(N, T, ctx=own, out=out), want)
    for (o, w), buf in zip(others, outs):
        g = job.captured(lambda b, o=o: job.encode(o[3], o[0], o[1], o[2], ctx=own, out=b), buf)
        for _ in range(3):
            assert _same(job.replay(g, buf), w), o
            assert _same(job.encode(N, T, ctx=own, out=out), want)
    own.close()
    job.close()


def test_an_encode_leaves_a_captured_decode_alone():
    V, d, N = 8000, 128, 40
    job = Job(V, d, N)
    want = job.decode(N, 64)
    out = torch.empty_like(want)
    graph = job.captured(lambda o: job.decode(N, 64, out=o), out)
    for T in (64, 200, 300):                              # (wants more rows of logits than the decode has)
        job.encode(N, T)
        assert torch.equal(job.replay(graph, out), want)
    job.close()


@pytest.mark.parametrize("V,d,N,ldt,top_k", [(8000, 512, 40, torch.bfloat16, 0), (8001, 128, 1100, torch.bfloat16, 20),
                                             (3000, 24, 1025, torch.float32, 0)])
def test_an_encode_does_with_the_workspace_of_a_decode(V, d, N, ldt, top_k):
    """Where its own is refused, and under a capture that comes before any encode: the same bits."""
    T = 90
    job = Job(V, d, N, ldt=ldt)
    job.tokens = torch.randint(0, V, (N, T), device="cuda", dtype=torch.int32)
    want = job.encode(N, T, top_k=top_k)
    small = job.context()
    small.set_tuning("workspace_mib", 30)                 # (a row per sequence fits: 17 MB)
    assert _same(job.encode(N, T, top_k=top_k, ctx=small), want)
    assert B.lib().as_last_error(small._h) == b""
    out = tuple(torch.empty_like(w) for w in want)
    graph = job.captured(lambda o: job.encode(N, T, top_k=top_k, ctx=small, out=o), out)
    assert _same(job.replay(graph, out), want)
    small.close()
    fresh = job.context()
    tokens = job.decode(N, T, ctx=fresh)
    graph = job.captured(lambda o: job.encode(N, T, top_k=top_k, ctx=fresh, out=o), out)
    for _ in range(3):
        assert _same(job.replay(graph, out), want)
        assert torch.equal(job.decode(N, T, ctx=fresh), tokens)
        assert _same(job.encode(N, T, top_k=top_k, ctx=fresh), want)     # (on its own from here on)
    fresh.close()
    job.close()


@pytest.mark.parametrize("V,d,N", [(201, 24, 60), (16, 8, 64)])
def test_a_decode_in_one_launch_leaves_the_workspace_of_its_size(V, d, N):
    """It needs none itself, but the same call truncated, or over one step, does, and can be captured after it."""
    job = Job(V, d, N, ldt=torch.float32, wdt=torch.float32)
    own = job.context()
    others = [(8, TEMP, 3), (1, TEMP, 0), (5, 0.2, 2), (8, 0.1, 0)]
    want = [job.decode(N, T, temp, top_k, ctx=own) for T, temp, top_k in others]
    job.decode(N, 8)
    for (T, temp, top_k), w in zip(others, want):
        out = torch.empty_like(w)
        graph = job.captured(lambda o: job.decode(N, T, temp, top_k, out=o), out)
        for _ in range(3):
            assert torch.equal(job.replay(graph, out), w)
            job.decode(N, 8)
    own.close()
    job.close()


def test_a_short_decode_makes_room_for_its_table_only_as_the_first_of_its_size():
    V, d, N = 32128, 512, 8000                            # rows kept: 1.5 GB over four steps, against 0.5 of a row per code
    job = Job(V, d, N)
    want = job.decode(N, 4)                               # (the first: with the table)
    job.close()
    job = Job(V, d, N)
    long = job.decode(N, 6)
    out = torch.empty_like(long)
    graph = job.captured(lambda o: job.decode(N, 6, out=o), out)
    got = torch.empty_like(want)
    before = _free()
    assert torch.equal(job.decode(N, 4, out=got), want) and torch.equal(job.decode(N, 3, out=got[:, :, :3].contiguous()), want[:, :, :3])
    assert abs(_free() - before) < 64 << 20
    assert torch.equal(job.replay(graph, out), long)
    job.close()
