"""The estimator over sequences of any number and length, against plain fp64 sums."""
import numpy as np
import pytest
import torch

from paper_2210_15458_amd import binding as B

pytestmark = pytest.mark.gpu


# one token, lengths that fill a share of a wave, a whole one, and more than one; more sequences than a block has places
@pytest.mark.parametrize("Bn,N,T", [(1, 1, 1), (3, 1100, 1), (2, 37, 3), (5, 70, 33), (2, 17, 64), (3, 5, 65), (1, 33, 200),
                                    # one wave and four a prompt, with more sequences than they hold
                                    (5000, 70, 1), (4097, 3, 40), (2000, 9, 40)])
@pytest.mark.parametrize("eos", [-1, 1])
def test_estimate_of_any_shape(Bn, N, T, eos):
    V = 50
    rng = np.random.default_rng(T)
    tokens = rng.integers(0, V, (Bn, N, T)).astype(np.int32)
    tokens[rng.random(tokens.shape) < 0.02] = V + 3              # outside: no score
    score = rng.standard_normal(V).astype(np.float32)
    alive = np.ones(tokens.shape, bool)
    if eos >= 0:
        alive[:, :, 1:] = np.cumsum(tokens == eos, axis=2)[:, :, :-1] == 0
    values = np.where(tokens < V, score.astype(np.float64)[np.minimum(tokens, V - 1)], 0.0)
    want = (values * alive).sum(axis=(1, 2)) / N
    ctx = B.Ctx(1, V, torch.float32)
    est = torch.empty(Bn, dtype=torch.float64, device="cuda")
    B.as_estimate_mean(ctx, torch.from_numpy(tokens).cuda(), torch.from_numpy(score).cuda(), eos, est)
    torch.cuda.synchronize()
    # fp64 sums of N*T terms of size 1 in another order
    assert np.allclose(est.cpu().numpy(), want, rtol=0, atol=N * T * 2.0 ** -50)
    ctx.close()
