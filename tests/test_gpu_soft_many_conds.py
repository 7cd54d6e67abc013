"""A population past 2^28 conditions (4 GiB of condition records): the relaxed
path reads each rule set's own parameters, in the forward and in the reverse
sweep of both heads.  The last rule sets, whose records lie past 4 GiB, give
the losses and gradients they give as a population of their own; the first
ones hold other parameters.  One feature and one tile of samples, so that the
run is the packing and a few launches."""
import numpy as np
import pytest

from paper_2406_01821_amd.population import Dataset, Population

pytestmark = pytest.mark.gpu

RULES, CONDS = 4, 255  # a rule set: the longest rules, 1020 conditions


def population(coef, n_sets):
    """Rule sets of threshold conditions coef * x > coef (on one feature, so
    the array that holds the coefficients holds the thresholds too)."""
    n = len(coef)
    zero = lambda m, t: np.zeros(m, t)  # pages of zeros: no memory behind them
    return Population(np.arange(n_sets + 1) * RULES, zero(n_sets, np.int32),
                      np.arange(n_sets * RULES + 1) * CONDS,
                      np.arange(n_sets * RULES) % RULES % 2, np.broadcast_to(np.uint8(2), n).copy(),
                      zero(n, np.uint8), zero(n, np.int32), zero(n, np.int32), coef, coef, coef)


def outputs(ctx, ds, pop, coef, last):
    """The last rule sets' losses and gradients under both heads."""
    import torch
    p = ctx.pack_population(pop, 1, 2)
    v = torch.tensor(coef, device=ctx.device)
    one = torch.ones(pop.n_sets, device=ctx.device)
    out = []
    for fwd, bwd in ((ctx.soft_forward(ds, p, v, v, v), lambda: ctx.soft_backward(ds, p, v, v, v, one)),
                     (ctx.softmax_forward(ds, p, v, v, v, 2.0),
                      lambda: ctx.softmax_backward(ds, p, v, v, v, 2.0, one))):
        out.append(fwd[-last:].cpu().numpy())
        g = bwd()
        out += [g[0][-last * RULES * CONDS:].cpu().numpy(), g[2][-last * RULES * CONDS:].cpu().numpy()]
        del g
    ctx.release_population(p)
    return out


def test_records_past_4_gib():
    import torch
    from paper_2406_01821_amd.aerl import Context
    ctx = Context(0)
    rng = np.random.default_rng(5)
    x = (1.0 + rng.exponential(size=(200, 1))).astype(np.float32)
    ds = ctx.upload_dataset(Dataset(x, (np.arange(200) % 2).astype(np.int32), 2))
    per, last = RULES * CONDS, 3
    n_sets = (1 << 28) // per + 1 + last
    coef = np.full(n_sets * per, np.float32(0.02))
    tail = rng.uniform(0.05, 0.15, last * per).astype(np.float32)
    coef[-last * per:] = tail
    assert n_sets * per - last * per >= 1 << 28
    small = outputs(ctx, ds, population(tail, last), tail, last)
    big = outputs(ctx, ds, population(coef, n_sets), coef, last)
    torch.cuda.synchronize()
    ctx.close()
    torch.cuda.empty_cache()
    for a, b in zip(big, small):
        # the plans may split the one tile's sums differently
        np.testing.assert_allclose(a, b, rtol=1e-5, atol=1e-6 * np.abs(b).max())
