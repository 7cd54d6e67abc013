"""Fine-tuning of small tables, where one block takes a rule set through every
epoch: one, two and four samples per lane and several rule sets per block (by
population size), one tile to the bound of eight and past it, the table in LDS
and not, rules past the product form, every condition kind, rule sets without
rules, runs longer than a launch; against the fp64 reference loop.

Bound: one epoch's gradient is within the soft-path tolerance (1e-4 of the
entry, floored at 1e-3 of the array's largest).  An update is smooth in the
gradient: gradient descent moves a parameter by lr per unit of gradient, Adam
with eps large against the gradients by at most 2 lr / eps (1/eps from the
mean, 1/eps from the root mean square).  So the parameters drift by at most
the sum over epochs of that times the tolerance, the reference's gradients
staying as they are to first order (twice that is allowed), plus an fp32
rounding per epoch."""
import numpy as np
import pytest

import oracle
from oracle import tune
from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import from_rule_lists

pytestmark = pytest.mark.gpu

LR, EPS = 1e-4, 1.0


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def run(ctx, w, epochs, optimizer, hist=False):
    import torch
    ds = ctx.upload_dataset(w.data)
    p = ctx.pack_population(w.pop, w.data.n_features, w.data.n_classes)
    v = [torch.tensor(a, device=ctx.device) for a in (w.pop.coef, w.pop.coef2, w.pop.theta)]
    h = ctx.finetune(ds, p, *v, epochs, optimizer=optimizer, lr=LR, eps=EPS, loss_history=hist)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in v], None if h is None else h.cpu().numpy()


def check(ctx, w, epochs, optimizer):
    x, y, nc = w.data.x, w.data.y, w.data.n_classes
    tau = oracle.tau(x)
    ps, ls = tune.finetune(x, y, tau, nc, w.pop, epochs, optimizer=optimizer, lr=LR, eps=EPS)
    got, hist = run(ctx, w, epochs, optimizer, hist=True)
    per = LR if optimizer == "sgd" else 2 * LR / EPS
    drift = [np.zeros(w.pop.n_conds) for _ in range(3)]
    for e in range(epochs):
        g = oracle.soft_backward(x, y, tau, nc, w.pop, None, *ps[e])
        drift = [d + per * 1e-4 * np.maximum(np.abs(a), 1e-3 * np.abs(a).max()) + 1.2e-7 * np.abs(q)
                 for d, a, q in zip(drift, g, ps[e])]
    for a, b, d in zip(got, ps[epochs], drift):
        assert np.all(np.abs(a - b) <= 2 * d + 1e-9), np.abs(a - b).max()
    for e in range(epochs + 1):
        np.testing.assert_allclose(hist[e], ls[e], rtol=2e-5, atol=1e-6)
    plain, _ = run(ctx, w, epochs, optimizer)
    for a, b in zip(got, plain):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n,nf,nc,n_sets,rules,conds", [
    (1, 3, 2, 4, (1, 3), (1, 3)),           # one sample
    (256, 8, 1, 5, (1, 8), (1, 4)),         # one tile
    (569, 30, 2, 40, (1, 8), (1, 4)),       # one sample per lane
    (569, 30, 2, 300, (1, 4), (1, 3)),      # two, two rule sets per block
    (500, 6, 2, 901, (1, 3), (1, 2)),       # four, three and a remainder
    (2048, 20, 1, 12, (1, 8), (1, 4)),      # eight tiles
    (2049, 20, 1, 12, (1, 8), (1, 4)),      # nine: the adjoint kernel
    (900, 60, 4, 10, (1, 8), (1, 4)),       # the table past LDS
    (700, 100, 2, 10, (1, 8), (1, 4)),      # two samples per lane at most
    (300, 200, 2, 6, (20, 40), (1, 3)),     # one, many rules
    (400, 12, 2, 4, (1, 2), (61, 70))])     # past the product form
@pytest.mark.parametrize("optimizer", ["adam", "sgd"])
def test_shapes(ctx, n, nf, nc, n_sets, rules, conds, optimizer):
    w = synth.tiny(n + nf, n=n, nf=nf, n_classes=nc, n_sets=n_sets, rules=rules, conds=conds,
                   ff_frac=0.3)
    sets = [w.pop.to_rule_list(s) for s in range(n_sets)]
    sets[0] = (0, [])                                    # no rules
    sets[1][1].insert(0, (0, []))                        # an empty rule first
    sets[-1][1].append((0, [dict(op=0, kind=2, f=0, mask=5), dict(op=2, kind=0, f=1, coef=0.5,
                                                                  theta=1.0)]))
    w.pop = from_rule_lists(sets)
    check(ctx, w, 3, optimizer)


def test_runs_longer_than_a_launch(ctx):
    """260 epochs: the optimizer state goes through the workspace once."""
    w = synth.tiny(31, n=300, nf=5, n_classes=2, n_sets=6, rules=(1, 4), conds=(1, 3), ff_frac=0.3)
    check(ctx, w, 260, "adam")
