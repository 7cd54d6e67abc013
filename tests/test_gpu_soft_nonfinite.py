"""A parameter that is not a number shows in the relaxed path's results on
every table size, also where tiles leave conditions out (16 tiles and more)
and where a rule's terms would be skipped as zeros: the samples of its rule
set take the capped loss and its own gradient is NaN, while the other rule
sets' results stay bit for bit as they are without it.

The NaN sits in the first rule, so every route to a class passes it: log P of
every sample is NaN or -inf, and its loss the cap of 100.  The condition's
term of the gradient is a factor 1 / (1 + u) with u = e^-|z| NaN.  Under the
softmax head every vote is NaN with it, and with it every gradient of the
rule set.  A second condition of the rule is far out of reach on every tile
(the rule is one that a tile rules out)."""
import numpy as np
import pytest

from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import from_rule_lists

pytestmark = pytest.mark.gpu

S = 2  # the rule set with the parameter


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def results(ctx, w, p, ds, params):
    import torch
    v = [torch.tensor(a, device=ctx.device) for a in params]
    one = torch.ones(w.pop.n_sets, device=ctx.device)
    out = [ctx.soft_forward(ds, p, *v), *ctx.soft_backward(ds, p, *v, one),
           ctx.softmax_forward(ds, p, *v, 2.0), *ctx.softmax_backward(ds, p, *v, 2.0, one)]
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("n,nf,rules,far", [(700, 9, (1, 8), False), (700, 9, (1, 8), True),
                                            (5000, 9, (1, 8), False), (5000, 9, (1, 8), True),
                                            (5000, 100, (9, 24), True), (9000, 200, (33, 40), True)])
@pytest.mark.parametrize("kind,which", [(0, "coef"), (0, "theta"), (1, "coef"), (1, "coef2")])
def test_nan_shows(ctx, n, nf, rules, far, kind, which):
    w = synth.tiny(n + nf, n=n, nf=nf, n_classes=3, n_sets=6, rules=rules, conds=(1, 4), ff_frac=0.3)
    sets = [w.pop.to_rule_list(s) for s in range(6)]
    odd = (dict(op=2, kind=0, f=1, coef=0.5, theta=1.0) if kind == 0 else
           dict(op=2, kind=1, f=1, g=2, coef=0.5, coef2=0.25))
    never = dict(op=2, kind=0, f=3, coef=1.0, theta=1e6)
    sets[S][1].insert(0, (1, [odd] + ([never] if far else [])))
    w.pop = from_rule_lists(sets)
    ds = ctx.upload_dataset(w.data)
    p = ctx.pack_population(w.pop, nf, 3)
    j0, j1 = (int(w.pop.rule_cond_off[w.pop.set_rule_off[s]]) for s in (S, S + 1))
    params = dict(coef=w.pop.coef, coef2=w.pop.coef2, theta=w.pop.theta)
    plain = results(ctx, w, p, ds, params.values())
    params[which] = params[which].copy()
    params[which][j0] = np.nan
    got = results(ctx, w, p, ds, params.values())
    others = np.arange(6) != S
    outside = np.r_[0:j0, j1:w.pop.n_conds]
    for head in (0, 4):
        assert got[head][S] == 100.0
        assert np.array_equal(got[head][others], plain[head][others])
        own = np.arange(j0, j0 + 1) if head == 0 else np.arange(j0, j1)
        ff = w.pop.kind[own] == 1
        assert np.isnan(got[head + 1][own]).all()
        assert np.isnan(got[head + 2][own[ff]]).all() and np.isnan(got[head + 3][own[~ff]]).all()
        for a, b in zip(got[head + 1:head + 4], plain[head + 1:head + 4]):
            assert np.array_equal(a[outside], b[outside])


@pytest.mark.parametrize("n", [700, 5000])
def test_a_run_that_diverges_is_one_run(ctx, n):
    """Gradient descent whose first step takes parameters past the float
    range: the records that the update writes for the next epoch mark such a
    rule set as the ones gathered anew after a loss pass do, so a run with a
    loss history and one without end in the same bits."""
    import torch
    w = synth.tiny(n, n=n, nf=9, n_classes=3, n_sets=30, rules=(0, 8), conds=(1, 4), ff_frac=0.3)
    ds = ctx.upload_dataset(w.data)
    p = ctx.pack_population(w.pop, 9, 3)
    out = []
    for hist in (False, True):
        v = [torch.tensor(a, device=ctx.device) for a in (w.pop.coef, w.pop.coef2, w.pop.theta)]
        ctx.finetune(ds, p, *v, 3, optimizer="sgd", lr=3e38, loss_history=hist)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in v])
    assert not all(np.isfinite(a).all() for a in out[0])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
