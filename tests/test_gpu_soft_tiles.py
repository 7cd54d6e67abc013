"""Tile classification of the relaxed path's conditions (tables of 16 tiles
and more): rules that a tile's feature extremes rule out and conditions that
they saturate are left out.  Parity with the fp64 oracle at rule sets that
cross the 64-condition window, one, two and four samples per lane, infinite
thresholds and both parametric condition kinds; and, bit for bit,
indifference to conditions that every sample passes by far and to rules that
no sample comes near, with rules up to past the window's 64 conditions."""
import numpy as np
import pytest

from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import from_rule_lists
from test_gpu_soft import run_case
from test_gpu_softmax import run_case as run_softmax

pytestmark = pytest.mark.gpu

N = 5000  # 20 tiles or more


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def workload(seed, rules, conds, nf, nc=3, n_sets=10, ff=0.3):
    """Thresholds over the columns' whole ranges, some of them infinite."""
    w = synth.tiny(seed, n=N, nf=nf, n_classes=nc, n_sets=n_sets, rules=rules, conds=conds,
                   ff_frac=ff)
    rng = np.random.default_rng(seed)
    t = w.pop.kind == 0
    pick = t & (rng.random(w.pop.n_conds) < 0.05)
    w.pop.theta[pick] = rng.choice(np.float32([np.inf, -np.inf]), int(pick.sum()))
    return w


@pytest.mark.parametrize("rules,conds,nf,ff", [
    ((1, 8), (1, 4), 9, 0.0), ((9, 16), (4, 8), 16, 0.3), ((17, 32), (1, 4), 8, 0.3),
    ((1, 8), (1, 4), 100, 0.3), ((1, 8), (1, 4), 200, 0.0)])
def test_parity(ctx, rules, conds, nf, ff):
    w = workload(40 + rules[1] + nf, rules, conds, nf, ff=ff)
    run_case(ctx, w.data, w.pop)
    run_softmax(ctx, w.data, w.pop, 2.0)


def _far(w, s):
    """Rule set s with a condition that holds by far added to every rule and a
    rule that no sample comes near after every rule."""
    d, rules = w.pop.to_rule_list(s)
    holds = dict(op=2, kind=0, f=s % w.data.n_features, coef=np.float32(1), theta=np.float32(-1e6))
    never = dict(op=2, kind=0, f=s % w.data.n_features, coef=np.float32(1), theta=np.float32(1e6))
    out = []
    for k, (c, conds) in enumerate(rules):
        at = k % (len(conds) + 1)
        out += [(c, conds[:at] + [holds] + conds[at:]), ((c + k) % w.data.n_classes, [never])]
    return d, out


@pytest.mark.parametrize("rules,conds", [((1, 8), (1, 4)), ((6, 8), (8, 12)), ((2, 4), (30, 50)),
                                         ((2, 3), (60, 70))])
def test_far_conditions_change_nothing(ctx, rules, conds):
    import torch
    w = synth.tiny(90 + conds[1], n=N, nf=12, n_classes=2, n_sets=8, rules=rules, conds=conds,
                   ff_frac=0.3)
    more = from_rule_lists([_far(w, s) for s in range(w.pop.n_sets)])
    ds = ctx.upload_dataset(w.data)
    got = []
    for pop in (w.pop, more):
        p = ctx.pack_population(pop, w.data.n_features, 2)
        v = [torch.tensor(a, device=ctx.device) for a in (pop.coef, pop.coef2, pop.theta)]
        one = torch.ones(pop.n_sets, device=ctx.device)
        kept = np.abs(pop.theta) != np.float32(1e6)
        r = [ctx.soft_forward(ds, p, *v), ctx.softmax_forward(ds, p, *v, 2.0)]
        g = list(ctx.soft_backward(ds, p, *v, one)) + list(ctx.softmax_backward(ds, p, *v, 2.0, one))
        torch.cuda.synchronize()
        got.append([t.cpu().numpy() for t in r] + [t.cpu().numpy()[kept] for t in g])
        assert all(not t.cpu().numpy()[~kept].any() for t in g)
    assert all(np.array_equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("n_rules,nc,nf", [(64, 3, 20), (65, 3, 20), (64, 16, 20), (33, 5, 70),
                                           (64, 4, 130)])
def test_rule_bound_of_the_private_state(ctx, n_rules, nc, nf):
    """Adjoints with 64 rules (state in private memory) and one more (state in
    LDS), at every sample count per lane."""
    w = synth.tiny(n_rules + nc + nf, n=700, nf=nf, n_classes=nc, n_sets=6,
                   rules=(n_rules, n_rules), conds=(1, 3), ff_frac=0.3)
    run_case(ctx, w.data, w.pop)
    run_softmax(ctx, w.data, w.pop, 2.0)


def test_refused_shapes_stay_refused(ctx):
    """512 features with 64 rules exceed the LDS-state adjoint, 320 features
    the softmax head's forward tile; 319 features pass it."""
    import torch
    from paper_2406_01821_amd.aerl import AerlError
    for nf, n_rules, soft, smax in ((512, 64, False, False), (320, 2, True, False),
                                    (319, 2, True, True)):
        w = synth.tiny(nf, n=300, nf=nf, n_classes=2, n_sets=2, rules=(n_rules, n_rules),
                       conds=(1, 2))
        ds = ctx.upload_dataset(w.data)
        p = ctx.pack_population(w.pop, nf, 2)
        v = [torch.tensor(a, device=ctx.device) for a in (w.pop.coef, w.pop.coef2, w.pop.theta)]
        one = torch.ones(2, device=ctx.device)
        for ok, call in ((soft, lambda: ctx.soft_backward(ds, p, *v, one)),
                         (smax, lambda: ctx.softmax_forward(ds, p, *v, 2.0)),
                         (smax, lambda: ctx.softmax_backward(ds, p, *v, 2.0, one))):
            if ok:
                call()
            else:
                with pytest.raises(AerlError):
                    call()
        if smax:
            run_softmax(ctx, w.data, w.pop, 2.0)
        torch.cuda.synchronize()
