"""The relaxed path on either side of the rules that decide whether tiles
classify the conditions and how many rule sets a block takes: the fp64 oracle,
and a rule set's loss is the same whether its population is small enough for
the plain sweep or large enough to classify (one rounding of the result: the
samples' terms are the same bits, the tiles' sums are added in fp64 in another
grouping)."""
import numpy as np
import pytest

import oracle
from paper_2406_01821_amd import synth
from test_gpu_soft import check_grad, check_loss

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def results(ctx, data, pop):
    import torch
    ds = ctx.upload_dataset(data)
    p = ctx.pack_population(pop, data.n_features, data.n_classes)
    v = [torch.tensor(a, device=ctx.device) for a in (pop.coef, pop.coef2, pop.theta)]
    out = [ctx.soft_forward(ds, p, *v).cpu().numpy(), ctx.softmax_forward(ds, p, *v, 2.0).cpu().numpy()]
    one = torch.ones(pop.n_sets, device=ctx.device)
    grads = [g.cpu().numpy() for g in ctx.soft_backward(ds, p, *v, one)]
    ctx.release_population(p)
    ctx.release_dataset(ds)
    return out, grads


# n, features, classes, rule sets of the large population, rules, conditions:
# four, two and one sample per lane, threshold-only and mixed, the product form
# and past it, two to sixteen padded classes, 15 and 16 tiles
@pytest.mark.parametrize("n,nf,nc,many,rules,conds,ff", [
    (9000, 9, 3, 300, (8, 16), (2, 6), 0.3), (9000, 16, 2, 400, (16, 16), (4, 4), 0.0),
    (6200, 60, 4, 500, (8, 24), (4, 6), 0.3), (6200, 110, 3, 700, (8, 24), (4, 6), 0.0),
    (5000, 200, 5, 900, (8, 24), (4, 6), 0.3), (9000, 9, 9, 300, (8, 16), (2, 6), 0.3),
    (6200, 12, 4, 300, (1, 3), (58, 66), 0.0), (6200, 12, 2, 100, (2, 3), (70, 80), 0.3),
    (3700, 20, 2, 900, (16, 32), (4, 8), 0.3), (4000, 20, 2, 900, (16, 32), (4, 8), 0.3)])
def test_plain_and_classifying_sweeps_agree(ctx, n, nf, nc, many, rules, conds, ff):
    w = synth.tiny(n + nf, n=n, nf=nf, n_classes=nc, n_sets=many, rules=rules, conds=conds, ff_frac=ff)
    few = w.pop.subset(range(6))
    (small, gs), (large, gl) = results(ctx, w.data, few), results(ctx, w.data, w.pop)
    x, y, tau = w.data.x, w.data.y, oracle.tau(w.data.x)
    check_loss(small[0], oracle.soft_forward(x, y, tau, nc, few))
    for a, b in zip(small, large):
        np.testing.assert_allclose(a, b[:6], rtol=1.2e-7, atol=0)
    if conds[1] > 8:  # rules that long have gradients below the fp32 range here
        return
    ref = oracle.soft_backward(x, y, tau, nc, few, dloss=np.ones(6))
    check_grad(gs, ref)
    check_grad([g[:few.n_conds] for g in gl], ref)
