"""Hard fitness of tables that one block holds: one tile to as many as its LDS
and the planner's limit allow, one row to full tiles, 1 to 64 classes, one
rule set to several per block with a short last block, rule sets past the 64
rules of the rule filter, empty rules and rule sets, categorical conditions;
stored (not added) over what the outputs held, with and without confusion
counts, from a replayed graph; bit-exact against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import Dataset, from_rule_lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("n,nf,nc,n_sets,rules", [
    (1, 1, 1, 1, (1, 1)), (256, 3, 1, 5, (1, 3)), (257, 7, 2, 300, (2, 9)), (569, 30, 2, 101, (1, 8)),
    (900, 39, 2, 40, (8, 17)), (900, 40, 2, 40, (8, 17)), (40, 512, 1, 9, (1, 8)),
    (2000, 2, 64, 3, (60, 70)), (40 * 256, 3, 1, 512, (1, 4)), (40 * 256, 3, 1, 513, (1, 4)),
    (700, 16, 4, 257, (30, 70))])
def test_edges(ctx, n, nf, nc, n_sets, rules):
    import torch
    rng = np.random.default_rng(100 * n + nf)
    x = synth.lognormal_features(rng, n, nf)
    x[::5] = np.float32(2)
    cat = 2 if nf >= 16 else 0
    if cat:
        x[:, -cat:] = rng.integers(0, 8, size=(n, cat))
        pop = synth.categorical_population(rng, x, cat, 8, n_sets, rules, (1, 5), nc, ff_frac=0.2)
    else:
        pop = synth.random_population(rng, x, n_sets, rules, (1, 5), nc, ff_frac=0.3 if nf > 1 else 0.0)
    sets = [pop.to_rule_list(s) for s in range(n_sets)]
    d, r = sets[0]
    sets[0] = (d, r[:1] + [(nc - 1, [])] + r[1:])  # an empty rule fires for every row
    if n_sets > 1:
        sets[-1] = (0, [])
    pop = from_rule_lists(sets)
    y = rng.integers(0, nc, size=n).astype(np.int32)
    want, conf = oracle.hard_eval(x, y, nc, pop)
    ds = ctx.upload_dataset(Dataset(x, y, nc, "edges"))
    p = ctx.pack_population(pop, nf, nc)
    out = ctx.eval_population(ds, p)
    for o in out:
        o.fill_(-7)
    ctx.eval_population(ds, p, out=out)
    np.testing.assert_array_equal(out[0].cpu().numpy(), want)
    np.testing.assert_array_equal(out[1].cpu().numpy(), conf)
    only, none = ctx.eval_population(ds, p, confusion=False)
    assert none is None
    np.testing.assert_array_equal(only.cpu().numpy(), want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.eval_population(ds, p, out=out)
    for _ in range(3):
        for o in out:
            o.fill_(-7)
        g.replay()
        np.testing.assert_array_equal(out[0].cpu().numpy(), want)
        np.testing.assert_array_equal(out[1].cpu().numpy(), conf)
