"""Predictions at the edges of the 64-row blocks and of the rule split over a
block's waves: one row to a few blocks, one feature to 512, one rule to more
than the waves take at once (and past 64), empty rules and rule sets, every
condition kind, non-finite rows; bit-exact against the CPU oracle, alone and
through the serving loop's batched kernel."""
import numpy as np
import pytest

import oracle
from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import from_rule_lists

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def rows_of(rng, n, nf):
    x = synth.lognormal_features(rng, max(n, 64), nf)
    ends = x.copy()
    x[::7, rng.integers(nf)] = np.nan
    x[1::11, rng.integers(nf)] = np.inf
    x[2::13, rng.integers(nf)] = np.float32(3)
    return x[:n].copy(), ends


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000])
@pytest.mark.parametrize("nf,rules", [(1, (1, 1)), (2, (3, 5)), (30, (8, 17)), (64, (16, 33)),
                                      (159, (1, 8)), (512, (60, 70))])
def test_edges(ctx, n, nf, rules):
    import torch
    rng = np.random.default_rng(1000 * nf + n)
    rows, ends = rows_of(rng, n, nf)
    cat = min(2, nf - 1)
    args = (rng, ends, 3, rules, (1, 6), 5)
    if cat:
        pop = synth.categorical_population(rng, ends, cat, 8, 3, rules, (1, 6), 5,
                                           ff_frac=0.2 if nf - cat > 1 else 0.0)
    else:
        pop = synth.random_population(*args, ff_frac=0.0)
    sets = [pop.to_rule_list(s) for s in range(3)]
    d, r = sets[1]
    sets[1] = (d, r[:2] + [(4, [])] + r[2:])  # an empty rule fires for every row
    sets.append((3, []))
    pop = from_rule_lists(sets)
    p = ctx.pack_population(pop, nf, 5)
    got = [ctx.predict(p, torch.tensor(rows, device=ctx.device), s) for s in range(4)]
    torch.cuda.synchronize()
    want = [oracle.predict(rows, pop, s) for s in range(4)]
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g.cpu().numpy(), w)
    ctx.serve_start(64 << 20)
    try:
        tickets = [ctx.serve_submit_predict(pop, rows, nf, 5, s) for s in range(4)]
        for t, w in zip(tickets, want):
            np.testing.assert_array_equal(t.wait()["pred"], w)
    finally:
        ctx.serve_stop()


def test_four_rows_per_lane(ctx):
    """From 2^18 rows on, on up to 32 features."""
    import torch
    rng = np.random.default_rng(5)
    rows, ends = rows_of(rng, (1 << 18) + 5, 32)
    pop = synth.categorical_population(rng, ends, 2, 8, 2, (16, 33), (1, 6), 5, ff_frac=0.2)
    p = ctx.pack_population(pop, 32, 5)
    got = ctx.predict(p, torch.tensor(rows, device=ctx.device), 1)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), oracle.predict(rows, pop, 1))
