"""Predictions around the sizes from which a wave per 256 rows walks the rules
in turn (2^15 rows of up to 5 features, 5 * 2^18 of up to 9): a row less, a
remainder of a wave's rows, one feature, rules past 64, empty rules and rule
sets, categorical and feature-vs-feature conditions, non-finite rows;
bit-exact against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import from_rule_lists

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,n", [(1, (1 << 15) + 1), (2, 1 << 15), (5, (1 << 15) - 1), (5, (1 << 15) + 255),
                                  (6, (5 << 18) - 1), (9, (5 << 18) + 257), (10, (5 << 18) + 3)])
def test_walk_edges(nf, n):
    import torch
    from paper_2406_01821_amd.aerl import Context
    rng = np.random.default_rng(nf + n)
    ends = synth.lognormal_features(rng, 4096, nf)
    rows = np.resize(ends, (n, nf)) * rng.uniform(0.5, 1.5, (n, 1)).astype(np.float32)
    rows[::7, rng.integers(nf)] = np.nan
    rows[1::11, rng.integers(nf)] = np.inf
    rows[2::13, rng.integers(nf)] = np.float32(3)
    if nf == 1:
        pop = synth.random_population(rng, ends, 2, (1, 70), (1, 6), 5, ff_frac=0.0)
    else:
        cat = min(2, nf - 1)
        pop = synth.categorical_population(rng, ends, cat, 8, 2, (66, 70), (1, 6), 5,
                                           ff_frac=0.2 if nf - cat > 1 else 0.0)
    sets = [pop.to_rule_list(s) for s in range(2)]
    d, r = sets[1]
    sets[1] = (d, r[:2] + [(4, [])] + r[2:])  # an empty rule fires for every row
    sets.append((3, []))
    pop = from_rule_lists(sets)
    ctx = Context(0)
    p = ctx.pack_population(pop, nf, 5)
    x = torch.tensor(rows, device=ctx.device)
    got = [ctx.predict(p, x, s).cpu().numpy() for s in range(3)]
    for s in range(3):
        np.testing.assert_array_equal(got[s], oracle.predict(rows, pop, s))
    ctx.close()
