"""Softmax gradients of rule sets past 64 rules that hold threshold conditions
alone, which have a kernel of their own: against the fp64 oracle, in the product
form and past 60 conditions per rule."""
import pytest

from paper_2406_01821_amd import synth
from paper_2406_01821_amd.population import from_rule_lists
from test_gpu_softmax import run_case as run_softmax

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("rules,long,nc", [((65, 70), False, 2), ((65, 70), True, 5), ((66, 66), False, 12)])
def test_threshold_rules(ctx, rules, long, nc):
    w = synth.tiny(rules[0] + nc, n=700, nf=9, n_classes=nc, n_sets=5, rules=rules, conds=(1, 3), ff_frac=0.0)
    pop = w.pop
    if long:
        sets = [pop.to_rule_list(s) for s in range(5)]
        d, r = sets[2]
        every = [c for _, conds in r for c in conds]
        sets[2] = (d, [(r[0][0], every[:62])] + r[1:])
        pop = from_rule_lists(sets)
    run_softmax(ctx, w.data, pop, 2.0)
