"""Fine-tuning where the rule sets' blocks outnumber the CUs: seven or eight tiles,
two rule sets per block, one block per CU by its registers.
257 blocks of uneven rule sets (the per-set kernel, a second turn of blocks),
twice as many, and 350 of even ones (the adjoint kernel); against the fp64
reference loop at test_gpu_tune_small's bound."""
import pytest

from paper_2406_01821_amd import synth
from test_gpu_tune_small import check, ctx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sets,rules,conds", [(514, (1, 4), (1, 3)), (1028, (1, 4), (1, 3)),
                                                (700, (2, 2), (3, 3))])
def test_more_blocks_than_cus(ctx, n_sets, rules, conds):  # noqa: F811
    w = synth.tiny(n_sets, n=1792, nf=6, n_classes=2, n_sets=n_sets, rules=rules, conds=conds, ff_frac=0.3)
    check(ctx, w, 2, "adam")
