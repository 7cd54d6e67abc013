"""Pools of an evolution run on both sides of the sizes where the packed image
is copied another way (256 KiB) and where a block of the fitness kernel takes
more than one rule set: every generation's fitness is the oracle's hard
evaluation of that generation's pool."""
import numpy as np
import pytest

import oracle
from paper_2406_01821_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("pool", [2, 255, 257, 320, 380, 6000])
def test_fitness_is_the_pools(ctx, pool):
    from paper_2406_01821_amd.aerl import evolve_cfg
    w = synth.small_hard(0)
    ds = ctx.upload_dataset(w.data)
    run = ctx.evolve(ds, evolve_cfg(pool=pool, elite=1, seed=pool), w.data.x.min(axis=0), w.data.x.max(axis=0))
    for g in range(3):
        st = run.state()
        assert st["generation"] == g
        want, _ = oracle.hard_eval(w.data.x, w.data.y, 2, st["pool"])
        np.testing.assert_array_equal(st["fitness"], want)
        run.run(1)
    run.release()
