"""Upload layout at the edges of its row groups: one row, group sizes (32 to
256 rows by feature count) and their neighbours, one feature to 512, rows
that are and are not whole 16-byte words, a pointer off 16-byte alignment,
one class to 64, a class without samples; each against a numpy layout, tau
within one rounding of the fp64 oracle, and refusals of bad values."""
from types import SimpleNamespace

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2406_01821_amd.aerl import Context
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def table(n, nf, nc, seed=0):
    rng = np.random.default_rng(1000 * n + 10 * nf + nc + seed)
    x = rng.standard_normal((n, nf)).astype(np.float32) * np.float32(3) + np.float32(100)
    y = rng.integers(0, nc, n).astype(np.int32)
    if nc > 2:
        y[y == 1] = 0  # a class without samples
    return x, y


def check(ctx, x, y, nc, dev_x=None):
    import torch
    n, nf = x.shape
    dev_x = torch.tensor(x, device=ctx.device) if dev_x is None else dev_x
    ds = ctx.upload_dataset(SimpleNamespace(x=dev_x, y=y, n_classes=nc))
    info = {k: v.cpu().numpy() if hasattr(v, "cpu") else v for k, v in ctx.dataset_info(ds).items()}
    ctx.release_dataset(ds)
    at, slots = 0, np.full(info["n_pad"], -1, np.int64)
    for c in range(nc):
        own = np.nonzero(y == c)[0]
        slots[at:at + len(own)] = own
        at += -(-len(own) // 256) * 256
    assert info["n_pad"] == at and info["class_count"] == list(np.bincount(y, minlength=nc))
    real = slots >= 0
    assert np.array_equal(info["perm"], slots)
    assert np.array_equal(info["y_pad"], np.where(real, y[np.maximum(slots, 0)], -1))
    assert np.array_equal(info["x_fm"], np.where(real, x[np.maximum(slots, 0)].T, 0))
    tau, ref = info["tau"], oracle.tau(x)
    assert np.abs(tau.view(np.int32) - ref.view(np.int32)).max() <= 1


@pytest.mark.parametrize("n,nf,nc", [
    (1, 1, 1), (255, 3, 2), (256, 4, 3), (257, 5, 2), (1023, 64, 4), (1025, 68, 64), (3000, 69, 4),
    (129, 140, 3), (4097, 141, 2), (2049, 284, 5), (1000, 285, 3), (65, 512, 4), (140_000, 8, 3)])
def test_layout(ctx, n, nf, nc):
    check(ctx, *table(n, nf, nc), nc)


def test_unaligned_features(ctx):
    """A feature pointer 4 bytes past a 16-byte boundary."""
    import torch
    x, y = table(777, 16, 3)
    buf = torch.empty(x.size + 1, device=ctx.device)
    buf[1:] = torch.tensor(x, device=ctx.device).view(-1)
    check(ctx, x, y, 3, buf[1:].view(x.shape))


@pytest.mark.parametrize("what", ["nan", "inf", "label", "negative", "both"])
def test_refusals(ctx, what):
    from paper_2406_01821_amd.aerl import AerlError
    x, y = table(5000, 12, 3)
    if what in ("nan", "both"):
        x[4999, 11] = np.nan
    if what == "inf":
        x[0, 0] = -np.inf
    if what in ("label", "both"):
        y[2500] = 3
    if what == "negative":
        y[0] = -1
    with pytest.raises(AerlError, match="non-finite" if what in ("nan", "inf", "both") else "label"):
        ctx.upload_dataset(SimpleNamespace(x=x, y=y, n_classes=3))
    check(ctx, *table(5000, 12, 3), 3)  # the context goes on
