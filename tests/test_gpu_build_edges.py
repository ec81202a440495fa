"""The builder's kernels where their strides, waves and blocks end, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import recd_oracle as orc
from paper_2211_05239_amd import synth
from tests import gpu_util as gu
from tests.test_gpu_weighted import _build as build_weighted

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def recd():
    from paper_2211_05239_amd import recd as mod
    return mod


@pytest.fixture(scope="module")
def ctx(recd):
    c = recd.Context(0)
    yield c
    c.close()


def _check(ik, batch):
    uv, uo, inv, fu = orc.build_ikjt(batch.F, batch.B, batch.values, batch.offsets)
    assert (ik.U, ik.M) == (int(fu[-1]), len(uv))
    for got, ref in zip(ik.numpy(), (uv, uo, inv, fu)):
        assert np.array_equal(got, ref)


@pytest.mark.parametrize("n", [1, 2, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 50, 63, 64, 65, 80, 81, 112, 113, 300])
@pytest.mark.parametrize("weighted", [False, True])
def test_lists_that_differ_in_one_place(ctx, n, weighted):
    """Neighbours of one length that agree, or differ in the first, the last or the last but one id, in an id's upper half
    or (weighted) in one weight only; every place of a list in its wave."""
    base = np.arange(n) * 7 + 3
    rows, weights = [], []
    for _ in range(3):
        for at, by in ((0, 0), (0, 0), (0, 1), (0, 0), (n - 1, 1), (n - 1, 1), (0, 0), (max(n - 2, 0), 2), (n // 2, 1 << 32), (0, 0), (0, 0)):
            ids = base.copy()
            ids[at] += by
            rows.append(ids)
            weights.append(np.ones(n))
    for at in (0, n // 2, n - 1, n - 1):
        w = np.ones(n)
        w[at] = 2.0
        rows.append(base)
        weights.append(w)
    rows += [base[:-1], base, np.append(base, 1), base]
    weights += [np.ones(n - 1), np.ones(n), np.ones(n + 1), np.ones(n)]
    batch = synth.batch_from_lists([[list(map(int, x)) for x in rows[k:] + rows[:k]] for k in range(8)])
    if weighted:
        build_weighted(ctx, batch, np.concatenate([x for k in range(8) for x in weights[k:] + weights[:k]]).astype(np.float32))
    else:
        _check(gu.gpu_build(ctx, batch)[2], batch)
