"""The one-launch grouping of small batches, whose blocks learn from each other through words that every launch leaves clear:
batches of one block, of a block a feature and of several features a block after each other on one context."""
import numpy as np
import pytest

from tests import test_gpu_group as grouping
from tests.test_gpu_group import recd  # noqa: F401  (the fixture)

pytestmark = grouping.pytestmark

SMALL = [k for k, c in enumerate(grouping.CASES) if sum(c[0]) <= 8189 and c[1] <= 8192]


@pytest.mark.parametrize("extra", [[], [[0] * 127 + [7]], [[5] + [0] * 128, [0] * 128 + [6], [0, 3] * 150], [[2, 0, 0, 40] * 64]])
def test_small_groupings_after_each_other(recd, extra, monkeypatch):  # noqa: F811
    cases = grouping.CASES + [(ids, 9, 8, 60, True) for ids in extra]
    monkeypatch.setattr(grouping, "CASES", cases)
    ctx = recd.Context(0)
    try:
        order = SMALL + list(range(len(cases) - len(extra), len(cases)))
        for k in order + order[::-1]:
            c = grouping.Batch(k)
            g = c.integers(c.F * c.B, c.D)
            R = ctx.backward_dedup(c.F, c.B, c.dev(g).view(c.F, c.B, c.D), *c.ikjt, *c.bounds, c.touched, c.froff, c.grad_rows,
                                   want_count=True)
            gu, most = c.list_sums(g)
            c.check(R, gu[c.list_of], most[c.list_of])
    finally:
        ctx.close()
