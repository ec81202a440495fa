"""The row sums with two pieces a lane and with four, plain and weighted: the same bits, at rows that end within a lane's pieces
and segments around one entry, the cut and the chunks."""
import numpy as np
import pytest
import torch

from paper_2211_05239_amd import synth
from tests import gpu_util as gu

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


@pytest.mark.parametrize("D", [32, 36, 60, 64, 68, 100, 128, 132, 200, 256, 512, 1024])
@pytest.mark.parametrize("cut", [16, 32, 128])
@pytest.mark.parametrize("weighted", [False, True])
def test_both_ways_give_the_same_bits(ctx, recd, D, cut, weighted):
    """Entries a row: 1 to 130 and some thousands; the bound on the positions is the number of them, and beyond that up to
    which the rows have two pieces a lane."""
    rng = np.random.default_rng(D + cut)
    F, rows = 2, 300
    feats = []
    for f in range(F):
        ids = np.concatenate([np.full(n, n) for n in range(1, 131, 1 if f else 3)] + [np.full(3000 if f else 257, 200)])
        ids = rng.permutation(np.concatenate([ids, np.full(513, 201), [299]]))
        ends = np.sort(rng.choice(len(ids) + 1, 399)).tolist()
        feats.append([x.tolist() for x in np.split(ids, ends)])
    batch = synth.batch_from_lists(feats)
    B = batch.B
    tabs = [rng.standard_normal((rows, D)).astype(np.float32) for _ in range(F)]
    gout = gu.to_dev(rng.standard_normal((F, B, D)).astype(np.float32))
    ctx.set_option(recd.RECD_OPT_LONG_SEGMENT_CUT, cut)
    try:
        values, offsets, ik = gu.gpu_build(ctx, batch)
        weights = gu.to_dev(rng.standard_normal(ik.M).astype(np.float32))
        got = []
        for M_cap in (ik.M, 512 * 1024, 512 * 1024 + 1):
            tables = gu.tables_to_dev(tabs, "f32")
            state = [torch.ones(rows, device="cuda") for _ in range(F)]
            touched = torch.zeros(M_cap, dtype=torch.int64, device="cuda")
            feat_roff = torch.zeros(F + 1, dtype=torch.int64, device="cuda")
            rest = ik.u_offsets, [rows] * F, ik.U, M_cap, touched, feat_roff, None
            update = dict(tables=tables, adagrad_state=state, lr=0.1, eps=1e-8, want_count=True)
            if weighted:
                R = ctx.backward_dedup_weighted(F, B, gout, ik.inverse, ik.feat_uoff, ik.u_values, weights, *rest, **update)
            else:
                R = ctx.backward_dedup(F, B, gout, ik.inverse, ik.feat_uoff, ik.u_values, *rest, **update)
            torch.cuda.synchronize()
            got.append([touched[:R], feat_roff, *tables, *state])
    finally:
        ctx.set_option(recd.RECD_OPT_LONG_SEGMENT_CUT, 32)
    for other in got[1:]:
        assert all(torch.equal(x, y) for x, y in zip(got[0], other))
