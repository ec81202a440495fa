"""Backward of the max-pooled lookup where its lane groups, windows and batches of entries end, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import recd_oracle as orc
from paper_2211_05239_amd import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 40, 47, 63, 64, 65, 66, 96, 127, 128, 129, 200, 300]


@pytest.fixture(scope="module")
def recd():
    from paper_2211_05239_amd import recd as mod
    return mod


@pytest.fixture(scope="module")
def ctx(recd):
    c = recd.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("D", [4, 12, 16, 48, 64, 96, 128, 160, 256, 512, 1024])
@pytest.mark.parametrize("cut", [16, 128])
def test_winners_of_every_length(ctx, recd, D, cut):
    """Every length at and around the lane groups', waves' and windows' ends; few distinct elements, so that ties between
    positions of one and of several groups are the rule, among them the type's lowest values, at all positions of some lists;
    table rows named once and up to some hundred times, below and above the cut."""
    rng = np.random.default_rng(D + cut)
    F, rows = 2, 160
    feats = []
    for f in range(F):
        lists = [rng.integers(0, 40 if n % 2 else rows, n).tolist() for n in LENGTHS]
        lists += [[159] * 70, [159, 158, 3], [5] * 33 + [6] * 33, list(range(130))]
        feats.append([lists[i] for i in rng.permutation(len(lists)).tolist() + [0, 0, 3]])
    batch = synth.batch_from_lists(feats)
    B = batch.B
    tabs = [rng.integers(-2, 3, size=(rows, D)).astype(np.float32) for _ in range(F)]
    for t in tabs:
        t[150:] = np.finfo(np.float32).min
        t[158:] = -np.inf
    gout = rng.standard_normal((F, B, D)).astype(np.float32)
    ctx.set_option(recd.RECD_OPT_LONG_SEGMENT_CUT, cut)
    try:
        values, offsets, ik = gu.gpu_build(ctx, batch)
        d_tabs = gu.tables_to_dev(tabs, "f32")
        touched = torch.zeros(ik.M, dtype=torch.int64, device="cuda")
        feat_roff = torch.zeros(F + 1, dtype=torch.int64, device="cuda")
        grad_rows = torch.full((ik.M, D), float("nan"), device="cuda")
        R = ctx.backward_dedup_max(F, B, gu.to_dev(gout), ik.inverse, ik.feat_uoff, ik.u_values, ik.u_offsets, [rows] * F, ik.U,
                                   ik.M, d_tabs, touched, feat_roff, grad_rows, want_count=True)
    finally:
        ctx.set_option(recd.RECD_OPT_LONG_SEGMENT_CUT, 32)
    tr, fr, gr = orc.backward_kjt_max(F, B, gout, batch.values, batch.offsets, tabs)
    assert R == len(tr) and np.array_equal(touched[:R].cpu().numpy(), tr) and np.array_equal(feat_roff.cpu().numpy(), fr)
    gu.assert_close_f32(gu.out_to_f64(grad_rows[:R]), gr, "grad_rows")
