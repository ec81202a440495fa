"""Backward passes of batches that hold lists but no id, too large for the one-launch grouping, under bounds that do not say
so: on a workspace that larger batches have written, and with ids again behind them."""
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


def _backward(ctx, kind, F, B, ik, rows, U_cap, M_cap, N, offsets, D=8):
    touched = torch.full((M_cap,), -1, dtype=torch.int64, device="cuda")
    feat_roff = torch.full((F + 1,), -1, dtype=torch.int64, device="cuda")
    grad_rows = torch.full((M_cap, D), 99.0, device="cuda")
    args = ik.inverse, ik.feat_uoff, ik.u_values, ik.u_offsets
    bounds = [rows] * F, U_cap, M_cap
    gout = torch.ones(F, B, D, device="cuda")
    if kind == "plan":
        ctx.backward_plan(F, B, D, *args, *bounds, touched, feat_roff)
        R = ctx.backward_apply(gout, grad_rows, want_count=True)
    elif kind == "sequence":
        emb = torch.full((M_cap, D), 99.0, device="cuda")
        R = ctx.backward_sequence_dedup(F, B, torch.ones(N, D, device="cuda"), offsets, *args, *bounds, emb, touched, feat_roff,
                                        grad_rows, want_count=True)
    elif kind == "weighted":
        R = ctx.backward_dedup_weighted(F, B, gout, *args[:3], torch.ones(M_cap, device="cuda"), args[3], *bounds, touched,
                                        feat_roff, grad_rows, want_count=True)
    elif kind == "max":
        R = ctx.backward_dedup_max(F, B, gout, *args, *bounds, [torch.ones(rows, D, device="cuda")] * F, touched, feat_roff,
                                   grad_rows, want_count=True)
    else:
        R = ctx.backward_dedup(F, B, gout, *args, *bounds, touched, feat_roff, grad_rows, want_count=True)
    return R, touched, feat_roff, grad_rows


@pytest.mark.parametrize("kind", ["sum", "plan", "sequence", "weighted", "max"])
@pytest.mark.parametrize("F,B,M_cap", [(1, 8193, 1), (3, 9000, 5), (20, 700, 9000), (9, 40000, 20000), (2, 250000, 9000)])
def test_lists_without_ids(recd, kind, F, B, M_cap):
    rows = 1 << 20
    ctx = recd.Context(0)
    try:
        rng = np.random.default_rng(F)
        # a feature of more small tiles than go by them; then of few
        full = [synth.batch_from_lists([rng.integers(0, rows, (600, n)).tolist(), [[]] * 600, rng.integers(0, rows, (600, 13)).tolist()])
                for n in (60, 20)]
        empty = synth.batch_from_lists([[[]] * B] * F)
        for batch in (*full, empty, *full, empty, empty, *full):
            values, offsets, ik = gu.gpu_build(ctx, batch)
            if batch.N:
                cap, ids = batch.N, [np.unique(batch.values[batch.offsets[f * batch.B]:batch.offsets[(f + 1) * batch.B]])
                                     for f in range(batch.F)]
            else:
                cap, ids = M_cap, [np.zeros(0, dtype=np.int64)] * F
                assert ik.M == 0
            R, touched, feat_roff, grad_rows = _backward(ctx, kind, batch.F, batch.B, ik, rows, batch.F * batch.B, cap, batch.N, offsets)
            assert feat_roff.tolist() == np.cumsum([0] + [len(x) for x in ids]).tolist() and R == feat_roff[-1]
            assert np.array_equal(touched[:R].cpu().numpy(), np.concatenate(ids))
            assert bool((touched[R:] == -1).all()) and bool((grad_rows[R:] == 99.0).all()) and not bool((grad_rows[:R] == 99.0).any())
    finally:
        ctx.close()
