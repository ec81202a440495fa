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


def _winners(ctx, recd, batch, tabs, tight):
    """The backward of a gradient of small integers, whose sums are exact, and what the rule gives element by element: the
    first position has it, and a later one takes it if its element is greater (a NaN never is, and nothing is greater than
    one at the first position)."""
    F, B, (rows, D) = batch.F, batch.B, tabs[0].shape
    rng = np.random.default_rng(D)
    gout = rng.integers(-4, 5, (F, B, D)).astype(np.float32)
    values, offsets, ik = gu.gpu_build(ctx, batch)
    U_cap, M_cap = (ik.U, ik.M) if tight else (F * B, batch.N)
    touched = torch.zeros(M_cap, dtype=torch.int64, device="cuda")
    feat_roff = torch.zeros(F + 1, dtype=torch.int64, device="cuda")
    grad_rows = torch.full((M_cap, D), 99.0, device="cuda")
    R = ctx.backward_dedup_max(F, B, gu.to_dev(gout), ik.inverse, ik.feat_uoff, ik.u_values, ik.u_offsets, [rows] * F, U_cap, M_cap,
                               gu.tables_to_dev(tabs, "f32"), touched, feat_roff, grad_rows, want_count=True)
    uv, uo, inv, fu = orc.build_ikjt(F, B, batch.values, batch.offsets)
    at, want = 0, []
    for f in range(F):
        g_u = np.zeros((fu[f + 1] - fu[f], D))
        np.add.at(g_u, inv[f * B:(f + 1) * B], gout[f].astype(np.float64))
        ref = np.zeros((rows, D))
        for u in range(fu[f], fu[f + 1]):
            ids = uv[uo[u]:uo[u + 1]]
            if len(ids) == 0:
                continue
            best, won = tabs[f][ids[0]].copy(), np.full(D, ids[0])
            for i in ids[1:]:
                more = tabs[f][i] > best
                best[more], won[more] = tabs[f][i][more], i
            np.add.at(ref, (won, np.arange(D)), g_u[u - fu[f]])
        rows_f = np.unique(uv[uo[fu[f]]:uo[fu[f + 1]]])
        assert np.array_equal(touched[at:at + len(rows_f)].cpu().numpy(), rows_f)
        want.append(ref[rows_f])
        at += len(rows_f)
    assert R == at and np.array_equal(grad_rows[:R].double().cpu().numpy(), np.concatenate(want))
    assert bool((grad_rows[R:] == 99.0).all())
    return ik.M / max(ik.U, 1)


def _shared_mean(D):
    """The mean length below which a wave owns several lists."""
    return 12 if D <= 64 else 4


SHORT = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 65]


@pytest.mark.parametrize("D", [4, 12, 16, 20, 32, 40, 64, 68, 128, 256])
@pytest.mark.parametrize("shared", [True, False])
def test_short_lists_share_waves(ctx, recd, D, shared):
    """Lists below and beyond the mean length up to which a wave owns several; features of one, of a few and of many lists, so
    that a wave's lists are of several; ties; tight and loose bounds."""
    rng = np.random.default_rng(D)
    F, rows, B = 140 if D == 16 else 9, 60, 61
    feats = []
    for f in range(F):
        n_pool = (1, 2, 5, B)[f % 4]
        lens = rng.choice(SHORT[:9 if D <= 64 else 5], B) if shared else rng.choice(SHORT[9:], B)
        lens[rng.integers(0, B, 3)] = rng.choice(SHORT, 3)
        pool = [rng.integers(0, rows, n).tolist() for n in lens[:n_pool]]
        feats.append([pool[b] if b < n_pool else pool[rng.integers(n_pool)] for b in range(B)])
    batch = synth.batch_from_lists(feats)
    tabs = [rng.integers(-2, 3, size=(rows, D)).astype(np.float32) for _ in range(F)]
    for tight in (True, False):
        mean = _winners(ctx, recd, batch, tabs, tight)
        assert (mean < _shared_mean(D)) == shared


@pytest.mark.parametrize("D", [4, 16, 32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("short", [True, False])
def test_nan_wins_at_the_first_position_only(ctx, recd, D, short):
    """NaNs of both signs in some or all elements of rows that lists name first, second, in other lane groups' parts, beyond 64
    positions, or everywhere; lists that begin with the type's lowest values and have a NaN behind them."""
    rng = np.random.default_rng(D)
    rows = 40
    tab = rng.integers(-3, 4, size=(rows, D)).astype(np.float32)
    tab[30:36] = np.nan
    tab[31] = -tab[31]
    tab[32, ::2] = 5.0
    tab[33, 1::3] = -np.inf
    tab[36:38] = -np.inf
    tab[38] = np.finfo(np.float32).min
    lists = [[36, 30], [36, 33, 37], [38, 36, 31, 38], [30], [32, 33], [33, 32], [36, 37]]
    for n in ([2, 3, 4, 5, 8, 9, 16] if short else [17, 33, 64, 65, 70, 130, 200]):
        for at in sorted({0, 1, min(n - 1, 2), n // 2, n - 1, min(n - 1, 7), min(n - 1, 31), min(n - 1, 63), min(n - 1, 64)}):
            for row in (30, 32, 33):
                ids = rng.integers(0, 30, n)
                ids[at] = row
                lists.append(ids.tolist())
        lists += [[30] * n, [36] * (n - 1) + [31], [31] + [5] * (n - 1), rng.choice([30, 32, 33, 36], n).tolist()]
    if not short:   # a mean length beyond which a wave owns one list
        lists += [rng.integers(0, rows, 40).tolist() for _ in range(40)]
    elif D > 64:
        lists += [rng.integers(0, rows, 2).tolist() for _ in range(400)]
    batch = synth.batch_from_lists([lists, lists[::-1]])
    mean = _winners(ctx, recd, batch, [tab, tab[::-1].copy()], True)
    assert (mean < _shared_mean(D)) == short
