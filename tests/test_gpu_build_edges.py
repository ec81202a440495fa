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


@pytest.mark.parametrize("F,B,S", [(1, 32, 4), (9, 3640, 4), (9, 3641, 4), (33, 993, 1), (17, 3856, 40), (31, 17000, 64),
                                   (11, 9973, 1), (7, 9973, 1)])
@pytest.mark.parametrize("slack", [0, 1, 20])
def test_lookups_under_tight_and_loose_bounds(ctx, F, B, S, slack):
    """Lists and runs fewer than waves, more, and more than twice as many: every bound gives what each list by itself does,
    and writes no row beyond the lists."""
    D = 8
    w = synth.scaled(synth.WORKLOADS["cfg2"], F=F, B=B, rows=500, D=D, S=S, len_max=9)
    batch = synth.make_batch(w, slack)
    tabs = gu.tables_to_dev(synth.make_tables(w), w.table_dtype)
    values, offsets = gu.to_dev(batch.values), gu.to_dev(batch.offsets)
    ik = gu.DeviceIKJT(F, B, batch.N)
    runs = torch.zeros(3 * (F * B + 2), dtype=torch.int64, device="cuda")
    ik.U, ik.M = ctx.build_ikjt_runs(F, B, values, offsets, ik.u_values, ik.u_offsets, ik.inverse, ik.feat_uoff, runs,
                                     want_counts=True)
    n_runs = int(runs[0])
    dt = gu.TORCH_DT[w.table_dtype]
    kjt = torch.empty(F, B, D, dtype=dt, device="cuda")
    ctx.kjt_pooled_lookup(tabs, B, values, offsets, kjt)
    bound = {0: ik.U, 1: min(F * B, 2 * ik.U), 20: F * B}[slack]
    pooled = torch.full((F * B, D), 7.0, dtype=dt, device="cuda")
    out = torch.empty(F, B, D, dtype=dt, device="cuda")
    ctx.pooled_lookup_unique(tabs, ik.u_values, ik.u_offsets, ik.feat_uoff, bound, pooled)
    ctx.expand_inverse(F, B, pooled, ik.feat_uoff, ik.inverse, out)
    assert torch.equal(out, kjt) and bool((pooled[ik.U:] == 7.0).all())
    both = torch.full((F * B, D), 7.0, dtype=dt, device="cuda")
    again = torch.full((F, B, D), float("nan"), dtype=dt, device="cuda")
    ctx.pooled_lookup_expand(tabs, B, ik.u_values, runs, min(F * B, n_runs if slack == 0 else bound), both, again)
    assert torch.equal(again, kjt) and torch.equal(both, pooled)


@pytest.mark.parametrize("F,B", [(1, 1025), (3, 4096), (5, 52429), (6, 43691), (8, 65537), (2, 262144 + 4096 * 3 + 1)])
def test_numbering_across_waves_and_blocks(ctx, F, B):
    """One row and four rows a thread; runs that begin a feature, a wave and a block or go on across several of them, lists
    that come back blocks later, and lists of 0, 1, 32, 33 and 70 ids to be copied."""
    rng = np.random.default_rng(F * B)
    base = [rng.integers(0, 1000, n) for n in (0, 1, 2, 32, 33, 70, 5, 4)]
    cuts = np.unique(np.concatenate([[0], rng.integers(0, B, 40), np.arange(0, B, 4096), np.arange(64, B, 9 * 1024) - 1]))
    cuts = cuts[(cuts < B) & ~((cuts > 20000) & (cuts < 33000))]
    lists = []
    for f in range(F):
        which = rng.integers(0, len(base), len(cuts))
        lists.append(np.repeat(which, np.diff(np.append(cuts, B))))
    which = np.concatenate(lists)
    lens = np.array([len(x) for x in base])[which]
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    flat, start = np.concatenate(base), np.concatenate([[0], np.cumsum([len(x) for x in base])])[:-1]
    values = flat[np.repeat(start[which] - offsets[:-1], lens) + np.arange(offsets[-1])].astype(np.int64)
    batch = synth.Batch(F, B, values, offsets, np.zeros(B, np.int32), 1.0)
    _check(gu.gpu_build(ctx, batch)[2], batch)


@pytest.mark.parametrize("seed", range(3))
def test_grouped_tuples_that_differ_in_one_place(recd, seed):
    """Groups of one to five features; neighbouring tuples that agree, differ in one id of one feature, or in one length; a
    plain build between the grouped ones, whose tables are others."""
    rng = np.random.default_rng(seed)
    lengths = [0, 1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 64, 65, 97]
    sizes = [1, 2, 3, 4, 5, 4]
    F, B, G = sum(sizes), 601, len(sizes)
    group_off = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    rows = []
    for b in range(B):
        if b and rng.random() < 0.7:
            row = [list(x) for x in (rows[-1] if rng.random() < 0.8 else rows[rng.integers(b)])]
            if rng.random() < 0.4:
                x = row[rng.integers(F)]
                if rng.random() < 0.3:
                    x.append(1)
                elif x:
                    x[rng.choice([0, len(x) - 1, rng.integers(len(x))])] += 1
        else:
            row = [rng.integers(0, 50, rng.choice(lengths)).tolist() for _ in range(F)]
        rows.append(row)
    batch = synth.batch_from_lists([[rows[b][f] for b in range(B)] for f in range(F)])
    c = recd.Context(0)
    try:
        for _ in range(2):
            values, offsets = gu.to_dev(batch.values), gu.to_dev(batch.offsets)
            ik = gu.DeviceIKJT(F, B, batch.N)
            inverse_g = torch.full((G * B,), -7, dtype=torch.int32, device="cuda")
            group_uoff = torch.full((G + 1,), -7, dtype=torch.int64, device="cuda")
            c.build_ikjt_grouped(F, B, group_off, values, offsets, ik.u_values, ik.u_offsets, inverse_g, group_uoff, ik.feat_uoff)
            at = 0
            for g in range(G):
                seen, first = {}, []
                inv = []
                for b in range(B):
                    key = tuple(tuple(rows[b][f]) for f in range(group_off[g], group_off[g + 1]))
                    if key not in seen:
                        seen[key] = len(first)
                        first.append(b)
                    inv.append(seen[key])
                assert inverse_g[g * B:(g + 1) * B].tolist() == inv
                assert group_uoff[g:g + 2].tolist() == [at, at + len(first)]
                at += len(first)
                for f in range(group_off[g], group_off[g + 1]):
                    u0, u1 = ik.feat_uoff[f:f + 2].tolist()
                    o = ik.u_offsets[u0:u1 + 1].tolist()
                    ids = ik.u_values[o[0]:o[-1]].tolist()
                    assert [ids[x - o[0]:y - o[0]] for x, y in zip(o, o[1:])] == [rows[b][f] for b in first]
            c.set_option(recd._OPT_INTERNAL_SMALL_PATH, 0)
            _check(gu.gpu_build(c, batch)[2], batch)
    finally:
        c.close()


def test_captured_grouped_build_outlives_larger_ones(recd):
    """A captured grouped build, replayed after eager builds, grouped and plain, whose tables are larger than its own."""
    def lists(F, B, seed):
        rng = np.random.default_rng(seed)
        pool = [rng.integers(0, 90, n).tolist() for n in (0, 1, 3, 16, 17, 40)]
        rows = [[pool[rng.integers(6)] for _ in range(B)] for _ in range(F)]
        for f in range(F):
            rows[f][0] = pool[5]
        return synth.batch_from_lists(rows)
    F, B, group_off, many = 5, 300, [0, 2, 5], 40 * 5 * 300
    stream = torch.cuda.Stream()
    z = lambda n, dt=torch.int64: torch.zeros(n, dtype=dt, device="cuda")
    with torch.cuda.stream(stream):
        c = recd.Context(0, workspace_hint_bytes=recd.workspace_bytes(F, 4096, many, 4))
        values, offsets = z(many), z(F * B + 1)
        out = [z(many), z(F * B + 1), z(2 * B, torch.int32), z(3), z(F + 1)]
    def build(values, offsets, B, out):
        c.build_ikjt_grouped(F, B, group_off, values, offsets, *out)
    def load(batch):
        values[:batch.N].copy_(torch.from_numpy(batch.values))
        offsets.copy_(torch.from_numpy(batch.offsets))
    try:
        with torch.cuda.stream(stream):
            load(lists(F, B, 0))
            build(values, offsets, B, out)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                build(values, offsets, B, out)
            for seed in range(1, 4):
                big = lists(F, 1000 * seed, seed)
                bv, bo = gu.to_dev(big.values), gu.to_dev(big.offsets)
                build(bv, bo, big.B, [z(big.N), z(F * big.B + 1), z(2 * big.B, torch.int32), z(3), z(F + 1)])
                c.set_option(recd._OPT_INTERNAL_SMALL_PATH, 0)
                _check(gu.gpu_build(c, big)[2], big)
                load(lists(F, B, 10 + seed))
                for x in out:
                    x.zero_()
                build(values, offsets, B, out)
                want = [x.clone() for x in out]
                for x in out:
                    x.zero_()
                graph.replay()
                torch.cuda.synchronize()
                assert all(torch.equal(x, y) for x, y in zip(out, want))
    finally:
        c.close()
