"""KJT lookup of batches whose neighbouring lists are equal or nearly so: a run of equal lists is summed once, and its
rows have the bits that every list gives on its own (one list a block)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _batch(seed, n_lists, rows, run):
    """Runs of equal lists of 0 to 130 ids; one list in ten has an id or a weight changed (at its ends and around its
    64th id), its ids rotated, or its last id left out."""
    rng = np.random.default_rng(seed)
    lists, weights = [], []
    while len(lists) < n_lists:
        n = int(rng.choice([0, 1, 2, 5, 17, 40, 63, 64, 65, 130], p=[.1, .15, .15, .2, .2, .1, .025, .025, .025, .025]))
        ids, wts = rng.integers(0, rows, n), rng.choice([0.25, 0.5, 1.0, 2.0], n).astype(np.float32)
        for _ in range(int(rng.geometric(1.0 / run))):
            x, w = ids.copy(), wts.copy()
            if n and rng.random() < 0.1:
                at = int(rng.choice([0, n - 1, min(n - 1, 63), min(n - 1, 64)]))
                kind = rng.integers(4)
                if kind == 0:
                    x[at] = (x[at] + 1) % rows
                elif kind == 1:
                    x = np.roll(x, 1)
                elif kind == 2:
                    w[at] = -w[at]
                else:
                    x, w = x[:-1], w[:-1]
            lists.append(x)
            weights.append(w)
    lists, weights = lists[:n_lists], weights[:n_lists]
    offsets = np.concatenate([[0], np.cumsum([len(x) for x in lists])])
    return np.concatenate(lists), np.concatenate(weights), offsets


# below and above the number of lists from which waves share sums, odd numbers of lists a feature; long and short runs
@pytest.mark.parametrize("F,B,run,D,dtype", [(3, 341, 6, 64, "f32"), (5, 6601, 8, 20, "f32"), (9, 11003, 8, 64, "bf16"),
                                             (5, 6601, 1, 32, "f16"), (2, 16411, 40, 512, "f32")])
def test_runs_of_equal_lists(F, B, run, D, dtype):
    from paper_2211_05239_amd import recd
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    rows = 3000
    v, w, off = _batch(F * B + run, F * B, rows, run)
    values, weights, offsets = (torch.from_numpy(a).cuda() for a in (v.astype(np.int64), w, off.astype(np.int64)))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    tables = [torch.empty(rows, D, dtype=dt, device="cuda").normal_(0.0, 0.5, generator=gen) for _ in range(F)]
    ctx = recd.Context(0)
    calls = [lambda o, m=m: ctx.kjt_pooled_lookup(tables, B, values, offsets, o, mode=m) for m in (None, "mean", "max")]
    calls.append(lambda o: ctx.kjt_pooled_lookup_weighted(tables, B, values, weights, offsets, o))
    for call in calls:
        got = {}
        for lists_a_block in (1, 0, 2, 4, 8, 16, 2_000_000):   # the last: no shared sums, the blocks as they come
            ctx.set_option(recd._OPT_INTERNAL_TUNE_SEGSUM, lists_a_block)
            got[lists_a_block] = torch.full((F, B, D), float("nan"), dtype=dt, device="cuda")
            call(got[lists_a_block])
        for lists_a_block, out in got.items():
            assert torch.equal(out, got[1]), lists_a_block
        ctx.set_option(recd._OPT_INTERNAL_TUNE_SEGSUM, 0)
        torch.cuda.synchronize()
        again = torch.full((F, B, D), float("nan"), dtype=dt, device="cuda")
        call(again)
        assert torch.equal(again, got[1])
    # the last call's sums, in 64 bits: fp32 additions of at most 130 terms and one rounding to the output's type
    lens = offsets[1:] - offsets[:-1]
    to = torch.repeat_interleave(torch.arange(F * B, device="cuda"), lens)
    for f in range(F):
        a, b = int(offsets[f * B]), int(offsets[(f + 1) * B])
        terms = tables[f][values[a:b]].double() * weights[a:b, None].double()
        ref = torch.zeros(B, D, dtype=torch.float64, device="cuda").index_add_(0, to[a:b] - f * B, terms)
        size = torch.zeros(B, D, dtype=torch.float64, device="cuda").index_add_(0, to[a:b] - f * B, terms.abs())
        bound = 130 * 2.0 ** -24 * size + {"f32": 0.0, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype] * ref.abs() + 1e-7
        assert bool(((got[0][f].double() - ref).abs() <= bound).all())
    ctx.close()


def test_captured_lookup_outlives_its_context():
    """A captured lookup holds the caller's tensors only: it is replayed after the context is gone, plain (captured
    first) and after eager calls, each replay with eager work before it."""
    from paper_2211_05239_amd import recd
    F, B, D, rows = 5, 6601, 32, 3000
    v, _, off = _batch(11, F * B, rows, 8)
    values, offsets = torch.from_numpy(v.astype(np.int64)).cuda(), torch.from_numpy(off.astype(np.int64)).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    tables = [torch.empty(rows, D, device="cuda").normal_(0.0, 0.5, generator=gen) for _ in range(F)]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx = recd.Context(0)
        want, graphs = torch.empty(F, B, D, device="cuda"), []
        for warm in (0, 2):
            for _ in range(warm):
                ctx.kjt_pooled_lookup(tables, B, values, offsets, want)
                side.synchronize()
            out, graph = torch.zeros(F, B, D, device="cuda"), torch.cuda.CUDAGraph()
            side.synchronize()
            with torch.cuda.graph(graph, stream=side):
                ctx.kjt_pooled_lookup(tables, B, values, offsets, out)
            graphs.append((graph, out))
        side.synchronize()
        ctx.close()
        for _ in range(3):
            for graph, out in graphs:
                out.zero_()
                side.synchronize()
                graph.replay()
                side.synchronize()
                assert torch.equal(out, want)


def _lists(F, B, fixed, run, rows):
    """Lists of `fixed` ids in runs of `run` equal ones."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(F * B + fixed)
    ids = torch.randint(0, rows, (F, (B + run - 1) // run, fixed), device="cuda", generator=gen)
    values = ids.repeat_interleave(run, dim=1)[:, :B].reshape(-1).contiguous()
    return values, torch.arange(F * B + 1, device="cuda") * fixed


def test_way_depends_on_the_sizes_alone():
    """Every call of a size is the same single kernel: a context's first one, one after batches of another kind, and
    one captured; lists of one length that hold different ids are summed as such."""
    from torch.profiler import ProfilerActivity, profile
    from paper_2211_05239_amd import recd
    F, B, D, rows = 5, 6601, 32, 3000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    tables = [torch.empty(rows, D, device="cuda").normal_(0.0, 0.5, generator=gen) for _ in range(F)]
    batches = [_lists(F, B, 5, 8, rows), _lists(F, B, 5, 1, rows), _lists(F, B, 70, 1, rows), _lists(F, B, 1, 1, rows)]
    out = torch.empty(F, B, D, device="cuda")
    with profile(activities=[ProfilerActivity.CUDA]):
        torch.cuda.synchronize()   # the profiler's own start is not measured
    ctx, seen = recd.Context(0), []
    for values, offsets in batches + batches[::-1]:
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            ctx.kjt_pooled_lookup(tables, B, values, offsets, out)
            torch.cuda.synchronize()
        seen.append([e.name for e in prof.events() if "k_" in e.name])
        n = values.numel() // (F * B)
        ref = torch.stack([tables[f][values.view(F, B, n)[f]].double().sum(1) for f in range(F)])
        size = torch.stack([tables[f][values.view(F, B, n)[f]].double().abs().sum(1) for f in range(F)])
        assert bool(((out.double() - ref).abs() <= n * 2.0 ** -24 * size).all())   # n fp32 additions
    assert len(seen[0]) == 1 and all(x == seen[0] for x in seen), seen
    ctx.close()


@pytest.mark.parametrize("D,dtype", [(64, torch.float32), (16, torch.bfloat16)])
def test_runs_of_lists_around_what_a_wave_stages(D, dtype):
    """Lists that end before, at and behind the 1024 ids that wait in LDS, begin behind them, or are longer by themselves;
    one in four differs from its neighbour in one id or weight, also at these ids."""
    from paper_2211_05239_amd import recd
    F, B, rows = 3, 167, 2000
    rng = np.random.default_rng(D)
    lists, weights = [], []
    while len(lists) < F * B:
        n = int(rng.choice([0, 1, 127, 128, 129, 511, 512, 513, 1023, 1024, 1025, 2500]))
        ids, wts = rng.integers(0, rows, n), rng.choice([0.5, 1.0, 2.0], n).astype(np.float32)
        for _ in range(int(rng.integers(1, 7))):
            x, w = ids.copy(), wts.copy()
            if n and rng.random() < 0.25:
                at = int(rng.choice([0, n - 1, min(n - 1, 511), min(n - 1, 512), min(n - 1, 1023), min(n - 1, 1024)]))
                if rng.random() < 0.5:
                    x[at] = (x[at] + 1) % rows
                else:
                    w[at] = -w[at]
            lists.append(x)
            weights.append(w)
    lists, weights = lists[:F * B], weights[:F * B]
    off = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    values, wts = torch.from_numpy(np.concatenate(lists).astype(np.int64)).cuda(), torch.from_numpy(np.concatenate(weights)).cuda()
    offsets = torch.from_numpy(off).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    tables = [torch.empty(rows, D, dtype=dtype, device="cuda").normal_(0.0, 0.5, generator=gen) for _ in range(F)]
    ctx = recd.Context(0)
    for call in (lambda o: ctx.kjt_pooled_lookup(tables, B, values, offsets, o),
                 lambda o: ctx.kjt_pooled_lookup_weighted(tables, B, values, wts, offsets, o)):
        got = {}
        for lists_a_block in (1, 2, 4, 8, 16):   # one: every list by itself
            ctx.set_option(recd._OPT_INTERNAL_TUNE_SEGSUM, lists_a_block)
            got[lists_a_block] = torch.full((F, B, D), float("nan"), dtype=dtype, device="cuda")
            call(got[lists_a_block])
        for lists_a_block, out in got.items():
            assert torch.equal(out, got[1]), lists_a_block
    ctx.close()
