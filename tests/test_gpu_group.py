"""The grouping of the backward pass (recd_group.hip) at the sizes where it can go wrong: features of no
id, one id, a tile less one, a whole tile, one more and several tiles; row ids of one, two and three
digits; slots of one and two digits; queues with more features than others."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

TILE = 4096


@pytest.fixture(scope="module")
def recd():
    from paper_2211_05239_amd import recd as m
    return m


def _case(seed, ids_per_feature, B, slots, rows, hot):
    """A batch's IKJT made directly: `slots` lists per feature that hold ids_per_feature[f] ids, every row of
    the batch naming one of them (some lists are named by no row)."""
    rng = np.random.default_rng(seed)
    F = len(ids_per_feature)
    lens, ids, inverse = [], [], []
    for n in ids_per_feature:
        cut = np.sort(rng.integers(0, n + 1, size=slots - 1))
        lens.append(np.diff(np.concatenate([[0], cut, [n]])))
        x = rng.integers(0, rows, size=n)
        if hot:  # a third of the ids name a few rows: long segments, also across tiles
            few = rng.integers(0, min(rows, 3), size=n)
            x = np.where(rng.random(n) < 1 / 3, few, x)
        ids.append(x)
        inverse.append(rng.integers(0, slots, size=B))
    lens = np.concatenate(lens)
    return (np.concatenate(ids).astype(np.int64), np.concatenate([[0], np.cumsum(lens)]).astype(np.int64),
            np.concatenate(inverse).astype(np.int32), np.arange(F + 1, dtype=np.int64) * slots)


CASES = [
    # ids per feature, B, slots, rows, hot
    ([0], 5, 3, 10, False),
    ([1, 0, 2], 1, 1, 1, False),
    ([0, 0, TILE - 1, 0], 17, 9, 1024, False),
    ([TILE, TILE + 1, 0, 5], TILE, 1024, 1025, True),
    ([TILE * 3 + 77, 1, TILE * 2], TILE + 1, 1025, 1 << 20, True),
    ([40000], 2 * TILE + 3, 4000, (1 << 20) + 1, True),
    ([300, 0, 9000, 5000, 1, 0, 0, 4097, 12000, 64, 8192], 700, 600, 50000, True),
    # at most 8192 ids and rows per feature: one launch
    ([8000 - 3, 0, 192], 8192, 8000, 1 << 17, True),   # with the bound M_cap = 8192 exactly
    ([0, 1024, 0, 1025, 3], 1025, 1024, 70000, True),
    ([8190], 8193, 90, 4000, True),                    # one row too many
    ([8190], 70, 60, 4000, True),                      # one id too many (M_cap = 8193)
    ([700, 0, 600], 2000, 7, (1 << 31) - 1, False),    # 31 + 2 bits of key: too many for one launch
    ([1400], 2000, 7, (1 << 31) - 1, False),           # 31 + 1 bits
    ([50] * 130, 40, 33, 5000, False),       # more features than one launch of the optimizer takes
    ([9] * 1024, 3, 3, 100, False),          # the most features
]


@pytest.mark.parametrize("k", range(len(CASES)))
@pytest.mark.parametrize("planned", [False, True])
def test_grouping_against_sums_in_64_bits(recd, k, planned):
    ids_per_feature, B, slots, rows, hot = CASES[k]
    F, D, n = len(ids_per_feature), 8, sum(ids_per_feature)
    uv, uo, inv, fu = _case(100 + k, ids_per_feature, B, slots, rows, hot)
    print(f"grouping case {k} planned={planned}", flush=True)
    g = np.random.default_rng(7 + k).standard_normal((F * B, D), dtype=np.float32) * np.float32(0.01)
    ctx = recd.Context(0)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    U = F * slots
    M_cap = n + 3                            # a bound, not the exact number
    touched = torch.full((M_cap,), -1, dtype=torch.int64, device="cuda")
    froff = torch.full((F + 1,), -1, dtype=torch.int64, device="cuda")
    grad_rows = torch.full((M_cap, D), 99.0, device="cuda")
    gout, d_uv, d_uo, d_inv, d_fu = dev(g), dev(np.concatenate([uv, [0, 0, 0]])), dev(uo), dev(inv), dev(fu)
    args = (F, B, D, d_inv, d_fu, d_uv, d_uo, [rows] * F, U, M_cap, touched, froff)
    if planned:
        ctx.backward_plan(*args)
        R = ctx.backward_apply(gout.view(F, B, D), grad_rows, want_count=True)
    else:
        R = ctx.backward_dedup(F, B, gout.view(F, B, D), d_inv, d_fu, d_uv, d_uo, [rows] * F, U, M_cap, touched,
                               froff, grad_rows, want_count=True)
    gu = np.zeros((U, D))
    np.add.at(gu, fu[np.arange(F * B) // B] + inv, g.astype(np.float64))
    lst = np.repeat(np.arange(U), np.diff(uo))
    key = (lst // slots) * (1 << 32) + uv
    want, back = np.unique(key, return_inverse=True)
    ref, size = np.zeros((len(want), D)), np.zeros((len(want), D))
    np.add.at(ref, back, gu[lst])
    gabs = np.zeros((U, D))
    np.add.at(gabs, fu[np.arange(F * B) // B] + inv, np.abs(g).astype(np.float64))
    np.add.at(size, back, gabs[lst])
    assert R == len(want)
    assert np.array_equal(touched[:R].cpu().numpy(), want & 0xffffffff)
    assert np.array_equal(froff.cpu().numpy(), np.searchsorted(want >> 32, np.arange(F + 1)))
    # fp32 sums through trees in which no term passes more than 2^12 additions (a list's rows in steps of 64
    # and a row's entries in chunks): 2^12 * 2^-24 of the sum of magnitudes, and the project's own bar
    bound = np.maximum(1e-5 * (1 + np.abs(ref)), 2.0 ** -12 * size)
    assert np.all(np.abs(grad_rows[:R].double().cpu().numpy() - ref) <= bound)
    ctx.close()
