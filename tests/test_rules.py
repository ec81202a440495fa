"""Sizes and bounds that host code and kernels share (csrc/recd_rules.h), built for the CPU and checked there."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2211_05239_amd", "csrc")

HARNESS = r"""
#include "recd_rules.h"
extern "C" {
int jagged_lists(int64_t N, int64_t U_cap, int64_t M_cap, int vecs) { return recd_jagged_lists(N, U_cap, M_cap, vecs, 256); }
bool short_grouping(int64_t rows, int64_t M_cap) { return recd_grouping_is_short(rows, M_cap); }
uint32_t divide(uint32_t by, uint32_t n) { return recd_divide_by(by).of(n); }
bool looks_back(int64_t rows, bool shared) { return recd_looks_back(rows, shared); }
void hash_pairs(const int64_t *a, const int64_t *b, int64_t n, uint32_t t, uint64_t *out, uint32_t *out32)
{
    for (int64_t i = 0; i < n; i++) {
        out[i] = recd_hash_pair(recd_hash_word(a[i], 0), recd_hash_word(b[i], 0), t);
        out32[i] = recd_hash_pair32(recd_hash_word(a[i], 0), recd_hash_word(b[i], 0), t);
    }
}
void share(uint32_t waves, uint32_t n, int32_t *taken, uint32_t *most)
{
    for (uint32_t w = 0; w < waves; w++) {
        const RecdShare s = recd_share(w, waves, n);
        for (uint32_t i = s.first; i < s.first + s.count; i++)
            taken[i]++;
        most[w >= waves / 2] = most[w >= waves / 2] < s.count ? s.count : most[w >= waves / 2];
    }
}
void next_items(int64_t waves, int64_t n, int32_t *taken, uint32_t *most)
{
    for (int64_t w = 0; w < waves; w++) {
        uint32_t count = 0;
        for (int64_t i = w; i >= 0 && i < n; i = recd_next_item(i, waves), count++)
            taken[i]++;
        most[w >= waves / 2] = most[w >= waves / 2] < count ? count : most[w >= waves / 2];
    }
}
uint32_t hash_key(uint32_t t) { return recd_hash_key(t); }
uint32_t row_named(uint32_t row, uint32_t rows) { return recd_row_named(row, rows); }

// a build per character of `steps`: p: a plan follows it, -: none, s: a short one; says of each p whether it had an event
// (counted) and of every build whether it recorded one
int events(const char *steps, int *records)
{
    RecdBuildEvent e;
    int had = 0;
    for (; *steps; steps++) {
        *records += e.at_build(*steps != 's');
        if (*steps == 'p')
            had += e.at_plan();
    }
    return had;
}
int64_t lists_held(int64_t F, int64_t B, int64_t U_cap, int64_t M_cap) { return recd_lists_held(F, B, U_cap, M_cap); }

// starts[slot] and how often each was written, of n >= 1 sorted keys; returns the writes outside [0, slots)
int64_t slot_starts(const uint32_t *keys, int64_t n, uint32_t bits, int64_t slots, int64_t *starts, int32_t *writes)
{
    int64_t outside = 0;
    for (int64_t i = 0; i < n; i++)
        recd_slot_starts(keys[i], i ? keys[i - 1] : 0u, i == 0, i == n - 1, bits, slots, [&](int64_t x, bool closed) {
            if (x < 0 || x >= slots) {
                outside++;
                return;
            }
            starts[x] = i + closed;
            writes[x]++;
        });
    return outside;
}

// work[q] of the lists that the blocks of queue q take, lists per block item lpb, `stride` blocks a queue
void deal(int64_t n, int F, int queues, int lpb, int64_t stride, const int64_t *len, int64_t *work, int32_t *taken)
{
    const int log = recd_deal_log_kjt(n, F, queues, 31 - __builtin_clz(lpb));
    for (int q = 0; q < queues; q++)
        for (int64_t b = 0; b < stride; b++)
            for (int64_t t = b * lpb;; t += stride * lpb) {
                const int64_t l0 = recd_dealt(t, q, queues, log);
                if (l0 >= n)
                    break;
                for (int64_t l = l0; l < n && l < l0 + lpb; l++) {
                    taken[l]++;
                    work[q] += len[l];
                }
            }
}

// the same for a KJT lookup whose waves share sums; returns the items of the queue that has the most
int64_t deal_items(int64_t n, int F, int queues, int lpb, int64_t stride, const int64_t *len, int64_t *work, int32_t *taken)
{
    const int log = recd_deal_log_kjt(n, F, queues, 31 - __builtin_clz(lpb));
    const int64_t most = recd_deal_most(n, queues, log), whole = recd_whole_items(most, queues, lpb);
    for (int q = 0; q < queues; q++)
        for (int64_t b = 0; b < stride; b++)
            for (int64_t i = b;; i += stride) {
                const int64_t l0 = recd_dealt(recd_item_start(i, whole, lpb), q, queues, log);
                if (l0 >= n)
                    break;
                for (int64_t l = l0; l < n && l < l0 + recd_item_lists(i, whole, lpb); l++) {
                    taken[l]++;
                    work[q] += len[l];
                }
            }
    return recd_items(most, whole, lpb);
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, lib = d / "rules.cpp", d / "rules.so"
    src.write_text(HARNESS)
    subprocess.check_call(["g++", "-std=c++20", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src),
                           "-o", str(lib)])
    return C.CDLL(str(lib))


def _ptr(a):
    return a.ctypes.data_as(C.c_void_p)


def test_room_for_every_unique_list(rules):
    rules.lists_held.restype = C.c_int64
    rules.lists_held.argtypes = [C.c_int64] * 4
    assert rules.lists_held(5, 600, 3000, 40) == 3000      # a group's empty lists
    assert rules.lists_held(5, 600, 3000, 10 ** 9) == 3000
    assert rules.lists_held(5, 600, 7, 40) == 45           # no fewer than a plain IKJT of M_cap ids can have
    assert rules.lists_held(5, 600, 10 ** 9, 40) == 3000


def test_division_by_a_number_of_rows(rules):
    """Quotients at and around multiples of the divisor, up to the largest row number."""
    rules.divide.restype = C.c_uint32
    rules.divide.argtypes = [C.c_uint32, C.c_uint32]
    rng = np.random.default_rng(5)
    most = (1 << 31) - 1
    for by in [1, 2, 3, 5, 7, 37, 255, 256, 257, 2500, 5003, 16384, 65537, (1 << 30) - 1, 1 << 30, most] + \
            [int(x) for x in 2 ** (rng.random(200) * 31)]:
        k = rng.integers(0, most // by + 1, 50)
        for n in {0, by - 1, by, most, most // by * by, *(k * by).tolist(), *(k * by + by - 1).tolist()}:
            if n <= most:
                assert rules.divide(by, n) == n // by, (by, n)


def test_short_groupings_fit_the_chip(rules):
    """Small tiles and plans in line up to fewer than two tiles of 1024 entries a CU, of both sides together."""
    rules.short_grouping.restype = C.c_bool
    rules.short_grouping.argtypes = [C.c_int64, C.c_int64]
    assert rules.short_grouping(65536, 425984) and not rules.short_grouping(65536, 425985)
    assert rules.short_grouping(425984, 65536) and not rules.short_grouping(1 << 19, 0)
    assert not rules.short_grouping(1 << 18, 1 << 18) and not rules.short_grouping(1 << 19, 1 << 19)


@pytest.mark.parametrize("steps", ["p" * 9, "-p" * 9, "p-" * 9, "--p" * 9, "s-p" * 9, "p" + "-" * 15 + "p" + "-" * 15 + "p",
                                   "-" * 100 + "ppp", "s" * 100 + "p", "-" * 100])
def test_plans_find_the_event_of_their_build(rules, steps):
    """Every plan starts where its build ended, whatever builds without a plan lie between, unless these are 16 and
    more in a row; builds that no plan ever follows record 16 events and no more."""
    records = C.c_int(0)
    rules.events.argtypes = [C.c_char_p, C.c_void_p]
    had = rules.events(steps.encode(), C.byref(records))
    many = "-" * 16 in steps
    assert had == steps.count("p") - many * ("p" in steps)
    assert records.value == (16 + max(steps.count("p") - 1, 0) if many else len(steps) - steps.count("s"))


def test_no_wait_between_blocks_on_shared_scratch(rules):
    """Overlapping recd_build_ikjt_noalloc calls may give wrong numbers; none may wait for words the other clears."""
    rules.looks_back.restype = C.c_bool
    rules.looks_back.argtypes = [C.c_int64, C.c_bool]
    for rows in (1, 1024, 1025, 65536, 1 << 18):
        assert rules.looks_back(rows, False) and not rules.looks_back(rows, True)
    assert not rules.looks_back((1 << 18) + 1, False)
    source = open(os.path.join(CSRC, "recd_build.hip")).read()
    call = source[source.index("recd_status recd_build_ikjt_noalloc("):]
    assert "carve_slots(c, F, B, n_lists, n_lists, true)" in call[:call.index("\n}\n")]


@pytest.mark.parametrize("t", [0, 2, 4, 46, 254, 3 << 20])
def test_no_id_hides_its_neighbour_from_the_hash(rules, t):
    """Lists that differ in one id, whatever its neighbour: among the neighbours the id that cancels its position's key, and
    those around it.  In 64 bits all differ, in 32 as good as all.  And pairs of any ids."""
    rules.hash_key.restype = C.c_uint32
    rules.hash_key.argtypes = [C.c_uint32]
    rules.hash_pairs.restype = None
    rules.hash_pairs.argtypes = [C.c_void_p, C.c_void_p, C.c_int64, C.c_uint32, C.c_void_p, C.c_void_p]

    def distinct(a, b):
        a, b = np.ascontiguousarray(a), np.ascontiguousarray(b)
        out, out32 = np.zeros(len(a), dtype=np.uint64), np.zeros(len(a), dtype=np.uint32)
        rules.hash_pairs(_ptr(a), _ptr(b), len(a), t, _ptr(out), _ptr(out32))
        return len(np.unique(out)), len(np.unique(out32))
    rng = np.random.default_rng(t)
    n = 20000
    others = rng.permutation(np.unique(np.concatenate([np.arange(n), rng.integers(0, 1 << 31, n)])))[:n].astype(np.int64)
    for at, swap in ((t, False), (t + 1, True)):
        zero = -rules.hash_key(at) % (1 << 32)
        for fixed in (zero, zero - 1, zero + 1, 0, 1, 12345, (1 << 31) - 1):
            pair = [np.full(n, fixed, dtype=np.int64), others]
            whole, folded = distinct(*(pair[::-1] if swap else pair))
            # the few alike cost the insertion a comparison each; half a percent of the lists would cost it half a percent
            assert whole == n and folded >= n - n // 200, (at, fixed)
    pairs = np.unique(rng.integers(0, 1 << 31, (n, 2)) % rng.choice([50, 10 ** 6, 1 << 31], (n, 1)), axis=0).astype(np.int64)
    whole, folded = distinct(pairs[:, 0], pairs[:, 1])
    assert whole == len(pairs) and folded >= len(pairs) - n // 200


def test_rows_that_tables_name_stay_inside_the_feature(rules):
    """Overlapping recd_build_ikjt_noalloc calls may clear or fill each other's tables: what the last kernel reads there it
    uses as a row only inside its feature."""
    rules.row_named.restype = C.c_uint32
    rules.row_named.argtypes = [C.c_uint32, C.c_uint32]
    for rows in (1, 2, 37, 1024, 65536, 1 << 30):
        for row in {0, rows - 1, rows, rows + 1, 65535, 1 << 31, 0xfffffffe, 0xffffffff}:
            assert rules.row_named(row, rows) == (row if row < rows else 0)
    source = open(os.path.join(CSRC, "recd_build.hip")).read()
    emit = source[source.index("void k_emit("):]
    emit = emit[:emit.index("\n}\n")]
    assert "number[row0 + recd_row_named((uint32_t)rep[l], rows.by)]" in emit and emit.count("number[") == 2


@pytest.mark.parametrize("seed", range(6))
@pytest.mark.parametrize("bad", [False, True])
def test_slot_starts_stay_inside_the_feature(rules, seed, bad):
    """Every slot's start is written exactly once and nowhere else, also where inverse entries are no slots
    (negative, or beyond the feature's last): sorted as the grouping sorts, by the low bits."""
    rng = np.random.default_rng(seed)
    slots, n = int(rng.integers(1, 40)), int(rng.integers(1, 120))
    bits = 0x3f
    keys = rng.integers(0, slots, n).astype(np.int64)
    if bad:
        at = rng.random(n) < 0.3
        keys[at] = rng.choice([-1, -2 ** 31, 2 ** 31 - 1, slots, slots + 1, 63], at.sum())
    keys = keys.astype(np.int64).astype(np.uint32)
    keys = keys[np.argsort(keys & bits, kind="stable")]
    starts, writes = np.full(slots, -1, dtype=np.int64), np.zeros(slots, dtype=np.int32)
    rules.slot_starts.restype = C.c_int64
    rules.slot_starts.argtypes = [C.c_void_p, C.c_int64, C.c_uint32, C.c_int64, C.c_void_p, C.c_void_p]
    assert rules.slot_starts(_ptr(keys), n, bits, slots, _ptr(starts), _ptr(writes)) == 0
    assert (writes == 1).all() and (np.diff(starts) >= 0).all() and starts[0] == 0
    if not bad:
        assert np.array_equal(starts, np.searchsorted(keys, np.arange(slots)))


def test_slot_starts_of_a_feature_without_slots(rules):
    keys = np.array([0, 5, 0xffffffff], dtype=np.uint32)
    none = np.zeros(1, dtype=np.int64)
    rules.slot_starts.restype = C.c_int64
    rules.slot_starts.argtypes = [C.c_void_p, C.c_int64, C.c_uint32, C.c_int64, C.c_void_p, C.c_void_p]
    assert rules.slot_starts(_ptr(keys), 3, 0x3ff, 0, _ptr(none), _ptr(none.astype(np.int32))) == 0


@pytest.mark.parametrize("means", [[16] * 32, [64] * 4 + [2] * 28, [100] + [2] * 5, [2] * 40 + [128] + [2] * 23,
                                   [4] * 50 + [150] + [4] * 14])
def test_lookup_lists_are_dealt_evenly(rules, means):
    """Every list goes to one block of one queue, and features of unequal mean length load the queues (the XCDs)
    alike: none has more than a quarter above its share of the ids."""
    rules.deal.restype = None
    rules.deal.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    lens = np.concatenate([np.full(1800, m, dtype=np.int64) for m in means])
    for lpb, stride in ((1, 3000), (2, 7), (4, 500), (16, 100)):
        work, taken = np.zeros(8, dtype=np.int64), np.zeros(len(lens), dtype=np.int32)
        rules.deal(len(lens), len(means), 8, lpb, stride, _ptr(lens), _ptr(work), _ptr(taken))
        assert (taken == 1).all()
        assert work.max() <= 1.25 * work.mean(), work


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 511, 512, 513, 5000])
def test_lookup_lists_of_any_number_are_all_dealt(rules, n):
    rules.deal.restype = None
    rules.deal.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    lens = np.ones(max(n, 1), dtype=np.int64)
    work, taken = np.zeros(8, dtype=np.int64), np.zeros(max(n, 1), dtype=np.int32)
    rules.deal(n, 8, 8, 4, 3, _ptr(lens), _ptr(work), _ptr(taken))
    assert (taken[:n] == 1).all() and work.sum() == n


@pytest.mark.parametrize("n,F", [(32768, 16), (32769, 3), (65535, 5), (65536, 8), (100003, 7), (1 << 19, 64),
                                 ((1 << 20) + 5, 8), (1030, 1), (9, 3)])
@pytest.mark.parametrize("lpb", [2, 4, 8, 16])
def test_items_of_several_and_of_two_lists_cover_every_list_once(rules, n, F, lpb):
    """Whole items and the short ones behind them take every list once, also by fewer blocks than items, and as many
    blocks a queue as the host launches are enough for one item each."""
    rules.deal_items.restype = C.c_int64
    rules.deal_items.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    lens = np.ones(n, dtype=np.int64)
    for queues in (8, 1):
        items = None
        for stride in (3 * n, 1013):
            work, taken = np.zeros(8, dtype=np.int64), np.zeros(n, dtype=np.int32)
            items = rules.deal_items(n, F, queues, lpb, min(stride, items or stride), _ptr(lens), _ptr(work), _ptr(taken))
            assert (taken == 1).all() and work.sum() == n
        work, taken = np.zeros(8, dtype=np.int64), np.zeros(n, dtype=np.int32)
        rules.deal_items(n, F, queues, lpb, items, _ptr(lens), _ptr(work), _ptr(taken))
        assert (taken == 1).all() and items * 2 >= n // queues // lpb
        assert items <= n // queues // lpb + 8192 // min(queues, 8) + 1024 // lpb + 2


@pytest.mark.parametrize("waves", [1, 2, 3, 7, 8, 1000, 6144])
@pytest.mark.parametrize("n", [0, 1, 2, 3, 5, 6, 7, 8, 9, 12, 999, 1000, 1001, 1500, 1501, 2500, 6145, 9215, 9216, 9217, 40000])
def test_waves_share_all_items(rules, waves, n):
    """Every item goes to one wave, and of more items than waves the second half of the waves has one each at most."""
    for share in (rules.share, rules.next_items):
        share.restype = None
        share.argtypes = [C.c_uint32, C.c_uint32, C.c_void_p, C.c_void_p] if share is rules.share else \
            [C.c_int64, C.c_int64, C.c_void_p, C.c_void_p]
        taken, most = np.zeros(n + 1, dtype=np.int32), np.zeros(2, dtype=np.uint32)
        share(waves, n, _ptr(taken), _ptr(most))
        assert (taken[:n] == 1).all() and taken[n] == 0
        assert waves == 1 or most[1] <= 1
        assert most[0] <= 2 + max(n - waves, 0) // max(waves // 2, 1)


@pytest.mark.parametrize("n", [8, 50, 100, 300, 530, 1000, 4000, 8191, 8192, 20000, 1 << 19, (1 << 20) + 5])
def test_few_lookup_lists_spread_over_all_queues(rules, n):
    rules.deal.restype = None
    rules.deal.argtypes = [C.c_int64, C.c_int, C.c_int, C.c_int, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p]
    work, taken = np.zeros(8, dtype=np.int64), np.zeros(n, dtype=np.int32)
    rules.deal(n, 8, 8, 1, n, _ptr(np.ones(n, dtype=np.int64)), _ptr(work), _ptr(taken))
    assert work.max() <= n / 8 * 1.0625 + 1


def test_lists_per_block_of_the_sequence_backward(rules):
    """A power of two up to 64 and at most 48 positions; twice that for short rows of many lists that are not
    known to have many rows: a block's threads would be idle for the most part."""
    rules.jagged_lists.argtypes = [C.c_int64] * 3 + [C.c_int]
    for U, M in ((1, 0), (0, 0), (10 ** 6, 16 * 10 ** 6), (10 ** 6, 10 ** 5), (7, 10 ** 9), (300, 300 * 30)):
        base = rules.jagged_lists(M, U, M, 16)
        assert base in (1, 2, 4, 8, 16, 32, 64) and (base == 1 or base * M <= 48 * max(U, 1))
        assert base == 64 or 2 * base * M > 48 * max(U, 1)
        assert rules.jagged_lists(9 * M + 9, U, M, 1) == base
    assert rules.jagged_lists(16 * 10 ** 6, 10 ** 6, 16 * 10 ** 6, 4) == 4
    assert rules.jagged_lists(16 * 10 ** 6, 10 ** 6, 16 * 10 ** 6, 16) == 2     # long rows
    assert rules.jagged_lists(16 * 10 ** 3, 10 ** 3, 16 * 10 ** 3, 4) == 2      # few lists
