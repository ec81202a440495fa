// Sizes and bounds that host code and kernels share.  Plain C++, so that they can be built and checked
// without a GPU.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define RECD_RULE __host__ __device__ inline
#else
#define RECD_RULE inline
#endif

// An id and the bit pattern of its weight (0: there are none) as 32 bits of hash input.
RECD_RULE uint32_t recd_hash_word(int64_t id, uint32_t wbits)
{
    const uint32_t hi = (uint32_t)((uint64_t)id >> 32);
    return (uint32_t)id ^ ((hi << 9) | (hi >> 23)) ^ (wbits * 0x85ebca6bu);
}

RECD_RULE uint32_t recd_hash_key(uint32_t t)
{
    const uint32_t k = (t + 1) * 0x9e3779b1u;
    return k ^ (k >> 15);
}

// What two adjacent ids, at positions t and t + 1, add to their list's hash: one product of 32 by 32 bits (two of 64 by 64
// before), and the keyed words beside each other, without which the id whose keyed word is zero would make lists that differ in
// its neighbour alike: x * y + x + y * 2^32 tells apart all y of an x and all x of a y.  That is enough: the sum goes through a
// mixer once a list, and an exact comparison follows every tag match.
RECD_RULE uint64_t recd_hash_pair(uint32_t a, uint32_t b, uint32_t t)
{
    const uint32_t x = a + recd_hash_key(t), y = b + recd_hash_key(t + 1);
    return (uint64_t)x * y + (((uint64_t)y << 32) | x);
}
// The same in 32 bits.  (The halves' exclusive or would be the same for every neighbour of the id whose keyed word is 2^32 - 1.)
RECD_RULE uint32_t recd_hash_pair32(uint32_t a, uint32_t b, uint32_t t)
{
    const uint64_t h = recd_hash_pair(a, b, t);
    return (uint32_t)h + (uint32_t)(h >> 32) * 0xc2b2ae35u;
}

// A row of the feature that the builder's tables name, whatever they hold: on scratch that calls of other streams share, an
// overlapping call may have cleared them, or filled in rows of a batch with more.
RECD_RULE uint32_t recd_row_named(uint32_t row, uint32_t rows) { return row < rows ? row : 0; }

// Division of a row number, below 2^31, by a number known to the host: a high product, an addition and a shift where the
// compiler's 64-bit division takes some hundred vector instructions (Granlund and Montgomery's method for 32-bit words; the
// sum stays below 2^32 as n does below 2^31).
struct RecdDiv {
    uint32_t by, mul, shift;
    RECD_RULE uint32_t of(uint32_t n) const { return (uint32_t)((((uint64_t)n * mul) >> 32) + n) >> shift; }
};
inline RecdDiv recd_divide_by(uint32_t by)  // 1 to 2^31
{
    uint32_t shift = 0;
    while (((uint64_t)1 << shift) < by)
        shift++;
    return RecdDiv{by, (uint32_t)((((((uint64_t)1 << shift) - by) << 32) / by) + 1), shift};
}

// Unique lists that the backward's workspace has room for (rows of g_u).  U_cap bounds their number; a
// plain IKJT has at most one empty list per feature and so at most M + F, but a grouped one stores an empty
// list for every slot of the group, so U_cap cannot be replaced by M_cap + F.
RECD_RULE int64_t recd_lists_held(int64_t F, int64_t B, int64_t U_cap, int64_t M_cap)
{
    const int64_t most = U_cap > M_cap + F ? U_cap : M_cap + F;
    return most < F * B ? most : F * B;
}

// Where the rows of a feature's unique lists start, from its rows sorted by slot: the row whose slot is `key`
// and its predecessor's `prev` (first: none) opens the slots after prev's up to its own, the last row also
// closes those that no row names.  put(slot, closed) is called once for every slot of the feature, whatever
// the keys hold: of an inverse entry that is no slot only the sorted bits count, and it counts as the last slot.
template <typename Put>
RECD_RULE void recd_slot_starts(uint32_t key, uint32_t prev, bool first, bool last, uint32_t sorted_bits, int64_t slots, Put put)
{
    const int64_t key_in = key & sorted_bits, prev_in = prev & sorted_bits;
    const int64_t k = key_in < slots ? key_in : slots - 1, p = first ? -1 : (prev_in < slots ? prev_in : slots - 1);
    for (int64_t x = p + 1; x <= k; x++)  // at most one turn where every slot is named
        put(x, false);
    for (int64_t x = k + 1; last && x < slots; x++)
        put(x, true);
}

// The lookups deal their n lists to the XCDs' block queues in turn, up to 1024 neighbours (2^10) at a time and at
// least 32 times round, but no fewer than the 2^lb_log lists of a block.  Neighbours (a session's lists, a
// feature's) stay together, features of unequal mean length load the queues alike, and a few lists spread over all
// of them.  (64 at a time at most is alike but for the largest: 1.05 M KJT lists of fp32 rows 1022 us, now 1005.)
RECD_RULE int recd_deal_log(int64_t n, int queues, int lb_log)
{
    const int64_t rounds = n / (queues * 64);
    const int bits = rounds > 0 ? 64 - __builtin_clzll((uint64_t)rounds) : 0, log = bits < 10 ? bits : 10;
    return log > lb_log ? log : lb_log;
}

// The same for the KJT's n lists, which the host knows.  Half a million and more of features that the queues can share
// evenly: up to 8192 at a time, 16 times round, so that a feature's hot rows are in fewer L2s (1.05 M lists of 64
// features, skewed ids 1038 -> 993 us; one feature of the 64 with half of the ids 297 -> 434, which a queue per
// feature took 636 for; 65 features, one with a third of the ids, would go from 242 to 324 where lists dealt one
// by one took 253).
RECD_RULE int recd_deal_log_kjt(int64_t n, int F, int queues, int lb_log)
{
    if (F % queues != 0 || n < (int64_t)1 << 19)
        return recd_deal_log(n, queues, lb_log);
    int log = 10;
    while (log < 13 && ((int64_t)queues * 16 << (log + 1)) <= n)
        log++;
    return log > lb_log ? log : lb_log;
}

// The items of wave w among `waves` that share n neighbouring items, which the waves find by themselves: of no more items than waves
// one each, of more the first waves have several neighbours, no more waves than half of them, and the others one each, so that
// the chip's last waves are short ones.  In the order of the waves, and so of time, the items follow each other.
struct RecdShare {
    uint32_t first, count;
};
RECD_RULE RecdShare recd_share(uint32_t w, uint32_t waves, uint32_t n)
{
    uint32_t first = w, several = 1;
    if (n > waves) {
        const uint32_t half = waves > 1 ? waves / 2 : 1, more = n - waves, extra = (more + half - 1) / half;
        const uint32_t whole = (more + extra - 1) / extra;  // waves of 1 + extra items
        several = w < whole ? 1 + extra : 1;
        first = w < whole ? w * (1 + extra) : whole * (1 + extra) + (w - whole);
    }
    return RecdShare{first, first >= n ? 0 : (n - first < several ? n - first : several)};
}

// The item that a wave takes after item i, of as many as it finds, on `waves` waves whose first items are their numbers; below 0:
// none.  The first half of the waves shares those beyond one each, for the same reason.
RECD_RULE int64_t recd_next_item(int64_t i, int64_t waves)
{
    const int64_t half = waves > 1 ? waves / 2 : 1;
    return i >= waves ? i + half : (i < half ? i + waves : -1);
}

// The t-th list of queue q.
RECD_RULE int64_t recd_dealt(int64_t t, int q, int queues, int deal_log)
{
    return ((((t >> deal_log) * queues) + q) << deal_log) + (t & (((int64_t)1 << deal_log) - 1));
}

// Lists of the queue that is dealt the most of n.
RECD_RULE int64_t recd_deal_most(int64_t n, int queues, int deal_log)
{
    const int64_t stretch = (int64_t)1 << deal_log, rest = n % (stretch * queues);
    return n / (stretch * queues) * stretch + (rest < stretch ? rest : stretch);
}

// Items of a queue of a KJT lookup whose waves share sums: `whole` items of lb lists, then items of two, so that the chip's
// last waves are short ones.  16384 lists, at most half of them, go two by two (65 K lists of 5 / 24 / 64 ids without
// sessions 40 -> 35, 156 -> 151, 362 -> 353 us; with sessions and of 262 K lists the same within 2 %).
enum { RECD_LAST_LISTS = 2 };
RECD_RULE int64_t recd_whole_items(int64_t lists, int queues, int lb)
{
    const int64_t tail = lists / 2 < 16384 / queues ? lists / 2 : 16384 / queues;
    return lb <= RECD_LAST_LISTS ? INT64_MAX : (lists - tail) / lb;
}
RECD_RULE int64_t recd_item_start(int64_t i, int64_t whole, int lb) { return i < whole ? i * lb : whole * lb + (i - whole) * RECD_LAST_LISTS; }
RECD_RULE int recd_item_lists(int64_t i, int64_t whole, int lb) { return i < whole ? lb : RECD_LAST_LISTS; }
RECD_RULE int64_t recd_items(int64_t lists, int64_t whole, int lb)
{
    return whole == INT64_MAX ? (lists + lb - 1) / lb : whole + (lists - whole * lb + RECD_LAST_LISTS - 1) / RECD_LAST_LISTS;
}

// Unique lists per block of the sequence backward's sum over their rows, of 16 * vecs bytes each: 24 to 48
// positions, and twice as many where rows are short, lists are neither short nor known to have many rows, and
// there are more blocks than the chip holds several times over (2.1 M positions, one row a list, whole call, us, by the
// bound 48 / 96: rows of 16 bytes 304 / 242, of 64 bytes 346 / 306, of 128 bytes 478 / 434).  Elsewhere the smaller
// block is the better or the safer one: eight rows a list, 0.26 M positions of 256 bytes 186 / 192; lists of 2
// positions 177 / 209; 0.3 M positions in lists of 1 to 400, 256 bytes, 205 / 250.
RECD_RULE int recd_jagged_lists(int64_t N, int64_t U_cap, int64_t M_cap, int vecs, int num_cu)
{
    const double positions = (double)M_cap / (double)(U_cap > 0 ? U_cap : 1);
    int lists = 1;
    while (lists < 64 && 2.0 * lists * positions <= 48.0)
        lists *= 2;
    if (vecs <= 8 && positions >= 8.0 && N <= 4 * M_cap && 2.0 * lists * positions <= 96.0 &&
        U_cap / (2 * lists) >= (int64_t)num_cu * 32)
        lists *= 2;
    return lists;
}

// Whether the builders number their rows one a thread in one launch whose blocks wait for what those before them hold
// (look-back): up to 256 blocks of 1024 rows.  Of more rows a thread takes four (k_number).  The stored lists of groups of
// features are then numbered too, of more in three launches: in groups of four build 65 K 38.9 / 27.4 us in three launches /
// by look-back, 262 K 44.7 / 36.8, 524 K 55.9 / 53.6.  Never on scratch that calls of other streams share: one that overlaps
// may give wrong numbers there, but as it clears the words that the blocks of the other wait for, neither might return.
RECD_RULE bool recd_looks_back(int64_t rows, bool shared_scratch) { return !shared_scratch && rows <= 256 * 1024; }

// Whether the grouping of a backward pass is short: its sides go by small tiles, and a plan goes in line, since the events
// that take it to the side stream and back cost more than the forward calls would hide of it.  480 K entries of both sides
// are fewer than two small tiles a CU; beyond that the chip is full either way and what the small tiles count again is
// lost.  Training step, us, F*B / M_cap in K, elements a row: beside by tiles of 4096 / in line by small tiles: 65 / 160,
// 128: 147 / 125; 180 / 180, 32: 150 / 138; 299 / 150, 64: 201 / 195; 376 / 84, 128: 241 / 239; 175 / 325, 128: 195 / 206;
// 325 / 175, 128: 241 / 249; 400 / 100, 64: 251 / 258; 494 / 248, 64: 218 / 240.  (Small tiles beside: 65 / 160, 128: 133;
// 256 / 256, 128: 216, in line 220, of 4096 beside 213.)
RECD_RULE bool recd_grouping_is_short(int64_t rows, int64_t M_cap) { return rows + M_cap <= 480 * 1024; }

// Whether a build records the event that a plan beside the forward calls starts at.  The record costs the kernel behind it
// 3 to 6 us, a plan without one up to some 90 us that the forward calls would hide: as many unused events as make up for one
// such plan are recorded before a context stops, until a plan asks for one again.  So plans that come after one build or
// after a few (two batches a step, an evaluation between) find theirs, and a context that only evaluates pays for 16.
struct RecdBuildEvent {
    int unused = 0;          // events in a row that no plan waited for
    bool recorded = false;   // of the last build
    bool used = false;
    bool at_build(bool plans_beside)  // whether this build records one
    {
        if (recorded && !used && unused < 16)
            unused++;
        recorded = plans_beside && unused < 16;
        used = false;
        return recorded;
    }
    bool at_plan()  // of the last build, beside the forward calls: whether there is one
    {
        used = true;
        unused = 0;
        return recorded;
    }
};
