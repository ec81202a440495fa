// Grouping for the backward pass: which entries go to which destination, in a fixed order.
//
//   side A   the rows (f,b) of every unique list, ascending              key = inverse[f*B+b]
//   side B   the positions j of every (feature, table row), ascending    key = u_values[j]
// Both are stable sorts of the entries *inside* a feature (the entries of a feature are one contiguous
// stretch on either side), so a key is a slot number or a row id and the feature needs no key bits:
// 20 bits for a million rows, two digits of 10.  The two sides go through the same launches:
//
//   k_group_count    digit counts of every feature and digit position -> where a digit starts
//   k_group_sweep    one launch per digit: a tile ranks its entries, learns from the tiles of its feature
//                    before it how many entries of each digit they hold (decoupled look-back), and
//                    writes its entries in order, regrouped in LDS so that neighbours go out together
//   k_group_segments side A: where every unique list's rows start (the slot number is the segment
//                    number); side B: the numbering of the distinct rows, the row ids, and the chunks
//                    of the rows with many entries
//
// A side of few entries goes by smaller tiles that need no look-back (sweep_small_tiles).
//
// Four launches for tables of up to 2^20 rows, where separate histogram, scan and scatter kernels per
// digit and side took 24 in two chains; with a dozen microseconds between dependent launches of two
// busy streams the chains, not their kernels, bounded every backward pass but the very largest.
//
// Look-back only ever waits for tiles of the same feature with a smaller number.  Tiles are handed out by
// tickets in that order (eight queues, feature f in queue f mod 8, which the blocks of one XCD serve
// first), so whoever is waited for has started and itself waits only further back: every wait ends.
#include "recd_internal.h"
#include "recd_scan.h"

namespace {

constexpr int kCountThreads = 256;
constexpr int kTileThreads = 512;
constexpr int kItems = 8;
constexpr int kTile = kTileThreads * kItems;  // entries of a tile
constexpr int kWaves = kTileThreads / 64;
constexpr int kMaxBits = 10;
constexpr int kMaxRadix = 1 << kMaxBits;
constexpr int kMaxPasses = 4;
constexpr int kQueues = 8;
constexpr int kMostChunks = 512;
constexpr int kSumChunks = 16;
// Small tiles (sweep_small_tiles): both sides of a short grouping (recd_grouping_is_short), where the features have at most
// kSmallTilesPer tiles each.
constexpr int kSmallItems = 2;
constexpr int kSmallTile = kTileThreads * kSmallItems;
constexpr int kSmallTileLog = 10;
static_assert(kSmallTile == 1 << kSmallTileLog, "chunks are powers of two");
constexpr int kSmallTilesPer = 32;
constexpr int64_t kSmallTilesMost = 480 << 10;  // entries of a side
static_assert(kTile % kSmallTile == 0 && kSmallTilesPer * kSmallTile < 1 << 16, "counts of other tiles are 16 bits");
static_assert(kMostChunks + 2 * RECD_MAX_FEATURES + 1 <= RECD_GROUP_ARRIVE, "a counter for every feature and every chunk");

__device__ __forceinline__ uint32_t ld_agent(const uint32_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint64_t ld_agent(const uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_agent(uint32_t *p, uint32_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_agent(uint64_t *p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Waits until the memory system has acknowledged this wave's stores.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Inclusive sums over a wave; of 64 bits those of the halves, whose totals fit them.
__device__ __forceinline__ uint32_t wave_incl(uint32_t v, int lane) { return wave_scan_add(v, lane); }
__device__ __forceinline__ uint64_t wave_incl(uint64_t v, int lane)
{
    return ((uint64_t)wave_scan_add((uint32_t)(v >> 32), lane) << 32) | wave_scan_add((uint32_t)v, lane);
}
__device__ __forceinline__ uint32_t row_incl(uint32_t v) { return row_scan_add(v); }
__device__ __forceinline__ uint64_t row_incl(uint64_t v) { return ((uint64_t)row_scan_add((uint32_t)(v >> 32)) << 32) | row_scan_add((uint32_t)v); }
__device__ __forceinline__ uint32_t of_lane(uint32_t v, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)v, lane); }
__device__ __forceinline__ uint64_t of_lane(uint64_t v, int lane) { return ((uint64_t)of_lane((uint32_t)(v >> 32), lane) << 32) | of_lane((uint32_t)v, lane); }

// Exclusive sum over the block's NW waves; every thread gets the total.  Every wave scans the waves' sums itself, in a row of
// 16 lanes.  (Shuffles through LDS and a loop over the waves before: blocks of 16 waves on one CU are bound by what they issue.)
template <typename T, int NW> __device__ __forceinline__ T block_excl(T v, T &total)
{
    static_assert(NW <= 16, "the waves' sums fit a row of lanes");
    __shared__ T s_w[NW];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const T inc = wave_incl(v, lane);
    __syncthreads();
    if (lane == 63)
        s_w[w] = inc;
    __syncthreads();
    const T sums = row_incl((lane & 15) < NW ? s_w[lane & 15] : (T)0);
    total = of_lane(sums, NW - 1);
    return (w > 0 ? of_lane(sums, w - 1) : (T)0) + inc - v;
}

struct SideParams {
    uint32_t *key[2], *pay[2];  // ping-pong buffers; pass p writes the pair p & 1
    int passes, dbits;
    uint32_t *base;             // [F][passes][radix]: where a digit starts inside the feature
    uint32_t *small_hist;       // [small tiles][radix] counts of the first digit
    uint32_t *chunk_hist;       // [chunks][passes][radix] (features of several chunks only)
    uint32_t *own, *upto;       // [tiles][radix] look-back: a tile's counts, and those of it and all before it
    uint32_t *flag;             // [passes][tiles] 0: nothing yet, 1: own is there, 2: upto is
    uint32_t *ticket;           // [kMaxPasses + 1][kQueues]
    uint32_t *arrive;           // [RECD_GROUP_ARRIVE] chunks (or sums of sixteen) of a feature that have been counted,
                                // and from RECD_MAX_FEATURES on the chunks of every sixteen; zero between launches
    int64_t chunk;              // entries per block of k_group_count
    int64_t tiles_cap;          // bound of the number of tiles
};

struct GroupParams {
    int F;
    int64_t B, M_cap, n_lists;
    const int32_t *inverse;
    const int64_t *feat_uoff, *u_values, *u_offsets;
    SideParams a, b;
    int tpf, cpf;               // side A: tiles and chunks of a feature
    unsigned a_blocks;          // blocks of the running launch that work on side A
    unsigned b_tiles;           // bound of side B's tiles
    unsigned list_block0;       // k_group_count: the first block that writes pos_list
    // side B
    uint32_t *pb;               // [F+1] first position of every feature
    uint32_t *queue_start;      // [kQueues+1] first tile of every queue
    uint2 *desc_queue;          // tile (in queue order) -> {feature, tile inside the feature}
    uint4 *desc_feat;           // tile (in feature order) -> {feature, tile inside the feature, the feature's first
                                // position, its positions}
    uint4 *desc_small;          // the same of the small tiles
    uint32_t *tile_total;       // [2] tiles; small tiles, 0: side B goes by tiles
    int small_a, small_b;       // whether side A goes by small tiles; whether side B may
    uint32_t *pos_list;         // list of every position, or null (then the payload is the position)
    int pay_positions;          // 1: the payload is the position also where pos_list is written
    const float *u_weights;     // weights of the positions, or null; sorted ones go to pay_w and the
    float *pay_w;               // payload of the last pass is pos_list of the position
    uint32_t *pay_pos;          // as pay_w, with the positions themselves; or null
    const int64_t *run_index;   // not null: only its count is compared with runs_cap
    int64_t runs_cap;
    int64_t *too_small_a, *too_small_b;  // whether the caller's bounds were too small
    int64_t lists_cap;          // no list at or beyond this is summed: a position of such a list names the last
    // segments
    uint64_t *seg_status;       // [tiles] look-back words of the numbering
    int64_t *seg_start_a, *list_off_a, *seg_start_b, *list_off_b;
    int64_t *touched_rows, *feat_roff;
    int32_t *seg_feat;
    int64_t *chunk_count;       // chunks of the segments that are cut
    RecdChunk *chunks;
    uint32_t *chunk_arrive;
    int long_seg;
};

// Side A's word about the caller's bounds, for U unique lists.
__device__ __forceinline__ void report_side_a(const GroupParams &g, int64_t U)
{
    g.too_small_a[0] = (g.run_index && g.run_index[0] > g.runs_cap ? RECD_GROUP_RUNS : 0) |
                       (U > g.lists_cap ? RECD_GROUP_LISTS : 0);
}

// The bits of a key that a side's digits cover.
__device__ __forceinline__ uint32_t sorted_bits(const SideParams &s) { return (uint32_t)((1ull << (s.passes * s.dbits)) - 1); }

// Digit starts of feature f from the block's counts in LDS.
__device__ __forceinline__ void write_bases(const SideParams &s, int f, const uint32_t *hist)
{
    const int radix = 1 << s.dbits;
    constexpr int kPer = kMaxRadix / kCountThreads;  // neighbouring digits of a thread
    for (int p = 0; p < s.passes; p++) {
        uint32_t v[kPer], sum = 0, total;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int d = threadIdx.x * kPer + i;
            v[i] = d < radix ? hist[p * radix + d] : 0;
            sum += v[i];
        }
        uint32_t e = block_excl<uint32_t, kCountThreads / 64>(sum, total);
        uint32_t *base = s.base + ((size_t)f * s.passes + p) * radix;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int d = threadIdx.x * kPer + i;
            if (d < radix)
                base[d] = e;
            e += v[i];
        }
    }
}

// ---- digit counts -----------------------------------------------------------------------------------
// A block takes a chunk of one feature's entries (a tile, or as many as keep the chunks below some 500),
// counts the digits of all passes in LDS and, where the feature is a single chunk, turns the counts into
// digit starts at once; else the block that arrives last adds up the feature's chunks (of more than 16 the
// last of every sixteen adds up these first).  The block also
// clears the look-back flags of its tiles; further blocks write the list of every position.  Of a side that goes by
// small tiles a block counts the first digit of one small tile, and the sweep adds up.  What is
// read is small (8 bytes an entry): the kernel is a few dependent round trips, the LDS atomics of a
// chunk, and what its waves issue: divisions by the chunk's size, four features and places of the queue order a thread,
// sixteen key slots where a small tile fills four were half of it (0.19 M ids 11.0 us, now 5.9).
__global__ __launch_bounds__(kCountThreads) void k_group_count(const GroupParams g)
{
    extern __shared__ uint32_t s_dyn[];          // the counts [passes * radix], side B also pb [F+1]: as little
    uint32_t *s_hist = s_dyn;                    // LDS as there is, so that blocks find room beside the lookup's
    __shared__ uint32_t s_pick[5];
    const int tid = threadIdx.x;
    if (blockIdx.x >= g.list_block0) {
        // the list of every position, 16 lanes to a list: blocks of their own, beside the chain of the others
        const int64_t U = g.feat_uoff[g.F], step = (int64_t)(gridDim.x - g.list_block0) * (kCountThreads / 16);
        for (int64_t u = (int64_t)(blockIdx.x - g.list_block0) * (kCountThreads / 16) + tid / 16; u < U; u += step) {
            const int64_t at = g.u_offsets[u], end = g.u_offsets[u + 1] < g.M_cap ? g.u_offsets[u + 1] : g.M_cap;
            const uint32_t name = (uint32_t)(u < g.lists_cap ? u : g.lists_cap - 1);
            for (int64_t j = at + tid % 16; j < end; j += 16)
                g.pos_list[j] = name;
        }
        return;
    }
    const bool side_a = blockIdx.x < g.a_blocks;
    const SideParams &s = side_a ? g.a : g.b;
    const unsigned blk = side_a ? blockIdx.x : blockIdx.x - g.a_blocks;
    int f, c, n_chunks;
    uint32_t begin, end;           // entries of the chunk
    size_t first_tile, chunk_row;  // in queue order; row of chunk_hist or small_hist
    bool small = g.small_a != 0;   // the chunk is a small tile, and only its first digit is counted
    if (blockIdx.x == 0 && tid < (kMaxPasses + 1) * kQueues) {
        g.a.ticket[tid] = 0;
        g.b.ticket[tid] = 0;
    }
    if (side_a) {
        f = (int)(blk / g.cpf);
        c = (int)(blk % g.cpf);
        n_chunks = g.cpf;
        const int64_t chunk = small ? kSmallTile : s.chunk;
        begin = (uint32_t)(f * g.B + c * chunk);
        end = (uint32_t)(c * chunk + chunk < g.B ? begin + chunk : (f + 1) * g.B);
        const int q = f % kQueues, per_q = g.F / kQueues, more = g.F % kQueues;
        first_tile = (size_t)(q * per_q + (q < more ? q : more) + f / kQueues) * g.tpf + (size_t)c * (s.chunk / kTile);
        chunk_row = blk;
        if (blk == 0 && tid == 0)
            report_side_a(g, g.feat_uoff[g.F]);
    } else {
        uint32_t *s_pb = s_dyn + (s.passes << s.dbits);
        // where every feature's positions lie; tiles and chunks of the features before each one
        for (int i = tid; i <= g.F; i += kCountThreads) {
            const int64_t at = g.u_offsets[g.feat_uoff[i]];
            s_pb[i] = (uint32_t)(at < g.M_cap ? at : g.M_cap);  // never past the caller's capacity
        }
        small = g.small_b != 0;
        if (tid == 0)
            s_pick[0] = ~0u;
        __syncthreads();
        if (small) {
            bool beyond = false;
            for (int x = tid; x < g.F; x += kCountThreads)
                beyond |= s_pb[x + 1] - s_pb[x] > (uint32_t)(kSmallTilesPer * kSmallTile);
            small = !__syncthreads_or(beyond);
        }
        const int chunk_log = small ? kSmallTileLog : 31 - __builtin_clz((uint32_t)s.chunk);  // a power of two
        const uint32_t chunk = 1u << chunk_log;
        auto tiles_of = [&](int x) { return (s_pb[x + 1] - s_pb[x] + kTile - 1) / kTile; };
        auto chunks_of = [&](int x) { return (s_pb[x + 1] - s_pb[x] + chunk - 1) >> chunk_log; };
        // the block's feature and chunk; a thread stands for one feature (of more than the block has threads, for one after
        // the other)
        uint64_t so_far = 0;  // tiles (high half) and chunks of the features before
        for (int x0 = 0; x0 < g.F; x0 += kCountThreads) {
            const int x = x0 + tid;
            uint64_t mine = 0, all;
            if (x < g.F)
                mine = ((uint64_t)tiles_of(x) << 32) | chunks_of(x);
            const uint64_t ex = so_far + block_excl<uint64_t, kCountThreads / 64>(mine, all);
            if (blk - (uint32_t)ex < (uint32_t)mine) {
                s_pick[0] = x;
                s_pick[1] = blk - (uint32_t)ex;
                s_pick[2] = (uint32_t)mine;
                s_pick[3] = (uint32_t)(ex >> 32);
            }
            so_far += all;
        }
        const uint32_t tiles = (uint32_t)(so_far >> 32);
        // Tiles go by queues: features 0, 8, 16, ..., then 1, 9, ...  The sweep looks for tiles there too where there is no id
        // at all, and so no small tile.
        if (!small || tiles == 0) {
            const int per_q = g.F / kQueues, more = g.F % kQueues;
            const int wide = more * (per_q + 1);  // places in the queues that hold one feature more
            uint32_t before = 0;
            __syncthreads();
            for (int x0 = 0; x0 < g.F; x0 += kCountThreads) {
                const int i = x0 + tid;  // place in the queue order
                uint32_t mine = 0, all;
                int q = 0, at = 0;
                if (i < g.F) {
                    q = i < wide ? i / (per_q + 1) : more + (i - wide) / per_q;
                    at = i < wide ? i % (per_q + 1) : (i - wide) % per_q;
                    mine = tiles_of(at * kQueues + q);
                }
                const uint32_t ex = before + block_excl<uint32_t, kCountThreads / 64>(mine, all);
                if (i < g.F && (uint32_t)(at * kQueues + q) == s_pick[0])
                    s_pick[4] = ex;
                if (i < g.F && blk == 0 && at == 0)
                    g.queue_start[q] = ex;
                before += all;
            }
            if (blk == 0 && tid >= (g.F < kQueues ? g.F : kQueues) && tid <= kQueues)
                g.queue_start[tid] = tiles;  // queues without a feature, and the end
        }
        if (blk == 0) {
            for (int i = tid; i <= g.F; i += kCountThreads)
                g.pb[i] = s_pb[i];
            if (tid == 0) {
                g.tile_total[0] = tiles;
                g.tile_total[1] = small ? (uint32_t)so_far : 0;
                const int64_t M = g.u_offsets[g.feat_uoff[g.F]];
                g.too_small_b[0] = M > g.M_cap ? 1 : 0;
                g.chunk_count[0] = 0;
            }
        }
        __syncthreads();
        if (s_pick[0] == ~0u)
            return;  // whole block: fewer chunks than the bound
        f = (int)s_pick[0];
        c = (int)s_pick[1];
        n_chunks = (int)s_pick[2];
        begin = s_pb[f] + ((uint32_t)c << chunk_log);
        end = s_pb[f + 1] - begin > chunk ? begin + chunk : s_pb[f + 1];
        const uint32_t k0 = ((uint32_t)c << chunk_log) / kTile;
        first_tile = (small ? 0 : s_pick[4]) + k0;
        chunk_row = blk;
        // tiles that start in the chunk
        const uint32_t my_tiles = small ? (((uint32_t)c << chunk_log) % kTile == 0 ? 1 : 0) : (end - begin + kTile - 1) / kTile;
        if (small && tid == 0)
            g.desc_small[blk] = make_uint4(f, c, s_pb[f], s_pb[f + 1] - s_pb[f]);
        for (uint32_t k = tid; k < my_tiles; k += kCountThreads) {
            if (!small)
                g.desc_queue[first_tile + k] = make_uint2(f, k0 + k);
            g.desc_feat[s_pick[3] + k0 + k] = make_uint4(f, k0 + k, s_pb[f], s_pb[f + 1] - s_pb[f]);
            g.seg_status[s_pick[3] + k0 + k] = 0;
        }
    }
    const uint32_t n = end - begin;
    const int radix = 1 << s.dbits;
    const uint32_t mask = radix - 1;
    const int passes = small ? 1 : s.passes;  // that are counted
    for (int i = tid; i < passes * radix; i += kCountThreads)
        s_hist[i] = 0;
    __syncthreads();
    for (uint32_t i0 = tid; i0 < n; i0 += 16 * kCountThreads) {
        uint32_t key[16];
#pragma unroll
        for (int u = 0; u < 16; u++) {
            if (i0 - tid + u * kCountThreads >= n)  // the same in every thread
                break;
            const uint32_t i = i0 + u * kCountThreads;
            key[u] = i < n ? (side_a ? (uint32_t)g.inverse[begin + i] : (uint32_t)g.u_values[begin + i]) : 0u;
        }
#pragma unroll
        for (int u = 0; u < 16; u++) {
            if (i0 - tid + u * kCountThreads >= n)
                break;
            // Side A comes in runs of one slot (the samples of a session): the first lane of a run counts for
            // all of it, where every lane's own atomic would queue at one address.
            const bool on = i0 + u * kCountThreads < n;
            uint32_t many = 1;
            bool count = on;
            if (side_a) {
                const uint32_t left = __shfl_up(key[u], 1);
                const int ln = tid & 63;
                count = on && (ln == 0 || left != key[u]);
                const uint64_t heads = __ballot(count), live = __ballot(on);
                const uint64_t above = ln == 63 ? 0 : heads >> (ln + 1);
                many = above ? (uint32_t)__builtin_ctzll(above) + 1 : (uint32_t)__popcll(live) - ln;
            }
            if (count)
                for (int p = 0; p < passes; p++)
                    atomicAdd(&s_hist[p * radix + ((key[u] >> (p * s.dbits)) & mask)], many);
        }
    }
    if (small) {  // the sweep adds up the counts of the feature's small tiles itself
        __syncthreads();
        for (int i = tid; i < radix; i += kCountThreads)
            s.small_hist[chunk_row * radix + i] = s_hist[i];
        return;
    }
    // look-back flags of the chunk's tiles
    for (int i = tid; i < (int)((n + kTile - 1) / kTile) * s.passes; i += kCountThreads)
        s.flag[(size_t)(i % s.passes) * s.tiles_cap + first_tile + i / s.passes] = 0;
    const int words = s.passes * radix;
    __syncthreads();
    if (n_chunks == 1) {
        write_bases(s, f, s_hist);
    } else {
        uint32_t *row = s.chunk_hist + chunk_row * words;
        for (int i = tid; i < words; i += kCountThreads)
            st_agent(row + i, s_hist[i]);
    }
    if (n_chunks == 1)
        return;
    // The counts are written through to where every XCD reads them; once the stores are acknowledged the
    // arrival may be counted.  A release here would write back the whole L2 of the XCD, once per block
    // (measured beside the forward kernels: 375 us for this kernel, and those slowed by half).
    stores_done();
    // whether this block is the last of `of` to arrive
    auto last_of = [&](uint32_t *counter, int of) {
        __syncthreads();
        if (tid == 0)
            s_pick[0] = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const bool last = s_pick[0] == (uint32_t)(of - 1);
        if (last && tid == 0)
            st_agent(counter, 0u);
        return last;
    };
    // the sum of `many` rows of counts, `stride` rows apart
    auto add_up = [&](const uint32_t *rows, int many, int stride) {
        constexpr int kPer = 8, kFly = 4;  // counts of a thread, and rows, in flight together
        for (int i0 = tid; i0 < words; i0 += kPer * kCountThreads) {
            uint32_t sum[kPer] = {};
            for (int k = 0; k < many; k += kFly) {
                uint32_t x[kFly][kPer];
#pragma unroll
                for (int j = 0; j < kFly; j++)
#pragma unroll
                    for (int i = 0; i < kPer; i++) {
                        const int at = i0 + i * kCountThreads;
                        x[j][i] = k + j < many && at < words ? ld_agent(rows + (size_t)(k + j) * stride * words + at) : 0;
                    }
#pragma unroll
                for (int j = 0; j < kFly; j++)
#pragma unroll
                    for (int i = 0; i < kPer; i++)
                        sum[i] += x[j][i];
            }
#pragma unroll
            for (int i = 0; i < kPer; i++)
                if (i0 + i * kCountThreads < words)
                    s_hist[i0 + i * kCountThreads] = sum[i];
        }
        __syncthreads();
    };
    uint32_t *rows = s.chunk_hist + (chunk_row - c) * words;
    int many = n_chunks, stride = 1;
    if (n_chunks > kSumChunks) {  // sums of sixteen first: one block adding up 320 rows took 91 us of kernel, now 24
        const int first = c / kSumChunks * kSumChunks, in = n_chunks - first < kSumChunks ? n_chunks - first : kSumChunks;
        if (!last_of(s.arrive + RECD_MAX_FEATURES + (chunk_row - c) + first, in))
            return;
        add_up(rows + (size_t)first * words, in, 1);
        for (int i = tid; i < words; i += kCountThreads)
            st_agent(rows + (size_t)first * words + i, s_hist[i]);
        stores_done();
        many = (n_chunks + kSumChunks - 1) / kSumChunks;
        stride = kSumChunks;
    }
    if (!last_of(s.arrive + f, many))
        return;
    add_up(rows, many, stride);
    write_bases(s, f, s_hist);
}

// ---- one digit ----------------------------------------------------------------------------------------
// A tile is 4096 entries (512 threads, 8 each; a wave owns 512 consecutive entries and walks them 64 at a
// time).  Ballots give a lane the lanes that hold its digit, a per-wave digit count in LDS the wave's
// earlier ones; a prefix over the waves completes the rank.  The entries are then laid out in LDS in
// digit order, so that a digit's entries (four on average with 10-bit digits) leave as one short run
// instead of as scattered words.  Bound by the latency of its chain (ticket, keys, ranks, look-back,
// stores); 40 KB of LDS keep four tiles on a CU.
union SweepShared {
    uint16_t run[kWaves][kMaxRadix];       // per wave: entries seen so far per digit
    struct { uint32_t key[kTile], pay[kTile]; } out;
    struct {
        uint16_t run[kWaves][kMaxRadix];
        uint32_t others[kMaxRadix];        // entries of a digit in the feature's tiles before this one (low half) and
        uint32_t key[kSmallTile], pay[kSmallTile];  // after it
    } small;
};

// The rank of an entry of digit d among its wave's entries of that digit so far, this round's included up to the lane;
// run: the wave's counts.
__device__ __forceinline__ uint32_t wave_rank(uint16_t *run, uint32_t d, bool valid, int dbits)
{
    const uint64_t all = __ballot(valid);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);  // lanes with my digit
#pragma unroll
    for (int bit = 0; bit < kMaxBits; bit++) {
        if (bit < dbits) {  // uniform
            const int one = (int)(d << (31 - bit)) >> 31;  // all ones where the bit is set
            const uint64_t bal = __ballot(one != 0);
            lo &= ~((uint32_t)bal ^ (uint32_t)one);
            hi &= ~((uint32_t)(bal >> 32) ^ (uint32_t)one);
        }
    }
    const uint32_t in_round = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
    const uint32_t of_digit = (uint32_t)(__popc(lo) + __popc(hi));
    // entries of this digit in the wave's earlier rounds; the first lane of each digit then adds this
    // round's (same wave: the read is complete before the write is issued)
    const uint32_t before = valid ? run[d] : 0;
    __builtin_amdgcn_wave_barrier();
    if (valid && in_round == 0)
        run[d] = (uint16_t)(before + of_digit);
    __builtin_amdgcn_wave_barrier();
    return before + in_round;
}

// One digit of a side of few entries.  Tiles of 4096 would leave most of the chip idle, and their ranks (a ballot per
// bit and 64 entries) and their look-back are then what a sweep takes; a tile of 1024 finds out for itself what the
// others of its feature hold, of the first digit from their counts, of a later one by counting their keys again, so
// that no tile waits for another.  The feature's digits start where the sum of all its tiles puts them.  0.19 M ids in
// 16 features: count 17.1 -> 11.6 us (its blocks no longer meet), a sweep 13.2 -> 9.8, weighted step 150 -> 137; tiles of
// 4096 without look-back: sweep 12.8.  With more tiles (and more entries a feature to count again) the chip is full either
// way: side A of 1.05 M rows in tiles of 4096 without look-back took the step from 797 to 818 us.
__device__ __forceinline__ void sweep_small_tiles(const GroupParams &g, const SideParams &s, bool side_a, uint32_t tile,
                                                  int pass, SweepShared &sh, uint32_t *s_from, uint16_t *s_loc)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint4 dsc;
    if (side_a) {
        const uint32_t per = (uint32_t)((g.B + kSmallTile - 1) / kSmallTile);
        dsc = make_uint4(tile / per, tile % per, (uint32_t)(tile / per * g.B), (uint32_t)g.B);
    } else {
        dsc = g.desc_small[tile];
    }
    const uint32_t k = dsc.y, f_begin = dsc.z, f_len = dsc.w, at0 = k * kSmallTile;
    const uint32_t n = f_len - at0 < (uint32_t)kSmallTile ? f_len - at0 : (uint32_t)kSmallTile;
    const uint32_t tiles_f = (f_len + kSmallTile - 1) / kSmallTile;
    const uint32_t *kin = s.key[(pass + 1) & 1] + f_begin, *pin = s.pay[(pass + 1) & 1] + f_begin;
    uint32_t *kout = s.key[pass & 1], *pout = s.pay[pass & 1];
    const int radix = 1 << s.dbits, shift = pass * s.dbits, d0 = 2 * tid;  // d0, d0 + 1: the thread's digits
    const uint32_t mask = radix - 1, i0 = w * (64 * kSmallItems) + lane;
    uint32_t key[kSmallItems], pay[kSmallItems], rank[kSmallItems];
#pragma unroll
    for (int u = 0; u < kSmallItems; u++) {
        const uint32_t i = at0 + i0 + u * 64;
        key[u] = pay[u] = 0;
        if (i0 + u * 64 < n) {
            if (pass > 0) {
                key[u] = kin[i];
                pay[u] = pin[i];
            } else if (side_a) {
                key[u] = (uint32_t)g.inverse[f_begin + i];
                pay[u] = f_begin + i;
            } else {
                key[u] = (uint32_t)g.u_values[f_begin + i];
                pay[u] = g.pay_positions ? f_begin + i : g.pos_list[f_begin + i];
            }
        }
    }
    uint32_t before[2] = {0, 0}, after[2] = {0, 0};
    constexpr int kFly = 8;
    if (pass == 0 && d0 < radix) {
        const uint32_t *rows = s.small_hist + (size_t)(tile - k) * radix + d0;
        for (uint32_t j0 = 0; j0 < tiles_f; j0 += kFly) {
            uint2 x[kFly];
#pragma unroll
            for (int u = 0; u < kFly; u++) {
                const uint32_t j = j0 + u;
                x[u] = j < tiles_f && j != k ? *reinterpret_cast<const uint2 *>(rows + (size_t)j * radix) : make_uint2(0, 0);
            }
#pragma unroll
            for (int u = 0; u < kFly; u++) {
                before[0] += j0 + u < k ? x[u].x : 0;
                before[1] += j0 + u < k ? x[u].y : 0;
                after[0] += j0 + u < k ? 0 : x[u].x;
                after[1] += j0 + u < k ? 0 : x[u].y;
            }
        }
    }
    for (int i = tid; i < (int)(offsetof(SweepShared, small.key) / sizeof(uint32_t)); i += kTileThreads)
        reinterpret_cast<uint32_t *>(&sh)[i] = 0;
    __syncthreads();
    if (pass > 0) {
        for (uint32_t j0 = 0; j0 < f_len; j0 += kFly * kTileThreads) {
            uint32_t x[kFly];
#pragma unroll
            for (int u = 0; u < kFly; u++) {
                const uint32_t i = j0 + u * kTileThreads + tid;
                x[u] = i < f_len ? kin[i] : 0;
            }
#pragma unroll
            for (int u = 0; u < kFly; u++) {
                // The lanes that hold the first lane's digit are counted by one atomic: skewed ids and the rows of a
                // session share their high digits, and a wave's atomics on one address queue.
                const uint32_t i = j0 + u * kTileThreads + tid;
                const bool on = i < f_len && i - at0 >= n;
                const uint32_t d = on ? (x[u] >> shift) & mask : ~0u, one = i < at0 ? 1u : 1u << 16;
                const uint64_t same = __ballot(d == (uint32_t)__builtin_amdgcn_readfirstlane(d));
                if (on && !((same >> lane) & 1))
                    atomicAdd(&sh.small.others[d], one);
                else if (on && lane == 0)
                    atomicAdd(&sh.small.others[d], one * (uint32_t)__popcll(same));
            }
        }
    }
#pragma unroll
    for (int u = 0; u < kSmallItems; u++)
        rank[u] = wave_rank(sh.small.run[w], (key[u] >> shift) & mask, i0 + u * 64 < n, s.dbits);
    __syncthreads();
    uint32_t cnt[2] = {0, 0}, of_digit[2];
#pragma unroll
    for (int e = 0; e < 2; e++) {
        if (d0 < radix) {
#pragma unroll
            for (int ww = 0; ww < kWaves; ww++) {
                const uint32_t x = sh.small.run[ww][d0 + e];
                sh.small.run[ww][d0 + e] = (uint16_t)cnt[e];
                cnt[e] += x;
            }
            if (pass > 0) {
                before[e] = sh.small.others[d0 + e] & 0xffff;
                after[e] = sh.small.others[d0 + e] >> 16;
            }
        }
        of_digit[e] = before[e] + cnt[e] + after[e];
    }
    uint64_t total;  // low half: where a digit starts in the tile, high half: in the feature
    const uint64_t starts = block_excl<uint64_t, kWaves>(((uint64_t)(of_digit[0] + of_digit[1]) << 32) | (cnt[0] + cnt[1]),
                                                         total);
#pragma unroll
    for (int e = 0; e < 2; e++)
        if (d0 < radix) {
            const uint32_t at = (uint32_t)starts + (e ? cnt[0] : 0);
            s_loc[d0 + e] = (uint16_t)at;
            s_from[d0 + e] = f_begin + (uint32_t)(starts >> 32) + (e ? of_digit[0] : 0) + before[e] - at;
        }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSmallItems; u++)
        if (i0 + u * 64 < n) {
            const uint32_t d = (key[u] >> shift) & mask, to = rank[u] + s_loc[d] + sh.small.run[w][d];
            sh.small.key[to] = key[u];
            sh.small.pay[to] = pay[u];
        }
    __syncthreads();
    const bool resolve = !side_a && (g.u_weights || g.pay_pos) && pass == s.passes - 1;
#pragma unroll
    for (int u = 0; u < kSmallItems; u++) {
        const uint32_t i = tid + u * kTileThreads;
        if (i < n) {
            const uint32_t kk = sh.small.key[i], pp = sh.small.pay[i];
            const uint32_t dst = s_from[(kk >> shift) & mask] + i;
            kout[dst] = kk;
            if (resolve) {  // the entry's source row and its weight or position, both in sorted order
                pout[dst] = g.pos_list[pp];
                if (g.u_weights)
                    g.pay_w[dst] = g.u_weights[pp];
                else
                    g.pay_pos[dst] = pp;
            } else {
                pout[dst] = pp;
            }
        }
    }
}

__global__ __launch_bounds__(kTileThreads) void k_group_sweep(const GroupParams g, int pass)
{
    __shared__ SweepShared sh;
    __shared__ uint32_t s_from[kMaxRadix];     // where the tile's entries of a digit go, less their place in LDS
    __shared__ uint16_t s_loc[kMaxRadix];      // where they start in LDS
    __shared__ uint32_t s_tile, s_window;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bool side_a = blockIdx.x < g.a_blocks;
    const SideParams &s = side_a ? g.a : g.b;
    const unsigned blk = side_a ? blockIdx.x : blockIdx.x - g.a_blocks;
    const uint32_t small_tiles = side_a ? (g.small_a ? g.a_blocks : 0) : g.tile_total[1];
    if (small_tiles) {
        if (blk < small_tiles)
            sweep_small_tiles(g, s, side_a, blk, pass, sh, s_from, s_loc);
        return;
    }
    if (!side_a && blk >= g.b_tiles)
        return;  // whole block: there for small tiles
    // ---- a tile: from the block's own queue while it has any, then from the others ------------------
    if (tid == 0) {
        uint32_t tile = ~0u;
        const int per_q = g.F / kQueues, more = g.F % kQueues;
        for (int i = 0; i < kQueues && tile == ~0u; i++) {
            const int q = (int)((blockIdx.x + i) % kQueues);
            uint32_t q0, q1;
            if (side_a) {
                q0 = (uint32_t)((q * per_q + (q < more ? q : more)) * g.tpf);
                q1 = q0 + (uint32_t)((per_q + (q < more ? 1 : 0)) * g.tpf);
            } else {
                q0 = g.queue_start[q];
                q1 = g.queue_start[q + 1];
            }
            if (q1 > q0) {
                const uint32_t t = __hip_atomic_fetch_add(s.ticket + pass * kQueues + q, 1u, __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT);
                if (t < q1 - q0)
                    tile = q0 + t;
            }
        }
        s_tile = tile;
    }
    const int radix = 1 << s.dbits;
    for (int i = tid; i < kWaves * kMaxRadix / 2; i += kTileThreads)
        reinterpret_cast<uint32_t *>(&sh.run[0][0])[i] = 0;
    __syncthreads();
    const uint32_t tile = s_tile;
    if (tile == ~0u)
        return;  // whole block: no tile left
    uint32_t f, k, begin, n, tiles_f, f_begin;
    if (side_a) {
        const int per_q = g.F / kQueues, more = g.F % kQueues;
        const uint32_t i = tile / g.tpf;  // the i-th feature in queue order
        const uint32_t wide = more * (per_q + 1);
        f = i < wide ? (i % (per_q + 1)) * kQueues + i / (per_q + 1)
                     : ((i - wide) % per_q) * kQueues + more + (i - wide) / per_q;
        k = tile % g.tpf;
        f_begin = (uint32_t)(f * g.B);
        begin = f_begin + k * kTile;
        n = (uint32_t)(g.B - (int64_t)k * kTile < kTile ? g.B - (int64_t)k * kTile : kTile);
        tiles_f = g.tpf;
    } else {
        const uint2 d = g.desc_queue[tile];
        f = d.x;
        k = d.y;
        f_begin = g.pb[f];
        const uint32_t f_end = g.pb[f + 1];
        begin = f_begin + k * kTile;
        n = f_end - begin < (uint32_t)kTile ? f_end - begin : (uint32_t)kTile;
        tiles_f = (f_end - f_begin + kTile - 1) / kTile;
    }
    const uint32_t *kin = s.key[(pass + 1) & 1], *pin = s.pay[(pass + 1) & 1];
    uint32_t *kout = s.key[pass & 1], *pout = s.pay[pass & 1];
    const int shift = pass * s.dbits;
    const uint32_t mask = radix - 1;

    // ---- ranks ------------------------------------------------------------------------------------------
    uint32_t key[kItems], pay[kItems], rank[kItems];
    const uint32_t wbase = w * (64 * kItems) + lane;
#pragma unroll
    for (int u = 0; u < kItems; u++) {
        const uint32_t i = wbase + u * 64;
        key[u] = pay[u] = 0;
        if (i < n) {
            if (pass > 0) {
                key[u] = kin[begin + i];
                pay[u] = pin[begin + i];
            } else if (side_a) {
                key[u] = (uint32_t)g.inverse[begin + i];
                pay[u] = begin + i;
            } else {
                key[u] = (uint32_t)g.u_values[begin + i];
                pay[u] = g.pay_positions ? begin + i : g.pos_list[begin + i];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < kItems; u++)
        rank[u] = wave_rank(sh.run[w], (key[u] >> shift) & mask, wbase + u * 64 < n, s.dbits);
    __syncthreads();
    // ---- digits d = 2 * tid, 2 * tid + 1: prefix over the waves, count of the tile --------------------------
    uint32_t cnt[2] = {0, 0};
    const int d0 = 2 * tid;
#pragma unroll
    for (int e = 0; e < 2; e++) {
        if (d0 + e < radix) {
            uint32_t run = 0;
#pragma unroll
            for (int ww = 0; ww < kWaves; ww++) {
                const uint32_t x = sh.run[ww][d0 + e];
                sh.run[ww][d0 + e] = (uint16_t)run;
                run += x;
            }
            cnt[e] = run;
        }
    }
    // Look-back: the counts go out first, a flag per tile behind them, so that whoever waits polls one word
    // a tile (polling the 1024 counts themselves kept the fabric busy: 37 us a sweep at 2.2 M entries).
    uint32_t *const own = s.own + (size_t)(tile - k) * radix, *const upto = s.upto + (size_t)(tile - k) * radix;
    uint32_t *const flag = s.flag + (size_t)pass * s.tiles_cap + (tile - k);  // of the feature's tiles
    if (tiles_f > 1) {
        uint32_t *dst = (k == 0 ? upto : own) + (size_t)k * radix;
#pragma unroll
        for (int e = 0; e < 2; e++)
            if (d0 + e < radix)
                st_agent(dst + d0 + e, cnt[e]);
    }
    uint32_t total;
    const uint32_t loc = block_excl<uint32_t, kWaves>(cnt[0] + cnt[1], total);
    if (tiles_f > 1) {
        stores_done();
        __syncthreads();
        if (tid == 0)
            st_agent(flag + k, k == 0 ? 2u : 1u);
    }
    uint32_t excl[2] = {0, 0};
    for (int64_t j = (int64_t)k - 1; j >= 0;) {
        if (w == 0) {
            // 64 tiles at a time, the nearest first: up to one that has the counts of all before it, or all
            const int window = j + 1 < 64 ? (int)j + 1 : 64;
            int take;
            bool last;
            for (;;) {
                const uint32_t x = lane < window ? ld_agent(flag + (j - lane)) : 0;
                const uint64_t none = __ballot(lane < window && x == 0), full = __ballot(x == 2);
                const int stop = none ? __builtin_ctzll(none) : window;
                const int fin = full ? __builtin_ctzll(full) : 64;
                last = fin < stop;
                take = last ? fin + 1 : window;
                if (last || stop == window)
                    break;
                __builtin_amdgcn_s_sleep(2);
            }
            if (lane == 0)
                s_window = (uint32_t)take | (last ? 256u : 0u);
        }
        __syncthreads();
        const uint32_t win = s_window;
        const int take = (int)(win & 255u);
        const bool last = (win & 256u) != 0;
        __syncthreads();
        constexpr int kFly = 8;
        for (int i = 0; i < take; i += kFly) {
            uint64_t x[kFly];  // both digits of a tile in one load (one feature, 320 tiles: 47 -> 41 us a sweep)
#pragma unroll
            for (int u = 0; u < kFly; u++) {
                const uint32_t *src = (last && i + u == take - 1 ? upto : own) + (size_t)(j - i - u) * radix + d0;
                x[u] = i + u < take && d0 < radix ? ld_agent(reinterpret_cast<const uint64_t *>(src)) : 0;
            }
#pragma unroll
            for (int u = 0; u < kFly; u++) {
                excl[0] += (uint32_t)x[u];
                excl[1] += (uint32_t)(x[u] >> 32);
            }
        }
        if (last)
            break;
        j -= take;
    }
    const bool pass_on = k > 0 && k + 1 < tiles_f;
#pragma unroll
    for (int e = 0; e < 2; e++) {
        const int d = d0 + e;
        if (d >= radix)
            continue;
        if (pass_on)
            st_agent(upto + (size_t)k * radix + d, excl[e] + cnt[e]);
        const uint32_t at = loc + (e ? cnt[0] : 0);
        s_loc[d] = (uint16_t)at;
        s_from[d] = f_begin + s.base[((size_t)f * s.passes + pass) * radix + d] + excl[e] - at;
    }
    __syncthreads();
    // ---- into LDS in digit order, then out ---------------------------------------------------------------
#pragma unroll
    for (int u = 0; u < kItems; u++)
        if (wbase + u * 64 < n) {
            const uint32_t d = (key[u] >> shift) & mask;
            rank[u] += (uint32_t)s_loc[d] + sh.run[w][d];
        }
    if (pass_on)
        stores_done();
    __syncthreads();  // the counts have been read: their memory takes the entries
    if (pass_on && tid == 0)
        st_agent(flag + k, 2u);
#pragma unroll
    for (int u = 0; u < kItems; u++)
        if (wbase + u * 64 < n) {
            sh.out.key[rank[u]] = key[u];
            sh.out.pay[rank[u]] = pay[u];
        }
    __syncthreads();
    const bool resolve = !side_a && (g.u_weights || g.pay_pos) && pass == s.passes - 1;
#pragma unroll
    for (int u = 0; u < kItems; u++) {
        const uint32_t i = tid + u * kTileThreads;
        if (i < n) {
            const uint32_t kk = sh.out.key[i], pp = sh.out.pay[i];
            const uint32_t dst = s_from[(kk >> shift) & mask] + i;
            kout[dst] = kk;
            if (resolve) {  // the entry's source row and its weight or position, both in sorted order
                pout[dst] = g.pos_list[pp];
                if (g.u_weights)
                    g.pay_w[dst] = g.u_weights[pp];
                else
                    g.pay_pos[dst] = pp;
            } else {
                pout[dst] = pp;
            }
        }
    }
}

// ---- segments of equal keys ---------------------------------------------------------------------------
// Side A: the segment number of a slot is feat_uoff[f] + slot, so starts are written without numbering
// (recd_slot_starts: a slot that no row names gets an empty segment).  Side B: a head is an entry whose key
// differs from its predecessor's in the feature; heads are numbered across all tiles in feature order by
// look-back words that carry the number of heads and the position of the last one, so the block that finds the
// next head also knows the length of the segment it closes: segments of more than long_seg entries are
// cut into chunks of 256 entries (larger ones if that would give more than 64).  The cut depends on the
// length only; the order in which segments and chunks are listed does not matter for the sums.
__global__ __launch_bounds__(kTileThreads) void k_group_segments(const GroupParams g)
{
    __shared__ uint32_t s_tile;
    __shared__ uint64_t s_wave[kWaves];  // heads of a wave (high half), position of its last head + 1
    __shared__ uint64_t s_before, s_chunk0;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (blockIdx.x < g.a_blocks) {
        const uint32_t *ks = g.a.key[(g.a.passes - 1) & 1];
        const uint32_t n = (uint32_t)g.n_lists, B = (uint32_t)g.B;
#pragma unroll
        for (int u = 0; u < kItems; u++) {
            const uint32_t i = blockIdx.x * kTile + u * kTileThreads + tid;
            if (i >= n)
                break;
            const uint32_t f = i / B;
            const bool last = i == f * B + (B - 1);
            const int64_t u0 = g.feat_uoff[f], u1 = g.feat_uoff[f + 1];
            recd_slot_starts(ks[i], i == f * B ? 0u : ks[i - 1], i == f * B, last, sorted_bits(g.a), u1 - u0,
                             [&](int64_t x, bool closed) { g.seg_start_a[u0 + x] = (int64_t)i + closed; });
            if (last && (int)f == g.F - 1) {
                g.seg_start_a[u1] = n;
                g.list_off_a[0] = 0;
                g.list_off_a[1] = u1 < g.lists_cap ? u1 : g.lists_cap;
            }
        }
        return;
    }
    const uint32_t total = g.tile_total[0];
    if (tid == 0)
        s_tile = __hip_atomic_fetch_add(g.b.ticket + kMaxPasses * kQueues, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const uint32_t tile = s_tile;
    if (tile >= total) {
        if (total == 0 && tile == 0) {  // no id anywhere
            for (int f = tid; f <= g.F; f += kTileThreads)
                g.feat_roff[f] = 0;
            if (tid == 0)
                g.seg_start_b[0] = g.list_off_b[0] = g.list_off_b[1] = 0;
        }
        return;
    }
    const uint4 dsc = g.desc_feat[tile];
    const uint32_t f = dsc.x, k = dsc.y;
    const uint32_t f_end = dsc.z + dsc.w, begin = dsc.z + k * kTile;
    const uint32_t n = f_end - begin < (uint32_t)kTile ? f_end - begin : (uint32_t)kTile;
    const uint32_t *ks = g.b.key[(g.b.passes - 1) & 1] + begin;
    // a wave owns 512 consecutive entries, 64 a round: heads are ballots, their numbers popcounts and the
    // nearest head before a lane a leading-zero count
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    const uint32_t wbase = w * (64 * kItems);
    uint32_t key[kItems], num[kItems], open[kItems];  // open: position + 1 of the nearest head before, 0: none in the wave
    uint32_t prev_last = wbase > 0 && wbase < n ? ks[wbase - 1] : (k > 0 && wbase == 0 ? ks[-1] : 0);
    uint64_t hm[kItems];
#pragma unroll
    for (int u = 0; u < kItems; u++) {
        const uint32_t i = wbase + u * 64 + lane;
        key[u] = i < n ? ks[i] : 0;
    }
    uint32_t heads = 0, last = 0;  // of the wave so far
#pragma unroll
    for (int u = 0; u < kItems; u++) {
        const uint32_t i = wbase + u * 64 + lane;
        uint32_t prev = __shfl_up(key[u], 1);
        if (lane == 0)
            prev = prev_last;
        prev_last = __shfl(key[u], 63);
        hm[u] = __ballot(i < n && ((k == 0 && i == 0) || key[u] != prev));
        const uint64_t below = hm[u] & lt_mask;
        num[u] = heads + (uint32_t)__popcll(below);
        open[u] = below ? begin + wbase + u * 64 + (63 - __builtin_clzll(below)) + 1 : last;
        heads += (uint32_t)__popcll(hm[u]);
        if (hm[u])
            last = begin + wbase + u * 64 + (63 - __builtin_clzll(hm[u])) + 1;
    }
    if (lane == 0)
        s_wave[w] = ((uint64_t)heads << 32) | last;
    __syncthreads();
    uint32_t wh = 0, wl = 0, all_h = 0, all_l = 0;  // the tile's waves before this one; the tile
#pragma unroll
    for (int i = 0; i < kWaves; i++) {
        const uint32_t h = (uint32_t)(s_wave[i] >> 32), l = (uint32_t)s_wave[i];
        if (i < w) {
            wh += h;
            wl = l > wl ? l : wl;
        }
        all_h += h;
        all_l = l > all_l ? l : all_l;
    }
    // look-back word: two bits, heads (31), position of the last head + 1 (31; positions stay below 2^31)
    constexpr uint64_t m31 = (1ull << 31) - 1;
    if (w == 0) {
        uint64_t bh = 0, bl = 0;
        if (lane == 0)
            st_agent(g.seg_status + tile, ((uint64_t)(tile == 0 ? 2 : 1) << 62) | ((uint64_t)all_h << 31) | all_l);
        int64_t j = (int64_t)tile - 1;
        while (j >= 0) {  // 64 tiles at a time
            const uint64_t x = j - lane >= 0 ? ld_agent(g.seg_status + (j - lane)) : 0;
            const uint64_t none = __ballot((x >> 62) == 0), full = __ballot((x >> 62) == 2);
            const int stop = none ? __builtin_ctzll(none) : 64;      // words from here on are not there yet
            const int fin = full ? __builtin_ctzll(full) : 64;
            const int take = fin < stop ? fin + 1 : stop;
            uint64_t h = lane < take ? (x >> 31) & m31 : 0, l = lane < take ? x & m31 : 0;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                h += __shfl_xor(h, d);
                const uint64_t y = __shfl_xor(l, d);
                l = y > l ? y : l;
            }
            bh += h;
            bl = l > bl ? l : bl;
            if (fin < stop)
                break;
            j -= take;
            if (take == 0)
                __builtin_amdgcn_s_sleep(1);
        }
        if (lane == 0) {
            if (tile > 0)
                st_agent(g.seg_status + tile, (2ull << 62) | ((bh + all_h) << 31) | (all_l > bl ? all_l : bl));
            s_before = (bh << 32) | bl;
        }
    }
    __syncthreads();
    const uint32_t bh = (uint32_t)(s_before >> 32), bl = (uint32_t)s_before;
    const uint32_t seg0 = bh + wh, open0 = wl > bl ? wl : bl;
    // chunks of a segment that is cut
    auto chunk_of = [&](uint32_t len) { return len > 64 * 256 ? (len + 63) / 64 : 256u; };
    auto chunks_of = [&](uint32_t len) { return len > (uint32_t)g.long_seg ? (len + chunk_of(len) - 1) / chunk_of(len) : 0u; };
    uint32_t mine = 0;  // chunks of the segments that this thread's entries close
#pragma unroll
    for (int u = 0; u < kItems; u++) {
        const uint32_t i = wbase + u * 64 + lane, at = begin + i;
        if ((hm[u] >> lane) & 1) {
            const uint32_t seg = seg0 + num[u];
            if (open[u] == 0)
                open[u] = open0;
            mine += open[u] ? chunks_of(at + 1 - open[u]) : 0;
            g.seg_start_b[seg] = at;
            g.touched_rows[seg] = key[u] & sorted_bits(g.b);  // of an id beyond the tables only these count
            g.seg_feat[seg] = (int32_t)f;
            if (k == 0 && i == 0) {
                const int first = tile == 0 ? 0 : (int)g.desc_feat[tile - 1].x + 1;
                for (int ff = first; ff <= (int)f; ff++)  // features without ids before this one
                    g.feat_roff[ff] = seg;
            }
        }
    }
    // the last entry of all closes the list
    uint32_t tail_seg = 0, tail_open = 0, tail_end = 0;
    if (tile == total - 1 && tid == 0) {
        tail_seg = bh + all_h - 1;
        tail_open = (all_l > bl ? all_l : bl) - 1;
        tail_end = begin + n;
        mine += chunks_of(tail_end - tail_open);
        g.seg_start_b[tail_seg + 1] = tail_end;
        g.list_off_b[0] = 0;
        g.list_off_b[1] = (int64_t)tail_seg + 1;
        for (int ff = (int)f + 1; ff <= g.F; ff++)
            g.feat_roff[ff] = (int64_t)tail_seg + 1;
    }
    // room for the tile's chunks: one atomic a tile
    uint32_t all;
    const uint32_t ex = block_excl<uint32_t, kWaves>(mine, all);
    if (all == 0)
        return;
    if (tid == 0)
        s_chunk0 = atomicAdd(reinterpret_cast<unsigned long long *>(g.chunk_count), (unsigned long long)all);
    __syncthreads();
    uint32_t item = (uint32_t)s_chunk0 + ex;
    auto put = [&](uint32_t seg, uint32_t start, uint32_t end) {
        const uint32_t nch = chunks_of(end - start), ch = chunk_of(end - start), first = item;
        if (nch == 0)
            return;
        g.chunk_arrive[first] = 0;
        for (uint32_t c = 0; c < nch; c++)
            g.chunks[item++] = RecdChunk{start + c * ch, c + 1 < nch ? start + (c + 1) * ch : end, seg, first, nch};
    };
#pragma unroll
    for (int u = 0; u < kItems; u++)
        if (((hm[u] >> lane) & 1) && open[u])
            put(seg0 + num[u] - 1, open[u] - 1, begin + wbase + u * 64 + lane);
    if (tail_end)
        put(tail_seg, tail_open, tail_end);
}

// ---- small batches: both sides in one launch -------------------------------------------------------
// Up to 8192 ids and 8192 rows per feature: the first blocks group `per` neighbouring features' ids each (key = feature and
// row), the others the rows of one feature, each by a radix sort in LDS, and write the segments straight from there.
// The blocks of the ids take their features by tickets and meet once, when they learn how many rows and chunks the features
// before theirs hold: a block waits for blocks that started before it only.  The last that has read the others' words
// clears them for the next launch.
// The four launches above cost such a batch their launches and a chain of dependent round trips each (2048 rows, 5 K ids:
// 38 us of kernels); here it is one chain.  (One block for all ids, and scans through
// LDS, 24 us; a block for each of the four features 16.0, with scans by lane shifts 13.9; one feature of 2.6 K ids 13.5 and 12.1.
// Blocks of 16 waves on a CU of their own are bound by what they issue.)
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / 64;
constexpr int kSmallRounds = 8;
constexpr int kSmallCap = kSmallThreads * kSmallRounds;
static_assert(RECD_MAX_FEATURES + 2 <= RECD_GROUP_ARRIVE, "a word a block, the ticket and the count of readers");

__global__ __launch_bounds__(kSmallThreads) void k_group_small(const GroupParams g, int b_blocks, int per, int row_bits,
                                                               int passes_b, int dbits_b)
{
    __shared__ uint32_t s_key[kSmallCap], s_pay[kSmallCap];
    __shared__ uint16_t s_run[kSmallWaves][kMaxRadix];
    __shared__ uint16_t s_loc[kMaxRadix];
    __shared__ uint64_t s_wave[kSmallWaves];
    __shared__ uint32_t s_fu[RECD_MAX_FEATURES + 1], s_chunks, s_blk, s_before[2];
    static_assert(kSmallWaves == 16, "a row of lanes scans the waves' sums");
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool side_a = (int)blockIdx.x >= b_blocks;
    const uint32_t f_a = blockIdx.x - b_blocks;
    const uint32_t row_mask = (uint32_t)((1ull << row_bits) - 1);  // with the features' bits it fits 32
    uint32_t *const words = g.b.arrive, *const ticket = words + RECD_MAX_FEATURES, *const readers = ticket + 1;
    uint32_t n, blk = 0, p0 = 0;  // p0: the first position
    uint32_t key[kSmallRounds], pay[kSmallRounds], rank[kSmallRounds];
    int f0 = 0, f1 = 0;           // the block's features
    if (side_a) {
        n = (uint32_t)g.B;
    } else {
        if (tid == 0)
            s_chunks = 0;
        if (b_blocks > 1) {
            if (tid == 0)
                s_blk = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            blk = s_blk;
        }
        f0 = (int)blk * per;
        f1 = f0 + per < g.F ? f0 + per : g.F;
        const uint32_t u0 = (uint32_t)g.feat_uoff[f0], u1 = (uint32_t)g.feat_uoff[f1];
        if (per > 1) {
            for (int i = tid; i <= f1 - f0; i += kSmallThreads)
                s_fu[i] = (uint32_t)g.feat_uoff[f0 + i];
            __syncthreads();
        }
        // one round trip: the block's positions and its first lists'
        int64_t a = 0, e = 0;
        if (u0 + tid < u1) {
            a = g.u_offsets[u0 + tid];
            e = g.u_offsets[u0 + tid + 1];
        }
        const int64_t P = g.u_offsets[u0], M = g.u_offsets[u1];
        p0 = (uint32_t)(P < g.M_cap ? P : g.M_cap);
        n = (uint32_t)(M < g.M_cap ? M : g.M_cap) - p0;
        if (f1 == g.F && tid == 0)
            g.too_small_b[0] = M > g.M_cap ? 1 : 0;
        // the ids are on their way meanwhile
        const uint32_t rounds = (n + kSmallThreads - 1) / kSmallThreads, i0 = w * (rounds * 64) + lane;
#pragma unroll
        for (int u = 0; u < kSmallRounds; u++) {
            if (u >= (int)rounds)  // the same in every thread, here and below
                break;
            key[u] = i0 + u * 64 < n ? (uint32_t)g.u_values[p0 + i0 + u * 64] : 0u;
        }
        // every list fills in its number and its feature at its positions (an empty list has none): a lane up to
        // 64 of them, the whole wave what lies beyond, list by list (a list of 7000 ids by one lane: backward 230 us,
        // now 44; with 16 instead of 64 the lists of 20 ids in a batch of 5 K took 1 us more)
        for (uint32_t v0 = u0; v0 < u1; v0 += kSmallThreads) {
            const uint32_t u = v0 + tid;
            uint32_t at = 0, end = 0, name = 0, fkey = 0;
            if (u < u1) {
                if (v0 > u0) {
                    a = g.u_offsets[u];
                    e = g.u_offsets[u + 1];
                }
                int f = 0;  // the last feature with s_fu[f] <= u
                for (int st = RECD_MAX_FEATURES / 2; per > 1 && st >= 1; st >>= 1)
                    if (f + st < f1 - f0 && s_fu[f + st] <= u)
                        f += st;
                at = a - p0 < (int64_t)n ? (uint32_t)(a - p0) : n;
                end = e - p0 < (int64_t)n ? (uint32_t)(e - p0) : n;
                name = (int64_t)u < g.lists_cap ? u : (uint32_t)(g.lists_cap - 1);
                fkey = per > 1 ? (uint32_t)f << row_bits : 0;
            }
            const uint32_t own = end > at + 64 ? at + 64 : end;
            for (uint32_t j = at; j < own; j++) {
                s_pay[j] = name;
                s_key[j] = fkey;
            }
            for (uint64_t longer = __ballot(own < end); longer; longer &= longer - 1) {
                const int l = __builtin_ctzll(longer);
                const uint32_t to = __shfl(end, l), list = __shfl(name, l), key_f = __shfl(fkey, l);
                for (uint32_t j = __shfl(own, l) + lane; j < to; j += 64) {
                    s_pay[j] = list;
                    s_key[j] = key_f;
                }
            }
        }
        __syncthreads();
    }
    // a wave owns `rounds` * 64 consecutive entries
    const int rounds = (int)((n + kSmallThreads - 1) / kSmallThreads);
    const uint32_t wbase = w * (rounds * 64) + lane;
#pragma unroll
    for (int u = 0; u < kSmallRounds; u++) {
        if (u >= rounds)
            break;
        const uint32_t i = wbase + u * 64;
        pay[u] = 0;
        if (i >= n) {
            key[u] = 0;
        } else if (side_a) {
            key[u] = (uint32_t)g.inverse[f_a * g.B + i];
            pay[u] = (uint32_t)(f_a * g.B + i);
        } else {
            key[u] = s_key[i] | (key[u] & row_mask);  // an id beyond the tables stays in its feature
            pay[u] = g.pay_positions ? p0 + i : s_pay[i];
            if (g.u_weights || g.pay_pos)
                g.pos_list[p0 + i] = s_pay[i];
        }
    }
    const int passes = side_a ? g.a.passes : passes_b, dbits = side_a ? g.a.dbits : dbits_b;
    const int radix = 1 << dbits;
    const uint32_t mask = radix - 1;
    for (int p = 0; p < passes; p++) {
        const int shift = p * dbits;
        __syncthreads();  // the previous pass is done with the shared arrays
        for (int i = tid; i < kSmallWaves * kMaxRadix / 2; i += kSmallThreads)
            reinterpret_cast<uint32_t *>(&s_run[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSmallRounds; u++) {
            if (u >= rounds || wbase - lane + u * 64 >= n)  // the same in every thread of the wave
                break;
            const bool valid = wbase + u * 64 < n;
            const uint32_t d = (key[u] >> shift) & mask;
            const uint64_t all = __ballot(valid);
            uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);  // lanes with my digit
#pragma unroll
            for (int bit = 0; bit < kMaxBits; bit++) {
                if (bit < dbits) {
                    const int one = (int)(d << (31 - bit)) >> 31;
                    const uint64_t bal = __ballot(one != 0);
                    lo &= ~((uint32_t)bal ^ (uint32_t)one);
                    hi &= ~((uint32_t)(bal >> 32) ^ (uint32_t)one);
                }
            }
            const uint32_t in_round = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0));
            const uint32_t before = valid ? s_run[w][d] : 0;
            __builtin_amdgcn_wave_barrier();
            if (valid && in_round == 0)
                s_run[w][d] = (uint16_t)(before + __popc(lo) + __popc(hi));
            __builtin_amdgcn_wave_barrier();
            rank[u] = before + in_round;
        }
        __syncthreads();
        uint32_t cnt = 0, total;
        if (tid < radix) {
#pragma unroll
            for (int ww = 0; ww < kSmallWaves; ww++) {
                const uint32_t x = s_run[ww][tid];
                s_run[ww][tid] = (uint16_t)cnt;
                cnt += x;
            }
        }
        const uint32_t at = block_excl<uint32_t, kSmallWaves>(cnt, total);
        if (tid < radix)
            s_loc[tid] = (uint16_t)at;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSmallRounds; u++) {
            if (u >= rounds)
                break;
            if (wbase + u * 64 < n) {
                const uint32_t d = (key[u] >> shift) & mask;
                const uint32_t to = (uint32_t)s_loc[d] + s_run[w][d] + rank[u];
                s_key[to] = key[u];
                s_pay[to] = pay[u];
            }
        }
        __syncthreads();
        if (p + 1 < passes) {
#pragma unroll
            for (int u = 0; u < kSmallRounds; u++) {
                if (u >= rounds)
                    break;
                if (wbase + u * 64 < n) {
                    key[u] = s_key[wbase + u * 64];
                    pay[u] = s_pay[wbase + u * 64];
                }
            }
        }
    }
    // ---- out, in the same order of threads ---------------------------------------------------------------
    if (side_a) {
        const int64_t u0 = g.feat_uoff[f_a], u1 = g.feat_uoff[f_a + 1];
        const uint32_t l0 = (uint32_t)(f_a * g.B);
        for (uint32_t i = tid; i < n; i += kSmallThreads) {
            g.a.pay[0][l0 + i] = s_pay[i];
            recd_slot_starts(s_key[i], i == 0 ? 0u : s_key[i - 1], i == 0, i == n - 1, sorted_bits(g.a), u1 - u0,
                             [&](int64_t x, bool closed) { g.seg_start_a[u0 + x] = (int64_t)l0 + i + closed; });
            if (i == n - 1 && (int)f_a == g.F - 1) {
                g.seg_start_a[u1] = g.n_lists;
                g.list_off_a[0] = 0;
                g.list_off_a[1] = u1 < g.lists_cap ? u1 : g.lists_cap;
                report_side_a(g, u1);
            }
        }
        return;
    }
    const uint64_t lt_mask = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    uint32_t heads = 0, last = 0;  // of the wave so far; last: place of its last head + 1
    uint32_t num[kSmallRounds], open[kSmallRounds], chunk[kSmallRounds];  // chunk: the first of the segment closed here
    uint64_t hm[kSmallRounds];
#pragma unroll
    for (int u = 0; u < kSmallRounds; u++) {
        if (u >= rounds)
            break;
        const uint32_t i = wbase + u * 64;
        hm[u] = __ballot(i < n && (i == 0 || s_key[i] != s_key[i - 1]));
        const uint64_t below = hm[u] & lt_mask;
        const uint32_t at0 = i - lane;
        num[u] = heads + (uint32_t)__popcll(below);
        open[u] = below ? at0 + (63 - __builtin_clzll(below)) + 1 : last;
        heads += (uint32_t)__popcll(hm[u]);
        if (hm[u])
            last = at0 + (63 - __builtin_clzll(hm[u])) + 1;
    }
    if (lane == 0)
        s_wave[w] = ((uint64_t)heads << 32) | last;
    __syncthreads();
    const uint64_t of_wave = s_wave[lane & 15];  // every wave scans the sixteen itself
    const uint32_t heads_to = row_scan_add((uint32_t)(of_wave >> 32));
    const int last_to = row_scan_max((int)(uint32_t)of_wave);
    const uint32_t R = of_lane(heads_to, 15), end_open = of_lane((uint32_t)last_to, 15);
    const uint32_t wh = w > 0 ? of_lane(heads_to, w - 1) : 0, wl = w > 0 ? of_lane((uint32_t)last_to, w - 1) : 0;
    // chunks of a segment that is cut
    static_assert(kSmallCap <= 64 * 256, "chunks of 256 entries, at most 64 of a segment");
    auto chunks_of = [&](uint32_t len) { return len > (uint32_t)g.long_seg ? (len + 255) / 256 : 0u; };
    uint32_t tail_chunk = 0;
#pragma unroll
    for (int u = 0; u < kSmallRounds; u++) {
        if (u >= rounds)
            break;
        const uint32_t i = wbase + u * 64;
        chunk[u] = 0;
        if (i >= n)
            continue;
        if ((hm[u] >> lane) & 1) {
            if (open[u] == 0)
                open[u] = wl;
            const uint32_t many = i > 0 ? chunks_of(i + 1 - open[u]) : 0;
            if (many)
                chunk[u] = atomicAdd(&s_chunks, many);
        }
        if (i == n - 1) {
            const uint32_t many = chunks_of(n + 1 - end_open);
            if (many)
                tail_chunk = atomicAdd(&s_chunks, many);
        }
    }
    __syncthreads();
    // rows and chunks of the blocks before this one: what needs neither goes out while the words travel
    if (tid == 0 && b_blocks > 1)
        st_agent(words + blk, (R + 1) | (s_chunks << 16));  // 8192 and 8192 / 17 at most
#pragma unroll
    for (int u = 0; u < kSmallRounds; u++) {
        if (u >= rounds)
            break;
        const uint32_t i = wbase + u * 64;
        if (i >= n)
            continue;
        const uint32_t pp = s_pay[i];
        if (g.u_weights || g.pay_pos) {  // the entry's source row and its weight or position, both in sorted order
            g.b.pay[0][p0 + i] = g.pos_list[pp];
            if (g.u_weights)
                g.pay_w[p0 + i] = g.u_weights[pp];
            else
                g.pay_pos[p0 + i] = pp;
        } else {
            g.b.pay[0][p0 + i] = pp;
        }
    }
    if (w == 0 && b_blocks > 1) {
        uint32_t r = 0, c = 0;
        for (uint32_t j = lane; j < blk; j += 64) {
            uint32_t x;
            while ((x = ld_agent(words + j)) == 0)
                __builtin_amdgcn_s_sleep(1);
            r += (x & 0xffff) - 1;
            c += x >> 16;
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            r += __shfl_xor(r, d);
            c += __shfl_xor(c, d);
        }
        if (lane == 0) {
            s_before[0] = r;
            s_before[1] = c;
        }
    }
    uint32_t seg0 = 0, chunk0 = 0;
    if (b_blocks > 1) {
        __syncthreads();
        seg0 = s_before[0];
        chunk0 = s_before[1];
    }
    auto list_chunks = [&](uint32_t seg, uint32_t start, uint32_t end, uint32_t first) {
        const uint32_t nch = chunks_of(end - start);
        if (nch == 0)
            return;
        g.chunk_arrive[first] = 0;
        for (uint32_t c = 0; c < nch; c++)
            g.chunks[first + c] = RecdChunk{p0 + start + c * 256, p0 + (c + 1 < nch ? start + (c + 1) * 256 : end), seg, first, nch};
    };
#pragma unroll
    for (int u = 0; u < kSmallRounds; u++) {
        if (u >= rounds)
            break;
        const uint32_t i = wbase + u * 64;
        if (i >= n)
            continue;
        const uint32_t seg = seg0 + wh + num[u];
        if ((hm[u] >> lane) & 1) {
            const uint32_t kk = s_key[i], f = per > 1 ? kk >> row_bits : 0;
            const int fprev = i == 0 ? -1 : (per > 1 ? (int)(s_key[i - 1] >> row_bits) : 0);
            g.seg_start_b[seg] = p0 + i;
            g.touched_rows[seg] = kk & row_mask;
            g.seg_feat[seg] = f0 + (int32_t)f;
            for (int ff = fprev + 1; ff <= (int)f; ff++)
                g.feat_roff[f0 + ff] = seg;
            if (i > 0)
                list_chunks(seg - 1, open[u] - 1, i, chunk0 + chunk[u]);
        }
        if (i == n - 1)
            list_chunks(seg0 + R - 1, end_open - 1, n, chunk0 + tail_chunk);
    }
    if (tid == 0) {
        const int held = n == 0 ? -1 : (per > 1 ? (int)(s_key[n - 1] >> row_bits) : 0);
        for (int ff = held + 1; ff < f1 - f0; ff++)  // the block's features without ids behind the last that has some
            g.feat_roff[f0 + ff] = seg0 + R;
        if (f1 == g.F) {
            g.feat_roff[g.F] = seg0 + R;
            g.seg_start_b[seg0 + R] = p0 + n;
            g.list_off_b[0] = 0;
            g.list_off_b[1] = seg0 + R;
            g.chunk_count[0] = chunk0 + s_chunks;
        }
    }
    if (w == 0 && b_blocks > 1) {
        uint32_t before = 0;
        if (lane == 0)
            before = __hip_atomic_fetch_add(readers, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) == (uint32_t)(b_blocks - 1)) {  // every block has read the words
            for (int i = lane; i < b_blocks; i += 64)
                st_agent(words + i, 0u);
            if (lane < 2)
                st_agent(ticket + lane, 0u);
        }
    }
}

int bits_for(uint64_t max_value)
{
    int b = 1;
    while (b < 64 && (max_value >> b) != 0)
        b++;
    return b;
}

// Bits of a slot number: a feature has at most B slots, all features U_cap.
int slot_bits(int64_t B, int64_t U_cap)
{
    const int64_t slots = U_cap < B ? U_cap : B;
    return bits_for((uint64_t)(slots > 1 ? slots - 1 : 1));
}

// The fewest digits of at most 10 bits, as even as possible.
void digits_for(int bits, int *passes, int *dbits)
{
    *passes = (bits + kMaxBits - 1) / kMaxBits;
    *dbits = (bits + *passes - 1) / *passes;
}

int64_t chunk_for(int64_t n)
{
    int64_t chunk = kTile;
    while (n / chunk > kMostChunks)
        chunk *= 2;
    return chunk;
}

// No fewer than n / chunk_for(n), for n itself and everything below it: a bound that grows with n, so that the
// workspace for a batch's ids also holds every smaller M_cap.
int64_t chunks_bound(int64_t n) { return n / kTile < kMostChunks ? n / kTile : kMostChunks; }

// Words (digit counts of all passes) of a feature or chunk whose keys have at most `bits` bits.  Fewer bits can
// need more words: 10 bits are one digit of 1024, 14 bits two of 128.
size_t words_for(int bits)
{
    size_t most = 0;
    for (int b = 1; b <= bits; b++) {
        int passes, dbits;
        digits_for(b, &passes, &dbits);
        const size_t n = (size_t)passes << dbits;
        most = n > most ? n : most;
    }
    return most;
}

}  // namespace

RecdGroupWs recd_group_carve(WsCarver &c, int F, int64_t B, int64_t M_cap)
{
    RecdGroupWs w{};
    const int64_t n_lists = (int64_t)F * B;
    auto side = [&](RecdGroupWs::Side &s, int64_t n, int64_t tiles, int64_t chunks, size_t words_per_tile) {
        for (int i = 0; i < 2; i++) {
            s.key[i] = c.take<uint32_t>(n);
            s.pay[i] = c.take<uint32_t>(n);
        }
        s.too_small = c.take<int64_t>(1);
        s.tiles_cap = tiles;
        s.base = c.take<uint32_t>((size_t)F * words_per_tile);
        s.chunk_hist = c.take<uint32_t>((size_t)chunks * words_per_tile);
        s.own = c.take<uint32_t>((size_t)tiles * kMaxRadix);
        s.upto = c.take<uint32_t>((size_t)tiles * kMaxRadix);
        s.flag = c.take<uint32_t>((size_t)tiles * kMaxPasses);
        s.ticket = c.take<uint32_t>((kMaxPasses + 1) * kQueues);
    };
    const int64_t tpf = (B + kTile - 1) / kTile, ch_a = chunk_for(n_lists);
    side(w.a, n_lists, (int64_t)F * tpf, (int64_t)F * ((B + ch_a - 1) / ch_a), words_for(bits_for((uint64_t)(B > 1 ? B - 1 : 1))));
    const int64_t tiles_b = M_cap / kTile + F + 1;
    // the number of rows of the tables is not known here: ids have at most 31 bits
    side(w.b, M_cap, tiles_b, chunks_bound(M_cap) + F + 1, words_for(31));
    w.pb = c.take<uint32_t>(F + 1);
    w.queue_start = c.take<uint32_t>(kQueues + 1);
    w.desc_queue = c.take<uint2>(tiles_b);
    w.desc_feat = c.take<uint4>(tiles_b);
    // room for the small tiles of every batch that has them and is no larger than this one
    const int64_t most_a = n_lists < kSmallTilesMost ? n_lists : kSmallTilesMost;
    const int64_t most_b = M_cap < kSmallTilesMost ? M_cap : kSmallTilesMost;
    w.a.small_hist = c.take<uint32_t>((size_t)(most_a / kSmallTile + F + 1) * kMaxRadix);
    w.b.small_hist = c.take<uint32_t>((size_t)(most_b / kSmallTile + F + 1) * kMaxRadix);
    w.desc_small = c.take<uint4>(most_b / kSmallTile + F + 1);
    w.seg_status = c.take<uint64_t>(tiles_b);
    w.tile_total = c.take<uint32_t>(2);
    return w;
}

bool recd_group_is_small(int F, int64_t B, int64_t M_cap, int64_t max_rows)
{
    return B <= kSmallCap && M_cap <= kSmallCap && bits_for((uint64_t)(max_rows > 1 ? max_rows - 1 : 1)) +
                                                           bits_for((uint64_t)(F > 1 ? F - 1 : 1)) <= 32;
}

const uint32_t *recd_group_rows(const RecdGroupWs &w, int F, int64_t B, int64_t U_cap, int64_t M_cap, int64_t max_rows)
{
    int passes, dbits;
    if (recd_group_is_small(F, B, M_cap, max_rows))
        return w.a.pay[0];
    digits_for(slot_bits(B, U_cap), &passes, &dbits);
    return w.a.pay[(passes - 1) & 1];
}

const uint32_t *recd_group_positions(const RecdGroupWs &w, int F, int64_t B, int64_t M_cap, int64_t max_rows)
{
    int passes, dbits;
    if (recd_group_is_small(F, B, M_cap, max_rows))
        return w.b.pay[0];
    digits_for(bits_for((uint64_t)(max_rows > 1 ? max_rows - 1 : 1)), &passes, &dbits);
    return w.b.pay[(passes - 1) & 1];
}

recd_status recd_group(recd_ctx *ctx, hipStream_t st, const RecdGroupWs &w, const RecdGroupArgs &a)
{
    GroupParams g{};
    g.F = a.F;
    g.B = a.B;
    g.M_cap = a.M_cap;
    g.n_lists = (int64_t)a.F * a.B;
    g.inverse = a.inverse;
    g.feat_uoff = a.feat_uoff;
    g.u_values = a.u_values;
    g.u_offsets = a.u_offsets;
    auto side = [&](SideParams &s, const RecdGroupWs::Side &v, int bits, int64_t n, uint32_t *arrive) {
        for (int i = 0; i < 2; i++) {
            s.key[i] = v.key[i];
            s.pay[i] = v.pay[i];
        }
        digits_for(bits, &s.passes, &s.dbits);
        s.base = v.base;
        s.chunk_hist = v.chunk_hist;
        s.small_hist = v.small_hist;
        s.own = v.own;
        s.upto = v.upto;
        s.flag = v.flag;
        s.ticket = v.ticket;
        s.arrive = arrive;
        s.chunk = chunk_for(n);
        s.tiles_cap = v.tiles_cap;
    };
    side(g.a, w.a, slot_bits(a.B, a.U_cap), g.n_lists, ctx->group_arrive);
    side(g.b, w.b, bits_for((uint64_t)(a.max_rows > 1 ? a.max_rows - 1 : 1)), a.M_cap, ctx->group_arrive + RECD_GROUP_ARRIVE);
    g.tpf = (int)((a.B + kTile - 1) / kTile);
    g.small_b = recd_grouping_is_short(g.n_lists, a.M_cap);
    g.small_a = g.small_b && a.B <= kSmallTilesPer * kSmallTile;
    const int64_t chunk_a = g.small_a ? kSmallTile : g.a.chunk, chunk_b = g.small_b ? kSmallTile : g.b.chunk;
    g.cpf = (int)((a.B + chunk_a - 1) / chunk_a);
    g.pb = w.pb;
    g.queue_start = w.queue_start;
    g.desc_queue = w.desc_queue;
    g.desc_feat = w.desc_feat;
    g.desc_small = w.desc_small;
    g.tile_total = w.tile_total;
    g.pos_list = a.pos_list;
    g.pay_positions = a.pay_positions;
    g.u_weights = a.u_weights;
    g.pay_w = a.pay_w;
    g.pay_pos = a.pay_pos;
    g.run_index = a.run_index;
    g.runs_cap = a.runs_cap;
    g.too_small_a = w.a.too_small;
    g.too_small_b = w.b.too_small;
    g.seg_status = w.seg_status;
    g.seg_start_a = a.seg_start_a;
    g.list_off_a = a.list_off_a;
    g.seg_start_b = a.seg_start_b;
    g.list_off_b = a.list_off_b;
    g.touched_rows = a.touched_rows;
    g.feat_roff = a.feat_roff;
    g.seg_feat = a.seg_feat;
    g.chunk_count = a.chunk_count;
    g.chunks = a.chunks;
    g.chunk_arrive = a.chunk_arrive;
    g.long_seg = a.long_seg;
    g.lists_cap = a.lists_cap;
    if (recd_group_is_small(a.F, a.B, a.M_cap, a.max_rows)) {
        const int row_bits = bits_for((uint64_t)(a.max_rows > 1 ? a.max_rows - 1 : 1));
        // a block's ids and rows take most of a CU's LDS: no more blocks than CUs as far as the features' rows allow it
        const int most = ctx->num_cu / 2 > 0 ? ctx->num_cu / 2 : 1, per = (a.F + most - 1) / most;
        const int b_blocks = (a.F + per - 1) / per;
        int passes, dbits;
        digits_for(row_bits + (per > 1 ? bits_for((uint64_t)(per - 1)) : 0), &passes, &dbits);
        hipLaunchKernelGGL(k_group_small, dim3(b_blocks + a.F), dim3(kSmallThreads), 0, st, g, b_blocks, per, row_bits, passes, dbits);
        RECD_HIP(ctx, hipGetLastError());
        return RECD_OK;
    }
    const unsigned a_tiles = g.small_a ? (unsigned)(a.F * g.cpf)
                                       : (unsigned)((g.a.tiles_cap + kQueues - 1) / kQueues * kQueues);
    g.b_tiles = (unsigned)(a.M_cap / kTile + a.F + 1);
    const unsigned b_blocks = g.small_b ? (unsigned)(a.M_cap / kSmallTile + a.F + 1) : g.b_tiles;
    g.a_blocks = (unsigned)((int64_t)a.F * g.cpf);
    g.list_block0 = g.a_blocks + (unsigned)(a.M_cap / chunk_b + a.F + 1);
    int64_t list_blocks = ((a.U_cap < g.n_lists ? a.U_cap : g.n_lists) + kCountThreads / 16 - 1) / (kCountThreads / 16);
    if (list_blocks > (int64_t)ctx->num_cu * 8)
        list_blocks = (int64_t)ctx->num_cu * 8;
    const unsigned cb = g.list_block0 + (a.pos_list ? (unsigned)(list_blocks < 1 ? 1 : list_blocks) : 0u);
    const size_t lds_a = (size_t)g.a.passes << g.a.dbits, lds_b = ((size_t)g.b.passes << g.b.dbits) + a.F + 1;
    const size_t lds = (lds_a > lds_b ? lds_a : lds_b) * sizeof(uint32_t);
    hipLaunchKernelGGL(k_group_count, dim3(cb), dim3(kCountThreads), lds, st, g);
    const int passes = g.a.passes > g.b.passes ? g.a.passes : g.b.passes;
    for (int p = 0; p < passes; p++) {
        g.a_blocks = p < g.a.passes ? a_tiles : 0;
        const unsigned nb = g.a_blocks + (p < g.b.passes ? b_blocks : 0);
        hipLaunchKernelGGL(k_group_sweep, dim3(nb), dim3(kTileThreads), 0, st, g, p);
    }
    g.a_blocks = (unsigned)((g.n_lists + kTile - 1) / kTile);
    hipLaunchKernelGGL(k_group_segments, dim3(g.a_blocks + g.b_tiles), dim3(kTileThreads), 0, st, g);
    RECD_HIP(ctx, hipGetLastError());
    return RECD_OK;
}
