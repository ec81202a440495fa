// Backward of expand + pooled lookup on an IKJT, and row-wise Adagrad on the touched rows.
//
//   step A  g_u[u,:] = sum_{b : inverse[f,b] = u} grad_out[f,b,:]            (b ascending)
//   step B  G_f[r,:] = sum_{j : u_values[j] = r} g_u[list of j,:]            (j ascending)
// Each step is "group the contributions by destination, then sum every group in a fixed order":
// recd_group.hip puts equal destinations next to each other with their sources still ascending and
// numbers the groups, and a segmented gather-sum adds each group's rows.  There are no
// floating-point atomics, so two runs give bit-identical gradients.
#include "recd_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

// ---------------------------------------------------------------- row-wise Adagrad
// One 32-lane group per touched row k (rows of features [f0, f0+nf) only):
//   m[r] += mean_d G[k,d]^2 ;  W[r,d] -= lr * G[k,d] / (sqrt(m[r]) + eps)
struct OptPtrs {
    float *w[RECD_F_PER_LAUNCH];
    float *m[RECD_F_PER_LAUNCH];
};

__global__ __launch_bounds__(256) void k_adagrad(const float *__restrict__ grad_rows,
                                                 const int64_t *__restrict__ touched_rows,
                                                 const int64_t *__restrict__ feat_roff, int f0, int nf,
                                                 int D, OptPtrs ptrs, float lr, float eps)
{
    constexpr int SG = 32;
    const int s = threadIdx.x % SG;
    const int64_t k0 = feat_roff[f0], k1 = feat_roff[f0 + nf];
    const int vecs = D / 4;
    for (int64_t k = k0 + (int64_t)blockIdx.x * (256 / SG) + threadIdx.x / SG; k < k1;
         k += (int64_t)gridDim.x * (256 / SG)) {
        int lo = f0, hi = f0 + nf;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (feat_roff[mid] <= k)
                lo = mid;
            else
                hi = mid;
        }
        const int64_t r = touched_rows[k];
        const float4 *g = reinterpret_cast<const float4 *>(grad_rows + k * D);
        float ss = 0.f;
        for (int v = s; v < vecs; v += SG) {
            const float4 x = g[v];
            ss += x.x * x.x;
            ss += x.y * x.y;
            ss += x.z * x.z;
            ss += x.w * x.w;
        }
#pragma unroll
        for (int m = SG / 2; m > 0; m >>= 1)
            ss += __shfl_xor(ss, m, SG);
        float *mp = ptrs.m[lo - f0] + r;
        const float mnew = *mp + ss / (float)D;
        const float scale = lr / (sqrtf(mnew) + eps);
        float4 *w = reinterpret_cast<float4 *>(ptrs.w[lo - f0] + r * D);
        for (int v = s; v < vecs; v += SG) {
            const float4 x = g[v];
            float4 y = w[v];
            y.x -= scale * x.x;
            y.y -= scale * x.y;
            y.z -= scale * x.z;
            y.w -= scale * x.w;
            w[v] = y;
        }
        // every lane has read *mp before any lane of the group overwrites it
        __builtin_amdgcn_wave_barrier();
        if (s == 0)
            *mp = mnew;
    }
}

// ---------------------------------------------------------------- row-gradient segment sum
// Step B has very many very short segments (a table row is named by a handful of unique lists, a
// few hot rows by thousands).  Here a group of LPR lanes owns a whole segment: G = 64/LPR segments
// advance side by side in one wave, each lane carries up to four 16-byte pieces of the row, no
// cross-lane fold is needed, and the Adagrad update of the destination row follows in the same
// lanes.  Order of additions inside such a segment: ascending position.
// A wave lasts as long as its longest segment, so segments longer than the cut (32 entries by default, see
// long_seg_cut) are cut into chunks, which whole blocks sum: the first blocks of the same launch.  A
// chunk's entries go to the block's lane groups in turn, the groups' sums are folded by a fixed
// butterfly and the four waves' in order.  A segment of one chunk is finished on the spot; else the
// block that arrives last adds the chunks' partial sums in chunk order: what is added in which order
// depends on the segment's length alone.
struct RowSumParams {
    const float *table;        // g_u [U, D]
    const uint32_t *pay;       // sorted payload: unique-list index of every position
    const float *pay_w;        // weighted lookup: the weight of every sorted entry, else nullptr
    const uint32_t *pay_pos;   // max pooling: the position of every sorted entry, else nullptr
    const uint32_t *won;       // max pooling [M, LPR]: byte w of word r: which elements of piece w * LPR + r the position won
    const int64_t *seg_start;  // [R+1]
    const int64_t *n_seg;      // device: R
    float *out;                // grad_rows [R, D] or nullptr
    int D;
    int pieces;                // D / 4
    // segments longer than long_seg entries are cut into chunks
    const int64_t *chunk_count;
    const RecdChunk *chunks;
    uint32_t *chunk_arrive;    // at a segment's first chunk: its chunks that are summed; zero before the launch
    float *partials;           // [chunks, D]: sums of the chunks of segments of several
    unsigned chunk_blocks;     // blocks of the launch that take chunks (a multiple of 8)
    int long_seg;              // segments with more entries than this are the cut ones
};

// Tail of a row-gradient segment held by a lane group: acc = the segment's sum (piece w of lane r).
// Applies row-wise Adagrad to the destination row (operands fetched earlier into wreg/mreg) and/or
// stores the gradient row.
template <int LPR, int VPL = 4>
__device__ __forceinline__ void finish_segment(const RowSumParams &p, const OptAdagrad &opt, int64_t t,
                                               const float4 *acc, const float4 *wreg, float mreg,
                                               float *wrow, float *mp, const bool *piece, int r,
                                               bool update)
{
    if (update) {
        float ss = 0.f;
        auto add_squares = [&](int w) {  // products and additions as written, not as the compiler would pair them
            if (piece[w]) {
                ss = __fmaf_rn(acc[w].x, acc[w].x, ss);
                ss = __fmaf_rn(acc[w].y, acc[w].y, ss);
                ss = __fmaf_rn(acc[w].z, acc[w].z, ss);
                ss = __fmaf_rn(acc[w].w, acc[w].w, ss);
            }
        };
        if constexpr (VPL == 4) {
#pragma unroll
            for (int w = 0; w < VPL; w++)
                add_squares(w);
#pragma unroll
            for (int s = 1; s < LPR; s <<= 1)
                ss += __shfl_xor(ss, s);
        } else {
            // the additions of half as many lanes with four pieces each: lane r's pieces take turns with lane r + LPR / 2's
            constexpr int H = LPR / 2;
            const bool upper = r >= H;
#pragma unroll
            for (int w = 0; w < 2 * VPL; w++) {
                if (upper == (w % 2 == 1))
                    add_squares(w / 2);
                const float other = __shfl_xor(ss, H);
                if (upper == (w % 2 == 0))
                    ss = other;
            }
#pragma unroll
            for (int s = 1; s < H; s <<= 1)
                ss += __shfl_xor(ss, s);
        }
        const float mnew = mreg + ss / (float)p.D;
        const float scale = opt.lr / (sqrtf(mnew) + opt.eps);
#pragma unroll
        for (int w = 0; w < VPL; w++)
            if (piece[w]) {
                float4 x = wreg[w];
                x.x -= scale * acc[w].x;
                x.y -= scale * acc[w].y;
                x.z -= scale * acc[w].z;
                x.w -= scale * acc[w].w;
                {
                    typedef float f32x4s __attribute__((ext_vector_type(4)));
                    const f32x4s xo = {x.x, x.y, x.z, x.w};
                    __builtin_nontemporal_store(xo, reinterpret_cast<f32x4s *>(wrow) + w * LPR + r);
                }
            }
        if (r == 0)
            *mp = mnew;
    }
    if (p.out) {
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        f32x4 *dst = reinterpret_cast<f32x4 *>(p.out + t * p.D);
#pragma unroll
        for (int w = 0; w < VPL; w++)
            if (piece[w]) {
                const f32x4 o = {acc[w].x, acc[w].y, acc[w].z, acc[w].w};
                __builtin_nontemporal_store(o, &dst[w * LPR + r]);
            }
    }
}

// Waits until the memory system has acknowledged this wave's stores.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Destination row of a segment for the update: pointers, and its operands fetched ahead of the sums.
template <int LPR, int VPL = 4>
__device__ __forceinline__ void fetch_row(const OptAdagrad &opt, int D, int f, int64_t row, const bool *piece, int r,
                                          float4 *wreg, float &mreg, float *&wrow, float *&mp)
{
    typedef float f32x4l __attribute__((ext_vector_type(4)));
    mp = opt.m[f] + row;
    wrow = opt.w[f] + row * D;
    mreg = *mp;
#pragma unroll
    for (int w = 0; w < VPL; w++)
        if (piece[w]) {
            const f32x4l t = __builtin_nontemporal_load(reinterpret_cast<const f32x4l *>(wrow) + w * LPR + r);
            wreg[w] = make_float4(t.x, t.y, t.z, t.w);
        }
}

// How a segment's entry counts: its source row, the row times the entry's weight, or (max pooling) the
// elements of the row that the entry's position won.
enum { ROWS_PLAIN = 0, ROWS_WEIGHTED = 1, ROWS_MAX = 2 };

// Piece w * LPR + r of an entry's source row.
template <int LPR>
__device__ __forceinline__ float4 entry_piece(const RowSumParams &p, uint32_t id, int w, int r)
{
    return reinterpret_cast<const float4 *>(p.table)[(int64_t)id * p.pieces + w * LPR + r];
}

// acc + what of v the four low bits of `won` leave.
__device__ __forceinline__ void add_masked(float4 &acc, const float4 &v, uint32_t won)
{
    auto left = [&](float x, int bit) { return __uint_as_float(__float_as_uint(x) & (uint32_t)((int)(won << (31 - bit)) >> 31)); };
    acc.x += left(v.x, 0);
    acc.y += left(v.y, 1);
    acc.z += left(v.z, 2);
    acc.w += left(v.w, 3);
}

// Max pooling: adds to acc what a lane group's segment's next one or two entries won (n of them count).  Lane lane0 + i holds
// the i-th one's source row (pre) and position (prex).  An entry of a list of 25 ids won one element in 25, so six lanes in
// seven have nothing to read of its row: those that have read both entries' pieces side by side.  (Every lane the whole row of
// one entry after the other, 0.3 M positions of 512 bytes: 76 us, now 52; each lane its own next of eight entries 67; what
// is left is the update's 120 MB of scattered table rows and the 32 bytes of every position's words.)
template <int LPR>
__device__ __forceinline__ void add_won(const RowSumParams &p, float4 *acc, uint32_t pre, uint32_t prex, int lane0, int n, int r)
{
    constexpr int VPL = 4;
    const uint32_t x0 = __shfl(prex, lane0), x1 = __shfl(prex, lane0 + (n > 1 ? 1 : 0));
    const uint32_t id0 = __shfl(pre, lane0), id1 = __shfl(pre, lane0 + (n > 1 ? 1 : 0));
    const uint32_t won0 = p.won[(int64_t)x0 * LPR + r], won1 = n > 1 ? p.won[(int64_t)x1 * LPR + r] : 0u;
    float4 v0[VPL], v1[VPL];
#pragma unroll
    for (int w = 0; w < VPL; w++) {
        if ((won0 >> (8 * w)) & 15u)
            v0[w] = entry_piece<LPR>(p, id0, w, r);
        if ((won1 >> (8 * w)) & 15u)
            v1[w] = entry_piece<LPR>(p, id1, w, r);
    }
#pragma unroll
    for (int w = 0; w < VPL; w++) {
        if ((won0 >> (8 * w)) & 15u)
            add_masked(acc[w], v0[w], won0 >> (8 * w));
        if ((won1 >> (8 * w)) & 15u)
            add_masked(acc[w], v1[w], won1 >> (8 * w));
    }
}

template <int MODE> __device__ __forceinline__ uint32_t entry_extra(const RowSumParams &p, int64_t i)
{
    return MODE == ROWS_WEIGHTED ? __float_as_uint(p.pay_w[i]) : (MODE == ROWS_MAX ? p.pay_pos[i] : 0u);
}

template <int MODE> __device__ __forceinline__ void add4(float4 &acc, const float4 &v, uint32_t x)
{
    constexpr bool WT = MODE == ROWS_WEIGHTED;
    const float wt = __uint_as_float(x);
    acc.x = WT ? __fmaf_rn(wt, v.x, acc.x) : acc.x + v.x;
    acc.y = WT ? __fmaf_rn(wt, v.y, acc.y) : acc.y + v.y;
    acc.z = WT ? __fmaf_rn(wt, v.z, acc.z) : acc.z + v.z;
    acc.w = WT ? __fmaf_rn(wt, v.w, acc.w) : acc.w + v.w;
}

// One chunk of a cut segment, summed by the block.
template <int LPR_, int MODE, bool WIDE>
__device__ __forceinline__ void sum_chunk(const RowSumParams &p, const OptAdagrad &opt, int64_t item, const bool *piece)
{
    constexpr int LPR = WIDE ? 2 * LPR_ : LPR_, VPL = WIDE ? 2 : 4, W = 256 / 64, G = 64 / LPR_;
    __shared__ float4 s_part[W][VPL][LPR];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int g = lane / LPR, r = lane % LPR;
    const RecdChunk c = p.chunks[item];
    float4 acc[VPL];
#pragma unroll
    for (int w = 0; w < VPL; w++)
        acc[w] = make_float4(0.f, 0.f, 0.f, 0.f);
    // A group takes the entries wv * G + g, + W * G, ...: LPR of them (256 of the block) are fetched by one
    // load, one per lane, and handed round by shuffles; two source rows in flight.
    const int gbase = lane - r;
    if constexpr (WIDE) {
        // the entries of two groups, 2g and 2g + 1, one of each in flight; each has its own sum, as it would alone
        float4 acc1[VPL];
#pragma unroll
        for (int w = 0; w < VPL; w++)
            acc1[w] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (uint32_t base = c.start + wv * G + 2 * g; base < c.end; base += W * G * LPR) {
            const uint32_t idx = base + r * (W * G);
            const uint32_t pre0 = idx < c.end ? p.pay[idx] : 0u, prex0 = idx < c.end ? entry_extra<MODE>(p, idx) : 0u;
            const uint32_t pre1 = idx + 1 < c.end ? p.pay[idx + 1] : 0u;
            const uint32_t prex1 = idx + 1 < c.end ? entry_extra<MODE>(p, idx + 1) : 0u;
            const int left0 = (int)((c.end - base + W * G - 1) / (W * G)), cnt0 = left0 < LPR ? left0 : LPR;
            const int left1 = (int)((c.end - base + W * G - 2) / (W * G)), cnt1 = left1 < LPR ? left1 : LPR;
            for (int i = 0; i < cnt0; i++) {
                const uint32_t id0 = __shfl(pre0, gbase + i), id1 = __shfl(pre1, gbase + i);
                const uint32_t x0 = __shfl(prex0, gbase + i), x1 = __shfl(prex1, gbase + i);
                float4 v0[VPL], v1[VPL];
#pragma unroll
                for (int w = 0; w < VPL; w++)
                    if (piece[w]) {
                        v0[w] = entry_piece<LPR>(p, id0, w, r);
                        v1[w] = entry_piece<LPR>(p, i < cnt1 ? id1 : id0, w, r);
                    }
#pragma unroll
                for (int w = 0; w < VPL; w++)
                    if (piece[w]) {
                        add4<MODE>(acc[w], v0[w], x0);
                        if (i < cnt1)
                            add4<MODE>(acc1[w], v1[w], x1);
                    }
            }
        }
#pragma unroll
        for (int w = 0; w < VPL; w++)
            add4<ROWS_PLAIN>(acc[w], acc1[w], 0);
    } else {
        for (uint32_t base = c.start + wv * G + g; base < c.end; base += W * G * LPR) {
            const uint32_t idx = base + r * (W * G);
            const uint32_t pre = idx < c.end ? p.pay[idx] : 0u, prex = idx < c.end ? entry_extra<MODE>(p, idx) : 0u;
            const int left = (int)((c.end - base + W * G - 1) / (W * G)), cnt = left < LPR ? left : LPR;
            if constexpr (MODE == ROWS_MAX) {
#pragma unroll 1
                for (int i0 = 0; i0 < cnt; i0 += 2)
                    add_won<LPR>(p, acc, pre, prex, gbase + i0, cnt - i0, r);
                continue;
            }
            for (int i0 = 0; i0 < cnt; i0 += 2) {
                const bool two = i0 + 1 < cnt;
                const int k1 = i0 + (two ? 1 : 0);
                const uint32_t id0 = __shfl(pre, gbase + i0), id1 = __shfl(pre, gbase + k1);
                const uint32_t x0 = __shfl(prex, gbase + i0), x1 = __shfl(prex, gbase + k1);
                float4 v0[VPL], v1[VPL];
#pragma unroll
                for (int w = 0; w < VPL; w++)
                    if (piece[w]) {
                        v0[w] = entry_piece<LPR>(p, id0, w, r);
                        v1[w] = entry_piece<LPR>(p, id1, w, r);
                    }
#pragma unroll
                for (int w = 0; w < VPL; w++)
                    if (piece[w]) {
                        add4<MODE>(acc[w], v0[w], x0);
                        if (two)
                            add4<MODE>(acc[w], v1[w], x1);
                    }
            }
        }
    }
#pragma unroll
    for (int s = LPR; s < 64; s <<= 1)
#pragma unroll
        for (int w = 0; w < VPL; w++) {
            acc[w].x += __shfl_xor(acc[w].x, s);
            acc[w].y += __shfl_xor(acc[w].y, s);
            acc[w].z += __shfl_xor(acc[w].z, s);
            acc[w].w += __shfl_xor(acc[w].w, s);
        }
    __syncthreads();  // the previous chunk is done with the shared arrays
    if (g == 0) {
#pragma unroll
        for (int w = 0; w < VPL; w++)
            s_part[wv][w][r] = acc[w];
    }
    __syncthreads();
    if (wv != 0)
        return;
    const bool update = opt.n_feat > 0;
    float4 wreg[VPL];
    float mreg = 0.f, *wrow = nullptr, *mp = nullptr;
#pragma unroll
    for (int w = 0; w < VPL; w++) {
        acc[w] = s_part[0][w][r];
#pragma unroll
        for (int k = 1; k < W; k++)
            add4<ROWS_PLAIN>(acc[w], s_part[k][w][r], 0);
    }
    if (c.n > 1) {
        // the partial sum goes where every XCD reads it, then the arrival is counted (see the grouping's
        // counting kernel: no release, which would write back the whole L2)
        if (g == 0) {
            uint32_t *dst = reinterpret_cast<uint32_t *>(p.partials + item * p.D);
#pragma unroll
            for (int w = 0; w < VPL; w++)
                if (piece[w]) {
                    const uint32_t v[4] = {__float_as_uint(acc[w].x), __float_as_uint(acc[w].y), __float_as_uint(acc[w].z),
                                           __float_as_uint(acc[w].w)};
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        __hip_atomic_store(dst + 4 * (w * LPR + r) + e, v[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
        }
        stores_done();
        uint32_t before = 0;
        if (lane == 0)
            before = __hip_atomic_fetch_add(p.chunk_arrive + c.first, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) != c.n - 1)
            return;
        asm volatile("" ::: "memory");
#pragma unroll
        for (int w = 0; w < VPL; w++)
            acc[w] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (uint32_t k = 0; k < c.n; k++) {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(p.partials + (int64_t)(c.first + k) * p.D);
#pragma unroll
            for (int w = 0; w < VPL; w++)
                if (piece[w]) {
                    uint32_t v[4];
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        v[e] = __hip_atomic_load(src + 4 * (w * LPR + r) + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    acc[w].x += __uint_as_float(v[0]);
                    acc[w].y += __uint_as_float(v[1]);
                    acc[w].z += __uint_as_float(v[2]);
                    acc[w].w += __uint_as_float(v[3]);
                }
        }
    }
    if (g != 0)
        return;
    if (update)
        fetch_row<LPR, VPL>(opt, p.D, opt.seg_feat[c.seg], opt.touched_rows[c.seg], piece, r, wreg, mreg, wrow, mp);
    finish_segment<LPR, VPL>(p, opt, c.seg, acc, wreg, mreg, wrow, mp, piece, r, update);
}

// WIDE: twice the lanes a segment, two pieces each.  What bounds a batch of some hundred thousand entries is the longest
// segment of a wave, whose entries follow each other at a round trip each, and the few waves there are: with half the
// segments a wave and 64 registers for 86 two entries are in flight, eight waves a SIMD.  us, four pieces a lane / WIDE: 0.19 M
// entries of skewed ids, rows of 512 bytes 33.2 / 25.3, weighted 24.6 / 19.5; 256 bytes 29.9 / 23.8, 1 KB 42.2 / 32.9.  (Two
// entries of four pieces a lane: 29.6, but uniform ids 66 -> 70; two pieces a lane in 85 registers 28.3, and uniform ids 66 -> 80.)
// The additions and their order are those of four pieces a lane, in the chunks and the update too: the same bits.
template <int LPR_, int MODE, bool WIDE>
__global__ __launch_bounds__(256) void k_segsum_rows(const RowSumParams p, const OptAdagrad opt)
{
    constexpr int LPR = WIDE ? 2 * LPR_ : LPR_, VPL = WIDE ? 2 : 4, G = 64 / LPR;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int g = lane / LPR, r = lane % LPR;
    bool piece[VPL];
#pragma unroll
    for (int w = 0; w < VPL; w++)
        piece[w] = w * LPR + r < p.pieces;
    if (blockIdx.x < p.chunk_blocks) {
        const int64_t n = *p.chunk_count;
        for (int64_t item = blockIdx.x; item < n; item += p.chunk_blocks)
            sum_chunk<LPR_, MODE, WIDE>(p, opt, item, piece);
        return;
    }
    const int64_t R = *p.n_seg;
    const int per_block = (256 / 64) * G;
    // The segments are ordered by (feature, row) and their entries name rows of the source array that
    // belong to the same feature.  Blocks go to the XCDs in turn; every XCD takes a contiguous eighth
    // of the segments and its blocks stride through it side by side, so that the source rows an XCD
    // gathers at one time are a few features' worth and stay in its L2.
    const unsigned blk = blockIdx.x - p.chunk_blocks;  // this part of the grid is a multiple of 8 blocks
    const int64_t groups = (R + per_block - 1) / per_block;
    const int64_t per_xcd = (groups + 7) / 8;
    const int64_t g_first = (int64_t)(blk % 8) * per_xcd;
    const int64_t g_count = per_xcd < groups - g_first ? per_xcd : groups - g_first;
    const int64_t g_step = (gridDim.x - p.chunk_blocks) / 8;
    for (int64_t gi = blk / 8; gi < g_count; gi += g_step) {
        const int64_t k = (g_first + gi) * per_block + wv * G + g;
        int64_t start = 0;
        int n = 0;
        int f_seg = 0;
        int64_t row_seg = 0;
        if (k < R) {
            // one round trip: where the segment lies, and (for the update) which row it is
            start = p.seg_start[k];
            const int64_t end = p.seg_start[k + 1];
            if (opt.n_feat > 0) {
                f_seg = opt.seg_feat[k];
                row_seg = opt.touched_rows[k];
            }
            const int64_t len = end - start;
            n = len <= p.long_seg ? (int)len : 0;  // longer segments were cut into chunks
        }
        const bool mine = n > 0;  // uniform inside the lane group
        const bool update = mine && opt.n_feat > 0;
        // second round trip: the segment's entries (the first kPre * LPR of them, one load per lane
        // and LPR entries) together with the destination row and its accumulator
        constexpr int kPre = MODE == ROWS_MAX ? 1 : VPL;
        uint32_t pre[kPre], prex[kPre];
#pragma unroll
        for (int u = 0; u < kPre; u++) {
            const int idx = u * LPR + r;
            pre[u] = idx < n ? p.pay[start + idx] : 0u;
            prex[u] = idx < n ? entry_extra<MODE>(p, start + idx) : 0u;
        }
        float4 wreg[VPL];
        float mreg = 0.f;
        float *wrow = nullptr, *mp = nullptr;
        if (update)
            fetch_row<LPR, VPL>(opt, p.D, f_seg, row_seg, piece, r, wreg, mreg, wrow, mp);
        float4 acc[VPL];
#pragma unroll
        for (int w = 0; w < VPL; w++)
            acc[w] = make_float4(0.f, 0.f, 0.f, 0.f);
        auto add_entry = [&](uint32_t id, uint32_t x) {
            float4 v[VPL];
#pragma unroll
            for (int w = 0; w < VPL; w++)
                if (piece[w])
                    v[w] = entry_piece<LPR>(p, id, w, r);
#pragma unroll
            for (int w = 0; w < VPL; w++)
                if (piece[w])
                    add4<MODE>(acc[w], v[w], x);
        };
        // entries in ascending order: the fetched ones come out of the lane group's registers, any
        // further ones (cuts above kPre * LPR entries) are read one by one, or again by all lanes
        const int gbase = lane - r;
        if constexpr (MODE == ROWS_MAX) {
            uint32_t id = pre[0], x = prex[0];
#pragma unroll 1
            for (int i1 = 0; i1 < n; i1 += LPR) {
                if (i1 > 0) {
                    id = i1 + r < n ? p.pay[start + i1 + r] : 0u;
                    x = i1 + r < n ? p.pay_pos[start + i1 + r] : 0u;
                }
                const int cnt = n - i1 < LPR ? n - i1 : LPR;
#pragma unroll 1
                for (int i0 = 0; i0 < cnt; i0 += 2)
                    add_won<LPR>(p, acc, id, x, gbase + i0, cnt - i0, r);
            }
        } else {
#pragma unroll
            for (int u = 0; u < kPre; u++) {
                const int cnt = n - u * LPR < LPR ? n - u * LPR : LPR;
                if constexpr (WIDE) {
                    constexpr int FLY = 2;
                    for (int i0 = 0; i0 < cnt; i0 += FLY) {
                        float4 v[FLY][VPL];
                        uint32_t x[FLY];
#pragma unroll
                        for (int k = 0; k < FLY; k++) {
                            const int from = gbase + (i0 + k < LPR ? i0 + k : LPR - 1);
                            const uint32_t id = __shfl(pre[u], from);
                            x[k] = MODE != ROWS_PLAIN ? __shfl(prex[u], from) : 0u;
                            if (k == 0 || i0 + k < cnt)
#pragma unroll
                                for (int w = 0; w < VPL; w++)
                                    if (piece[w])
                                        v[k][w] = entry_piece<LPR>(p, id, w, r);
                        }
#pragma unroll
                        for (int k = 0; k < FLY; k++)
                            if (k == 0 || i0 + k < cnt)
#pragma unroll
                                for (int w = 0; w < VPL; w++)
                                    if (piece[w])
                                        add4<MODE>(acc[w], v[k][w], x[k]);
                    }
                } else {
                    for (int ii = 0; ii < cnt; ii++) {
                        const uint32_t id = __shfl(pre[u], gbase + ii);
                        add_entry(id, MODE != ROWS_PLAIN ? __shfl(prex[u], gbase + ii) : 0u);
                    }
                }
            }
            for (int i = kPre * LPR; i < n; i++) {
                const uint32_t x = entry_extra<MODE>(p, start + i);
                add_entry(p.pay[start + i], x);
            }
        }
        if (mine)
            finish_segment<LPR, VPL>(p, opt, k, acc, wreg, mreg, wrow, mp, piece, r, update);
    }
}

// ---------------------------------------------------------------- max pooling: who won
// Backward of the max-pooled lookup: element d of g_u[u] belongs to the position of list u that holds
// the largest table element d (the first such position).  A wave owns a unique list: the lane groups of LPR lanes
// (lane r: pieces r, r + LPR, ... of the row, 16 bytes each; one piece per lane up to 1 KiB rows) take a part of every 64
// positions each, eight rows in flight per lane, and agree at the end (of equal elements the smaller position).  For every
// position and piece the kernel writes which elements it won, four bits in a byte: a few of the bytes are not zero, so they
// are put together in LDS and leave as whole words.  The row-gradient sum then takes of g_u[u] what the entry's position won;
// the rows of g_u stay in L2.  (One masked row per position went to memory and back once; then a lane group walked a list
// alone, the ids of eight rows fetched by every lane before them, and stored a byte a lane and position: 0.3 M positions of
// 512 bytes in 12 K lists 43.4 us, now 19.4; a lookup of the same lists takes 21.)
// Of short lists a wave owns NL, a lane group or more each: a wave for every list left most groups idle (whole backward, us, a
// lane group a list as it was / a wave / NL = 64 / LPR: 108 K lists of one id, rows of 64 bytes 164 / 221 / 153, 198 K of 3 ids
// 204 / 308 / 194, of 256 bytes 286 / 313 / 255; 57 K of 10 ids, 64 bytes 140 / 157 / 128; 24 K of 25, 512 bytes 256 / 179 / 194).
// With NL = 1 the list's number must not hang on the lane, or its offsets and loops leave the scalar unit (12 K lists 25 for 19).
struct MaxTables {
    const float *w[RECD_F_PER_LAUNCH];
};
constexpr int kWonWords = 512;  // of a window of a list's positions in LDS

template <int LPR, int VPL, int NL>
__global__ __launch_bounds__(64) void k_max_winner(const int64_t *__restrict__ u_values,
                                                   const int64_t *__restrict__ u_offsets,
                                                   const int64_t *__restrict__ feat_uoff, int f0, int nf,
                                                   MaxTables tabs, uint32_t *__restrict__ won, int won_lpr, int pieces,
                                                   int64_t lists_cap, int64_t m_cap)
{
    constexpr int W = 64 / NL, G = W / LPR, US = 8 / VPL;  // lanes and lane groups of a list; positions in flight per lane
    __shared__ uint4 s_won[kWonWords / 4];
    const int lane = threadIdx.x, n_own = NL > 1 ? lane / W : 0, in = NL > 1 ? lane % W : lane, g = in / LPR, r = lane % LPR;
    uint4 *const own = s_won + n_own * (kWonWords / 4 / NL);
    uint32_t *const words = reinterpret_cast<uint32_t *>(own);
    const int64_t u_lo = feat_uoff[f0];
    int64_t u_hi = feat_uoff[f0 + nf];
    u_hi = u_hi < lists_cap ? u_hi : lists_cap;
    const int64_t fo0 = lane < nf ? feat_uoff[f0 + lane] : INT64_MAX, fo1 = 64 + lane < nf ? feat_uoff[f0 + 64 + lane] : INT64_MAX;
    const int win = kWonWords / NL / won_lpr;  // positions of a window
    for (int64_t u0 = u_lo + (int64_t)blockIdx.x * NL; u0 < u_hi; u0 += (int64_t)gridDim.x * NL) {
        int f = (int)(__popcll(__ballot(fo0 <= u0)) + __popcll(__ballot(fo1 <= u0))) - 1;
        const int64_t u = u0 + n_own;
        int64_t j0 = 0;
        int len = 0;
        if (NL == 1 || u < u_hi) {
            while (NL > 1 && f + 1 < nf && feat_uoff[f0 + f + 1] <= u)
                f++;
            j0 = u_offsets[u];
            const int64_t j1 = u_offsets[u + 1], end = j1 < m_cap ? j1 : m_cap;
            len = j0 < end ? (int)(end - j0) : 0;  // m_cap is below 2^31
        }
        const float4 *table = reinterpret_cast<const float4 *>(tabs.w[f]);
        int most = len;  // of the wave's lists
#pragma unroll
        for (int s = W; s < 64; s <<= 1) {
            const int y = __shfl_xor(most, s);
            most = y > most ? y : most;
        }
        most = __builtin_amdgcn_readfirstlane(most);
        float best[VPL][4];
        int arg[VPL][4];
#pragma unroll
        for (int w = 0; w < VPL; w++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                best[w][e] = -INFINITY;
                arg[w][e] = INT32_MAX;
            }
        for (int c0 = 0; c0 < most; c0 += W) {
            const int nc = len - c0 < W ? len - c0 : W, per = (nc + G - 1) / G;  // of the list; the longest's:
            const int per_most = (most - c0 < W ? most - c0 + G - 1 : W) / G;
            const uint32_t id = in < nc ? (uint32_t)u_values[j0 + c0 + in] : 0u;
            for (int k0 = 0; k0 < per_most; k0 += US) {
                float4 v[US][VPL];
#pragma unroll
                for (int k = 0; k < US; k++) {
                    const int t = g * per + k0 + k;
                    const uint32_t row = __shfl(id, n_own * W + (t & (W - 1)));
                    if (k0 + k < per && t < nc)
#pragma unroll
                        for (int w = 0; w < VPL; w++)
                            if (w * LPR + r < pieces)
                                v[k][w] = table[(int64_t)row * pieces + w * LPR + r];
                }
#pragma unroll
                for (int k = 0; k < US; k++) {
                    const int t = g * per + k0 + k, pos = c0 + t;
                    if (k0 + k < per && t < nc)
#pragma unroll
                        for (int w = 0; w < VPL; w++) {
                            const float x[4] = {v[k][w].x, v[k][w].y, v[k][w].z, v[k][w].w};
#pragma unroll
                            for (int e = 0; e < 4; e++)
                                if (pos == 0 || x[e] > best[w][e]) {  // a NaN wins at the first position only, and stays
                                    best[w][e] = x[e];
                                    arg[w][e] = pos;
                                }
                        }
                }
            }
        }
#pragma unroll
        for (int s = LPR; s < W; s <<= 1)
#pragma unroll
            for (int w = 0; w < VPL; w++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const float y = __shfl_xor(best[w][e], s);
                    const int a = __shfl_xor(arg[w][e], s);
                    const bool low = (lane & s) == 0;  // only a lower group's can be NaN
                    const float lx = low ? best[w][e] : y, hx = low ? y : best[w][e];
                    const int la = low ? arg[w][e] : a, ha = low ? a : arg[w][e];
                    const bool high = hx > lx || (hx == lx && ha < la);
                    best[w][e] = high ? hx : lx;
                    arg[w][e] = high ? ha : la;
                }
        for (int w0 = 0; w0 < most; w0 += win) {
            const int left = len - w0 < win ? len - w0 : win, n = left > 0 ? left : 0, vecs = n * won_lpr / 4;
            for (int i = in; i < vecs; i += W)
                own[i] = make_uint4(0, 0, 0, 0);
            __syncthreads();
#pragma unroll
            for (int w = 0; w < VPL; w++) {
                const int piece = w * LPR + r;
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const int at = arg[w][e] - w0;
                    if (e % G == g && piece < pieces && at >= 0 && at < n)
                        atomicOr(&words[at * won_lpr + piece % won_lpr], 1u << (8 * (piece / won_lpr) + e));
                }
            }
            __syncthreads();
            uint4 *dst = reinterpret_cast<uint4 *>(won + (j0 + w0) * won_lpr);
            for (int i = in; i < vecs; i += W)
                dst[i] = own[i];
            __syncthreads();
        }
    }
}

__global__ void k_no_rows(int F, int64_t *feat_roff, int64_t *list_off)
{
    for (int f = threadIdx.x; f <= F; f += blockDim.x)
        feat_roff[f] = 0;
    if (threadIdx.x == 0) {
        list_off[0] = 0;
        list_off[1] = 0;
    }
}

// ---------------------------------------------------------------- sequence path, step A
// g_emb[u_offsets[u] + t, :] = sum over the rows l (ascending) of unique list u of
// grad_out[offsets[l] + t, :].  The rows of u are ps[seg_start[u] .. seg_start[u+1]) (rows sorted by
// unique list; every list has at least one row, so segment number = list number).  A block owns
// LISTS consecutive unique lists and numbers their positions flat, so long and short lists load
// the threads alike.  The start offsets of up to 64 source rows per list are staged in LDS, so
// the inner loop is row loads only, eight in flight per thread (a thread = one 16-byte piece of
// one position); lists with more rows take further rounds that continue from the stored partial
// sum - the same additions in the same order.
//
// Eight loads in flight are worth what the list has rows for: with one or two rows a list, six or
// seven of the eight load the last row again and a thread waits a whole trip for each position.  Where
// no list of the block has more than two (four) rows, FEW takes four (two) positions side by side
// instead, two (four) rows of each: the same eight loads, all of them wanted.  Of 2 rows a list
// 339 -> 231 us (rows of 1 KB, 1.2 GB in all), of 3 68 -> 65, of 1 211 -> 151.  Its loads are unconditional, of a row
// of the list again where there is none: loads under a condition took 109 registers, and the 72 us of a batch of
// 8 rows a list became 134.  Batches with more rows a list run the kernel without it (8 rows 72.5 us either way,
// 32 rows 162 against 170).
template <int LISTS, bool FEW>
__global__ __launch_bounds__(256) void k_jagged_reduce(const float4 *__restrict__ grad_out,
                                                       const int64_t *__restrict__ offsets,
                                                       const uint32_t *__restrict__ ps,
                                                       const int64_t *__restrict__ seg_start,
                                                       const int64_t *__restrict__ n_seg,
                                                       const int64_t *__restrict__ u_offsets,
                                                       float4 *__restrict__ g_emb, int vecs,
                                                       int64_t n_rows, int64_t m_cap)
{
    static_assert(LISTS <= 64 && (LISTS & (LISTS - 1)) == 0, "one wave prepares the block's lists");
    constexpr int kRound = 64;  // source rows per list and round
    constexpr int kFly = 8;     // row loads in flight per thread
    __shared__ uint32_t rel_s[LISTS + 1];
    __shared__ int64_t pos_s[LISTS], seg_s[LISTS];
    __shared__ uint32_t cnt_s[LISTS];
    __shared__ uint32_t cmax_s;
    __shared__ int64_t off_s[LISTS][kRound];
    const int64_t U = *n_seg;
    const uint32_t rows_per_sweep = 256 / vecs;
    const uint32_t piece = threadIdx.x % vecs, sub = threadIdx.x / vecs;
    for (int64_t u0 = (int64_t)blockIdx.x * LISTS; u0 < U; u0 += (int64_t)gridDim.x * LISTS) {
        const uint32_t nl = U - u0 < LISTS ? (uint32_t)(U - u0) : (uint32_t)LISTS;
        __syncthreads();  // the previous lists are done with the shared arrays
        if (threadIdx.x < 64) {
            const uint32_t i = threadIdx.x;
            int64_t start = 0, s0 = 0;
            uint32_t len = 0, c = 0;
            if (i < nl) {
                start = u_offsets[u0 + i];
                len = (uint32_t)(u_offsets[u0 + i + 1] - start);
                s0 = seg_start[u0 + i];
                c = (uint32_t)(seg_start[u0 + i + 1] - s0);
            }
            uint32_t incl = len, cmax = c;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t x = __shfl_up(incl, d);
                if (i >= (uint32_t)d)
                    incl += x;
                const uint32_t y = __shfl_xor(cmax, d);
                cmax = y > cmax ? y : cmax;
            }
            if (i < nl) {
                rel_s[i] = incl - len;
                pos_s[i] = start;
                seg_s[i] = s0;
                cnt_s[i] = c;
            }
            if (i == 63) {
                rel_s[nl] = incl;
                cmax_s = cmax;
            }
        }
        __syncthreads();
        const uint32_t total = rel_s[nl];
        const uint32_t cmax = cmax_s;
        for (uint32_t c0 = 0; c0 < cmax; c0 += kRound) {
            if (c0 > 0)
                __syncthreads();  // the previous round's offsets have been used
            for (uint32_t idx = threadIdx.x; idx < nl * kRound; idx += 256) {
                const uint32_t a = idx / kRound, i = idx % kRound;
                if (c0 + i < cnt_s[a])
                    off_s[a][i] = offsets[ps[seg_s[a] + c0 + i]];
            }
            __syncthreads();
            if (sub >= rows_per_sweep)
                continue;
            // Lists of few rows: AT positions of a thread side by side, ROWS rows of each
            auto add_few = [&](auto rows_, auto at_) {
                constexpr int ROWS = decltype(rows_)::value, AT = decltype(at_)::value;
                for (uint32_t r0 = sub; r0 < total; r0 += rows_per_sweep * AT) {
                    uint32_t j[AT], n[AT];
                    bool in[AT];
                    uint32_t src[AT][ROWS];  // below 2^31, as all rows
#pragma unroll
                    for (int x = 0; x < AT; x++) {
                        const uint32_t r = r0 + x * rows_per_sweep, rc = r < total ? r : total - 1;
                        uint32_t a = 0;  // the last list with rel_s[a] <= rc
#pragma unroll
                        for (uint32_t s = LISTS / 2; s >= 1; s >>= 1)
                            if (a + s < nl && rel_s[a + s] <= rc)
                                a += s;
                        const uint32_t t = rc - rel_s[a], c = cnt_s[a];
                        const int64_t at = pos_s[a] + t;
                        j[x] = (uint32_t)at;
                        n[x] = c;
                        in[x] = r < total && at < m_cap;
#pragma unroll
                        for (int k = 0; k < ROWS; k++) {
                            const int64_t from = c > 0 ? off_s[a][k < (int)c ? k : c - 1] + t : 0;
                            src[x][k] = (uint32_t)(from < n_rows ? from : n_rows - 1);  // only a malformed IKJT gets here
                        }
                    }
                    float4 v[AT][ROWS];
#pragma unroll
                    for (int x = 0; x < AT; x++)
#pragma unroll
                        for (int k = 0; k < ROWS; k++) {
                            typedef float f32x4g __attribute__((ext_vector_type(4)));
                            const f32x4g t4 = __builtin_nontemporal_load(reinterpret_cast<const f32x4g *>(grad_out) +
                                                                         (int64_t)src[x][k] * vecs + piece);
                            v[x][k] = make_float4(t4.x, t4.y, t4.z, t4.w);
                        }
#pragma unroll
                    for (int x = 0; x < AT; x++) {
                        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                        for (int k = 0; k < ROWS; k++)
                            if (k < (int)n[x]) {
                                acc.x += v[x][k].x;
                                acc.y += v[x][k].y;
                                acc.z += v[x][k].z;
                                acc.w += v[x][k].w;
                            }
                        if (in[x])
                            g_emb[(int64_t)j[x] * vecs + piece] = acc;
                    }
                }
            };
            if (FEW && cmax <= 2) {
                add_few(std::integral_constant<int, 2>(), std::integral_constant<int, 4>());
                continue;
            }
            if (FEW && cmax <= 4) {
                add_few(std::integral_constant<int, 4>(), std::integral_constant<int, 2>());
                continue;
            }
            for (uint32_t r = sub; r < total; r += rows_per_sweep) {
                uint32_t a = 0;  // the last list with rel_s[a] <= r; r < rel_s[nl], so it is not empty
#pragma unroll
                for (uint32_t s = LISTS / 2; s >= 1; s >>= 1)
                    if (a + s < nl && rel_s[a + s] <= r)
                        a += s;
                const uint32_t c = cnt_s[a];
                if (c <= c0)
                    continue;  // this list has no rows left in this round
                const uint32_t n = c - c0 < (uint32_t)kRound ? c - c0 : (uint32_t)kRound;
                const int64_t t = r - rel_s[a];
                const int64_t j = pos_s[a] + t;
                if (j >= m_cap)
                    continue;
                float4 acc = c0 == 0 ? make_float4(0.f, 0.f, 0.f, 0.f) : g_emb[j * vecs + piece];
                for (uint32_t i = 0; i < n; i += kFly) {
                    float4 v[kFly];
#pragma unroll
                    for (int k = 0; k < kFly; k++) {
                        int64_t src = off_s[a][i + k < n ? i + k : n - 1] + t;
                        src = src < n_rows ? src : n_rows - 1;  // only a malformed IKJT gets here
                        {   // every gradient row is read once: a streaming load
                            typedef float f32x4g __attribute__((ext_vector_type(4)));
                            const f32x4g t4 = __builtin_nontemporal_load(
                                reinterpret_cast<const f32x4g *>(grad_out) + src * vecs + piece);
                            v[k] = make_float4(t4.x, t4.y, t4.z, t4.w);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < kFly; k++)
                        if (i + k < n) {
                            acc.x += v[k].x;
                            acc.y += v[k].y;
                            acc.z += v[k].z;
                            acc.w += v[k].w;
                        }
                }
                g_emb[j * vecs + piece] = acc;
            }
        }
    }
}

struct BwdWs {
    RecdGroupWs group;
    // segments of step A (list_off, seg_start) and of step B (the _b arrays and what follows)
    int64_t *list_off, *seg_start;
    int64_t *list_off_b, *seg_start_b;
    int32_t *seg_feat;
    int64_t *chunk_count;
    RecdChunk *chunks;
    uint32_t *chunk_arrive;
    float *g_u, *partials;
    int64_t lists_cap;   // rows of g_u
    uint32_t *pos_list;  // unique list of every position of u_values
    float *pay_w;        // weighted lookup: weight of every sorted entry of step B
    uint32_t *won;       // max pooling [M, row_lanes(D)]: which elements of every piece the position won
    int long_seg;        // step B: segments with more entries are cut into chunks
    size_t bytes;
};

// Step B's lane groups walk a segment entry by entry, several segments to a wave, so a wave lasts as
// long as its longest segment; segments with more entries than the context's cut
// (RECD_OPT_LONG_SEGMENT_CUT, default 32) are cut into chunks, which the first blocks of the launch sum.
// Whole backward, us, with a cut of 16 / 32 / 64 / 128: 2.2 M entries of 512 bytes 482 / 474 / 501 / 538, 0.19 M
// 127 / 132 / 148 / 184, 0.3 M 139 / 142 / 159 / 192; 35 M of 256 bytes (no deduplication, where the chunks are
// the larger part) 3410 / 3220 / 3125 / 3185; uniform ids alike.
constexpr int kDefaultLongSeg = 32;

// Lanes that carry a row in the row-gradient sum (up to four 16-byte pieces each).
int row_lanes(int D)
{
    const int P = D / 4;
    return P <= 16 ? 4 : (P <= 32 ? 8 : (P <= 64 ? 16 : (P <= 128 ? 32 : 64)));
}

BwdWs carve_bwd(char *base, int F, int64_t B, int64_t U_cap, int64_t M_cap, int D, int long_seg, bool with_won = false)
{
    WsCarver c(base);
    BwdWs w;
    (void)c.take<char>(1024);  // the head of the workspace stays with the validation passes' flags
    const int64_t n_lists = (int64_t)F * B;
    w.lists_cap = recd_lists_held(F, B, U_cap, M_cap);
    w.group = recd_group_carve(c, F, B, M_cap);
    w.list_off = c.take<int64_t>(2);
    w.seg_start = c.take<int64_t>(n_lists + 1);
    w.list_off_b = c.take<int64_t>(2);
    w.seg_start_b = c.take<int64_t>(M_cap + 1);
    w.seg_feat = c.take<int32_t>(M_cap);
    // at most n/(long_seg+1) segments of more than long_seg entries, in at most n/256 + n/(long_seg+1) chunks
    w.long_seg = long_seg;
    const int64_t item_cap = M_cap / 256 + M_cap / (w.long_seg + 1) + 16;
    w.chunk_count = c.take<int64_t>(1);
    w.chunks = c.take<RecdChunk>(item_cap);
    w.chunk_arrive = c.take<uint32_t>(item_cap);
    w.partials = c.take<float>((size_t)item_cap * D);
    w.g_u = c.take<float>((size_t)w.lists_cap * D);
    w.pos_list = c.take<uint32_t>(M_cap);
    w.pay_w = c.take<float>(M_cap);
    w.won = with_won ? c.take<uint32_t>((size_t)M_cap * row_lanes(D)) : nullptr;
    w.bytes = c.off;
    return w;
}

// What the row-gradient kernels of step B need to know about its segments.
RowSumParams row_params(const BwdWs &w, const uint32_t *ps, const float *pay_w, const void *table, int D, void *out)
{
    RowSumParams rp;
    rp.table = static_cast<const float *>(table);
    rp.pay = ps;
    rp.pay_w = pay_w;
    rp.seg_start = w.seg_start_b;
    rp.n_seg = w.list_off_b + 1;
    rp.out = static_cast<float *>(out);
    rp.D = D;
    rp.pieces = D / 4;
    rp.chunk_count = w.chunk_count;
    rp.chunks = w.chunks;
    rp.chunk_arrive = w.chunk_arrive;
    rp.partials = w.partials;
    rp.long_seg = w.long_seg;
    return rp;
}

// Step A: the sum of every unique list's grad_out rows (ps, grouped) into out.
recd_status sum_lists(recd_ctx *ctx, const BwdWs &w, const uint32_t *ps, int64_t U_cap, const float *grad_out, int D,
                      const int64_t *div_off)
{
    SegSumArgs a{};
    a.site = RECD_SITE_GRAD_STREAM;  // every grad_out row is read exactly once
    a.F = 1;
    a.D = D;
    a.table_dt = RECD_F32;
    a.out_dt = RECD_F32;
    a.tables.p[0] = grad_out;
    a.values = ps;
    a.values_are_i32 = 1;
    a.offsets = w.seg_start;
    a.list_off = w.list_off;
    a.lists_bound = U_cap;
    a.flat = 1;
    a.out = w.g_u;
    a.div_off = div_off;
    return recd_launch_segsum(ctx, a);
}

// What the grouping writes for a backward pass in the workspace w.
RecdGroupArgs group_args(const BwdWs &w, int F, int64_t B, int64_t U_cap, int64_t M_cap, int64_t max_rows,
                         const int32_t *inverse, const int64_t *feat_uoff, const int64_t *u_values,
                         const int64_t *u_offsets, int64_t *touched_rows, int64_t *feat_roff)
{
    RecdGroupArgs a{};
    a.F = F;
    a.B = B;
    a.U_cap = U_cap;
    a.M_cap = M_cap;
    a.max_rows = max_rows;
    a.inverse = inverse;
    a.feat_uoff = feat_uoff;
    a.u_values = u_values;
    a.u_offsets = u_offsets;
    a.pos_list = w.pos_list;
    a.seg_start_a = w.seg_start;
    a.list_off_a = w.list_off;
    a.seg_start_b = w.seg_start_b;
    a.list_off_b = w.list_off_b;
    a.touched_rows = touched_rows;
    a.feat_roff = feat_roff;
    a.seg_feat = w.seg_feat;
    a.chunk_count = w.chunk_count;
    a.chunks = w.chunks;
    a.chunk_arrive = w.chunk_arrive;
    a.long_seg = w.long_seg;
    a.lists_cap = w.lists_cap;
    return a;
}

// Ids a list on average, by the caller's bounds, below which the lists of a max-pooled backward share waves (k_max_winner): of
// rows of up to 256 bytes, four lists a wave or more, and of 512 bytes, two.  Whole backward, us, a wave a list / shared: rows of
// 64 and 256 bytes, uniform lengths, 8 ids 173 / 135, 186 / 173; 14 ids 138 / 122, 155 / 157; 25 ids 117 / 118, 137 / 145; Zipf's,
// 7 of at most 30 152 / 126, 161 / 155, 15 of at most 256 180 / 221, 203 / 265.  Rows of 512 bytes, 1.5 ids 366 / 344, 4 ids
// 288 / 284, 6 ids 239 / 246, 14 ids 191 / 206.
constexpr int64_t kSharedMean = 12, kSharedMeanWide = 4;

constexpr int64_t kWideRows = 512 * 1024;  // entries up to which k_segsum_rows has two pieces a lane

// Step B after the grouping: all segments in one launch, optimizer fused.
recd_status sum_rows(recd_ctx *ctx, const BwdWs &w, const uint32_t *ps, int64_t M_cap, const void *table,
                     int D, void *out, int64_t *touched_rows, const OptAdagrad *opt, const float *pay_w,
                     const uint32_t *won = nullptr)
{
    hipStream_t st = ctx->stream;
    RowSumParams rp = row_params(w, ps, pay_w, table, D, out);
    rp.pay_pos = reinterpret_cast<const uint32_t *>(pay_w);  // what lies beside the entries: weights or positions
    rp.won = won;
    OptAdagrad o;
    if (opt)
        o = *opt;
    else
        o.n_feat = 0;
    o.touched_rows = touched_rows;
    o.seg_feat = w.seg_feat;
    const int lpr = row_lanes(D);
    // Rows of 9 to 128 pieces, and not so many entries that what counts is the memory's rate: us, four pieces a lane / two,
    // rows of 512 bytes, 0.34 M entries of uniform ids 32.2 / 30.2, 0.69 M 66.1 / 72.1 (of skewed ids 87.8 / 82.7), 2.2 M of
    // skewed ids 214.9 / 212.9.
    const bool wide = !won && D > 32 && D <= 512 && M_cap <= kWideRows;
    const int per_block = 4 * (64 / lpr) / (wide ? 2 : 1);
    int64_t nblk = (M_cap + per_block - 1) / per_block;
    const int64_t cap = (int64_t)ctx->num_cu * 64;
    if (nblk > cap)
        nblk = cap;
    nblk = (nblk + 7) / 8 * 8;  // the kernel deals its blocks to 8 XCDs
    if (nblk < 8)
        nblk = 8;
    // blocks for the chunks: their number is on the device, usually far below the bound: at most what the
    // chip holds at once, striding
    int64_t cblk = M_cap / 256 + M_cap / (w.long_seg + 1);
    if (cblk > (int64_t)ctx->num_cu * 8)
        cblk = (int64_t)ctx->num_cu * 8;
    rp.chunk_blocks = (unsigned)((cblk + 7) / 8 * 8);
    const dim3 grid((unsigned)(nblk + rp.chunk_blocks)), block(256);
    recd_time_begin(ctx, RECD_T_GRAD_ROWS, st);
#define RECD_ROWS(L, WIDE) hipLaunchKernelGGL((k_segsum_rows<L, MODE, WIDE>), grid, block, 0, st, rp, o)
    auto launch = [&](auto mode) {
        constexpr int MODE = decltype(mode)::value;
        if constexpr (MODE != ROWS_MAX)
            if (wide) {
                switch (lpr) {
                case 4: RECD_ROWS(4, true); break;
                case 8: RECD_ROWS(8, true); break;
                case 16: RECD_ROWS(16, true); break;
                default: RECD_ROWS(32, true); break;
                }
                return;
            }
        switch (lpr) {
        case 4: RECD_ROWS(4, false); break;
        case 8: RECD_ROWS(8, false); break;
        case 16: RECD_ROWS(16, false); break;
        case 32: RECD_ROWS(32, false); break;
        default: RECD_ROWS(64, false); break;
        }
    };
#undef RECD_ROWS
    if (won)
        launch(std::integral_constant<int, ROWS_MAX>());
    else if (pay_w)
        launch(std::integral_constant<int, ROWS_WEIGHTED>());
    else
        launch(std::integral_constant<int, ROWS_PLAIN>());
    recd_time_end(ctx, RECD_T_GRAD_ROWS, st);
    RECD_HIP(ctx, hipGetLastError());
    return RECD_OK;
}

} // namespace

size_t recd_backward_workspace(int F, int64_t B, int64_t M_cap, int D)
{
    return carve_bwd(nullptr, F, B, (int64_t)F * B, M_cap, D, kDefaultLongSeg).bytes;
}

// The fused update reads and writes a table row (and its accumulator) once per (feature, row)
// segment, from different lane groups at the same time: two features must not name the same table or
// the same accumulator array.
static recd_status check_distinct_tables(recd_ctx *ctx, int F, void *const *tables, float *const *state)
{
    if (!tables)
        return RECD_OK;
    std::vector<const void *> t(tables, tables + F), m(state, state + F);
    std::sort(t.begin(), t.end());
    std::sort(m.begin(), m.end());
    for (int f = 1; f < F; f++)
        if (t[f] == t[f - 1] || m[f] == m[f - 1])
            return recd_fail(ctx, RECD_EINVAL,
                             "tables[] and adagrad_state[] must each hold pairwise distinct pointers "
                             "(one table per feature)");
    return RECD_OK;
}

// What the grouping found about the caller's bounds (host_pinned[1]: side B's word, [2]: side A's).
static recd_status check_bounds(recd_ctx *ctx, int64_t U_cap, int64_t M_cap)
{
    if (ctx->host_pinned[1])
        return recd_fail(ctx, RECD_ECAPACITY, "M_cap=%lld is smaller than M", (long long)M_cap);
    if (ctx->host_pinned[2] & RECD_GROUP_LISTS)
        return recd_fail(ctx, RECD_ECAPACITY, "U_cap=%lld is smaller than U", (long long)U_cap);
    if (ctx->host_pinned[2] & RECD_GROUP_RUNS)
        return recd_fail(ctx, RECD_ECAPACITY, "runs_cap is smaller than the number of runs");
    return RECD_OK;
}

// Backward of the pooled path (seq = false: grad_out is [F,B,D]) and of the sequence path (seq =
// true: grad_out is [N,D], one row per KJT position; kjt_offsets, N and grad_emb are used).
// mean: the pooled path averaged, so g_u[u] is divided by the length of unique list u (every
// segment of step A is one unique list, in order: each has at least one row).
// u_weights: the pooled path's lookup was the weighted sum: position j hands u_weights[j] * g_u on.
// max_tables: the pooled path's lookup was the maximum over these fp32 tables: element d of g_u
// goes to the position that won it (k_max_winner); step B takes of g_u what each position won.
static recd_status backward_common(recd_ctx *ctx, bool seq, bool mean, int F, int64_t B, int64_t N, int D,
                                   const float *grad_out, const int64_t *kjt_offsets,
                                   const int32_t *inverse, const int64_t *feat_uoff,
                                   const int64_t *u_values, const float *u_weights,
                                   const void *const *max_tables, const int64_t *u_offsets,
                                   const int64_t *rows, int64_t U_cap, int64_t M_cap, float *grad_emb,
                                   int64_t *touched_rows, int64_t *feat_roff, float *grad_rows,
                                   void *const *tables, float *const *adagrad_state, float lr,
                                   float eps, int64_t *host_R)
{
    if (!ctx)
        return RECD_EINVAL;
    if (seq && (N < 0 || N >= (int64_t)1 << 31 || !kjt_offsets || (M_cap > 0 && !grad_emb)))
        return recd_fail(ctx, RECD_EINVAL, "sequence backward: bad N or null offsets / grad_emb");
    if (F < 0 || F > RECD_MAX_FEATURES || B < 0 || M_cap < 0 || U_cap < 0)
        return recd_fail(ctx, RECD_EINVAL, "bad sizes");
    if (U_cap > (int64_t)F * B)
        U_cap = (int64_t)F * B;
    if (D <= 0 || D % 4 != 0 || (size_t)D * 4 > RECD_MAX_ROW_BYTES ||
        (D * 4 / 16 > 64 && D * 4 / 16 != 128 && D * 4 / 16 != 256))
        return recd_fail(ctx, RECD_EINVAL, "unsupported D=%d", D);
    const int64_t n_lists = (int64_t)F * B;
    if (n_lists >= (int64_t)1 << 31 || M_cap >= (int64_t)1 << 31)
        return recd_fail(ctx, RECD_EINVAL, "F*B and M_cap must stay below 2^31");
    if (!feat_roff || !feat_uoff || !u_offsets || (F > 0 && !rows))
        return recd_fail(ctx, RECD_EINVAL, "null pointer argument");
    if (n_lists > 0 && ((!grad_out && !(seq && N == 0)) || !inverse))
        return recd_fail(ctx, RECD_EINVAL, "null pointer argument");
    if (M_cap > 0 && (!u_values || !touched_rows))
        return recd_fail(ctx, RECD_EINVAL, "null pointer argument");
    if (M_cap > 0 && !grad_rows && !(tables && F <= RECD_F_PER_LAUNCH))
        return recd_fail(ctx, RECD_EINVAL,
                         "grad_rows may be NULL only with the optimizer and at most %d features",
                         RECD_F_PER_LAUNCH);
    if ((tables == nullptr) != (adagrad_state == nullptr))
        return recd_fail(ctx, RECD_EINVAL, "tables and adagrad_state must be given together");
    RECD_TRY(recd_check_rows(ctx, F, rows));
    int64_t max_rows = 1;
    for (int f = 0; f < F; f++) {
        if (rows[f] <= 0)
            return recd_fail(ctx, RECD_EINVAL, "rows[%d] <= 0", f);
        if (rows[f] > max_rows)
            max_rows = rows[f];
        if (tables && (!tables[f] || !adagrad_state[f]))
            return recd_fail(ctx, RECD_EINVAL, "tables[%d] or adagrad_state[%d] is null", f, f);
    }
    RECD_TRY(check_distinct_tables(ctx, F, tables, adagrad_state));
    RECD_HIP(ctx, hipSetDevice(ctx->device));
    if (ctx->validate && n_lists > 0)
        RECD_TRY(recd_validate_inverse(ctx, F, B, feat_uoff, inverse));
    const bool maxmode = max_tables != nullptr;
    ctx->plan.valid = false;  // this call reuses the workspace a plan would live in
    RECD_TRY(recd_reserve(ctx, carve_bwd(nullptr, F, B, U_cap, M_cap, D, ctx->long_seg_cut, maxmode).bytes));
    const BwdWs w = carve_bwd(ctx->ws, F, B, U_cap, M_cap, D, ctx->long_seg_cut, maxmode);
    hipStream_t st = ctx->stream;

    if (n_lists == 0 || M_cap == 0) {
        // no id anywhere: no row is touched
        hipLaunchKernelGGL(k_no_rows, dim3(1), dim3(64), 0, st, F, feat_roff, w.list_off);
        RECD_HIP(ctx, hipGetLastError());
        if (host_R) {
            RECD_HIP(ctx, hipStreamSynchronize(st));
            host_R[0] = 0;
        }
        return RECD_OK;
    }

    // Row-wise Adagrad runs inside the row-gradient segment sum while the sum is still in
    // registers; with more features than one launch carries it runs as a kernel of its own.
    const bool fused = tables != nullptr && F <= RECD_F_PER_LAUNCH;
    OptAdagrad oa;
    oa.n_feat = 0;
    if (fused) {
        oa.n_feat = F;
        for (int f = 0; f < F; f++) {
            oa.w[f] = static_cast<float *>(tables[f]);
            oa.m[f] = adagrad_state[f];
        }
        oa.lr = lr;
        oa.eps = eps;
    }
    // ---- both groupings ----------------------------------------------------------------------------
    RecdGroupArgs ga = group_args(w, F, B, U_cap, M_cap, max_rows, inverse, feat_uoff, u_values, u_offsets,
                                  touched_rows, feat_roff);
    ga.pay_positions = seq || u_weights || maxmode ? 1 : 0;  // the later sum's source row: position or list
    if (seq)
        ga.pos_list = nullptr;
    if (maxmode)
        ga.pay_pos = reinterpret_cast<uint32_t *>(w.pay_w);  // the sorted positions take the place of weights
    ga.u_weights = u_weights;
    ga.pay_w = w.pay_w;
    RECD_TRY(recd_group(ctx, st, w.group, ga));
    const uint32_t *ps_a = recd_group_rows(w.group, F, B, U_cap, M_cap, max_rows);
    const uint32_t *ps_b = recd_group_positions(w.group, F, B, M_cap, max_rows);
    // ---- step A: sum grad_out rows into g_u (or, for sequences, into grad_emb) ---------------------------
    {
        if (!seq) {
            RECD_TRY(sum_lists(ctx, w, ps_a, U_cap, grad_out, D, mean ? u_offsets : nullptr));
        } else {
            const int lists = recd_jagged_lists(N, U_cap, M_cap, D / 4, ctx->num_cu);
            int64_t blocks = (U_cap + lists - 1) / lists;
            if (blocks > (int64_t)ctx->num_cu * 64)
                blocks = (int64_t)ctx->num_cu * 64;
            if (blocks < 1)
                blocks = 1;
            // At most four rows a list, on average over its positions: blocks without a longer list are
            // likely.  Beyond, few are, and the plain kernel is the quicker one (figures at the kernel).
            // A loose M_cap only makes the average smaller than it is.  With M_cap = N, which cannot be told from
            // lists of one row each, whole calls with / without FEW, us, 0.65 M ids, 512-byte rows: of 1 row 306 / 419, of 3
            // 186 / 197, of 8 to 32 173 / 173, of 64 254 / 251, of 200 394 / 386.
            const bool few = N <= 4 * M_cap;
#define RECD_JR_(L, FEW)                                                                              \
    hipLaunchKernelGGL((k_jagged_reduce<L, FEW>), dim3((unsigned)blocks), dim3(256), 0, st,           \
                       reinterpret_cast<const float4 *>(grad_out), kjt_offsets, ps_a, w.seg_start,    \
                       w.list_off + 1, u_offsets, reinterpret_cast<float4 *>(grad_emb), D / 4, N, M_cap)
#define RECD_JR(L) if (few) RECD_JR_(L, true); else RECD_JR_(L, false)
            switch (lists) {
            case 1: RECD_JR(1); break;
            case 2: RECD_JR(2); break;
            case 4: RECD_JR(4); break;
            case 8: RECD_JR(8); break;
            case 16: RECD_JR(16); break;
            case 32: RECD_JR(32); break;
            default: RECD_JR(64); break;
            }
#undef RECD_JR
#undef RECD_JR_
            RECD_HIP(ctx, hipGetLastError());
        }
    }
    if (maxmode) {
        const int P = D / 4;  // 16-byte pieces of a row: up to 64 one per lane, else 128 or 256
        const int lpr = P <= 4 ? 4 : (P <= 8 ? 8 : (P <= 16 ? 16 : (P <= 32 ? 32 : 64)));
        const int vpl = P <= 64 ? 1 : (P == 128 ? 2 : 4);
        for (int f0 = 0; f0 < F; f0 += RECD_F_PER_LAUNCH) {
            MaxTables mt;
            const int nf = F - f0 < RECD_F_PER_LAUNCH ? F - f0 : RECD_F_PER_LAUNCH;
            for (int f = 0; f < nf; f++)
                mt.w[f] = static_cast<const float *>(max_tables[f0 + f]);
            const int nl = M_cap < (lpr < 32 ? kSharedMean : kSharedMeanWide) * U_cap ? 64 / lpr : 1;
            const int64_t waves = (U_cap + nl - 1) / nl, nblk = waves < (int64_t)ctx->num_cu * 256 ? waves : (int64_t)ctx->num_cu * 256;
            const dim3 grid((unsigned)(nblk < 1 ? 1 : nblk)), block(64);
#define RECD_MR(L, V, N)                                                                                    \
    hipLaunchKernelGGL((k_max_winner<L, V, N>), grid, block, 0, st, u_values, u_offsets, feat_uoff, f0, nf, mt,  \
                       w.won, row_lanes(D), P, U_cap, M_cap)
#define RECD_MR_(L) if (nl > 1) RECD_MR(L, 1, 64 / L); else RECD_MR(L, 1, 1)
            switch (vpl > 1 ? P : lpr) {
            case 256: RECD_MR(64, 4, 1); break;
            case 128: RECD_MR(64, 2, 1); break;
            case 4: RECD_MR_(4); break;
            case 8: RECD_MR_(8); break;
            case 16: RECD_MR_(16); break;
            case 32: RECD_MR_(32); break;
            default: RECD_MR(64, 1, 1); break;
            }
#undef RECD_MR_
#undef RECD_MR
        }
        RECD_HIP(ctx, hipGetLastError());
    }
    const float *b_table = seq ? grad_emb : w.g_u;
    // ---- step B: sum the source rows of every (feature, row) into grad_rows -------------------------
    RECD_TRY(sum_rows(ctx, w, ps_b, M_cap, b_table, D, grad_rows, touched_rows, fused ? &oa : nullptr,
                      u_weights || maxmode ? w.pay_w : nullptr, maxmode ? w.won : nullptr));
    // ---- optimizer -------------------------------------------------------------------------------
    if (tables && !fused) {
        for (int f0 = 0; f0 < F; f0 += RECD_F_PER_LAUNCH) {
            OptPtrs ptrs;
            const int nf = F - f0 < RECD_F_PER_LAUNCH ? F - f0 : RECD_F_PER_LAUNCH;
            for (int f = 0; f < nf; f++) {
                ptrs.w[f] = static_cast<float *>(tables[f0 + f]);
                ptrs.m[f] = adagrad_state[f0 + f];
            }
            hipLaunchKernelGGL(k_adagrad, dim3(ctx->num_cu * 8), dim3(256), 0, st, grad_rows,
                               touched_rows, feat_roff, f0, nf, D, ptrs, lr, eps);
        }
        RECD_HIP(ctx, hipGetLastError());
    }
    if (host_R) {
        RECD_HIP(ctx, hipMemcpyAsync(ctx->host_pinned, w.list_off_b + 1, sizeof(int64_t),
                                     hipMemcpyDeviceToHost, st));
        RECD_HIP(ctx, hipMemcpyAsync(ctx->host_pinned + 1, w.group.b.too_small, sizeof(int64_t),
                                     hipMemcpyDeviceToHost, st));
        RECD_HIP(ctx, hipMemcpyAsync(ctx->host_pinned + 2, w.group.a.too_small, sizeof(int64_t),
                                     hipMemcpyDeviceToHost, st));
        RECD_HIP(ctx, hipStreamSynchronize(st));
        host_R[0] = ctx->host_pinned[0];
        RECD_TRY(check_bounds(ctx, U_cap, M_cap));
    }
    return RECD_OK;
}

// ---------------------------------------------------------------- planned backward
// The backward's grouping work depends on the IKJT only, not on the gradient.  recd_backward_plan runs it
// on the side stream (a short one on the stream itself), starting where the IKJT's build ended, so
// that it overlaps the forward calls (which are bandwidth-bound, while the plan is a chain of short
// latency-bound kernels);
// recd_backward_apply then waits for the plan on the main stream and runs the two segment sums with
// the fused update.  Same kernels, same inputs, same results as the one-call form.
// run_index: null, or the batch's run index, whose number of runs is checked against runs_cap (the
// grouping itself reads `inverse`: sorting the runs instead of the rows took fewer keys and more
// launches).
static recd_status plan_common(recd_ctx *ctx, int F, int64_t B, int D, const int32_t *inverse,
                               const int64_t *feat_uoff, const int64_t *u_values, const int64_t *u_offsets,
                               const int64_t *rows, int64_t U_cap, int64_t M_cap, const int64_t *run_index,
                               int64_t runs_cap, int64_t *touched_rows, int64_t *feat_roff)
{
    if (!ctx)
        return RECD_EINVAL;
    ctx->plan.valid = false;
    if (run_index && runs_cap < 0)
        return recd_fail(ctx, RECD_EINVAL, "runs_cap < 0");
    if (F < 0 || F > RECD_MAX_FEATURES || B < 0 || M_cap < 0 || U_cap < 0)
        return recd_fail(ctx, RECD_EINVAL, "bad sizes");
    if (U_cap > (int64_t)F * B)
        U_cap = (int64_t)F * B;
    if (D <= 0 || D % 4 != 0 || (size_t)D * 4 > RECD_MAX_ROW_BYTES ||
        (D * 4 / 16 > 64 && D * 4 / 16 != 128 && D * 4 / 16 != 256))
        return recd_fail(ctx, RECD_EINVAL, "unsupported D=%d", D);
    const int64_t n_lists = (int64_t)F * B;
    if (n_lists >= (int64_t)1 << 31 || M_cap >= (int64_t)1 << 31)
        return recd_fail(ctx, RECD_EINVAL, "F*B and M_cap must stay below 2^31");
    if (!feat_roff || !feat_uoff || !u_offsets || (F > 0 && !rows) || (n_lists > 0 && !inverse) ||
        (M_cap > 0 && (!u_values || !touched_rows)))
        return recd_fail(ctx, RECD_EINVAL, "null pointer argument");
    RECD_TRY(recd_check_rows(ctx, F, rows));
    int64_t max_rows = 1;
    for (int f = 0; f < F; f++) {
        if (rows[f] <= 0)
            return recd_fail(ctx, RECD_EINVAL, "rows[%d] <= 0", f);
        if (rows[f] > max_rows)
            max_rows = rows[f];
    }
    RECD_HIP(ctx, hipSetDevice(ctx->device));
    if (ctx->validate && n_lists > 0)
        RECD_TRY(recd_validate_inverse(ctx, F, B, feat_uoff, inverse));
    // the side stream may start at the end of the build only if nothing on the stream has used the
    // workspace since (this call's own reservation does not count)
    const bool ws_idle_since_build = !ctx->ws_used_since_build;
    RECD_TRY(recd_reserve(ctx, carve_bwd(nullptr, F, B, U_cap, M_cap, D, ctx->long_seg_cut).bytes));
    const BwdWs w = carve_bwd(ctx->ws, F, B, U_cap, M_cap, D, ctx->long_seg_cut);
    recd_ctx::BackwardPlan &pl = ctx->plan;
    pl.F = F;
    pl.B = B;
    pl.D = D;
    pl.U_cap = U_cap;
    pl.M_cap = M_cap;
    pl.u_offsets = u_offsets;
    pl.touched_rows = touched_rows;
    pl.feat_roff = feat_roff;
    pl.ws = ctx->ws;
    pl.empty = n_lists == 0 || M_cap == 0;
    // A short grouping costs less on the stream itself than the events that would take it to the side stream and back.
    hipStream_t st = ctx->stream;
    const bool own_stream = pl.empty || recd_group_is_small(F, B, M_cap, max_rows) || recd_grouping_is_short((int64_t)F * B, M_cap);
    hipStream_t side = own_stream ? st : ctx->side_stream;
    // Where the side stream may start: at the end of the build that produced this IKJT if it is the
    // context's most recent one, else at the main stream's current position.
    hipEvent_t from = ctx->ev_fork;
    if (own_stream)
        from = nullptr;
    else if (ctx->build_valid && ws_idle_since_build && ctx->built_inverse == inverse &&
        ctx->built_u_values == u_values && n_lists > 0) {
        if (ctx->build_event.at_plan())
            from = ctx->ev_built;
    }
    if (from == ctx->ev_fork)
        RECD_HIP(ctx, hipEventRecord(ctx->ev_fork, st));
    if (from)
        RECD_HIP(ctx, hipStreamWaitEvent(side, from, 0));
    if (!pl.empty) {
        RecdGroupArgs ga = group_args(w, F, B, U_cap, M_cap, max_rows, inverse, feat_uoff, u_values, u_offsets,
                                      touched_rows, feat_roff);
        ga.run_index = run_index;
        ga.runs_cap = runs_cap > n_lists || runs_cap == 0 ? n_lists : runs_cap;
        RECD_TRY(recd_group(ctx, side, w.group, ga));
        pl.ps_a = recd_group_rows(w.group, F, B, U_cap, M_cap, max_rows);
        pl.ps_b = recd_group_positions(w.group, F, B, M_cap, max_rows);
    }
    if (!own_stream) {
        RECD_HIP(ctx, hipEventRecord(ctx->ev_plan, side));
        pl.pending = true;
    }
    pl.valid = true;
    return RECD_OK;
}

extern "C" recd_status recd_backward_plan(recd_ctx *ctx, int F, int64_t B, int D, const int32_t *inverse,
                                          const int64_t *feat_uoff, const int64_t *u_values,
                                          const int64_t *u_offsets, const int64_t *rows, int64_t U_cap,
                                          int64_t M_cap, int64_t *touched_rows, int64_t *feat_roff)
{
    return plan_common(ctx, F, B, D, inverse, feat_uoff, u_values, u_offsets, rows, U_cap, M_cap, nullptr, 0,
                       touched_rows, feat_roff);
}

extern "C" recd_status recd_backward_plan_runs(recd_ctx *ctx, int F, int64_t B, int D, const int32_t *inverse,
                                               const int64_t *feat_uoff, const int64_t *u_values,
                                               const int64_t *u_offsets, const int64_t *rows, int64_t U_cap,
                                               int64_t M_cap, const int64_t *run_index, int64_t runs_cap,
                                               int64_t *touched_rows, int64_t *feat_roff)
{
    if (ctx && !run_index && (int64_t)F * B > 0)
        return recd_fail(ctx, RECD_EINVAL, "null run_index");
    return plan_common(ctx, F, B, D, inverse, feat_uoff, u_values, u_offsets, rows, U_cap, M_cap, run_index,
                       runs_cap, touched_rows, feat_roff);
}

extern "C" recd_status recd_backward_apply(recd_ctx *ctx, recd_pooling mode, const float *grad_out,
                                           float *grad_rows, void *const *tables,
                                           float *const *adagrad_state, float lr, float eps,
                                           int64_t *host_R)
{
    if (!ctx)
        return RECD_EINVAL;
    recd_ctx::BackwardPlan &pl = ctx->plan;
    if (!pl.valid || pl.ws != ctx->ws)
        return recd_fail(ctx, RECD_EINVAL,
                         "no valid plan: recd_backward_plan must be the context's last workspace-using call");
    pl.valid = false;
    if (mode != RECD_POOL_SUM && mode != RECD_POOL_MEAN)
        return recd_fail(ctx, RECD_EINVAL, "planned backward: pooling mode %d is not supported", (int)mode);
    const int F = pl.F, D = pl.D;
    const int64_t B = pl.B, n_lists = (int64_t)F * B, M_cap = pl.M_cap;
    if (n_lists > 0 && !grad_out)
        return recd_fail(ctx, RECD_EINVAL, "null grad_out");
    if ((tables == nullptr) != (adagrad_state == nullptr))
        return recd_fail(ctx, RECD_EINVAL, "tables and adagrad_state must be given together");
    if (M_cap > 0 && !grad_rows && !(tables && F <= RECD_F_PER_LAUNCH))
        return recd_fail(ctx, RECD_EINVAL,
                         "grad_rows may be NULL only with the optimizer and at most %d features",
                         RECD_F_PER_LAUNCH);
    for (int f = 0; f < F && tables; f++)
        if (!tables[f] || !adagrad_state[f])
            return recd_fail(ctx, RECD_EINVAL, "tables[%d] or adagrad_state[%d] is null", f, f);
    RECD_TRY(check_distinct_tables(ctx, F, tables, adagrad_state));
    RECD_HIP(ctx, hipSetDevice(ctx->device));
    hipStream_t st = ctx->stream;
    const BwdWs w = carve_bwd(ctx->ws, F, B, pl.U_cap, M_cap, D, ctx->long_seg_cut);
    if (pl.pending)
        RECD_HIP(ctx, hipStreamWaitEvent(st, ctx->ev_plan, 0));
    pl.pending = false;  // the stream now waits for everything the plan enqueued
    if (pl.empty) {
        hipLaunchKernelGGL(k_no_rows, dim3(1), dim3(64), 0, st, F, pl.feat_roff, w.list_off_b);
        RECD_HIP(ctx, hipGetLastError());
        if (host_R) {
            RECD_HIP(ctx, hipStreamSynchronize(st));
            host_R[0] = 0;
        }
        return RECD_OK;
    }
    const bool fused = tables != nullptr && F <= RECD_F_PER_LAUNCH;
    OptAdagrad oa;
    oa.n_feat = 0;
    if (fused) {
        oa.n_feat = F;
        for (int f = 0; f < F; f++) {
            oa.w[f] = static_cast<float *>(tables[f]);
            oa.m[f] = adagrad_state[f];
        }
        oa.lr = lr;
        oa.eps = eps;
    }
    RECD_TRY(sum_lists(ctx, w, pl.ps_a, pl.U_cap, grad_out, D, mode == RECD_POOL_MEAN ? pl.u_offsets : nullptr));
    RECD_TRY(sum_rows(ctx, w, pl.ps_b, M_cap, w.g_u, D, grad_rows, pl.touched_rows, fused ? &oa : nullptr,
                      nullptr));
    if (tables && !fused) {
        for (int f0 = 0; f0 < F; f0 += RECD_F_PER_LAUNCH) {
            OptPtrs ptrs;
            const int nf = F - f0 < RECD_F_PER_LAUNCH ? F - f0 : RECD_F_PER_LAUNCH;
            for (int f = 0; f < nf; f++) {
                ptrs.w[f] = static_cast<float *>(tables[f0 + f]);
                ptrs.m[f] = adagrad_state[f0 + f];
            }
            hipLaunchKernelGGL(k_adagrad, dim3(ctx->num_cu * 8), dim3(256), 0, st, grad_rows, pl.touched_rows,
                               pl.feat_roff, f0, nf, D, ptrs, lr, eps);
        }
        RECD_HIP(ctx, hipGetLastError());
    }
    if (host_R) {
        RECD_HIP(ctx, hipMemcpyAsync(ctx->host_pinned, w.list_off_b + 1, sizeof(int64_t), hipMemcpyDeviceToHost, st));
        RECD_HIP(ctx, hipMemcpyAsync(ctx->host_pinned + 1, w.group.b.too_small, sizeof(int64_t), hipMemcpyDeviceToHost,
                                     st));
        RECD_HIP(ctx, hipMemcpyAsync(ctx->host_pinned + 2, w.group.a.too_small, sizeof(int64_t), hipMemcpyDeviceToHost,
                                     st));
        RECD_HIP(ctx, hipStreamSynchronize(st));
        host_R[0] = ctx->host_pinned[0];
        RECD_TRY(check_bounds(ctx, pl.U_cap, M_cap));
    }
    return RECD_OK;
}

extern "C" recd_status recd_backward_dedup(recd_ctx *ctx, int F, int64_t B, int D,
                                           const float *grad_out, const int32_t *inverse,
                                           const int64_t *feat_uoff, const int64_t *u_values,
                                           const int64_t *u_offsets, const int64_t *rows,
                                           int64_t U_cap, int64_t M_cap, int64_t *touched_rows,
                                           int64_t *feat_roff, float *grad_rows, void *const *tables,
                                           float *const *adagrad_state, float lr, float eps,
                                           int64_t *host_R)
{
    return backward_common(ctx, false, false, F, B, 0, D, grad_out, nullptr, inverse, feat_uoff, u_values,
                           nullptr, nullptr, u_offsets, rows, U_cap, M_cap, nullptr, touched_rows, feat_roff, grad_rows, tables,
                           adagrad_state, lr, eps, host_R);
}

extern "C" recd_status recd_backward_dedup_mode(recd_ctx *ctx, recd_pooling mode, int F, int64_t B, int D,
                                                const float *grad_out, const int32_t *inverse,
                                                const int64_t *feat_uoff, const int64_t *u_values,
                                                const int64_t *u_offsets, const int64_t *rows,
                                                int64_t U_cap, int64_t M_cap, int64_t *touched_rows,
                                                int64_t *feat_roff, float *grad_rows, void *const *tables,
                                                float *const *adagrad_state, float lr, float eps,
                                                int64_t *host_R)
{
    if (!ctx)
        return RECD_EINVAL;
    if (mode != RECD_POOL_SUM && mode != RECD_POOL_MEAN)
        return recd_fail(ctx, RECD_EINVAL,
                         "backward: pooling mode %d is not supported (sum and mean are)", (int)mode);
    return backward_common(ctx, false, mode == RECD_POOL_MEAN, F, B, 0, D, grad_out, nullptr, inverse,
                           feat_uoff, u_values, nullptr, nullptr, u_offsets, rows, U_cap, M_cap, nullptr, touched_rows,
                           feat_roff, grad_rows, tables, adagrad_state, lr, eps, host_R);
}

extern "C" recd_status recd_backward_sequence_dedup(recd_ctx *ctx, int F, int64_t B, int64_t N, int D,
                                                    const float *grad_out, const int64_t *offsets,
                                                    const int32_t *inverse, const int64_t *feat_uoff,
                                                    const int64_t *u_values, const int64_t *u_offsets,
                                                    const int64_t *rows, int64_t U_cap, int64_t M_cap,
                                                    float *grad_emb, int64_t *touched_rows,
                                                    int64_t *feat_roff, float *grad_rows,
                                                    void *const *tables, float *const *adagrad_state,
                                                    float lr, float eps, int64_t *host_R)
{
    return backward_common(ctx, true, false, F, B, N, D, grad_out, offsets, inverse, feat_uoff, u_values, nullptr,
                           nullptr, u_offsets, rows, U_cap, M_cap, grad_emb, touched_rows, feat_roff, grad_rows, tables,
                           adagrad_state, lr, eps, host_R);
}

extern "C" recd_status recd_backward_dedup_weighted(recd_ctx *ctx, int F, int64_t B, int D,
                                                    const float *grad_out, const int32_t *inverse,
                                                    const int64_t *feat_uoff, const int64_t *u_values,
                                                    const float *u_weights, const int64_t *u_offsets,
                                                    const int64_t *rows, int64_t U_cap, int64_t M_cap,
                                                    int64_t *touched_rows, int64_t *feat_roff,
                                                    float *grad_rows, void *const *tables,
                                                    float *const *adagrad_state, float lr, float eps,
                                                    int64_t *host_R)
{
    if (!ctx)
        return RECD_EINVAL;
    if (M_cap > 0 && !u_weights)
        return recd_fail(ctx, RECD_EINVAL, "null u_weights");
    return backward_common(ctx, false, false, F, B, 0, D, grad_out, nullptr, inverse, feat_uoff, u_values,
                           M_cap > 0 ? u_weights : nullptr, nullptr, u_offsets, rows, U_cap, M_cap, nullptr,
                           touched_rows, feat_roff, grad_rows, tables, adagrad_state, lr, eps, host_R);
}

extern "C" recd_status recd_backward_dedup_max(recd_ctx *ctx, int F, int64_t B, int D,
                                               const float *grad_out, const int32_t *inverse,
                                               const int64_t *feat_uoff, const int64_t *u_values,
                                               const int64_t *u_offsets, const int64_t *rows,
                                               int64_t U_cap, int64_t M_cap,
                                               const void *const *lookup_tables, int64_t *touched_rows,
                                               int64_t *feat_roff, float *grad_rows, void *const *tables,
                                               float *const *adagrad_state, float lr, float eps,
                                               int64_t *host_R)
{
    if (!ctx)
        return RECD_EINVAL;
    if (F > 0 && !lookup_tables)
        return recd_fail(ctx, RECD_EINVAL, "null lookup_tables");
    for (int f = 0; f < F; f++)
        if (!lookup_tables[f])
            return recd_fail(ctx, RECD_EINVAL, "lookup_tables[%d] is null", f);
    return backward_common(ctx, false, false, F, B, 0, D, grad_out, nullptr, inverse, feat_uoff, u_values,
                           nullptr, M_cap > 0 && F > 0 ? lookup_tables : nullptr, u_offsets, rows, U_cap, M_cap,
                           nullptr, touched_rows, feat_roff, grad_rows, tables, adagrad_state, lr, eps, host_R);
}

size_t recd_build_workspace(int F, int64_t B);

extern "C" recd_status recd_workspace_bytes(int F, int64_t B, int64_t N, int D, size_t *out_bytes)
{
    if (!out_bytes || F < 0 || B < 0 || N < 0 || D <= 0)
        return RECD_EINVAL;
    const size_t a = recd_build_workspace(F, B);
    const size_t b = recd_backward_workspace(F, B, N, D);
    *out_bytes = (a > b ? a : b) + 4096;
    return RECD_OK;
}
