// bload_plan: seeded order + next-fit block assignment on the device
// (BLoad, Methods section: blocks of T_max frames made of randomly ordered
// whole sequences, each closed as near T_max as the order allows).
//
// Next-fit is a sequential recurrence (whether a sequence opens a new block
// depends on everything before it).  Its exact parallel form, all in integers:
//   P        exclusive prefix sum of the lengths in shuffled order
//   next[p]  the position that would open the next block if p opened one:
//            the smallest q > p with P[q+1] - P[p] > T_blk (binary search in P)
//   heads    the orbit of position 0 under next[], marked by pointer jumping
//            (round k: every marked p marks jump[p], then jump = jump o jump)
//   block    inclusive count of heads up to p, minus one
//   offset   P[p] - P[head of p's block]
// Up to 2048 sequences one workgroup does all of it in one launch, a position to a lane (plan_wave_kernel and
// plan_waves_kernel); up to 12288, one of 16 waves does, between a launch that finds the order, which is work for the
// whole chip, and one that writes the tables (plan_mid_kernel).
// Beyond that the scans work on tiles of 2048 positions (many small workgroups)
// and the orbit is found on tiles of 2048 to 8192 in three steps that need no launch per
// jumping round: every tile jumps inside its own LDS until each of its positions
// has left the tile (exit[p]); the orbit's entry into each tile is found by following
// exit[] from position 0 (one hop per tile; from 40 tiles on over groups of 8 or 16 tiles, whose
// exits a small kernel composes first; beyond 1024 tiles one thread finds all entries); every
// tile then marks its heads from its entry by jumping in LDS again.  Six launches up to 40 tiles,
// seven beyond, one more where the sequences fetch what they get (plan_gather_kernel).  (Blocks so long that prefix sums
// of 12288 sequences leave 32 bits: the tiles from 2049 sequences on, five launches where the one tile is entered at
// position 0.)
// Bound by launches and latencies: 10^6 documents 125 -> 111 us per call with smaller jump tiles (exit kernel 17 -> 13 us;
// the marking kernel's shorter rounds pay for its longer walk: 23 -> 25), tables fetched instead of scattered (32 -> 11 +
// 12) and next[] searched in LDS (16 -> 10).
#include "bload_common.hpp"
#include "bload_order.hpp"

#include <algorithm>
#include <type_traits>

namespace bload {

constexpr int kItems = 8;                         // consecutive positions per thread in the scans
constexpr int kTile = kThreads * kItems;          // positions per workgroup in the scans: 2048
constexpr int kJumpItems = 16;                    // positions per thread where a workgroup jumps in LDS
// Such a workgroup takes a jump tile of 16 positions for each of its NT threads: 2048, 4096 or 8192 of them.  Small ones
// spread over more compute units and their rounds are shorter, but the walk over them is longer: 20000
// sequences 74 us in tiles of 8192, 69 in tiles of 4096, 66 of 2048; 10^6 114.8, 111.2, 113; 2 * 10^6 213, 216, 219.
// Up to 8192 sequences one tile needs no exits (those of which the sums leave 32 bits come here: 2049 and 8192 in blocks of
// 2^24 slots 51 and 58 us, 64 and 67 in tiles of 2048).
constexpr int kJumpTile = 8192;                   // the largest
template <int NT> __host__ __device__ constexpr int jump_tile() { return NT * kJumpItems; }
constexpr int64_t kSmallTilesUpTo = 160000, kMidTilesUpTo = (int64_t)1 << 20;
constexpr int kPlanWaves = 16;                    // one launch and up to this many waves do for 64 to kWavesMost sequences (256: 23.4
constexpr int kWavesMost = 2 * kPlanWaves * kWave;     // -> 18.5 us a call; 300: 28.1 -> 20.3; 2048, 125 and 1 to a block: 29.3 -> 26.3,
                                                  // 33.5 -> 26.1.  At 4096 three launches are faster: 31.8 and 39.0, 33.8 and 33.0 in one)
constexpr int kWalkTiles = 1024;                  // up to this many jump tiles, each finds its own entry (see plan_mark_kernel),
constexpr int kGroupFrom = 40;                    // and from this many on with the exits of groups of tiles: their launch
                                                  // costs 5 us, a hop of the walk 0.24
constexpr int64_t kGatherFrom = (int64_t)1 << 19;      // see plan_gather_kernel
constexpr int64_t kSingleItems = (int64_t)1 << 20;     // up to this many sequences the order kernel takes one per thread
constexpr int kJumpRounds = 13;                   // 2^13 = kJumpTile: rounds that cross a whole tile
constexpr int kWavesPerScanTile = kTile / (kWave * kJumpItems);     // waves of the marking kernel per scan tile

// ---- workgroup scans --------------------------------------------------------

// (number of heads, position of the last head): combined by sum and max.
struct HeadPair { int32_t cnt; int32_t head; };
struct HeadOp {
    __device__ HeadPair operator()(HeadPair a, HeadPair b) const
    {
        return HeadPair{a.cnt + b.cnt, max(a.head, b.head)};
    }
};
struct SumI64 { __device__ int64_t operator()(int64_t a, int64_t b) const { return a + b; } };

// How a value of each scanned type comes from another lane (DPP), with the operation's
// identity where there is no such lane.
struct LaneMove {
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ int64_t at(int64_t v) const
    {
        return (int64_t)dpp_move<CTRL, ROW_MASK>((long long)v, 0ll);
    }
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ HeadPair at(HeadPair v) const
    {
        return HeadPair{dpp_move<CTRL, ROW_MASK>(v.cnt, 0), dpp_move<CTRL, ROW_MASK>(v.head, -1)};
    }
};

// Exclusive scan of one value per thread across the workgroup; `total` gets
// the reduction of all values.  `ident` is the identity of `op`.
template <typename T, typename Op>
__device__ __forceinline__ T block_exclusive_scan(T x, T ident, Op op, T* total)
{
    __shared__ T wave_tot[kThreads / kWave];
    const int lane = lane_id(), wave = wave_id();
    const T incl = wave_scan(x, op, LaneMove());
    const T excl = LaneMove().template at<kDppWaveShr1, 0xF>(incl);     // lane 0: the identity
    __syncthreads();                                  // wave_tot may still be read by a previous call
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    T before = ident, all = ident;
#pragma unroll
    for (int w = 0; w < kThreads / kWave; ++w) {
        const T t = wave_tot[w];
        if (w < wave) before = op(before, t);
        all = op(all, t);
    }
    *total = all;
    return op(before, excl);
}

// ---- steps shared by the plans of one workgroup and the tiled one --------------------------

// next[p]: smallest q > p with P[q+1] - P[p] > t_blk, n_seq if there is none; P is read
// through `prefix_at`.  Every length is >= 1, so q - p <= t_blk bounds the search window.
template <typename PrefixAt>
__device__ __forceinline__ int32_t next_head(PrefixAt prefix_at, int32_t p, int32_t n_seq, int32_t t_blk)
{
    const int64_t limit = prefix_at(p) + t_blk;
    // first index e in (p+1, min(n_seq, p+1+t_blk)] with P[e] > limit; q = e - 1
    int64_t lo = (int64_t)p + 2, hi = min((int64_t)n_seq, (int64_t)p + 1 + (int64_t)t_blk) + 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (prefix_at((int32_t)mid) > limit) hi = mid; else lo = mid + 1;
    }
    return (lo <= n_seq) ? (int32_t)(lo - 1) : n_seq;
}

// One round of pointer jumping over the `count` positions from lo on that a jump tile holds in LDS (`from` and `to` are
// different arrays): a pointer that points behind them stays.  Four neighbouring
// positions per thread and step: their pointers come and go as one 16-byte LDS access, only the
// look-ups behind them are single words (24 LDS instructions per thread and round instead of
// 48), and all first accesses are made before the second ones, so that they are in flight together.  Positions from
// `count` on must hold pointers that point behind the tile.  Returns whether a pointer of the calling thread still
// pointed into the tile (when none of the workgroup does, further rounds change nothing).  The caller puts a barrier
// between rounds.
template <int NT>
__device__ __forceinline__ bool jump_round_tile(const int32_t* __restrict__ from, int32_t* __restrict__ to,
                                                int32_t lo, int32_t count)
{
    typedef int32_t int4v __attribute__((ext_vector_type(4)));
    constexpr int kQuads = kJumpItems / 4;        // quads of positions per thread
    int4v at[kQuads], then[kQuads];
#pragma unroll
    for (int u = 0; u < kQuads; ++u)
        at[u] = *reinterpret_cast<const int4v*>(from + 4 * ((int)threadIdx.x + u * NT));
    bool inside_any = false;
#pragma unroll
    for (int u = 0; u < kQuads; ++u) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool inside = at[u][j] - lo < count;
            inside_any |= inside;
            then[u][j] = inside ? from[at[u][j] - lo] : at[u][j];
        }
    }
#pragma unroll
    for (int u = 0; u < kQuads; ++u)
        *reinterpret_cast<int4v*>(to + 4 * ((int)threadIdx.x + u * NT)) = then[u];
    return inside_any;
}

// Pointers behind the tile for the positions of a jump tile that lie behind the last sequence.
template <int NT>
__device__ __forceinline__ void pad_tile(int32_t* tile, int32_t lo, int32_t count)
{
    for (int32_t k = count + (int32_t)threadIdx.x; k < jump_tile<NT>(); k += NT) tile[k] = lo + count;
}

// ---- kernels ------------------------------------------------------------------

// order[p], the shuffled lengths, and per workgroup of ITEMS * 256 positions: the sum of its lengths, and
// whether one of them is outside [1, t_blk].  One position per thread where that makes few sums: a
// walk through the order is a long chain of integer operations whose length differs from lane to
// lane, and eight in a row by few waves took 10 us at 10^4 sequences and 17 at 10^6.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void plan_order_kernel(
    const int32_t* __restrict__ lengths, int32_t n_seq, int32_t t_blk, OrderKey key,
    int32_t* __restrict__ order, int32_t* __restrict__ shuffled_len,
    int64_t* __restrict__ sums, int32_t* __restrict__ bads)
{
    const int64_t base = (int64_t)blockIdx.x * (kThreads * ITEMS) + (int64_t)threadIdx.x * ITEMS;
    int64_t sum = 0;
    int bad = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const int64_t p = base + j;
        if (p < n_seq) {
            const int32_t i = order_at((uint32_t)p, (uint32_t)n_seq, key);
            int32_t len = lengths[i];
            order[p] = i;
            // (a length out of range is refused in the end; as a 1 it keeps next[] rising until then)
            if ((len < 1) | (len > t_blk)) { bad = 1; len = 1; }
            shuffled_len[p] = len;
            sum += len;
        }
    }
    int64_t total;
    block_exclusive_scan<int64_t>(sum, 0, SumI64(), &total);
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) { sums[blockIdx.x] = total; bads[blockIdx.x] = bad; }
}

// P[p] = frames before shuffled position p; P[n_seq] = total.  Every tile adds up the sums
// in front of it by itself (`sums_per_tile` of the `n_sums` to a tile), and keeps whether a length of its own
// is out of range.
__global__ __launch_bounds__(kThreads) void plan_prefix_kernel(
    const int32_t* __restrict__ shuffled_len, int32_t n_seq, const int64_t* __restrict__ sums,
    const int32_t* __restrict__ bads, int32_t n_sums, int32_t sums_per_tile, int64_t* __restrict__ prefix,
    int32_t* __restrict__ tile_bad)
{
    const int32_t first_sum = (int32_t)blockIdx.x * sums_per_tile;
    if (wave_id() == 0) {
        const int32_t t = first_sum + lane_id();
        const uint64_t bad = __ballot(lane_id() < sums_per_tile && t < n_sums && bads[t] != 0);
        if (lane_id() == 0) tile_bad[blockIdx.x] = bad != 0;
    }
    int64_t mine = 0;
    constexpr int kBatch = 8;          // in flight together
    for (int32_t t0 = (int32_t)threadIdx.x; t0 < first_sum; t0 += kBatch * kThreads) {
        int64_t v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) v[u] = sums[min(t0 + u * kThreads, first_sum - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) mine += t0 + u * kThreads < first_sum ? v[u] : 0;
    }
    int64_t before;
    block_exclusive_scan<int64_t>(mine, 0, SumI64(), &before);

    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    int32_t len[kItems];
    int64_t sum = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        len[j] = (base + j < n_seq) ? shuffled_len[base + j] : 0;
        sum += len[j];
    }
    int64_t total;
    int64_t run = before + block_exclusive_scan<int64_t>(sum, 0, SumI64(), &total);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        if (base + j < n_seq) {
            prefix[base + j] = run;
            run += len[j];
            if (base + j == (int64_t)n_seq - 1) prefix[n_seq] = run;
        }
    }
}

// next[p] for every position, one thread each: a chain of dependent look-ups in P, of which the next kNextWindow
// positions (or t_blk of them, beyond which no block reaches) lie in LDS and hold the answer where blocks are of fewer
// sequences.  Where the first position's block is of more, so are the others', and P is searched where it lies.  (10^6
// documents 16 us without the window, 10 with it.  5 * 10^6 sequences: documents 58 and 44, 64 to a block at most 32 and 20;
// blocks of 50000, which it does not hold, 75 and 79, with the window fetched all the same 89; blocks of one 14, 15 and 40.)
constexpr int kNextWindow = 1024;
constexpr int kNextLeast = 16;                    // shorter blocks: four look-ups at most

__global__ __launch_bounds__(kThreads) void plan_next_kernel(const int64_t* __restrict__ prefix,
                                                             int32_t n_seq, int32_t t_blk,
                                                             int32_t* __restrict__ next)
{
    __shared__ int64_t s_prefix[kNextWindow + kThreads + 1];
    const int64_t first = (int64_t)blockIdx.x * kThreads, p = first + threadIdx.x;
    const int32_t held = (int32_t)min((int64_t)(min(kNextWindow, t_blk) + kThreads + 1), (int64_t)n_seq + 1 - first);    // from `first` on
    const int64_t own = prefix[min(p, (int64_t)n_seq)], limit = own + t_blk;
    // is an answer among them (next[] never falls), and worth bringing them here
    const bool within = t_blk >= kNextLeast && prefix[first + held - 1] - prefix[first] > t_blk;
    if (within) {
        s_prefix[threadIdx.x] = own;
        for (int32_t k = (int32_t)threadIdx.x + kThreads; k < held; k += kThreads) s_prefix[k] = prefix[first + k];
        __syncthreads();
    }
    if (p >= n_seq) return;
    // the first entry above the limit is next[p] + 1; P[p + 1] never is
    if (within && s_prefix[held - 1] > limit) {
        int32_t lo = (int32_t)threadIdx.x + 2, hi = (int32_t)min((int64_t)held - 1, (int64_t)threadIdx.x + 1 + t_blk);
        while (lo < hi) {
            const int32_t mid = (lo + hi) >> 1;
            if (s_prefix[mid] > limit) hi = mid; else lo = mid + 1;
        }
        next[p] = (int32_t)(first + lo - 1);
    } else {
        next[p] = next_head([&](int32_t q) { return prefix[q]; }, (int32_t)p, n_seq, t_blk);
    }
}

// Copy `count` ints between global memory and LDS, thread t taking elements t, t + NT, ...,
// eight loads in flight per thread.
template <int NT>
__device__ __forceinline__ void copy_tile(const int32_t* __restrict__ from, int32_t* __restrict__ to,
                                          int32_t count)
{
    constexpr int kBatch = 8;
    for (int32_t k0 = (int32_t)threadIdx.x; k0 < count; k0 += kBatch * NT) {
        int32_t v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) v[u] = k0 + u * NT < count ? from[k0 + u * NT] : 0;
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (k0 + u * NT < count) to[k0 + u * NT] = v[u];
    }
}

// For each position of a jump tile, where the orbit that passes through it leaves the tile:
// exit[p] = the first position at or behind the tile's end reached from p under next[].
template <int NT>
__global__ __launch_bounds__(NT) void plan_exit_kernel(const int32_t* __restrict__ next,
                                                                 int32_t n_seq,
                                                                 int32_t* __restrict__ exit_of)
{
    __shared__ __attribute__((aligned(16))) int32_t s_jump[2][jump_tile<NT>()];
    const int32_t lo = (int32_t)blockIdx.x * jump_tile<NT>();
    const int32_t count = min(jump_tile<NT>(), n_seq - lo);
    copy_tile<NT>(next + lo, s_jump[0], count);
    pad_tile<NT>(s_jump[0], lo, count);
    int cur = 0;
    for (int r = 0; r < kJumpRounds; ++r) {
        __syncthreads();
        const bool more = jump_round_tile<NT>(s_jump[cur], s_jump[cur ^ 1], lo, count);
        cur ^= 1;
        if (!__syncthreads_or(more ? 1 : 0)) break;       // every pointer has left the tile
    }
    __syncthreads();
    copy_tile<NT>(s_jump[cur], exit_of + lo, count);
}

// The same over 8 jump tiles at a time (16 of the smallest), for the positions where an orbit can enter such a
// group (next[] never falls, so those are at most next[the position in front of the group]; the
// first group is entered at 0).  A tile that looks for its entry then takes a hop per group and a
// few per tile instead of one per tile.
template <int NT> constexpr int kGroupTiles = NT == 128 ? 16 : 8;
constexpr int kGroupSpread = 64;                  // workgroups side by side over a group's entries (all its positions where blocks are
                                                  // longer: 300000 sequences 5.0 us with 16 of them, 3.0 like this; few entries 4.0 both)

template <int NT>
__global__ __launch_bounds__(kThreads) void plan_group_exit_kernel(const int32_t* __restrict__ next,
                                                                   const int32_t* __restrict__ exit_of, int32_t n_seq,
                                                                   int32_t* __restrict__ group_exit)
{
    const int32_t lo = (int32_t)blockIdx.x * (kGroupTiles<NT> * jump_tile<NT>());
    const int32_t end = min((int64_t)lo + kGroupTiles<NT> * jump_tile<NT>(), (int64_t)n_seq);
    const int32_t most = min(lo == 0 ? 0 : next[lo - 1], end - 1);
    for (int64_t p = (int64_t)lo + blockIdx.y * kThreads + threadIdx.x; p <= most; p += kGroupSpread * kThreads) {
        int32_t e = (int32_t)p;
        while (e < end) e = exit_of[e];           // exit[e] lies in a later tile than e: at most a hop per tile
        group_exit[p] = e;
    }
}

// Where the orbit of position 0 enters each jump tile (-1: it passes over the tile): one hop
// per tile along exit[].  One workgroup; thread 0 walks.
__global__ __launch_bounds__(kThreads) void plan_chain_kernel(const int32_t* __restrict__ exit_of,
                                                              int32_t n_seq, int32_t n_jump_tiles, int32_t tile,
                                                              int32_t* __restrict__ tile_entry)
{
    for (int32_t t = (int32_t)threadIdx.x; t < n_jump_tiles; t += kThreads) tile_entry[t] = -1;
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t e = 0;
        while (e < n_seq) {               // exit[e] lies in a later tile: at most n_jump_tiles hops
            tile_entry[e / tile] = e;
            e = exit_of[e];
        }
    }
}

// The heads inside a jump tile, from the position where the orbit enters it: tile_entry[tile],
// or, with `tile_entry` null, found here by following group_exit[] and exit[] from position 0 (one hop
// per group of tiles and per tile of the last group: quicker than a launch that does it for all;
// `group_exit` null: exit[] alone;
// `exit_of` null as well: there is one tile only, entered at position 0).  The heads found so far are kept as a list in
// orbit order, h_0 = the entry: round r jumps every position of the tile from next^(2^r) to
// next^(2^(r+1)) as the exit kernel does, and before that the first 2^r heads look up theirs,
// which are h_(2^r) .. h_(2^(r+1) - 1) where those still lie inside the tile (an orbit only
// moves forward, so they leave the tile in order and the list has no holes).  A round that
// adds no head ends the search.  Also, for each of its scan tiles (one per wave), the number of heads
// and the last head.
template <int NT>
__global__ __launch_bounds__(NT) void plan_mark_kernel(
    const int32_t* __restrict__ next, const int32_t* __restrict__ tile_entry,
    const int32_t* __restrict__ exit_of, const int32_t* __restrict__ group_exit, int32_t n_seq,
    uint8_t* __restrict__ mark, int32_t* __restrict__ tile_cnt, int32_t* __restrict__ tile_head)
{
    __shared__ __attribute__((aligned(16))) int32_t s_jump[2][jump_tile<NT>()];
    __shared__ __attribute__((aligned(16))) uint8_t s_mark[jump_tile<NT>()];
    __shared__ uint16_t s_heads[jump_tile<NT>()];           // positions inside the tile, relative to its first
    __shared__ int32_t s_n_heads;
    __shared__ HeadPair s_wave[NT / kWave];
    constexpr int kScans = jump_tile<NT>() / kTile;    // scan tiles in the jump tile
    static_assert(kScans * kWavesPerScanTile == NT / kWave, "the waves tile the scan tiles");
    static_assert(kJumpTile <= 65536, "a head's place inside the tile is kept in 16 bits");
    const int32_t lo = (int32_t)blockIdx.x * jump_tile<NT>();
    const int32_t count = min(jump_tile<NT>(), n_seq - lo);
    __shared__ int32_t s_entry;
    copy_tile<NT>(next + lo, s_jump[0], count);
    pad_tile<NT>(s_jump[0], lo, count);
    if (threadIdx.x == 0) {
        int32_t e = 0;
        if (tile_entry) {
            e = tile_entry[blockIdx.x];
        } else if (exit_of) {
            // group by group up to this tile's group, then tile by tile: every hop leads into a later one
            const int32_t group_lo = group_exit ? lo - lo % (kGroupTiles<NT> * jump_tile<NT>()) : 0;
            while (e < group_lo) e = group_exit[e];
            while (e < lo) e = exit_of[e];
            if (e >= lo + count) e = -1;              // the orbit passes over this tile
        }
        s_entry = e;
    }
    __syncthreads();
    const int32_t entry = s_entry;
    for (int32_t k = (int32_t)threadIdx.x; k < count; k += NT) s_mark[k] = (uint8_t)(lo + k == entry);
    if (threadIdx.x == 0) {
        s_heads[0] = (uint16_t)max(entry - lo, 0);
        s_n_heads = entry >= 0 ? 1 : 0;
    }
    __syncthreads();
    int32_t n_heads = entry >= 0 ? 1 : 0;            // the same in every thread
    if (n_heads > 0) {
        int cur = 0;
        for (int r = 0; r < kJumpRounds; ++r) {
            const int32_t* jump = s_jump[cur];
            for (int32_t i0 = (int32_t)threadIdx.x - lane_id(); i0 < n_heads; i0 += NT) {   // wave-uniform
                const int32_t i = i0 + lane_id();
                const int32_t to = i < n_heads ? jump[s_heads[i]] - lo : count;
                const bool inside = to < count;
                if (inside) {
                    s_heads[n_heads + i] = (uint16_t)to;
                    s_mark[to] = 1;
                }
                // the new heads of a round are the first so many of its candidates: the last lane
                // that found one speaks for its wave
                const unsigned long long found = __ballot(inside);
                if (found != 0ull && lane_id() == 63 - __builtin_clzll(found)) atomicMax(&s_n_heads, n_heads + i + 1);
            }
            const bool more = jump_round_tile<NT>(s_jump[cur], s_jump[cur ^ 1], lo, count);
            cur ^= 1;
            const bool any_inside = __syncthreads_or(more ? 1 : 0) != 0;
            const int32_t now = s_n_heads;
            const bool grew = now > n_heads;
            n_heads = now;
            if (!grew || !any_inside) break;
            __syncthreads();                          // everyone has read s_n_heads before the next round updates it
        }
    }
    __syncthreads();
    // thread t: positions 16 t .. 16 t + 15 (one 16-byte vector of marks)
    static_assert(kJumpItems == 16, "a thread's marks are one 16-byte vector");
    const int32_t base = (int32_t)threadIdx.x * kJumpItems;
    HeadPair v{0, -1};
    if (base + kJumpItems <= count) {
        union { vec16 q; uint8_t b[16]; } u;
        u.q = *reinterpret_cast<const vec16*>(s_mark + base);
        *reinterpret_cast<vec16*>(mark + lo + base) = u.q;
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (u.b[j]) { v.cnt += 1; v.head = lo + base + j; }
    } else {
        for (int j = 0; base + j < count; ++j) {
            const uint8_t m = s_mark[base + j];
            mark[lo + base + j] = m;
            if (m) { v.cnt += 1; v.head = lo + base + j; }
        }
    }
    // heads per scan tile: kWavesPerScanTile consecutive waves each
    const HeadPair upto = wave_scan(v, HeadOp(), LaneMove());
    if (lane_id() == kWave - 1) s_wave[wave_id()] = upto;
    __syncthreads();
    if (threadIdx.x < kScans) {
        const int32_t scan_tile = (int32_t)blockIdx.x * kScans + (int32_t)threadIdx.x;
        if ((int64_t)scan_tile * kTile < n_seq) {
            HeadPair sum{0, -1};
            for (int w = 0; w < kWavesPerScanTile; ++w)
                sum = HeadOp()(sum, s_wave[threadIdx.x * kWavesPerScanTile + w]);
            tile_cnt[scan_tile] = sum.cnt;
            tile_head[scan_tile] = sum.head;
        }
    }
}

// Block and offset of every sequence, first position of every block, totals.  Every tile
// adds up the head counts of the tiles before it by itself.  GATHER: what the sequences get is left in `at_position`, in
// the order of the positions, for plan_gather_kernel.  (Not asked at run time: 5 * 10^6 sequences, which are not gathered,
// took 198 us with the question between the loads, 184 without.)
template <bool GATHER>
__global__ __launch_bounds__(kThreads) void plan_assign_kernel(
    const uint8_t* __restrict__ mark, const int32_t* __restrict__ order,
    const int64_t* __restrict__ prefix, int32_t n_seq, const int32_t* __restrict__ tile_cnt,
    const int32_t* __restrict__ tile_head, const int32_t* __restrict__ tile_bad,
    int32_t* __restrict__ block_of_seq, int32_t* __restrict__ offset_of_seq, int2* __restrict__ at_position,
    int32_t* __restrict__ block_first, PlanResult* __restrict__ result)
{
    // heads in front of this tile and the last of them; the last tile also collects the
    // length checks of all tiles
    HeadPair mine{0, -1};
    int bad = 0;
    const bool last_tile = blockIdx.x == gridDim.x - 1;
    for (int32_t t = (int32_t)threadIdx.x; t < (int32_t)gridDim.x; t += kThreads) {
        if (t < (int32_t)blockIdx.x) mine = HeadOp()(mine, HeadPair{tile_cnt[t], tile_head[t]});
        if (last_tile) bad |= tile_bad[t];
    }
    HeadPair before;
    block_exclusive_scan<HeadPair>(mine, HeadPair{0, -1}, HeadOp(), &before);
    if (last_tile) bad = __syncthreads_or(bad);

    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kItems;
    uint8_t m[kItems];
    HeadPair v{0, -1};
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        m[j] = (base + j < n_seq) ? mark[base + j] : (uint8_t)0;
        if (m[j]) { v.cnt += 1; v.head = (int32_t)(base + j); }
    }
    HeadPair total;
    HeadPair run = block_exclusive_scan<HeadPair>(v, HeadPair{0, -1}, HeadOp(), &total);
    run = HeadOp()(before, run);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
        const int64_t p = base + j;
        if (p < n_seq) {
            if (m[j]) {
                run.cnt += 1;
                run.head = (int32_t)p;
                block_first[run.cnt - 1] = (int32_t)p;
            }
            const int32_t offset = (int32_t)(prefix[p] - prefix[run.head]);
            if (GATHER) {
                at_position[p] = make_int2(run.cnt - 1, offset);
            } else {
                const int32_t i = order[p];
                block_of_seq[i] = run.cnt - 1;
                offset_of_seq[i] = offset;
            }
            if (p == (int64_t)n_seq - 1) {
                block_first[run.cnt] = n_seq;
                result->num_blocks = run.cnt;
                result->total_frames = prefix[n_seq];
                result->bad_length = bad;
                result->pad_ = 0;
            }
        }
    }
}

// From the positions to the sequences: every sequence finds its position (the order is a permutation that runs backwards
// as well) and fetches what lies there.  Two tables written in order and one look-up of 8 bytes, instead of two
// stores of 4 bytes at random places, of which every compute die keeps lines of its own to write back: 10^6 sequences
// 32 us, 11 + 12 like this.  Where the permutation's domain is more than 2.25 times the sequences the walks get too long
// (300000: 97 us the call, 105 like this), and below 2^19 the launch costs what it saves.
__global__ __launch_bounds__(kThreads) void plan_gather_kernel(const int2* __restrict__ at_position, int32_t n_seq, OrderKey key,
                                                               int32_t* __restrict__ block_of_seq,
                                                               int32_t* __restrict__ offset_of_seq)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n_seq) return;
    const int2 v = at_position[position_of((uint32_t)i, (uint32_t)n_seq, key)];
    block_of_seq[i] = v.x;
    offset_of_seq[i] = v.y;
}

// The whole plan of at most 64 sequences in one wave, a position to a lane: prefix sums by DPP, next[] searched in the other
// lanes' sums, and the orbit as masks of 64 positions (round k: the positions that 2^k steps from a lane reach), of which
// lane 0 ends with the heads; block and offset are then a count and the highest bit below the lane.  No barrier and no LDS
// array: what bounds it is the chain of look-ups in other lanes, seven for next[] and two a round for the masks.  (In four
// waves with the pointers in LDS, as up to 256 sequences were planned before, a round costs a barrier and three trips
// there: 64 sequences 21.7 -> 17.0 us the call, of which the launch and the wait for it are 16.)
__global__ __launch_bounds__(kWave) void plan_wave_kernel(
    const int32_t* __restrict__ lengths, int32_t n_seq, int32_t t_blk, OrderKey key, int rounds,
    int32_t* __restrict__ order, int32_t* __restrict__ block_of_seq,
    int32_t* __restrict__ offset_of_seq, int32_t* __restrict__ block_first,
    PlanResult* __restrict__ result)
{
    const int p = (int)threadIdx.x;
    const bool mine = p < n_seq;
    int32_t i = 0, len = 0;
    if (key.half_bits > 0) {                          // (a domain of at most 64: every lane has one step of the walks)
        const int step = (int)(feistel((uint32_t)p & ((1u << 2 * key.half_bits) - 1u), key));
        i = step;
        while (__any(mine && i >= n_seq)) {
            const int on = __shfl(step, i, kWave);
            if (i >= n_seq) i = on;
        }
    }
    if (mine) {
        len = lengths[i];
        order[p] = i;
    }
    const bool bad = __any(mine && (len < 1 || len > t_blk));
    const int64_t upto = wave_scan((int64_t)len, SumI64(), LaneMove());
    const int64_t front = upto - len, limit = front + t_blk;

    // next[p]: the number of positions whose sum the limit covers (lanes behind the last one repeat the total)
    int next = 0;
#pragma unroll
    for (int step = kWave / 2; step > 0; step >>= 1)
        if (__shfl((long long)upto, next + step - 1, kWave) <= limit) next += step;
    if (__shfl((long long)upto, next, kWave) <= limit) ++next;
    next = min(max(next, p + 1), n_seq);              // (lengths that are refused: the sums need not rise)

    unsigned long long reach = mine ? 1ull << p : 0ull;
    for (int r = 0; r < rounds; ++r) {                // 2^rounds >= n_seq
        const int at = min(next, kWave - 1);
        const unsigned long long there = __shfl(reach, at, kWave);
        const int beyond = __shfl(next, at, kWave);
        if (next < n_seq) {
            reach |= there;
            next = beyond;
        }
    }
    const unsigned long long heads = __shfl(reach, 0, kWave);
    const unsigned long long own = heads & (~0ull >> (kWave - 1 - p));       // heads up to this position: bit 0 at least
    const int head = kWave - 1 - __clzll((long long)own), block = __popcll(own) - 1, blocks = __popcll(heads);
    const int64_t head_front = __shfl((long long)front, head, kWave);
    if (mine) {
        if (head == p) block_first[block] = p;
        block_of_seq[i] = block;
        offset_of_seq[i] = (int32_t)(front - head_front);
    }
    if (p == kWave - 1) {
        block_first[blocks] = n_seq;
        result->num_blocks = blocks;
        result->total_frames = upto;
        result->bad_length = bad;
        result->pad_ = 0;
    }
}

// The same with several waves, J chunks of 64 positions to each, for at most 1024 * J sequences: the walks of the order are
// look-ups in a table of the permutation's whole domain, a chunk's masks stop at its end, every wave then follows the
// orbit of position 0 from chunk to chunk (a look-up each), and lane c holds the heads of chunk c.
template <int J>
__global__ __launch_bounds__(kPlanWaves * kWave) void plan_waves_kernel(
    const int32_t* __restrict__ lengths, int32_t n_seq, int32_t t_blk, OrderKey key,
    int32_t* __restrict__ order, int32_t* __restrict__ block_of_seq,
    int32_t* __restrict__ offset_of_seq, int32_t* __restrict__ block_first,
    PlanResult* __restrict__ result)
{
    constexpr int kMost = J * kPlanWaves * kWave;
    __shared__ int64_t s_front[kMost + 1];
    __shared__ unsigned long long s_reach[kMost];
    __shared__ uint16_t s_exit[kMost];
    __shared__ uint16_t s_step[J == 1 ? 1024 : 4096];        // the smallest power of four that holds kMost
    __shared__ int64_t s_sums[kPlanWaves];
    const int lane = lane_id(), wave = wave_id(), threads = (int)blockDim.x;
    const int domain = 1 << 2 * key.half_bits;
    for (int x = (int)threadIdx.x; x < domain; x += threads) s_step[x] = (uint16_t)feistel((uint32_t)x, key);
    __syncthreads();

    int32_t i[J], len[J];
    int64_t front[J], sum = 0;
    int bad = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = (wave * J + j) * kWave + lane;
        i[j] = len[j] = 0;
        if (p < n_seq) {
            i[j] = s_step[p];
            while (i[j] >= n_seq) i[j] = s_step[i[j]];
            len[j] = lengths[i[j]];
            order[p] = i[j];
            bad |= (len[j] < 1) | (len[j] > t_blk);
        }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int64_t upto = wave_scan((int64_t)len[j], SumI64(), LaneMove());
        front[j] = sum + upto - len[j];
        sum += __shfl((long long)upto, kWave - 1, kWave);
    }
    if (lane == 0) s_sums[wave] = sum;
    bad = __syncthreads_or(bad);
    int64_t before = 0, total = 0;
    for (int w = 0; w < threads / kWave; ++w) {
        const int64_t t = s_sums[w];
        if (w < wave) before += t;
        total += t;
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = (wave * J + j) * kWave + lane;
        front[j] += before;
        if (p < n_seq) s_front[p] = front[j];
    }
    if (threadIdx.x == 0) s_front[n_seq] = total;
    __syncthreads();

    int next[J];
    unsigned long long reach[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = (wave * J + j) * kWave + lane;
        next[j] = n_seq;
        if (p < n_seq) next[j] = next_head([&](int32_t q) { return s_front[q]; }, p, n_seq, t_blk);
        reach[j] = 1ull << lane;
    }
    for (int r = 0; r < 6; ++r) {                     // 2^6 positions in a chunk
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int stop = min((wave * J + j + 1) * kWave, n_seq), at = next[j] & (kWave - 1);
            const unsigned long long there = __shfl(reach[j], at, kWave);
            const int beyond = __shfl(next[j], at, kWave);
            if (next[j] < stop) {
                reach[j] |= there;
                next[j] = beyond;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int p = (wave * J + j) * kWave + lane;
        if (p < n_seq) {
            s_exit[p] = (uint16_t)next[j];
            s_reach[p] = reach[j];
        }
    }
    __syncthreads();

    int entry = -1;
    for (int e = 0; e < n_seq; e = s_exit[e])
        if (e >> 6 == lane) entry = e;
    const unsigned long long heads = entry >= 0 ? s_reach[entry] : 0ull;
    const HeadPair here{(int32_t)__popcll(heads),
                        entry >= 0 ? lane * kWave + kWave - 1 - (int32_t)__clzll((long long)heads) : -1};
    const HeadPair upto = wave_scan(here, HeadOp(), LaneMove());
    const HeadPair front_of = LaneMove().template at<kDppWaveShr1, 0xF>(upto);
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int chunk = wave * J + j, p = chunk * kWave + lane;
        const unsigned long long own = __shfl(heads, chunk, kWave) & (~0ull >> (kWave - 1 - lane));
        const int earlier = __shfl(front_of.cnt, chunk, kWave), last = __shfl(front_of.head, chunk, kWave);
        if (p < n_seq) {
            const int block = earlier + __popcll(own) - 1;
            const int head = own ? chunk * kWave + kWave - 1 - __clzll((long long)own) : last;
            if (head == p) block_first[block] = p;
            block_of_seq[i[j]] = block;
            offset_of_seq[i[j]] = (int32_t)(front[j] - s_front[head]);
        }
    }
    if (threadIdx.x == kWave - 1) {
        block_first[upto.cnt] = n_seq;
        result->num_blocks = upto.cnt;
        result->total_frames = total;
        result->bad_length = bad;
        result->pad_ = 0;
    }
}

// The plan of up to kMidMost sequences behind plan_order_kernel: the steps of the tiled path in one workgroup of 16
// waves, with everything in LDS and a barrier where that has a kernel boundary.  Positions are kept in 16 bits and
// prefix sums in 32 (the host sees to it that they fit).  Thread t takes `per` (3 to 13) consecutive positions, so that a
// wave's positions are a jump tile of its own, whose rounds need no barrier:
//   next      by binary search, a thread's first position in the whole window, the others between that one and
//             the next thread's (next[] never falls)
//   exits     each wave jumps inside its positions until every pointer has left them (in place: a wave's look-ups of a
//             round are all made before its stores)
//   entries   one thread follows the exits, a hop per wave
//   heads     each wave from its entry, as plan_mark_kernel does
// What the sequences get is left in the order of the positions; plan_scatter_kernel brings it to them, which one
// compute unit would take longer for than the launch does.
// Bound by the latency of LDS.  Whole call, before and after: 10^4 sequences of heavy-tailed length in blocks of 3000, six launches -> three,
// 56 -> 40 us, nearly full blocks 74 -> 61; 3001 sequences, one to six to a block, 52 -> 34.
constexpr int kMidThreads = 1024;
constexpr int kMidWaves = kMidThreads / kWave;
constexpr int kMidPer = 13;                       // an odd number, so that the threads' places in LDS spread over the banks
constexpr int kMidMost = 12 * kMidThreads;        // about there the tiled path is as fast (nearly full blocks: 12288 sequences 68.2 us,
                                                  // 12289 by tiles 67.7; documents 57 and 62; 13312 is what the threads hold)

struct MidShared {
    alignas(16) int32_t prefix[kMidThreads * kMidPer + 4];     // lengths, then their prefix sums, in the end the offsets
    union {
        struct {
            uint16_t heads[kMidThreads * kMidPer];       // every wave's, in its positions' part
            uint16_t jump[kMidThreads * kMidPer];
        };
        int32_t blocks[kMidThreads * kMidPer];           // in the end
    };
    uint32_t mark[kMidThreads * kMidPer / 32];
    uint16_t first[kMidThreads + 1];              // next[] of every thread's first position
    uint16_t entry[kMidWaves];
    int32_t wave_sum[kMidWaves];
    HeadPair wave_heads[kMidWaves];
};
static_assert(kMidMost < 1 << 16 && sizeof(MidShared) <= 150 * 1024, "positions in 16 bits, one workgroup's LDS");

struct SumI32 { __device__ int32_t operator()(int32_t a, int32_t b) const { return a + b; } };
struct LaneMoveI32 {
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ int32_t at(int32_t v) const { return dpp_move<CTRL, ROW_MASK>(v, 0); }
};

// PER: positions per thread.
template <int PER>
__global__ __launch_bounds__(kMidThreads) void plan_mid_kernel(
    const int32_t* __restrict__ shuffled_len, int32_t n_seq, int32_t t_blk, const int32_t* __restrict__ bads,
    int32_t n_bads, int32_t* __restrict__ block_at, int32_t* __restrict__ offset_at, int32_t* __restrict__ block_first,
    PlanResult* __restrict__ result)
{
    __shared__ MidShared sh;
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
    constexpr int per = PER;
    const int base = tid * per, mine = max(min(per, n_seq - base), 0);
    const int wave_lo = min(wave * kWave * per, n_seq), wave_hi = min((wave + 1) * kWave * per, n_seq);

    int bad = 0;
    for (int k = tid; k < n_bads; k += kMidThreads) bad |= bads[k];
    int32_t x[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) x[j] = shuffled_len[min(tid + j * kMidThreads, n_seq - 1)];      // all asked for at once
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (tid + j * kMidThreads < n_seq) sh.prefix[tid + j * kMidThreads] = x[j];
    for (int w = tid; w < kMidThreads * kMidPer / 32; w += kMidThreads) sh.mark[w] = 0;
    bad = __syncthreads_or(bad);

    // prefix sums, in place
    int32_t sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        x[j] = j < mine ? sh.prefix[base + j] : 0;
        sum += x[j];
    }
    const int32_t upto = wave_scan(sum, SumI32(), LaneMoveI32());
    if (lane == kWave - 1) sh.wave_sum[wave] = upto;
    __syncthreads();
    int32_t run = upto - sum, total = 0;
#pragma unroll
    for (int w = 0; w < kMidWaves; ++w) {
        const int32_t t = sh.wave_sum[w];
        run += w < wave ? t : 0;
        total += t;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j < mine) sh.prefix[base + j] = run;
        run += x[j];
    }
    if (tid == 0) sh.prefix[n_seq] = total;
    __syncthreads();

    // next[]: the smallest q behind p with P[q + 1] - P[p] > t_blk, n_seq if there is none.  (Every length is 1 or more.)
    {
        int lo = base + 1, hi = (int)min((int64_t)n_seq, (int64_t)base + t_blk);
        const int32_t limit = mine > 0 ? sh.prefix[base] + t_blk : 0;
        while (mine > 0 && lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sh.prefix[mid + 1] > limit) hi = mid; else lo = mid + 1;
        }
        sh.first[tid] = (uint16_t)(mine > 0 ? lo : n_seq);
        if (tid == 0) sh.first[kMidThreads] = (uint16_t)n_seq;
    }
    __syncthreads();
    int32_t next[PER];
    {
        const int from = sh.first[tid], to = sh.first[tid + 1];
        int32_t high[PER], limit[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            next[j] = j < mine ? max(from, base + j + 1) : n_seq;
            high[j] = j < mine && j > 0 ? max(to, next[j]) : next[j];
            limit[j] = j < mine ? sh.prefix[base + j] + t_blk : 0;
        }
        for (;;) {
            bool more = false;
#pragma unroll
            for (int j = 1; j < PER; ++j) {
                const int mid = (next[j] + high[j]) >> 1;
                const bool open = next[j] < high[j];
                const bool beyond = sh.prefix[open ? mid + 1 : 0] > limit[j];
                high[j] = open && beyond ? mid : high[j];
                next[j] = open && !beyond ? mid + 1 : next[j];
                more |= next[j] < high[j];
            }
            if (__ballot(more) == 0) break;
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (j < mine) sh.jump[base + j] = (uint16_t)next[j];
        }
    }

    // one round of jumping over the wave's positions: x = the lane's pointers, what they are after it
    auto jump_round = [&]() {
        int32_t then[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j)
            then[j] = x[j] < wave_hi ? (int32_t)sh.jump[x[j]] : x[j];
        bool inside = false;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            x[j] = then[j];
            inside |= x[j] < wave_hi;
            if (j < mine) sh.jump[base + j] = (uint16_t)x[j];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        return __ballot(inside) != 0;
    };
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < PER; ++j) x[j] = next[j];
    // (pointers rise, so 2^10 hops leave the wave's 1024 positions)
    for (int r = 0; r < 10 && jump_round(); ++r) {}
    __syncthreads();
    if (tid == 0) {
        int e = 0;
        for (int w = 0; w < kMidWaves; ++w) {
            const bool in = e < min((w + 1) * kWave * per, n_seq);
            sh.entry[w] = (uint16_t)(in ? e : kMidMost);
            if (in) e = sh.jump[e];
        }
    }
    __syncthreads();

    // the wave's heads: the list so far, and twice as many with every round
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        x[j] = next[j];
        if (j < mine) sh.jump[base + j] = (uint16_t)x[j];
    }
    const int entry = __builtin_amdgcn_readfirstlane((int)sh.entry[wave]);
    uint16_t* heads = sh.heads + wave_lo;
    int n_heads = entry < kMidMost ? 1 : 0;
    if (n_heads > 0) {
        if (lane == 0) {
            heads[0] = (uint16_t)entry;
            atomicOr(&sh.mark[entry >> 5], 1u << (entry & 31));
        }
        for (int r = 0; r < 11; ++r) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int found = 0;
            for (int i0 = 0; i0 < n_heads; i0 += kWave) {
                const int i = i0 + lane;
                const int to = i < n_heads ? (int)sh.jump[heads[i]] : wave_hi;
                const bool inside = to < wave_hi;
                if (inside) {
                    heads[n_heads + i] = (uint16_t)to;
                    atomicOr(&sh.mark[to >> 5], 1u << (to & 31));
                }
                found += (int)__popcll(__ballot(inside));        // (the first so many of the list: an orbit leaves in order)
            }
            if (found == 0) break;
            n_heads += found;
            jump_round();
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();

    // blocks and offsets
    uint32_t marks = 0;
    if (mine > 0) {
        const int word = base >> 5, more = min(word + 1, kMidThreads * kMidPer / 32 - 1);
        marks = (uint32_t)(((uint64_t)sh.mark[more] << 32 | sh.mark[word]) >> (base & 31)) & ((1u << mine) - 1u);
    }
    HeadPair own{(int32_t)__popc(marks), marks ? base + 31 - __clz((int)marks) : -1};
    const HeadPair heads_upto = wave_scan(own, HeadOp(), LaneMove());
    HeadPair at = LaneMove().template at<kDppWaveShr1, 0xF>(heads_upto);
    if (lane == 0) at = HeadPair{0, -1};
    if (lane == kWave - 1) sh.wave_heads[wave] = heads_upto;
    __syncthreads();
    HeadPair all{0, -1}, before{0, -1};
#pragma unroll
    for (int w = 0; w < kMidWaves; ++w) {
        if (w == wave) before = all;
        all = HeadOp()(all, sh.wave_heads[w]);
    }
    at = HeadOp()(before, at);
    int32_t offset[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j < mine) {
            if ((marks >> j) & 1u) {
                at.cnt += 1;
                at.head = base + j;
                block_first[at.cnt - 1] = base + j;
            }
            x[j] = at.cnt - 1;
            offset[j] = sh.prefix[base + j] - sh.prefix[at.head];
        }
    }
    __syncthreads();                                     // the prefix sums and pointers have been read
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j < mine) {
            sh.blocks[base + j] = x[j];
            sh.prefix[base + j] = offset[j];
        }
    }
    __syncthreads();
    for (int p = tid; p < n_seq; p += kMidThreads) {
        block_at[p] = sh.blocks[p];
        offset_at[p] = sh.prefix[p];
    }
    if (tid == 0) {
        block_first[all.cnt] = n_seq;
        result->num_blocks = all.cnt;
        result->total_frames = total;
        result->bad_length = bad;
        result->pad_ = 0;
    }
}

// What is known per position, to the sequences.
__global__ __launch_bounds__(kThreads) void plan_scatter_kernel(
    const int32_t* __restrict__ order, const int32_t* __restrict__ block_at, const int32_t* __restrict__ offset_at,
    int32_t n_seq, int32_t* __restrict__ block_of_seq, int32_t* __restrict__ offset_of_seq)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= n_seq) return;
    const int32_t i = order[p];
    block_of_seq[i] = block_at[p];
    offset_of_seq[i] = offset_at[p];
}

// Workspace layout (every part 16-byte aligned).
struct PlanLayout {
    size_t result, shuffled_len, prefix, next, exit_of, mark, tile_cnt, tile_head, tile_entry, tile_bad, bytes;
    size_t sums, bads;         // of the order kernel's workgroups: in the bytes of exit_of, which is written after their use
    int32_t n_tiles;           // scan tiles
    int32_t sums_per_tile;     // workgroups of the order kernel to a scan tile
    int32_t n_sums;
    int32_t n_jump_tiles, jump_threads;
};

static PlanLayout plan_layout(int64_t n_seq)
{
    PlanLayout l{};
    const size_t n = (size_t)(n_seq > 0 ? n_seq : 0);
    l.n_tiles = (int32_t)ceil_div((int64_t)n, kTile);
    l.jump_threads = (int64_t)n <= kJumpTile ? 512 : (int64_t)n <= kSmallTilesUpTo ? 128 : (int64_t)n <= kMidTilesUpTo ? 256 : 512;
    l.n_jump_tiles = (int32_t)ceil_div((int64_t)n, l.jump_threads * kJumpItems);
    l.sums_per_tile = (int64_t)n <= kSingleItems ? kItems : 1;
    l.n_sums = (int32_t)ceil_div((int64_t)n, kTile / l.sums_per_tile);
    size_t off = 0;
    auto take = [&off](size_t bytes) { const size_t at = off; off += round_up(bytes, 16); return at; };
    l.result = take(sizeof(PlanResult));
    l.shuffled_len = take(n * 4);
    l.prefix = take((n + 1) * 8);
    l.next = take(n * 4);
    l.exit_of = take(n * 4);           // (right behind `next`: the two are one table of 8 bytes per position in the end)
    l.mark = take(n);
    l.tile_cnt = take((size_t)l.n_tiles * 4);
    l.tile_head = take((size_t)l.n_tiles * 4);
    l.tile_entry = take((size_t)ceil_div((int64_t)n, kJumpTile) * 4);      // (only the largest tiles are so many that it is used)
    l.tile_bad = take((size_t)l.n_tiles * 4);
    l.bytes = off;
    // (12 bytes per 256 positions and a rest, beyond 2048 positions of 4 bytes: they fit)
    l.sums = l.exit_of;
    l.bads = l.exit_of + (size_t)l.n_sums * 8;
    return l;
}

}  // namespace bload

using namespace bload;

extern "C" size_t bload_plan_workspace_bytes(int64_t n_seq)
{
    if (n_seq < 0 || n_seq > BLOAD_MAX_SEQ) return 0;
    return plan_layout(n_seq).bytes;
}

extern "C" bload_status bload_plan(const int32_t* d_lengths, int64_t n_seq, int32_t t_blk,
                                   uint64_t seed, int32_t* d_order, int32_t* d_block_of_seq,
                                   int32_t* d_offset_of_seq, int32_t* d_block_first,
                                   int64_t* h_num_blocks, int64_t* h_total_frames,
                                   void* d_workspace, size_t workspace_bytes, void* hip_stream)
{
    if (!h_num_blocks || !h_total_frames || n_seq < 0 || t_blk < 1) return BLOAD_EINVAL;
    *h_num_blocks = 0;
    *h_total_frames = 0;
    if (n_seq > BLOAD_MAX_SEQ) return BLOAD_EOVERFLOW;
    if (n_seq == 0) return BLOAD_OK;
    if (!d_lengths || !d_order || !d_block_of_seq || !d_offset_of_seq || !d_block_first ||
        !d_workspace)
        return BLOAD_EINVAL;
    if (!aligned_to(d_lengths, 4) || !aligned_to(d_order, 4) || !aligned_to(d_block_of_seq, 4) ||
        !aligned_to(d_offset_of_seq, 4) || !aligned_to(d_block_first, 4) ||
        !aligned_to(d_workspace, 16))
        return BLOAD_EALIGN;
    const PlanLayout l = plan_layout(n_seq);
    if (workspace_bytes < l.bytes) return BLOAD_EWORKSPACE;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    // the numbers the host waits for go straight into pinned host memory where there is some,
    // else into the workspace, from where they are copied back
    static_assert(sizeof(PlanResult) <= 64, "the pinned buffer holds 64 bytes");
    PlanResult* pinned = static_cast<PlanResult*>(host_result_buffer());
    PlanResult* result = pinned ? pinned : reinterpret_cast<PlanResult*>(ws + l.result);
    int32_t* shuffled_len = reinterpret_cast<int32_t*>(ws + l.shuffled_len);
    int64_t* prefix = reinterpret_cast<int64_t*>(ws + l.prefix);
    int32_t* next = reinterpret_cast<int32_t*>(ws + l.next);
    int32_t* exit_of = reinterpret_cast<int32_t*>(ws + l.exit_of);
    uint8_t* mark = ws + l.mark;
    int64_t* sum_of = reinterpret_cast<int64_t*>(ws + l.sums);
    int32_t* bad_of = reinterpret_cast<int32_t*>(ws + l.bads);
    int32_t* tile_cnt = reinterpret_cast<int32_t*>(ws + l.tile_cnt);
    int32_t* tile_head = reinterpret_cast<int32_t*>(ws + l.tile_head);
    int32_t* tile_entry = reinterpret_cast<int32_t*>(ws + l.tile_entry);
    int32_t* tile_bad = reinterpret_cast<int32_t*>(ws + l.tile_bad);

    const int32_t n = (int32_t)n_seq;
    const OrderKey key = make_order_key(n_seq, seed);
    const dim3 block(kThreads);
    const dim3 tiles((uint32_t)l.n_tiles), jump_tiles((uint32_t)l.n_jump_tiles);

    // (the workgroup of 16 waves keeps its prefix sums in 32 bits)
    const bool mid_fits = n_seq <= kMidMost && n_seq * (int64_t)t_blk <= INT32_MAX - t_blk;
    if (n_seq <= kWave) {
        // 2^rounds >= n_seq >= number of heads
        int rounds = 0;
        while (((int64_t)1 << rounds) < n_seq) ++rounds;
        hipLaunchKernelGGL(plan_wave_kernel, dim3(1), dim3(kWave), 0, stream, d_lengths, n, t_blk, key, rounds, d_order,
                           d_block_of_seq, d_offset_of_seq, d_block_first, result);
    } else if (n_seq <= kWavesMost) {
        const dim3 waves((uint32_t)std::min<int64_t>((int64_t)1 << 2 * key.half_bits, kPlanWaves * kWave));
        const auto kernel = n_seq <= kPlanWaves * kWave ? plan_waves_kernel<1> : plan_waves_kernel<2>;
        hipLaunchKernelGGL(kernel, dim3(1), waves, 0, stream, d_lengths, n, t_blk, key, d_order, d_block_of_seq,
                           d_offset_of_seq, d_block_first, result);
    } else if (mid_fits) {
        const dim3 sums((uint32_t)l.n_sums), per_item((uint32_t)ceil_div(n_seq, kThreads));
        int32_t* block_at = next;
        int32_t* offset_at = reinterpret_cast<int32_t*>(prefix);
        hipLaunchKernelGGL(plan_order_kernel<1>, sums, block, 0, stream, d_lengths, n, t_blk, key, d_order,
                           shuffled_len, sum_of, bad_of);
        const int per = (int)ceil_div(n_seq, kMidThreads) | 1;
        const auto mid = per == 3 ? plan_mid_kernel<3> : per == 5 ? plan_mid_kernel<5> : per == 7 ? plan_mid_kernel<7>
                         : per == 9 ? plan_mid_kernel<9> : per == 11 ? plan_mid_kernel<11> : plan_mid_kernel<13>;
        static_assert(kMidPer == 13 && kMidMost <= kMidThreads * kMidPer, "3 to 13 positions per thread");
        hipLaunchKernelGGL(mid, dim3(1), dim3(kMidThreads), 0, stream, shuffled_len, n, t_blk, bad_of, l.n_sums, block_at,
                           offset_at, d_block_first, result);
        hipLaunchKernelGGL(plan_scatter_kernel, per_item, block, 0, stream, d_order, block_at, offset_at, n, d_block_of_seq,
                           d_offset_of_seq);
    } else {
        const dim3 sums((uint32_t)l.n_sums);
        if (l.sums_per_tile == 1)
            hipLaunchKernelGGL(plan_order_kernel<kItems>, sums, block, 0, stream, d_lengths, n, t_blk, key, d_order,
                               shuffled_len, sum_of, bad_of);
        else
            hipLaunchKernelGGL(plan_order_kernel<1>, sums, block, 0, stream, d_lengths, n, t_blk, key, d_order,
                               shuffled_len, sum_of, bad_of);
        hipLaunchKernelGGL(plan_prefix_kernel, tiles, block, 0, stream, shuffled_len, n, sum_of, bad_of, l.n_sums,
                           l.sums_per_tile, prefix, tile_bad);
        hipLaunchKernelGGL(plan_next_kernel, dim3((uint32_t)ceil_div(n_seq, kThreads)), block, 0, stream,
                           prefix, n, t_blk, next);
        // where the orbit of position 0 enters each jump tile: a single tile it enters at 0; up to
        // kWalkTiles tiles every tile finds its own entry; beyond, one thread finds them all
        const bool one_jump_tile = l.n_jump_tiles == 1, tiles_walk = l.n_jump_tiles <= kWalkTiles;
        const bool grouped = tiles_walk && l.n_jump_tiles >= kGroupFrom;
        int32_t* group_exit = shuffled_len;       // (the shuffled lengths are not needed any more)
        auto jump = [&](auto threads) {
            constexpr int NT = decltype(threads)::value;
            if (!one_jump_tile)
                hipLaunchKernelGGL(plan_exit_kernel<NT>, jump_tiles, dim3(NT), 0, stream, next, n, exit_of);
            if (grouped)
                hipLaunchKernelGGL(plan_group_exit_kernel<NT>, dim3((uint32_t)ceil_div(l.n_jump_tiles, kGroupTiles<NT>), kGroupSpread),
                                   block, 0, stream, next, exit_of, n, group_exit);
            if (!tiles_walk)
                hipLaunchKernelGGL(plan_chain_kernel, dim3(1), block, 0, stream, exit_of, n, l.n_jump_tiles, jump_tile<NT>(),
                                   tile_entry);
            hipLaunchKernelGGL(plan_mark_kernel<NT>, jump_tiles, dim3(NT), 0, stream, next, tiles_walk ? nullptr : tile_entry,
                               one_jump_tile ? nullptr : exit_of, grouped ? group_exit : nullptr, n, mark, tile_cnt, tile_head);
        };
        if (l.jump_threads == 128) jump(std::integral_constant<int, 128>());
        else if (l.jump_threads == 256) jump(std::integral_constant<int, 256>());
        else jump(std::integral_constant<int, 512>());
        // (`next` and `exit_of` behind it, 8 bytes per position, are not needed any more)
        const bool gathers = n_seq >= kGatherFrom && ((int64_t)1 << (2 * key.half_bits)) * 4 <= n_seq * 9;
        int2* at_position = reinterpret_cast<int2*>(next);
        const auto assign = gathers ? plan_assign_kernel<true> : plan_assign_kernel<false>;
        hipLaunchKernelGGL(assign, tiles, block, 0, stream, mark, d_order, prefix, n,
                           tile_cnt, tile_head, tile_bad, d_block_of_seq, d_offset_of_seq, at_position,
                           d_block_first, result);
        if (gathers)
            hipLaunchKernelGGL(plan_gather_kernel, dim3((uint32_t)ceil_div(n_seq, kThreads)), block, 0, stream, at_position, n,
                               key, d_block_of_seq, d_offset_of_seq);
    }
    if (launch_status() != BLOAD_OK) return BLOAD_EHIP;

    PlanResult host{};
    if (!pinned && !hip_ok(hipMemcpyAsync(&host, result, sizeof(host), hipMemcpyDeviceToHost, stream)))
        return BLOAD_EHIP;
    if (!hip_ok(hipStreamSynchronize(stream))) return BLOAD_EHIP;
    if (pinned) host = *pinned;
    if (host.bad_length) return BLOAD_ELENGTH;
    *h_num_blocks = host.num_blocks;
    *h_total_frames = host.total_frames;
    return BLOAD_OK;
}
