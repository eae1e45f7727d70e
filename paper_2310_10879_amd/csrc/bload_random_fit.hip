// bload_plan_random_fit: the block builder with the paper's own sampler (BLoad,
// caption of the pseudocode figure: a random entry of the length dictionary L_dict
// among those no longer than the frames remaining in the open block).
//
// The draws are a chain: what fits, and how many of each length are left, depends on
// every earlier draw.  So the chain itself runs on ONE wavefront and is kept as short
// as the hardware allows, and everything around it is parallel:
//   rf_order_kernel    seeded position p -> sequence, its length, checks, frame total
//   rf_count_kernel, rf_offsets_kernel, rf_scatter_kernel
//                      L_dict: where each length's list starts, the lists themselves in
//                      seeded order, and the running counts the chain starts from; the
//                      seeded positions are cut into chunks, one workgroup each, that
//                      count their lengths, learn where their part of every list
//                      begins, and fill it in order
//   rf_draw_kernel     the chain: per placement only (length, rank in its list, block,
//                      offset) - no global load on the chain
//   rf_assign_kernel   placement p -> sequence, and the per-sequence tables
//
// Counts per length live as two levels of running sums: inside groups of 64 lengths
// (rows in LDS) and over the groups (two registers per lane).  "How many fit" is one
// LDS read plus one lane read; "which length holds the k-th" is two compare-and-vote
// steps; taking a sequence out lowers the sums behind it.
#include "bload_common.hpp"
#include "bload_order.hpp"

#include <algorithm>

namespace bload {

constexpr int kRfMaxT = BLOAD_RANDOM_FIT_MAX_T_BLK;   // lengths 1..kRfMaxT
constexpr int kRfGroups = kRfMaxT / kWave;            // groups of 64 lengths
constexpr int kRfStride = kWave + 1;                  // a group's row: 65 running sums
static_assert(kRfGroups == 2 * kWave, "two group sums per lane");

// One placement, as the chain leaves it: its block is the one whose range of placements holds it.
struct RfPick {
    int32_t where;        // length - 1 << 16 | what was free in the block - 1
    int32_t left;         // how many of that length were left: it takes the last of them
};
static_assert(kRfMaxT <= 1 << 15, "lengths and offsets, counted from 0, take 15 bits");

__global__ void rf_clear_kernel(PlanResult* result)
{
    result->num_blocks = 0;
    result->total_frames = 0;
    result->bad_length = 0;
    result->pad_ = 0;
}

// seeded[p], the length found there (0 where it is outside [1, t_blk]), the frame total.
__global__ __launch_bounds__(kThreads) void rf_order_kernel(
    const int32_t* __restrict__ lengths, int32_t n_seq, int32_t t_blk, OrderKey key,
    int32_t* __restrict__ seeded, int32_t* __restrict__ seeded_len, PlanResult* __restrict__ result)
{
    __shared__ unsigned long long s_sum;
    if (threadIdx.x == 0) s_sum = 0;
    __syncthreads();
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p < n_seq) {
        const int32_t i = order_at((uint32_t)p, (uint32_t)n_seq, key);
        const int32_t len = lengths[i];
        const bool bad = (len < 1) | (len > t_blk);
        seeded[p] = i;
        seeded_len[p] = bad ? 0 : len;
        if (bad) atomicOr(&result->bad_length, 1);
        else atomicAdd(&s_sum, (unsigned long long)len);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_sum)
        atomicAdd(reinterpret_cast<unsigned long long*>(&result->total_frames), s_sum);
}

// L_dict.  first[e] = start of the list of length e+1 in entry[]; entry[first[e] + r] =
// the r-th sequence of that length in seeded order.  For the chain: within[g * 65 + j] =
// sequences of the lengths g*64+1 .. g*64+j (j = 0..64, lengths taken in groups of 64) and
// group_before[g] = sequences shorter than group g's lengths (the total for g past the end).
//
// The lists must come out in seeded order.  The seeded positions are cut into chunks of
// `per_chunk` consecutive positions (a multiple of 256).  Step 1, one workgroup per chunk:
// how many sequences of each length the chunk holds.
constexpr int kRfMaxChunks = 128;

__global__ __launch_bounds__(kThreads) void rf_count_kernel(const int32_t* __restrict__ seeded_len,
                                                            int32_t n_seq, int32_t t_blk, int32_t per_chunk,
                                                            int32_t* __restrict__ chunk_count)
{
    __shared__ int32_t s_fill[kRfMaxT];
    const int tid = (int)threadIdx.x;
    const int lengths_kept = ((t_blk + kWave - 1) / kWave) * kWave;
    for (int e = tid; e < lengths_kept; e += kThreads) s_fill[e] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * per_chunk;
    const int64_t hi = min((int64_t)n_seq, lo + per_chunk);
    for (int64_t p = lo + tid; p < hi; p += kThreads) {
        const int32_t len = seeded_len[p];
        if (len) atomicAdd(&s_fill[len - 1], 1);
    }
    __syncthreads();
    for (int e = tid; e < lengths_kept; e += kThreads) chunk_count[(int64_t)blockIdx.x * kRfMaxT + e] = s_fill[e];
}

// Step 2, one workgroup of 16 waves: the totals per length, from them first[], within[] and
// group_before[], and in place of every chunk's counts the place where its part of each list
// begins.  A wave takes a group of 64 lengths at a time, a lane each (one thread per group walking its
// lengths took 43 us at 3000 lengths, this 9).
constexpr int kRfOffsetThreads = 1024;
constexpr int kRfOffsetRounds = kRfGroups / (kRfOffsetThreads / kWave);

struct RfSum { __device__ int32_t operator()(int32_t a, int32_t b) const { return a + b; } };
struct RfMove {
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ int32_t at(int32_t v) const { return dpp_move<CTRL, ROW_MASK>(v, 0); }
};

__global__ __launch_bounds__(kRfOffsetThreads) void rf_offsets_kernel(
    int32_t n_chunks, int32_t t_blk, int32_t* __restrict__ chunk_count, int32_t* __restrict__ first,
    int32_t* __restrict__ within, int32_t* __restrict__ group_before)
{
    __shared__ int32_t s_group[kRfGroups];
    const int lane = lane_id(), wave = wave_id();
    constexpr int kWaves = kRfOffsetThreads / kWave;
    const int groups = (t_blk + kWave - 1) / kWave;
    int32_t mine[kRfOffsetRounds], upto[kRfOffsetRounds];      // sequences of the lane's length; up to it in its group
#pragma unroll
    for (int r = 0; r < kRfOffsetRounds; ++r) {
        const int g = wave + r * kWaves, e = g * kWave + lane;
        mine[r] = upto[r] = 0;
        if (g < groups) {
            int32_t total = 0;
#pragma unroll 8
            for (int c = 0; c < n_chunks; ++c) total += chunk_count[(int64_t)c * kRfMaxT + e];
            mine[r] = total;
            upto[r] = wave_scan(total, RfSum(), RfMove());
            within[g * kRfStride + lane + 1] = upto[r];
            if (lane == 0) within[g * kRfStride] = 0;
        }
        if (lane == kWave - 1) s_group[g] = upto[r];
    }
    __syncthreads();
    // sequences in the groups before each one: every wave adds them up for itself
    static_assert(kRfGroups == 2 * kWave, "two groups per lane");
    const int32_t lo = s_group[lane], hi = s_group[kWave + lane];
    const int32_t lo_upto = wave_scan(lo, RfSum(), RfMove()), hi_upto = wave_scan(hi, RfSum(), RfMove());
    const int32_t lo_all = __builtin_amdgcn_readlane(lo_upto, kWave - 1);
    if (wave == 0) {
        group_before[lane] = lo_upto - lo;
        group_before[kWave + lane] = lo_all + hi_upto - hi;
    }
#pragma unroll
    for (int r = 0; r < kRfOffsetRounds; ++r) {
        const int g = wave + r * kWaves, e = g * kWave + lane;
        if (g >= groups) break;
        const int32_t before = g < kWave ? __shfl(lo_upto - lo, g & 63, kWave) : lo_all + __shfl(hi_upto - hi, g & 63, kWave);
        int32_t at = before + upto[r] - mine[r];
        if (e < t_blk) first[e] = at;
        // a chunk's part of a list begins behind the parts of the chunks before it
        for (int c0 = 0; c0 < n_chunks; c0 += 8) {
            int32_t count[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) count[c] = c0 + c < n_chunks ? chunk_count[(int64_t)(c0 + c) * kRfMaxT + e] : 0;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if (c0 + c < n_chunks) chunk_count[(int64_t)(c0 + c) * kRfMaxT + e] = at;
                at += count[c];
            }
        }
    }
}

// Step 3, one workgroup per chunk: its sequences into their lists, in seeded order: tile by
// tile of 256 positions.  The lanes of a wave that hold the same length find each other by votes on its bits, and the
// waves take their places in the lists one after another.  (Each thread ranking itself among the keys in front, read
// from LDS, took 7 us a tile: 29 us at 10^4 sequences.)
__global__ __launch_bounds__(kThreads) void rf_scatter_kernel(
    const int32_t* __restrict__ seeded, const int32_t* __restrict__ seeded_len, int32_t n_seq,
    int32_t t_blk, int32_t per_chunk, const int32_t* __restrict__ chunk_start, int32_t* __restrict__ entry)
{
    __shared__ int32_t s_fill[kRfMaxT];         // next free place of every list, for this chunk
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = wave_id();
    const int lengths_kept = ((t_blk + kWave - 1) / kWave) * kWave;
    const int bits = 32 - __clz(t_blk);
    for (int e = tid; e < lengths_kept; e += kThreads) s_fill[e] = chunk_start[(int64_t)blockIdx.x * kRfMaxT + e];
    const int64_t lo = (int64_t)blockIdx.x * per_chunk;
    const int64_t hi = min((int64_t)n_seq, lo + per_chunk);
    for (int64_t tile = lo; tile < hi; tile += kThreads) {
        const int64_t p = tile + tid;
        const int32_t len = p < hi ? seeded_len[p] : 0;
        const int32_t sequence = p < hi ? seeded[p] : 0;
        uint64_t same = ~0ull;                   // the lanes with this length
        for (int b = 0; b < bits; ++b) {
            const bool one = (len >> b) & 1;
            const uint64_t vote = __ballot(one);
            same &= one ? vote : ~vote;
        }
        const int rank = (int)__popcll(same & ((1ull << lane) - 1ull));
        for (int w = 0; w < kThreads / kWave; ++w) {
            __syncthreads();
            if (wave == w && len) {
                const int32_t at = s_fill[len - 1] + rank;
                if ((same >> lane) == 1ull) s_fill[len - 1] = at + 1;        // the last of them
                entry[at] = sequence;
            }
        }
    }
}

// The chain of draws, on one wavefront, everything wave-uniform except: the running sums of a
// group's lengths (a row: lane j holds how many of the group's first j + 1 lengths are left),
// the sums over the groups (lane j holds groups j and 64 + j), the next 64 random numbers and the
// last 64 placements.
//   how many fit    = groups below the room's group (a lane read) + the row entry of the room
//   the group of k  = the last group with "shorter sequences" <= k (compare, vote, find last)
//   the length of k = the first lane of the group's row above k's place in it
//   taking it out   = one less in the lanes from there on and in the groups behind
// A single wavefront issues a dependent instruction every seven cycles or so (3 ns), whatever it is;
// so what counts is the number of instructions of a draw (75 -> 60: 273 -> 217 ns a draw at lengths
// up to 3000): placements are kept in registers, a lane each, and stored 64 at a time without their
// block (rf_assign_kernel finds it).  REGISTERS (t_blk <= 2048): the rows lie in 32 vector registers,
// picked with an indexed register move, which saves the two waits for LDS of a draw (256 -> 233 ns);
// more than 32 registers cannot be indexed as one, and choosing between two sets costs more
// instructions than the waits (83 in all, 270 ns).  GROUPS_HI: more than 64 groups (t_blk > 4096).
constexpr int kRfRegisterRows = 32;
typedef int32_t rf_rows __attribute__((ext_vector_type(kRfRegisterRows)));

template <bool REGISTERS, bool GROUPS_HI>
__global__ __launch_bounds__(kWave) void rf_draw_kernel(
    const int32_t* __restrict__ within, const int32_t* __restrict__ group_before, int32_t n_seq,
    int32_t t_blk, uint64_t seed, RfPick* __restrict__ pick, int32_t* __restrict__ block_first,
    PlanResult* __restrict__ result, PlanResult* __restrict__ host_result)
{
    __shared__ int32_t s_rows[REGISTERS ? 1 : (GROUPS_HI ? kRfGroups : kWave) * kWave];
    const int lane = (int)threadIdx.x;
    const int groups = (t_blk + kWave - 1) / kWave;
    rf_rows rows = {};
    if (REGISTERS) {
#pragma unroll
        for (int k = 0; k < kRfRegisterRows; ++k)        // (behind the last group never picked; they repeat it)
            rows[k] = within[min(k, groups - 1) * kRfStride + lane + 1];
    } else {
        for (int g = 0; g < groups; ++g) s_rows[g * kWave + lane] = within[g * kRfStride + lane + 1];
    }
    int32_t before_lo = group_before[lane];
    int32_t before_hi = GROUPS_HI ? group_before[kWave + lane] : 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int32_t bad = result->bad_length;
    if (bad) {
        if (lane == 0 && host_result) host_result->bad_length = bad;
        return;
    }

    // Every block takes at least one sequence (all of them fit an empty block), every placement
    // uses up room, and at most n_seq blocks are begun: the loop ends whatever the sums hold.
    int32_t placed = 0, blocks = 0;
    int32_t last = -1;                                   // the longest length that fits, counted from 0; -1: none
    uint32_t u_lo = 0, u_hi = 0;
    int32_t kept_where = 0, kept_left = 0;               // placement (placed & ~63) + lane
    while (placed < n_seq && blocks < n_seq && last >= -1) {
      if (lane == 0) block_first[blocks] = placed;
      blocks += 1;
      last = t_blk - 1;
      while (last >= 0) {
        const int g_room = last >> 6;
        int32_t fit = REGISTERS ? __builtin_amdgcn_readlane(rows[g_room & (kRfRegisterRows - 1)], last & 63)
                                : __builtin_amdgcn_readfirstlane(s_rows[last]);
        if (GROUPS_HI && g_room >= kWave) fit += __builtin_amdgcn_readlane(before_hi, g_room - kWave);
        else fit += __builtin_amdgcn_readlane(before_lo, g_room);
        if (fit <= 0) break;

        const int turn = placed & (kWave - 1);
        if (turn == 0) {                                 // the next 64 random numbers, one per lane
            const uint64_t u = splitmix64_at(seed, (uint64_t)(6 + placed + lane));
            u_lo = (uint32_t)u;
            u_hi = (uint32_t)(u >> 32);
            if (placed > 0) pick[placed - kWave + lane] = RfPick{kept_where, kept_left};
        }
        const uint64_t u = ((uint64_t)__builtin_amdgcn_readlane(u_hi, turn) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane(u_lo, turn);
        const int32_t k = (int32_t)__umul64hi(u, (uint64_t)(uint32_t)fit);        // uniform in [0, fit)

        int g = 63 - __builtin_clzll(__ballot(before_lo <= k));                   // lane 0 holds 0 <= k
        int32_t in_row = k - __builtin_amdgcn_readlane(before_lo, g);
        if (GROUPS_HI) {
            const uint64_t vote_hi = __ballot(before_hi <= k);
            if (vote_hi) {
                const int j = 63 - __builtin_clzll(vote_hi);
                g = kWave + j;
                in_row = k - __builtin_amdgcn_readlane(before_hi, j);
            }
        }
        const int32_t upto = REGISTERS ? rows[g & (kRfRegisterRows - 1)] : s_rows[g * kWave + lane];
        const bool above = upto > in_row;                // running sums do not fall: the lanes from k's length on
        const int j = __builtin_ctzll(__ballot(above));
        // (two lane reads: a difference in the vector unit, folded into the move, comes out negated)
        const int32_t shorter = dpp_move<kDppWaveShr1>(upto, 0);
        const int32_t left = __builtin_amdgcn_readlane(upto, j) - __builtin_amdgcn_readlane(shorter, j);

        // the last remaining sequence of that length leaves
        if (REGISTERS) rows[g & (kRfRegisterRows - 1)] = upto - (int32_t)above;
        else s_rows[g * kWave + lane] = upto - (int32_t)above;
        before_lo -= (lane > g);
        if (GROUPS_HI) before_hi -= (kWave + lane > g);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");

        const int32_t drawn = g * kWave + j;             // its length, counted from 0
        const int32_t where = drawn << 16 | last;
        kept_where = lane == turn ? where : kept_where;
        kept_left = lane == turn ? left : kept_left;
        last -= drawn + 1;                               // (below -1 only if the sums were wrong)
        placed += 1;
      }
    }
    const int32_t rest = (placed - 1) & (kWave - 1);     // the last set of placements
    if (placed > 0 && lane <= rest) pick[placed - 1 - rest + lane] = RfPick{kept_where, kept_left};
    if (lane == 0) {
        if (last >= -1 && placed == n_seq) {
            block_first[blocks] = n_seq;
            result->num_blocks = blocks;
        } else {
            result->bad_length = 2;
        }
        if (host_result) {
            host_result->num_blocks = blocks;
            host_result->total_frames = result->total_frames;
            host_result->bad_length = last >= -1 && placed == n_seq ? 0 : 2;
        }
    }
}

__global__ __launch_bounds__(kThreads) void rf_assign_kernel(
    const RfPick* __restrict__ pick, const int32_t* __restrict__ first,
    const int32_t* __restrict__ entry, int32_t n_seq, int32_t t_blk, const int32_t* __restrict__ block_first,
    int32_t* __restrict__ order, int32_t* __restrict__ block_of_seq, int32_t* __restrict__ offset_of_seq,
    PlanResult* __restrict__ result, PlanResult* __restrict__ host_result)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= n_seq || result->bad_length) return;
    const RfPick k = pick[p];
    const int32_t rank = k.left - 1;
    const int64_t at = (int64_t)first[k.where >> 16] + rank;
    if (rank < 0 || at >= n_seq) {                      // cannot happen with consistent sums
        result->bad_length = 2;
        if (host_result) host_result->bad_length = 2;
        return;
    }
    const int32_t i = entry[at];
    // the last block that begins at or before placement p
    int32_t lo = 0, hi = (int32_t)result->num_blocks;
    while (hi - lo > 1) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (block_first[mid] <= p) lo = mid; else hi = mid;
    }
    order[p] = i;
    block_of_seq[i] = lo;
    offset_of_seq[i] = t_blk - 1 - (k.where & 0xffff);
}

struct RfLayout {
    size_t result, seeded, seeded_len, entry, pick, first, within, group_before, chunk_count, bytes;
    int32_t n_chunks, per_chunk;
};

static RfLayout rf_layout(int64_t n_seq)
{
    RfLayout l{};
    const size_t n = (size_t)(n_seq > 0 ? n_seq : 0);
    size_t off = 0;
    auto take = [&off](size_t bytes) { const size_t at = off; off += round_up(bytes, 16); return at; };
    l.result = take(sizeof(PlanResult));
    l.seeded = take(n * 4);
    l.seeded_len = take(n * 4);
    l.entry = take(n * 4);
    l.pick = take(n * sizeof(RfPick));
    take(n * 8);              // not used: the answer stays at the 28 bytes per sequence that the layout always had
    l.first = take((size_t)kRfMaxT * 4);
    l.within = take((size_t)kRfGroups * kRfStride * 4);
    l.group_before = take((size_t)kRfGroups * 4);
    // chunks of whole 256-position tiles, at most kRfMaxChunks of them, at least 4 tiles each
    const int64_t tiles = ceil_div((int64_t)n, kThreads);
    const int64_t tiles_per_chunk = std::max<int64_t>(4, ceil_div(tiles, kRfMaxChunks));
    l.per_chunk = (int32_t)(tiles_per_chunk * kThreads);
    l.n_chunks = (int32_t)std::max<int64_t>(1, ceil_div((int64_t)n, l.per_chunk));
    l.chunk_count = take((size_t)l.n_chunks * kRfMaxT * 4);
    l.bytes = off;
    return l;
}

}  // namespace bload

using namespace bload;

extern "C" size_t bload_plan_random_fit_workspace_bytes(int64_t n_seq)
{
    if (n_seq < 0 || n_seq > BLOAD_MAX_SEQ) return 0;
    return rf_layout(n_seq).bytes;
}

extern "C" bload_status bload_plan_random_fit(const int32_t* d_lengths, int64_t n_seq, int32_t t_blk,
                                              uint64_t seed, int32_t* d_order,
                                              int32_t* d_block_of_seq, int32_t* d_offset_of_seq,
                                              int32_t* d_block_first, int64_t* h_num_blocks,
                                              int64_t* h_total_frames, void* d_workspace,
                                              size_t workspace_bytes, void* hip_stream)
{
    if (!h_num_blocks || !h_total_frames || n_seq < 0 || t_blk < 1) return BLOAD_EINVAL;
    *h_num_blocks = 0;
    *h_total_frames = 0;
    if (n_seq > BLOAD_MAX_SEQ || t_blk > kRfMaxT) return BLOAD_EOVERFLOW;
    if (n_seq == 0) return BLOAD_OK;
    if (!d_lengths || !d_order || !d_block_of_seq || !d_offset_of_seq || !d_block_first ||
        !d_workspace)
        return BLOAD_EINVAL;
    if (!aligned_to(d_lengths, 4) || !aligned_to(d_order, 4) || !aligned_to(d_block_of_seq, 4) ||
        !aligned_to(d_offset_of_seq, 4) || !aligned_to(d_block_first, 4) ||
        !aligned_to(d_workspace, 16))
        return BLOAD_EALIGN;
    const RfLayout l = rf_layout(n_seq);
    if (workspace_bytes < l.bytes) return BLOAD_EWORKSPACE;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    uint8_t* ws = static_cast<uint8_t*>(d_workspace);
    PlanResult* result = reinterpret_cast<PlanResult*>(ws + l.result);
    // the numbers the host waits for also go into pinned host memory where there is some (plain stores of
    // the last kernels), else they are copied back from the workspace
    static_assert(sizeof(PlanResult) <= 64, "the pinned buffer holds 64 bytes");
    PlanResult* pinned = static_cast<PlanResult*>(host_result_buffer());
    int32_t* seeded = reinterpret_cast<int32_t*>(ws + l.seeded);
    int32_t* seeded_len = reinterpret_cast<int32_t*>(ws + l.seeded_len);
    int32_t* entry = reinterpret_cast<int32_t*>(ws + l.entry);
    RfPick* pick = reinterpret_cast<RfPick*>(ws + l.pick);
    int32_t* first = reinterpret_cast<int32_t*>(ws + l.first);
    int32_t* within = reinterpret_cast<int32_t*>(ws + l.within);
    int32_t* group_before = reinterpret_cast<int32_t*>(ws + l.group_before);
    int32_t* chunk_count = reinterpret_cast<int32_t*>(ws + l.chunk_count);

    const int32_t n = (int32_t)n_seq;
    const OrderKey key = make_order_key(n_seq, seed);
    const dim3 block(kThreads);
    const dim3 per_item((uint32_t)ceil_div(n_seq, kThreads));

    hipLaunchKernelGGL(rf_clear_kernel, dim3(1), dim3(1), 0, stream, result);
    hipLaunchKernelGGL(rf_order_kernel, per_item, block, 0, stream, d_lengths, n, t_blk, key, seeded,
                       seeded_len, result);
    hipLaunchKernelGGL(rf_count_kernel, dim3((uint32_t)l.n_chunks), block, 0, stream, seeded_len, n, t_blk,
                       l.per_chunk, chunk_count);
    hipLaunchKernelGGL(rf_offsets_kernel, dim3(1), dim3(kRfOffsetThreads), 0, stream, l.n_chunks, t_blk, chunk_count, first,
                       within, group_before);
    hipLaunchKernelGGL(rf_scatter_kernel, dim3((uint32_t)l.n_chunks), block, 0, stream, seeded, seeded_len,
                       n, t_blk, l.per_chunk, chunk_count, entry);
    // after a length outside [1, t_blk] the last two kernels return at once
    const dim3 wave(kWave);
    if (t_blk <= kRfRegisterRows * kWave)
        hipLaunchKernelGGL((rf_draw_kernel<true, false>), dim3(1), wave, 0, stream, within, group_before, n, t_blk,
                           seed, pick, d_block_first, result, pinned);
    else if (t_blk <= kWave * kWave)
        hipLaunchKernelGGL((rf_draw_kernel<false, false>), dim3(1), wave, 0, stream, within, group_before, n, t_blk,
                           seed, pick, d_block_first, result, pinned);
    else
        hipLaunchKernelGGL((rf_draw_kernel<false, true>), dim3(1), wave, 0, stream, within, group_before, n, t_blk,
                           seed, pick, d_block_first, result, pinned);
    hipLaunchKernelGGL(rf_assign_kernel, per_item, block, 0, stream, pick, first, entry, n, t_blk, d_block_first, d_order,
                       d_block_of_seq, d_offset_of_seq, result, pinned);
    if (launch_status() != BLOAD_OK) return BLOAD_EHIP;
    PlanResult host{};
    if (!pinned && !hip_ok(hipMemcpyAsync(&host, result, sizeof(host), hipMemcpyDeviceToHost, stream)))
        return BLOAD_EHIP;
    if (!hip_ok(hipStreamSynchronize(stream))) return BLOAD_EHIP;
    if (pinned) host = *pinned;
    if (host.bad_length == 1) return BLOAD_ELENGTH;
    if (host.bad_length) return BLOAD_EHIP;            // the chain found its sums inconsistent
    *h_num_blocks = host.num_blocks;
    *h_total_frames = host.total_frames;
    return BLOAD_OK;
}
