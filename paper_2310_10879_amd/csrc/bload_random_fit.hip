// bload_plan_random_fit: the block builder with the paper's own sampler (BLoad,
// caption of the pseudocode figure: a random entry of the length dictionary L_dict
// among those no longer than the frames remaining in the open block).
//
// The draws are a chain: what fits, and how many of each length are left, depends on
// every earlier draw.  So the draws are made by one workgroup that guesses many at a time and
// goes over them until the guesses are right, or, where that does not pay, by ONE wavefront
// whose chain is kept as short as the hardware allows, and everything around is parallel:
//   rf_order_kernel    seeded position p -> sequence, its length, checks, frame total
//   rf_count_kernel, rf_offsets_kernel, rf_scatter_kernel
//                      L_dict: where each length's list starts, the lists themselves in
//                      seeded order, and the running counts the chain starts from; the
//                      seeded positions are cut into chunks, one workgroup each, that
//                      count their lengths, learn where their part of every list
//                      begins, and fill it in order
//                      (up to 4096 sequences rf_prepare_kernel does all of this in one workgroup)
//                      (up to 64 sequences rf_wave_kernel makes the whole plan)
//   rf_draw_batches_kernel, rf_draw_kernel
//                      the draws: per placement only (length, free room, how many were left) - no
//                      global load on the chain
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

// Where the chain of draws goes on behind those that were made in batches.
struct RfState {
    int32_t placed, blocks;   // draws made, blocks begun
    int32_t room;             // what is free in the last of them
    int32_t pad_;
};

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

__device__ __forceinline__ void rf_offsets(int32_t n_chunks, int32_t t_blk, int32_t* chunk_count, int32_t* s_group,
                                           int32_t* __restrict__ first, int32_t* __restrict__ within,
                                           int32_t* __restrict__ group_before)
{
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

__global__ __launch_bounds__(kRfOffsetThreads) void rf_offsets_kernel(
    int32_t n_chunks, int32_t t_blk, int32_t* __restrict__ chunk_count, int32_t* __restrict__ first,
    int32_t* __restrict__ within, int32_t* __restrict__ group_before)
{
    __shared__ int32_t s_group[kRfGroups];
    rf_offsets(n_chunks, t_blk, chunk_count, s_group, first, within, group_before);
}

// Step 3, one workgroup per chunk: its sequences into their lists, in seeded order: tile by
// tile of 256 positions.  The lanes of a wave that hold the same length find each other by votes on its bits, and the
// waves take their places in the lists one after another.  (Each thread ranking itself among the keys in front, read
// from LDS, took 7 us a tile: 29 us at 10^4 sequences.)
// `waves` waves take turns: the barriers are the workgroup's.
__device__ __forceinline__ void rf_scatter_tile(int32_t len, int32_t sequence, int bits, int waves, int32_t* s_fill,
                                                int32_t* __restrict__ entry, uint16_t* __restrict__ sorted_len)
{
    const int lane = lane_id(), wave = wave_id();
    uint64_t same = ~0ull;                       // the lanes with this length
    for (int b = 0; b < bits; ++b) {
        const bool one = (len >> b) & 1;
        const uint64_t vote = __ballot(one);
        same &= one ? vote : ~vote;
    }
    const int rank = (int)__popcll(same & ((1ull << lane) - 1ull));
    for (int w = 0; w < waves; ++w) {
        __syncthreads();
        if (wave == w && len) {
            const int32_t at = s_fill[len - 1] + rank;
            if ((same >> lane) == 1ull) s_fill[len - 1] = at + 1;        // the last of them
            entry[at] = sequence;
            sorted_len[at] = (uint16_t)len;
        }
    }
}

__global__ __launch_bounds__(kThreads) void rf_scatter_kernel(
    const int32_t* __restrict__ seeded, const int32_t* __restrict__ seeded_len, int32_t n_seq,
    int32_t t_blk, int32_t per_chunk, const int32_t* __restrict__ chunk_start, int32_t* __restrict__ entry,
    uint16_t* __restrict__ sorted_len)
{
    __shared__ int32_t s_fill[kRfMaxT];         // next free place of every list, for this chunk
    const int tid = (int)threadIdx.x;
    const int lengths_kept = ((t_blk + kWave - 1) / kWave) * kWave;
    const int bits = 32 - __clz(t_blk);
    for (int e = tid; e < lengths_kept; e += kThreads) s_fill[e] = chunk_start[(int64_t)blockIdx.x * kRfMaxT + e];
    const int64_t lo = (int64_t)blockIdx.x * per_chunk;
    const int64_t hi = min((int64_t)n_seq, lo + per_chunk);
    for (int64_t tile = lo; tile < hi; tile += kThreads) {
        const int64_t p = tile + tid;
        const int32_t len = p < hi ? seeded_len[p] : 0;
        const int32_t sequence = p < hi ? seeded[p] : 0;
        rf_scatter_tile(len, sequence, bits, kThreads / kWave, s_fill, entry, sorted_len);
    }
}

// All steps for at most kRfPrepareMost sequences, in one workgroup: a position to a thread, kRfPrepareTiles times, the one
// chunk's counts in LDS, and the walks of the order as look-ups in a table of the permutation's domain (one compute unit
// would pay for the longest walk of every wave).  Bound by barriers and latencies; what it saves is four launches: a call for 128
// sequences 67 -> 56 us, 300: 107 -> 95, 1000: 142 -> 125, 4096: 434 -> 421.  (Every further 1024 positions cost some 2 us
// of the 16 that it saves at 2048, and beyond 4096 the table is four times as large.)
constexpr int kRfPrepareTiles = 4;
constexpr int kRfPrepareMost = kRfPrepareTiles * kRfOffsetThreads;

__global__ __launch_bounds__(kRfOffsetThreads) void rf_prepare_kernel(
    const int32_t* __restrict__ lengths, int32_t n_seq, int32_t t_blk, OrderKey key, int32_t* __restrict__ first,
    int32_t* __restrict__ within, int32_t* __restrict__ group_before, int32_t* __restrict__ entry,
    uint16_t* __restrict__ sorted_len, PlanResult* __restrict__ result)
{
    __shared__ int32_t s_fill[kRfMaxT];         // sequences of every length, then the next free place of every list
    __shared__ int32_t s_group[kRfGroups];
    __shared__ uint16_t s_step[kRfPrepareMost];
    __shared__ unsigned long long s_sum;
    const int tid = (int)threadIdx.x;
    const int lengths_kept = ((t_blk + kWave - 1) / kWave) * kWave;
    const int bits = 32 - __clz(t_blk);
    const int domain = 1 << 2 * key.half_bits;
    for (int e = tid; e < lengths_kept; e += kRfOffsetThreads) s_fill[e] = 0;
    for (int x = tid; x < domain; x += kRfOffsetThreads) s_step[x] = (uint16_t)feistel((uint32_t)x, key);
    if (tid == 0) s_sum = 0;
    __syncthreads();
    int32_t sequence[kRfPrepareTiles], len[kRfPrepareTiles];
    int32_t bad = 0, sum = 0;
#pragma unroll
    for (int j = 0; j < kRfPrepareTiles; ++j) {
        const int p = tid + j * kRfOffsetThreads;
        sequence[j] = len[j] = 0;
        if (p < n_seq) {
            int i = s_step[p];
            while (i >= n_seq) i = s_step[i];
            const int32_t found = lengths[i];
            sequence[j] = i;
            if (found < 1 || found > t_blk) bad = 1;
            else len[j] = found;
        }
    }
#pragma unroll
    for (int j = 0; j < kRfPrepareTiles; ++j) {
        sum += len[j];
        if (len[j]) atomicAdd(&s_fill[len[j] - 1], 1);
    }
    if (sum) atomicAdd(&s_sum, (unsigned long long)sum);
    bad = __syncthreads_or(bad);
    if (tid == 0) {
        result->num_blocks = 0;
        result->total_frames = (int64_t)s_sum;
        result->bad_length = bad;
        result->pad_ = 0;
    }
    rf_offsets(1, t_blk, s_fill, s_group, first, within, group_before);
#pragma unroll
    for (int j = 0; j < kRfPrepareTiles; ++j) {
        const int here = n_seq - j * kRfOffsetThreads;
        if (here <= 0) break;
        rf_scatter_tile(len[j], sequence[j], bits, min((here + kWave - 1) / kWave, kRfOffsetThreads / kWave), s_fill, entry,
                        sorted_len);
    }
}

// ---- the draws --------------------------------------------------------------------
//
// Two ways to make them, with the same result: many at a time by a workgroup as long as that pays,
// and one after another by one wavefront.
//
// Many at a time.  The sequences left are kept as a list of their lengths in ascending order (`len`)
// with, per length, how many are not longer (`upto`).  Draw i of a batch of 64 then is, with j over
// the draws in front of it in the batch and ranks counted in the list as the batch finds it:
//   fit_i  = upto[room_i] - #{j < i: rank_j < upto[room_i]}     (none fits: a new block, all left fit)
//   k_i    = floor(u_i * fit_i / 2^64)
//   rank_i = k_i + #{j < i: rank_j <= rank_i}                   (the k-th of those not yet taken)
//   room_(i+1) = room_i - len[rank_i]
// All 64 are guessed, the right sides computed from the guesses, and that again with what came out until
// nothing changes.  A value that depends on right values in front of it alone is right, so after every
// round the draws up to the first one that changed are exactly those of the chain: the rounds end, and
// how many they are only depends on how far a wrong guess is carried on.  10^4 sequences of heavy-tailed
// lengths take 5 rounds per 64 draws, lengths near the block's 3, clips of a sixteenth of it and more 26, and 6 where
// blocks are guessed ahead (below); lengths spread evenly over it 20 to 40, guessed ahead or not.
// (rank_i is a fixed point of its own equation as well.  One on a rank already taken can be reached from
// above only and has nothing but taken ranks down to the right one: it is then lowered by one.)
// Bound by latency, like the chain: a round is 0.6 us of some 180 dependent instructions and three look-ups in LDS, on a
// workgroup whose 8 waves share the counting (64 x 63 / 2 comparisons of two limits, 16 bits each); what follows the
// rounds of a batch (taking the ranks out of the list and the counts) 2.6 us; 64 draws one after another 14 us.  Whole
// call, before and after, 10^4 sequences in blocks of 3000: heavy-tailed lengths 2250 -> 930 us, nearly full blocks
// 3540 -> 705, clips 3110 -> 1505; lengths spread evenly, which give up after the trial, 3055 -> 2985.
// Where they stop paying, batches end at once and the chain goes on within the block.  (Ones and halves of a block of 8192: 3060
// us by the chain alone, 3030 like this, 5300 where batches went on until a block began in the middle of one.)
//
// One after another (rf_draw_kernel): what is left where batches cost more than they bring, and sequences beyond
// kRfBatchMost.

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
// With `state`, the draws behind it, in the block that is open there: the loop is entered in the middle of a block and
// needs to know nothing else (a flag in it, or the loop behind the batches in one kernel: 7 to 13 % slower).
constexpr int kRfRegisterRows = 32;
typedef int32_t rf_rows __attribute__((ext_vector_type(kRfRegisterRows)));

template <bool REGISTERS, bool GROUPS_HI>
__global__ __launch_bounds__(kWave) void rf_draw_kernel(
    const int32_t* __restrict__ within, const int32_t* __restrict__ group_before, const RfState* __restrict__ state,
    int32_t n_seq, int32_t t_blk, uint64_t seed, RfPick* __restrict__ pick, int32_t* __restrict__ block_first,
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
    const RfState from = state ? *state : RfState{0, 0, 0, 0};
    if (from.placed == n_seq) return;                    // the batches were all

    // Every block takes at least one sequence (all of them fit an empty block), every placement
    // uses up room, and at most n_seq blocks are begun: the loop ends whatever the sums hold.
    int32_t placed = from.placed, blocks = from.blocks;
    int32_t last = from.room - 1;                        // the longest length that fits, counted from 0; -1: none
    int32_t least = -1;                                  // of these at the blocks' ends: below -1 only if the sums were wrong
    uint32_t u_lo = 0, u_hi = 0;
    int32_t kept_where = 0, kept_left = 0;               // placement (placed & ~63) + lane
    if (placed > 0) {
        const uint64_t u = splitmix64_at(seed, (uint64_t)(6 + (placed & ~(kWave - 1)) + lane));
        u_lo = (uint32_t)u;
        u_hi = (uint32_t)(u >> 32);
        const RfPick k = pick[min(((placed - 1) & ~(kWave - 1)) + lane, placed - 1)];      // (lanes behind are set before they are stored)
        kept_where = k.where;
        kept_left = k.left;
    }
    __builtin_amdgcn_s_waitcnt(0);                       // (or every draw waits for what is loaded above)
    for (;;) {
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
        last -= drawn + 1;
        placed += 1;
      }
      least = min(least, last);
      if (max(placed, blocks) >= n_seq) break;           // (one test a block: three cost 3 % where blocks hold a sequence or two)
      if (lane == 0) block_first[blocks] = placed;
      blocks += 1;
      last = t_blk - 1;
    }
    const int32_t rest = (placed - 1) & (kWave - 1);     // the last set of placements
    if (placed > 0 && lane <= rest) pick[placed - 1 - rest + lane] = RfPick{kept_where, kept_left};
    if (lane == 0) {
        if (least == -1 && placed == n_seq) {
            block_first[blocks] = n_seq;
            result->num_blocks = blocks;
        } else {
            result->bad_length = 2;
        }
        if (host_result) {
            host_result->num_blocks = blocks;
            host_result->total_frames = result->total_frames;
            host_result->bad_length = least == -1 && placed == n_seq ? 0 : 2;
        }
    }
}

constexpr int kRfBatch = kWave;                   // draws at a time, a lane each
constexpr int kRfBatchWaves = 8;                  // two per SIMD hide each other's latencies
constexpr int kRfBatchThreads = kRfBatchWaves * kWave;
constexpr int kRfBatchMost = 24576;               // sequences: what is kept of them in LDS, 35 bits each, is 129 KiB with the rest
// From so many sequences on.  A trial that brings nothing and the second launch cost 8 us, 3 % of a call here, and batches that
// pay until few sequences are left up to 20 (lengths of some tenth of a block of 40: 218 -> 235 us); lengths near the
// block's gain half (304 -> 136), heavy-tailed ones in blocks of 3000 40 % (226 -> 138).
constexpr int kRfBatchLeast = 768;
// From so few on where what is left nearly all fits or hardly any of it, which the frame total tells: lengths of a fiftieth of
// the block on average or less (from kRfShortLeast on), or of three quarters of it and more.  256 nearly full blocks 107 -> 70 us
// a call, 767 271 -> 120; heavy-tailed lengths in blocks of 3000, 320 of them 100 -> 80, 700 184 -> 104.  (At a 41st of the
// block 320 and 400 exponential lengths took 116 and 133 us, 100 and 118 by the chain; lengths of a tenth 96 and 111 us at 256
// and 384, 81 and 111 by the chain.)  Where the total tells that batches don't pay, the launch costs 2 us.
constexpr int kRfFewest = 192, kRfShortLeast = 320, kRfShortPart = 50;
// The first batch is a trial: it ends, with nothing drawn, if after so many rounds not so many of its draws are settled.
// Of many sequences it is guessed ahead and lasts longer, which costs 10 us where it fails: 1 % of 4096 draws.
constexpr int kRfTryRounds = 4, kRfTryDraws = 6, kRfTryLong = 8, kRfTryLongDraws = 16, kRfTryLongFrom = 4096;
constexpr int kRfBatchRounds = 48;                // of a batch, before what is settled of it is taken
constexpr int kRfGuessSteps = 16;                 // draws that a guess of a block's contents goes ahead
constexpr int kRfPlainBatches = 16;               // batches without one after one that told of less than half the draws
constexpr int kRfGuessFrom = 8;                   // rounds of a batch from which on the next are guessed so
// What a batch costs and brings, in units of 1/64 us: a round, the rest of a batch (and a unit for so many entries of the
// lists), a step of a guess; a draw of the chain in blocks of up to 2048 (longer ones 18).
constexpr int kRfCostRound = 40, kRfCostBatch = 100, kRfCostEntries = 120, kRfCostGuess = 16, kRfCostDraw = 14;

struct RfShared {
    alignas(16) uint16_t len[2][kRfBatchMost + 8 * kWave];   // lengths that are left, ascending
    alignas(16) uint16_t upto[kRfMaxT + 8];              // [7 + l]: sequences left of at most length l
    unsigned long long gone[kRfBatchMost / 64 + 1];      // ranks that the batch takes, a bit each
    uint2 taken[kRfBatchMost / 32 + 2];                  // the same, 32 ranks at a time: bits, and how many in front
    uint32_t count[3][kRfBatch];                         // what the waves count, in turn; the next one is 0
    unsigned long long random[kRfBatch];
    uint16_t guess[kRfBatch][kRfGuessSteps];
    uint16_t rank[kRfBatch];
    unsigned long long opens;
    int32_t known, steps;
    uint16_t nowhere;                                    // where lengths that leave the list are stored
};
static_assert(sizeof(RfShared) <= 156 * 1024, "one workgroup's LDS");
static_assert(kRfBatchWaves == 8 && kRfBatch == 64, "a wave counts eight draws");
static_assert(kRfBatchMost < 1 << 15, "ranks and their limits are compared in 16 bits");

struct RfMax { __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return max(a, b); } };
struct RfMoveU {
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ uint32_t at(uint32_t v) const { return dpp_move<CTRL, ROW_MASK>(v, 0u); }
};

typedef uint16_t rf_two __attribute__((ext_vector_type(2)));

// One to each half of `sum` where the value in that half of `v` is below the one of `limits`.  (`one` is 1 in each
// half, and not known to be: three packed instructions, not two comparisons and their bits put together.)
__device__ __forceinline__ rf_two rf_add_below(rf_two sum, rf_two limits, uint32_t v, uint32_t one)
{
    return sum + __builtin_elementwise_min(__builtin_elementwise_sub_sat(limits, __builtin_bit_cast(rf_two, v)),
                                           __builtin_bit_cast(rf_two, one));
}

// The wave's share of: how many of the draws in front of the lane's have a value below each of the two limits
// (16 bits each, and so are the counts).  Wave w < 7 counts draws 8 w .. 8 w + 7 for the draws of later eights, the
// last one the draws of the lane's own eight.
__device__ __forceinline__ uint32_t rf_count_below(uint32_t value, uint32_t limits, int wave)
{
    const uint32_t both = value | value << 16;
    uint32_t one = 0x10001u;
    asm("" : "+v"(one));
    rf_two sum = {0, 0};
    if (wave < kRfBatchWaves - 1) {
        const rf_two limit = __builtin_bit_cast(rf_two, lane_id() >= 8 * wave + 8 ? limits : 0u);
#pragma unroll
        for (int j = 0; j < 8; ++j) sum = rf_add_below(sum, limit, (uint32_t)__builtin_amdgcn_readlane((int)both, 8 * wave + j), one);
    } else {
        const rf_two limit = __builtin_bit_cast(rf_two, limits);
        // (every lane moves, whatever becomes of it)
        const uint32_t moved[7] = {dpp_move<kDppRowShr1>(both, ~0u), dpp_move<kDppRowShr1 + 1>(both, ~0u),
                                   dpp_move<kDppRowShr1 + 2>(both, ~0u), dpp_move<kDppRowShr1 + 3>(both, ~0u),
                                   dpp_move<kDppRowShr1 + 4>(both, ~0u), dpp_move<kDppRowShr1 + 5>(both, ~0u),
                                   dpp_move<kDppRowShr1 + 6>(both, ~0u)};
#pragma unroll
        for (int j = 0; j < 7; ++j) sum = rf_add_below(sum, limit, (lane_id() & 7) > j ? moved[j] : ~0u, one);
    }
    return __builtin_bit_cast(uint32_t, sum);
}

// The sum of the waves' counts of the lane's draw; one barrier.  `turn` goes round over three sets, so that one is
// cleared while another one is added to and the third may still be read.
__device__ __forceinline__ uint32_t rf_all_counts(RfShared& sh, uint32_t mine, int wave, int& turn)
{
    const int lane = lane_id(), next = turn == 2 ? 0 : turn + 1;
    atomicAdd(&sh.count[turn][lane], mine);
    if (wave == kRfBatchWaves - 2) sh.count[next][lane] = 0;
    __syncthreads();
    const uint32_t all = sh.count[turn][lane];
    turn = next;
    return all;
}

// Every wave holds all 64 draws, a lane each, and does the same with them; a wave by itself only counts over its
// eight draws, and moves its part of the list.
__global__ __launch_bounds__(kRfBatchThreads) void rf_draw_batches_kernel(
    const uint16_t* __restrict__ sorted_len, int32_t* __restrict__ within, int32_t* __restrict__ group_before,
    RfState* __restrict__ state, int32_t n_seq, int32_t t_blk, uint64_t seed, RfPick* __restrict__ pick, int32_t* __restrict__ block_first,
    PlanResult* __restrict__ result, PlanResult* __restrict__ host_result)
{
    __shared__ RfShared sh;
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
    const int32_t bad = result->bad_length;
    if (bad) {
        if (tid == 0 && host_result) host_result->bad_length = bad;
        return;
    }
    if (n_seq < kRfBatchLeast) {
        const int64_t frames = result->total_frames, most = (int64_t)n_seq * t_blk;
        if (!(n_seq >= kRfShortLeast && kRfShortPart * frames <= most) && 4 * frames < 3 * most) {
            if (tid == 0) *state = RfState{0, 0, 0, 0};
            return;
        }
    }
    const int groups = (t_blk + kWave - 1) / kWave, kept = groups * kWave;
    const uint16_t* upto = sh.upto + 7;
    for (int e = tid; e < kept; e += kRfBatchThreads)
        sh.upto[8 + e] = (uint16_t)(group_before[e >> 6] + within[(e >> 6) * kRfStride + (e & 63) + 1]);
    if (tid == 0) sh.upto[7] = 0;
    for (int i = tid; i < (n_seq + 7) / 8; i += kRfBatchThreads)
        reinterpret_cast<vec16*>(sh.len[0])[i] = reinterpret_cast<const vec16*>(sorted_len)[i];
    for (int w = tid; w <= n_seq / 64; w += kRfBatchThreads) sh.gone[w] = 0;
    if (tid < kRfBatch) {
        sh.random[tid] = splitmix64_at(seed, (uint64_t)(6 + tid));
        sh.count[0][tid] = 0;
    }
    __syncthreads();

    int cur = 0, turn = 0;
    int32_t placed = 0, blocks = 0;
    int32_t room = 0;                                    // in the open block, in front of the batch (no block yet: 0)
    int32_t left = n_seq;                                // sequences
    int32_t credit = 4 * 64 + n_seq / 8;                 // batches may cost 4 us and some 1 % of a chain of all draws
    const int32_t most_credit = credit + 4 * 64;
    const bool long_try = n_seq >= kRfTryLongFrom;
    bool guesses = long_try;
    int plain = 0;                                       // batches to come that are not guessed ahead
    while (left > 0 && credit >= 0) {
        const uint16_t* len = sh.len[cur];
        const int32_t w = min(kRfBatch, left);
        const uint64_t in_batch = w == 64 ? ~0ull : (1ull << w) - 1ull;
        // The first guess: all that is left fits, and of the draws in front the usual share lies below.
        // Of the lane's draw: `rank`, `length`, and whether it `opens` a block.
        const uint64_t u = sh.random[lane];
        const uint32_t u_lo = (uint32_t)u, u_hi = (uint32_t)(u >> 32);
        int32_t rank, length;
        const bool opens_first = upto[room] == 0;
        bool opens = lane == 0 && opens_first;
        const float per_draw = __builtin_amdgcn_rcpf((float)left);
        {
            const int32_t k = (int32_t)__umulhi(u_hi, (uint32_t)max(left - lane, 1));
            rank = min(k + (int32_t)((float)k * ((float)lane * per_draw)), left - 1);
        }
        const bool ahead = guesses && plain == 0;
        if (ahead) {
            // Every lane draws the contents of a block that begins with its draw (the first: that goes
            // on with it), from counts that the batch does not lower.  The blocks that follow one
            // another from the first draw on are then the guess.
            if (wave == 0) {
                int32_t free = lane == 0 && !opens_first ? room : t_blk, at = lane;
                int step = 0;
#pragma nounroll
                for (; step < kRfGuessSteps; ++step) {
                    const bool draws = at < w && free > 0 && at - lane == step;
                    const int32_t all = draws ? (int32_t)upto[free] : 0;
                    const float part = (float)at * per_draw;
                    const int32_t fit = all - (int32_t)((float)all * part);
                    if (__ballot(draws && fit > 0) == 0) break;
                    if (draws && fit > 0) {
                        const int32_t k = (int32_t)__umulhi((uint32_t)(sh.random[at] >> 32), (uint32_t)fit);
                        const int32_t r = min(k + (int32_t)((float)k * part), left - 1);
                        sh.guess[lane][step] = (uint16_t)r;
                        free = max(free - (int32_t)len[r], 0);
                        at += 1;
                    }
                }
                uint64_t heads = 0;
                int32_t head = 0, known = 0;             // first draw of a block, draws guessed so far
                while (head < w) {
                    heads |= 1ull << head;
                    known = __builtin_amdgcn_readlane(at, head);
                    if (known <= head || known - head >= kRfGuessSteps) break;
                    head = known;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                const int mine = 63 - __builtin_clzll(heads & (~0ull >> (63 - lane)));       // (draw 0 is a head)
                sh.rank[lane] = lane < known ? sh.guess[mine][lane - mine] : (uint16_t)rank;
                if (lane == 0) {
                    sh.opens = (heads & ~1ull) | (opens_first ? 1ull : 0ull);
                    sh.known = known;
                    sh.steps = step;
                }
            }
            __syncthreads();
            rank = sh.rank[lane];
            opens = (sh.opens >> lane) & 1ull;
            if (sh.known < kRfBatch / 2) plain = kRfPlainBatches;        // blocks of many sequences: not worth it
        } else if (plain > 0) {
            plain -= 1;
        }
        length = len[rank];

        int32_t accepted = 0, room_at, same = 0;
        int rounds = 0, until = placed == 0 && !long_try ? kRfTryRounds : kRfTryLong;
        for (;;) {
            // rooms, from the lengths in front in the block: a block that begins at draw j is full when the sum
            // reaches t_blk + the sum in front of j
            const int32_t own = lane < w ? length : 0;
            const int32_t sum = wave_scan(own, RfSum(), RfMove()), front = sum - own;
            const uint32_t full = opens ? (uint32_t)(t_blk + front) : 0u;
            const uint32_t full_at = dpp_move<kDppWaveShr1>(wave_scan(full, RfMax(), RfMoveU()), 0u);
            room_at = max(max((int32_t)full_at, room) - front, 0);
            const uint32_t all = upto[room_at];
            // what the right sides give
            const uint32_t count = rf_all_counts(sh, rf_count_below((uint32_t)rank, all | (uint32_t)(rank + 1) << 16, wave), wave, turn);
            rounds += 1;
            int32_t fit = (int32_t)(all - (count & 0xffffu));
            const bool opening = fit <= 0;
            if (opening) fit = max(left - lane, 1);
            // floor(u * fit / 2^64), fit < 2^16
            const int32_t k = (int32_t)(((uint64_t)u_hi * (uint32_t)fit + __umulhi(u_lo, (uint32_t)fit)) >> 32);
            const int32_t now = min(k + (int32_t)(count >> 16), left - 1);
            const uint64_t changed = __ballot((now != rank) | (opening != opens)) & in_batch;
            int32_t lowered = 0;
            if (changed == 0 || --until == 0) {
                until = 8;
                const int32_t settled = changed ? __builtin_ctzll(changed) : w;
                if (placed == 0 && changed != 0 && rounds <= kRfTryLong && settled < (long_try ? kRfTryLongDraws : kRfTryDraws)) break;
                const bool ends = changed == 0 || rounds >= kRfBatchRounds || settled < 2 * rounds ||
                                  credit + kRfCostDraw * settled < kRfCostRound * rounds + kRfCostBatch;
                if (ends) {
                    // settled, unless a draw has come to rest on a rank that one in front has taken
                    const bool mine = lane < settled;
                    if (wave == 0 && mine) atomicOr(&sh.gone[rank >> 6], 1ull << (rank & 63));
                    const uint32_t of_length = rf_count_below((uint32_t)length, (uint32_t)length | (uint32_t)(length + 1) << 16, wave);
                    const uint32_t of_rank = rf_count_below((uint32_t)rank, (uint32_t)rank, wave) & 0xffffu;
                    const uint32_t more = rf_all_counts(sh, (of_length & 0xffffu) | (of_length >> 16) << 8 | of_rank << 16, wave, turn);
                    same = (int32_t)((more >> 8) & 0xffu) - (int32_t)(more & 0xffu);
                    const uint64_t twice = __ballot(mine && (count >> 16) != (more >> 16));
                    if (twice == 0) { accepted = settled; break; }
                    __syncthreads();                     // (no wave reads `gone` before this batch is accepted)
                    if (wave == 0 && mine) atomicAnd(&sh.gone[rank >> 6], ~(1ull << (rank & 63)));
                    if (changed != 0 || rounds >= kRfBatchRounds) {
                        accepted = __builtin_ctzll(twice);
                        if (wave == 0 && lane < accepted) atomicOr(&sh.gone[rank >> 6], 1ull << (rank & 63));
                        __syncthreads();
                        break;
                    }
                    lowered = (int32_t)((twice >> lane) & 1ull);
                }
            }
            rank = max(now - lowered, 0);
            opens = opening;
            length = len[rank];
        }

        if (accepted == 0) break;                        // (of the first batch only)
        // Goes on while batches bring more than they cost, within what has been gained or was given.
        credit += kRfCostDraw * accepted - kRfCostRound * rounds - kRfCostBatch - (left + kept) / kRfCostEntries -
                  (ahead ? kRfCostGuess * sh.steps : 0);
        credit = min(credit, most_credit);
        // (a long trial says nothing about rounds without a guess)
        guesses = !(placed == 0 && long_try) && (guesses || rounds >= kRfGuessFrom);

        // The draws settled leave the list: every length moves down by the ranks taken in front of it.  Eight
        // consecutive ranks per lane, eight lanes to a word of `gone`.
        const int32_t in_block = opens ? t_blk : room_at;
        const uint64_t opened = __ballot(opens && lane < accepted);
        const int32_t rank_taken = lane < accepted ? rank : INT32_MAX;
        uint16_t* to = sh.len[cur ^ 1];
        for (int32_t r0 = (kRfBatchWaves - 1 - wave) * (8 * kWave); r0 <= left; r0 += kRfBatchWaves * 8 * kWave) {
            int32_t in_front = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int32_t c = (int32_t)__popcll(__ballot(rank_taken < r0 + i * 64));
                if ((lane >> 3) == i) in_front = c;
            }
            const int32_t r = r0 + 8 * lane;
            if (r <= left) {
                const unsigned long long word = sh.gone[r >> 6];
                const vec16 l = *reinterpret_cast<const vec16*>(len + r);
                const uint32_t half = (r & 32) ? (uint32_t)(word >> 32) : (uint32_t)word;
                if (r & 32) in_front += (int32_t)__popc((uint32_t)word);
                if ((lane & 3) == 0) sh.taken[r >> 5] = make_uint2(half, (uint32_t)in_front);
                int32_t at = r - in_front - (int32_t)__popc(half & ((1u << (r & 31)) - 1u));
                const uint32_t bits = half >> (r & 31);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    // (without a branch)
                    const bool stays = (bits & (1u << i)) == 0;
                    uint16_t* place = stays ? to + at : &sh.nowhere;
                    *place = (uint16_t)((i & 1) ? l[i / 2] >> 16 : l[i / 2]);
                    at += stays ? 1 : 0;
                }
            }
        }
        if (wave == 0) {
            if (lane < accepted) {
                // how many of its length are left: of those that the batch finds, less the draws in front
                pick[placed + lane] = RfPick{(length - 1) << 16 | (in_block - 1), (int32_t)upto[length] - (int32_t)upto[length - 1] - same};
                if (opens) block_first[blocks + (int32_t)__popcll(opened & ((1ull << lane) - 1ull))] = placed + lane;
            }
        }
        if (wave == 1) sh.random[lane] = splitmix64_at(seed, (uint64_t)(6 + placed + accepted + lane));
        __syncthreads();
        for (int e = 8 * tid; e < kept; e += 8 * kRfBatchThreads) {
            vec16 counts = *reinterpret_cast<const vec16*>(sh.upto + 8 + e);
            uint2 taken[8];                              // (all look-ups before the first use)
#pragma unroll
            for (int i = 0; i < 8; ++i) taken[i] = sh.taken[((i & 1) ? counts[i / 2] >> 16 : counts[i / 2] & 0xffffu) >> 5];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t lo = counts[i] & 0xffffu, hi = counts[i] >> 16;
                const uint32_t lo_now = lo - taken[2 * i].y - (uint32_t)__popc(taken[2 * i].x & ((1u << (lo & 31)) - 1u));
                const uint32_t hi_now = hi - taken[2 * i + 1].y - (uint32_t)__popc(taken[2 * i + 1].x & ((1u << (hi & 31)) - 1u));
                counts[i] = lo_now | hi_now << 16;
            }
            *reinterpret_cast<vec16*>(sh.upto + 8 + e) = counts;
        }
        for (int32_t word = tid; word <= left / 64; word += kRfBatchThreads) sh.gone[word] = 0;
        blocks += (int32_t)__popcll(opened);
        room = __builtin_amdgcn_readlane(in_block - length, accepted - 1);
        placed += accepted;
        left -= accepted;
        cur ^= 1;
        __syncthreads();
    }

    if (tid == 0) {
        *state = RfState{placed, blocks, room, 0};
        if (left == 0) {
            block_first[blocks] = n_seq;
            result->num_blocks = blocks;
            if (host_result) {
                host_result->num_blocks = blocks;
                host_result->total_frames = result->total_frames;
                host_result->bad_length = 0;
            }
        }
    }
    if (left == 0 || placed == 0) return;
    // the rest is drawn one after another (a kernel of its own: behind the batches in this one, the chain was 13 %
    // slower): the counts that it begins with
    for (int e = tid; e < kept; e += kRfBatchThreads)
        within[(e >> 6) * kRfStride + (e & 63) + 1] = (int32_t)upto[e + 1] - (int32_t)upto[e & ~63];
    if (tid < kRfGroups) group_before[tid] = upto[min(tid, groups) * kWave];
}

// ---- few sequences ------------------------------------------------------------------
//
// The whole plan of at most 64 sequences in one wave and one launch: the sequences lie in the lanes, in ascending order of their
// lengths and those of one length in seeded order, and what is left of them is a mask.  How many fit is a vote and a count, the
// k-th of them the lane with k fitting ones below it, and of its length the last one left is taken, as from the lists of
// L_dict.  No table of lengths, so nothing depends on t_blk.  Bound by the launch, the wait for it (16 us together)
// and some 30 dependent instructions a draw, 0.13 us where the chain over L_dict takes 0.26: a call for 64
// sequences in three launches 42 to 51 us (nine, before those: 47 to 63), like this 26; 30: 22.
__global__ __launch_bounds__(kWave) void rf_wave_kernel(
    const int32_t* __restrict__ lengths, int32_t n_seq, int32_t t_blk, OrderKey key, uint64_t seed,
    int32_t* __restrict__ order, int32_t* __restrict__ block_of_seq, int32_t* __restrict__ offset_of_seq,
    int32_t* __restrict__ block_first, PlanResult* __restrict__ result)
{
    const int lane = (int)threadIdx.x;
    const bool mine = lane < n_seq;
    int32_t i = 0, len = INT32_MAX;
    if (key.half_bits > 0) {                             // (a domain of at most 64: every lane has one step of the walks)
        const int step = (int)feistel((uint32_t)lane & ((1u << 2 * key.half_bits) - 1u), key);
        i = step;
        while (__any(mine && i >= n_seq)) {
            const int on = __shfl(step, i, kWave);
            if (i >= n_seq) i = on;
        }
    }
    if (mine) len = lengths[i];
    if (__any(mine && (len < 1 || len > t_blk))) {
        if (lane == 0) {
            result->num_blocks = 0;
            result->total_frames = 0;
            result->bad_length = 1;
            result->pad_ = 0;
        }
        return;
    }
    const int32_t total = __builtin_amdgcn_readlane(wave_scan(mine ? len : 0, RfSum(), RfMove()), kWave - 1);

    int rank = 0;                                        // (lanes without a sequence come last, in their order)
#pragma unroll 8
    for (int j = 0; j < kWave; ++j) {
        const int32_t other = __builtin_amdgcn_readlane(len, j);
        rank += other < len || (other == len && j < lane) ? 1 : 0;
    }
    len = __builtin_amdgcn_ds_permute(rank * 4, len);
    i = __builtin_amdgcn_ds_permute(rank * 4, i);

    const uint64_t random = splitmix64_at(seed, (uint64_t)(6 + lane));
    const uint32_t u_lo = (uint32_t)random, u_hi = (uint32_t)(random >> 32);
    unsigned long long left = ~0ull >> (kWave - n_seq);
    int32_t room = 0, blocks = 0;
    int32_t first = 0, place = 0, block = 0, offset = 0; // of block `lane`; of the lane's sequence
    for (int32_t placed = 0; placed < n_seq; ++placed) {
        unsigned long long fits = __ballot(len <= room) & left;
        if (fits == 0) {                                 // a new block: all that is left fits
            first = lane == blocks ? placed : first;
            ++blocks;
            room = t_blk;
            fits = left;
        }
        const uint32_t fit = (uint32_t)__popcll(fits);
        const uint32_t lo = __builtin_amdgcn_readlane(u_lo, placed), hi = __builtin_amdgcn_readlane(u_hi, placed);
        const uint32_t k = (uint32_t)(((uint64_t)hi * fit + ((uint64_t)lo * fit >> 32)) >> 32);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(fits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)fits, 0u));
        const unsigned long long chosen = __ballot(below == k) & fits;
        const int32_t length = __builtin_amdgcn_readlane(len, __ffsll((long long)chosen) - 1);
        const int last = kWave - 1 - __clzll((long long)(__ballot(len == length) & left));
        if (lane == last) {
            place = placed;
            block = blocks - 1;
            offset = t_blk - room;
        }
        left &= ~(1ull << last);
        room -= length;
    }
    if (mine) {
        order[place] = i;
        block_of_seq[i] = block;
        offset_of_seq[i] = offset;
        if (lane < blocks) block_first[lane] = first;
    }
    if (lane == 0) {
        block_first[blocks] = n_seq;
        result->num_blocks = blocks;
        result->total_frames = total;
        result->bad_length = 0;
        result->pad_ = 0;
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
    size_t result, seeded, seeded_len, entry, pick, sorted_len, first, within, group_before, chunk_count, bytes;
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
    l.sorted_len = take(n * 8);      // (2 of them used: the answer stays at the 28 bytes per sequence that the layout always had)
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
    uint16_t* sorted_len = reinterpret_cast<uint16_t*>(ws + l.sorted_len);
    int32_t* first = reinterpret_cast<int32_t*>(ws + l.first);
    int32_t* within = reinterpret_cast<int32_t*>(ws + l.within);
    int32_t* group_before = reinterpret_cast<int32_t*>(ws + l.group_before);
    int32_t* chunk_count = reinterpret_cast<int32_t*>(ws + l.chunk_count);

    const int32_t n = (int32_t)n_seq;
    const OrderKey key = make_order_key(n_seq, seed);
    const dim3 block(kThreads);
    const dim3 per_item((uint32_t)ceil_div(n_seq, kThreads));

    if (n_seq <= kWave) {
        hipLaunchKernelGGL(rf_wave_kernel, dim3(1), dim3(kWave), 0, stream, d_lengths, n, t_blk, key, seed, d_order,
                           d_block_of_seq, d_offset_of_seq, d_block_first, pinned ? pinned : result);
    } else {
        if (n_seq <= kRfPrepareMost) {
            hipLaunchKernelGGL(rf_prepare_kernel, dim3(1), dim3(kRfOffsetThreads), 0, stream, d_lengths, n, t_blk, key, first,
                               within, group_before, entry, sorted_len, result);
        } else {
            hipLaunchKernelGGL(rf_clear_kernel, dim3(1), dim3(1), 0, stream, result);
            hipLaunchKernelGGL(rf_order_kernel, per_item, block, 0, stream, d_lengths, n, t_blk, key, seeded,
                               seeded_len, result);
            hipLaunchKernelGGL(rf_count_kernel, dim3((uint32_t)l.n_chunks), block, 0, stream, seeded_len, n, t_blk,
                               l.per_chunk, chunk_count);
            hipLaunchKernelGGL(rf_offsets_kernel, dim3(1), dim3(kRfOffsetThreads), 0, stream, l.n_chunks, t_blk, chunk_count, first,
                               within, group_before);
            hipLaunchKernelGGL(rf_scatter_kernel, dim3((uint32_t)l.n_chunks), block, 0, stream, seeded, seeded_len,
                               n, t_blk, l.per_chunk, chunk_count, entry, sorted_len);
        }
        // after a length outside [1, t_blk] the last kernels return at once
        const bool batches = n_seq >= kRfFewest && n_seq <= kRfBatchMost;
        // (behind the sorted lengths, 2 of the 8 bytes per sequence that their part of the workspace has)
        RfState* state = reinterpret_cast<RfState*>(ws + l.sorted_len + round_up((size_t)n_seq * 2, 16));
        if (batches)
            hipLaunchKernelGGL(rf_draw_batches_kernel, dim3(1), dim3(kRfBatchThreads), 0, stream, sorted_len, within,
                               group_before, state, n, t_blk, seed, pick, d_block_first, result, pinned);
        const auto draw = t_blk <= kRfRegisterRows * kWave ? rf_draw_kernel<true, false>
                          : t_blk <= kWave * kWave ? rf_draw_kernel<false, false> : rf_draw_kernel<false, true>;
        hipLaunchKernelGGL(draw, dim3(1), dim3(kWave), 0, stream, within, group_before, batches ? state : nullptr, n, t_blk,
                           seed, pick, d_block_first, result, pinned);
        hipLaunchKernelGGL(rf_assign_kernel, per_item, block, 0, stream, pick, first, entry, n, t_blk, d_block_first, d_order,
                           d_block_of_seq, d_offset_of_seq, result, pinned);
    }
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
