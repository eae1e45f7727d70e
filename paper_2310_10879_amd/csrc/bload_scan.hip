// bload_segment_scan: the recurrent consumer of the start table (BLoad, Methods section and
// the figure of the DDS model: what frame n-1 produced is part of the input of frame n, and
// the table says where that carried state belongs to another sequence and is dropped).
// Per feature:  h = x at the first frame of a sequence,  h = decay * h + x afterwards;
// padding slots yield 0.  Output float32 [B, t_blk, feat_dim].
//
// HBM bound, and write heavy (4 output bytes per element): what a plain copy in tile order
// reaches (6.3-6.4 TB/s) is the mark, and a wave that walks a row of its own from end to end
// stays at 5 (it keeps thousands of far-apart places open at a time).  So the tensor is cut into
// tiles of a few hundred slots that short workgroups take nearly in memory order, every slot read
// once and written once, and the state travels from tile to tile:
//   - a tile computes its recurrence from a state of 0.  If it holds a boundary (a slot that
//     starts a sequence, or padding: nothing in front of it matters) the state it ends in is
//     final and is published, a word per feature
//   - a tile whose first slot continues a sequence looks for the state in front of it: the final
//     one of the tile before, or, going back over the tiles of its block as many at a time as it
//     has groups of lanes, the nearest final one and the partial ones behind it: state =
//     decay^chunk * state + partial.  It publishes its own end state: partial while it waits, final then
//   - the recurrence over the tile's own slots from that state, kept in registers meanwhile, is
//     what leaves for the output
// (The hand-over is the decoupled look-back of Merrill and Garland's single-pass scan, here with boundaries that make
// most states final at once, and with an end to the wait.)
// A state travels as a double whose last two mantissa bits are its mark (partial / final): one 8-byte
// word, written and read by atomics of device scope, so no order between different words is needed.
// Every state is cut to 50 mantissa bits when it is made, and the states are combined in the
// same order whichever tile finishes first: equal inputs give equal bits.  A hand-over in float32
// would add a rounding at every border (10000 sequences of log-mel frames: error against 64 bits
// 6.36e-8 instead of 6.17e-8 of the recurrence from end to end).
// Tiles that wait hold their registers, so the order of the tiles is that of memory only in
// the large: 32 blocks are taken side by side, chunk by chunk, and the tile in front has mostly
// finished (6900 blocks of 3000 slots x 320 bytes, one run on other pages than the figures below: 3.75 ms block by
// block, 2.75 with 8 side by side, 2.41 with 32 as with 128; without any hand-over, which is not the
// right result, 2.39).
//
// The wait ends.  A tile waits only for tiles in front of it in the same block, which publish
// their partial state without waiting for anything and have lower workgroup numbers on the same
// XCD (or, with few blocks, lower numbers in all), so they were started before.  Should one not
// have been heard of after BLOAD_SCAN_POLLS looks (some ten milliseconds), the workgroup computes
// all tiles in front of it in its block itself, the same way, and gets the same bits.
//
// Two kernels:
//   scan_direct_kernel  frames of 64 elements or more.  A lane holds 32 slots of one quad (4
//                       elements); up to 64 quads side by side, 4 to 16 groups of lanes one
//                       behind the other in time
//   scan_staged_kernel  smaller frames, whose rows are too short to be read lane by lane: the
//                       tile goes through LDS in both directions, whole 16-byte vectors to
//                       and from memory; a lane holds 9 to 33 slots, by what fills the tile
// Measured against the form before (a row of lanes walking a stretch of time, behind a pass over
// the open ends of the stretches): 6900 blocks of 3000 x 80 floats 3.07 -> 2.32 ms (5.0 TB/s),
// 79 blocks of 3000 x 2048 halfs 0.62 -> 0.49 ms, 300 videos of 37632 bytes a frame 1.34 -> 1.04 ms,
// 1.5 * 10^8 slots of one float 6.9 -> 0.26 ms, 37 halfs a frame 0.74 -> 0.63 ms.
#include "bload_common.hpp"

#include <hip/hip_fp16.h>
#include <cmath>

#include <algorithm>

namespace bload {

#ifndef BLOAD_SCAN_POLLS
#define BLOAD_SCAN_POLLS 16384         // looks at the tiles in front before a workgroup computes them itself
#endif

constexpr int kScanSmallFrame = 64;    // frames of fewer elements go through LDS
constexpr int kScanRow = 64;           // units (quads or elements) of a frame side by side in a workgroup
constexpr int kStagedElems = 8448;     // elements of a staged tile: 33 KiB of LDS, four workgroups per CU
constexpr int kScanLong = 32, kScanShort = 8;                  // slots per lane, and where tiles are few
constexpr int kScanStagedLong = 33, kScanStagedHalf = 17, kScanStagedShort = 9;      // odd, see scan_staged_kernel
constexpr int kScanStagedWalk = 25;    // what a walking workgroup has the registers for
constexpr int kScanGroup = 32;         // blocks whose tiles are taken side by side
constexpr int kScanLine = 32;          // floats of a cache line

// Direct tiles, how they pass the caches (scan_traffic).
enum ScanTraffic : int { kScanStream = 0, kScanCached = 1, kScanPlain = 2 };

struct ScanArgs {
    const uint8_t* packed;
    const uint8_t* reset;
    const uint8_t* valid;
    float* out;
    unsigned long long* words;         // [B, chunks - 1, feat_dim]: published states (null: chunks == 1)
    int64_t num_blocks;
    int64_t n_units;                   // blocks, or groups of blocks_per_tile blocks
    int32_t t_blk;
    int32_t feat_dim;
    int32_t chunk;                     // slots per tile = subs * K
    int32_t chunks;                    // tiles per block
    int32_t blocks_per_tile;           // chunks == 1: whole blocks per tile
    int32_t row;                       // units side by side: lanes of a group
    int32_t subs;                      // groups of lanes one behind the other in time
    int32_t slices;                    // rows needed to cover a frame
    int32_t frame_units;               // units of a frame
    int32_t group;                     // units whose tiles are taken side by side
    int32_t by_xcd;                    // every XCD takes whole blocks of its own
    uint32_t polls;
    float decay;
    double decay_sub[8];               // decay ^ (K * 2^i)
    double decay_chunk;                // decay ^ chunk
    uint32_t plain;                    // bit i: decay_sub[i] is finite and not 0; bit 8: decay_chunk
};

template <typename ElemT> struct ScanElem;
template <> struct ScanElem<uint8_t> {
    __device__ static float get(uint8_t v) { return (float)v; }
};
struct scan_half { uint16_t bits; };   // IEEE binary16 storage
template <> struct ScanElem<scan_half> {
    __device__ static float get(scan_half v) { return __half2float(__ushort_as_half(v.bits)); }
};
template <> struct ScanElem<float> {
    __device__ static float get(float v) { return v; }
};

typedef float float4v __attribute__((ext_vector_type(4)));
typedef float4v __attribute__((aligned(4))) float4v_any;
typedef vec16 __attribute__((aligned(1))) vec16_any;

// Four consecutive elements ("quad") as loaded: 4, 8 or 16 bytes in one instruction, at any address.
typedef unsigned int vec8 __attribute__((ext_vector_type(2)));
template <int BYTES> struct ScanBits;
template <> struct ScanBits<4> { typedef unsigned int T; typedef T __attribute__((aligned(1))) Any; };
template <> struct ScanBits<8> { typedef vec8 T; typedef T __attribute__((aligned(1))) Any; };
template <> struct ScanBits<16> { typedef vec16 T; typedef T __attribute__((aligned(1))) Any; };
template <typename ElemT> union ScanQuad {
    typename ScanBits<sizeof(ElemT) * 4>::T bits;
    ElemT e[4];
};

// A state and its mark in one word.
__device__ __forceinline__ unsigned long long scan_word(double v, uint32_t mark)
{
    return ((unsigned long long)__double_as_longlong(v) & ~3ull) | mark;
}
__device__ __forceinline__ double scan_value(unsigned long long w) { return __longlong_as_double((long long)(w & ~3ull)); }
__device__ __forceinline__ uint32_t scan_mark(unsigned long long w) { return (uint32_t)w & 3u; }

// The state `n` slots on: own = what those slots make of a state of 0, power = decay^n.  In 64
// bits, so that a power that float32 cannot hold does no harm.  A state of exactly 0 leaves
// `own` whatever the power is; an infinite one stays infinite when the power has become 0.  `plain`: the
// power is finite and not 0, and the multiplication does both by itself.
__device__ __forceinline__ double scan_join(double power, bool plain, double handed, double own)
{
    if (!plain) {
        if (handed == 0.0) return own;
        if (power == 0.0 && __builtin_isinf(handed)) power = __builtin_copysign(1.0, power);
    }
    return __builtin_fma(power, handed, own);
}

// A state that leaves a tile or enters a lane: what has left the range of float32 is infinite, as it is in the
// recurrence, and the mantissa is cut as a word cuts it.
__device__ __forceinline__ double scan_state(double v)
{
    return __builtin_isinf((float)v) ? (double)(float)v : scan_value(scan_word(v, 0));
}

// The recurrence at a lane's first slot, from a state in 64 bits: rounded once.
__device__ __forceinline__ float scan_first(float decay, double state, float x)
{
    return (float)__builtin_fma((double)decay, state, (double)x);
}

// Where a workgroup's tile lies: `unit` = block (or group of blocks), tile `c` of it, feature slice.
struct ScanTile {
    int64_t unit;
    int32_t c, slice;
};

// (WALK: the first tile of a block)
template <bool WALK>
__device__ __forceinline__ ScanTile scan_tile(const ScanArgs& a)
{
    const uint32_t slices = (uint32_t)a.slices, chunks = WALK ? 1u : (uint32_t)a.chunks, per_unit = chunks * slices;
    uint32_t y = blockIdx.x, first = 0, units = (uint32_t)a.n_units;
    if (a.by_xcd) {
        // workgroup b runs on XCD b mod 8: every XCD takes units of its own
        const uint32_t x = y % kXcds, most = (units + kXcds - 1) / kXcds;
        y /= kXcds;
        first = x * most;
        units = first < units ? min(most, units - first) : 0u;
    }
    const uint32_t G = (uint32_t)a.group;
    const uint32_t g = y / (G * per_unit), in_group = y - g * (G * per_unit);
    if (g * G >= units) return ScanTile{a.n_units, 0, 0};
    const uint32_t here = min(G, units - g * G);                 // units of this group
    const uint32_t c = in_group / (here * slices), rest = in_group - c * (here * slices);
    if (c >= chunks) return ScanTile{a.n_units, 0, 0};
    const uint32_t u = rest / slices;
    return ScanTile{(int64_t)(first + g * G + u), (int32_t)c, (int32_t)(rest - u * slices)};
}

// Slots of tile c of a unit: first slot (counted over all blocks), slots, place in its block.
struct ScanSpan {
    int64_t g0;
    int32_t n, rem0;
};

__device__ __forceinline__ ScanSpan scan_span(const ScanArgs& a, int64_t unit, int32_t c)
{
    ScanSpan s;
    if (a.chunks > 1) {
        s.rem0 = c * a.chunk;
        s.g0 = unit * (int64_t)a.t_blk + s.rem0;
        s.n = min(a.chunk, a.t_blk - s.rem0);
    } else {
        const int64_t b0 = unit * a.blocks_per_tile;
        s.rem0 = 0;
        s.g0 = b0 * (int64_t)a.t_blk;
        s.n = (int32_t)min((int64_t)a.blocks_per_tile, a.num_blocks - b0) * a.t_blk;
    }
    return s;
}

// What the lanes of a workgroup exchange.  Lane `tid` = group s, place q in the row.
template <int UNIT> struct ScanShared {
    alignas(16) unsigned long long word[2][kThreads][UNIT];
};

// Inclusive scan over the groups: in, v = what the lane's own slots make of a state of 0 and
// `closed` = they hold a boundary; out, the same for all slots of the tile up to the lane's last
// (left in sh.word [return value], the mark being `closed`, with a barrier behind it).
template <int UNIT>
__device__ __forceinline__ int scan_groups(const ScanArgs& a, ScanShared<UNIT>& sh, int s, const float (&own)[UNIT],
                                           uint32_t closed)
{
    const int tid = (int)threadIdx.x;
    int buf = 0;
    double v[UNIT];
#pragma unroll
    for (int k = 0; k < UNIT; ++k) v[k] = (double)own[k];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int step = 1 << i;
        if (step >= a.subs) break;
#pragma unroll
        for (int k = 0; k < UNIT; ++k) sh.word[buf][tid][k] = scan_word(v[k], closed);
        __syncthreads();
        if (s >= step && s < a.subs) {
            const int other = tid - step * a.row;
            if (!closed) {
#pragma unroll
                for (int k = 0; k < UNIT; ++k)
                    v[k] = scan_join(a.decay_sub[i], (a.plain >> i) & 1u, scan_value(sh.word[buf][other][k]), v[k]);
                closed = scan_mark(sh.word[buf][other][0]);
            }
        }
        buf ^= 1;
    }
#pragma unroll
    for (int k = 0; k < UNIT; ++k) sh.word[buf][tid][k] = scan_word(v[k], closed);
    __syncthreads();
    return buf;
}

// The state a tile on.
__device__ __forceinline__ double scan_over_tile(const ScanArgs& a, double handed, double own)
{
    return scan_state(scan_join(a.decay_chunk, (a.plain >> 8) & 1u, handed, own));
}

constexpr uint32_t kPartial = 1, kFinal = 2;

__device__ __forceinline__ void scan_publish(unsigned long long* word, double v, uint32_t mark)
{
    __hip_atomic_store(word, scan_word(v, mark), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What group s sees of tile c - 1 - s: the words of the lane's features.
template <int UNIT> struct ScanSeen {
    unsigned long long w[UNIT];
};

template <int UNIT>
__device__ __forceinline__ void scan_look(const ScanArgs& a, const unsigned long long* words, int s, bool looks,
                                          ScanSeen<UNIT>& seen)
{
#pragma unroll
    for (int k = 0; k < UNIT; ++k) seen.w[k] = 0;
    if (looks) {
        const unsigned long long* from = words - (int64_t)(1 + s) * a.feat_dim;
#pragma unroll
        for (int k = 0; k < UNIT; ++k) seen.w[k] = __hip_atomic_load(from + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The state tile c is handed, for the features of place q: true if it was found.  `words` = the
// tile's own words at the lane's first feature.  The first look is at tile c - 1 alone, whose state
// is final most of the time; where it is not, `not_yet` is called before the wait begins.  Uses
// sh.word[buf]; all lanes of the workgroup call it together and get the same answer.
template <int UNIT, typename NotYet>
__device__ __forceinline__ bool scan_look_back(const ScanArgs& a, ScanShared<UNIT>& sh, int buf,
                                               const unsigned long long* words, int s, int q, int window, bool active,
                                               double (&handed)[UNIT], NotYet not_yet)
{
    const int tid = (int)threadIdx.x;
    for (uint32_t look = 0; look < a.polls; ++look) {
        ScanSeen<UNIT> seen;
        scan_look<UNIT>(a, words, s, active && s < (look == 0 ? 1 : window), seen);
        // words that are seen half way from partial to final are none yet
        uint32_t mark = scan_mark(seen.w[0]);
#pragma unroll
        for (int k = 1; k < UNIT; ++k) mark = scan_mark(seen.w[k]) == mark ? mark : 0u;
#pragma unroll
        for (int k = 0; k < UNIT; ++k) sh.word[buf][tid][k] = (seen.w[k] & ~3ull) | mark;
        __syncthreads();
        int found = -1;
        if (active) {
            for (int j = 0; j < window; ++j) {
                const uint32_t m = scan_mark(sh.word[buf][j * a.row + q][0]);
                if (m == kFinal) found = j;
                if (m != kPartial) break;
            }
        }
        if (__syncthreads_and(!active || found >= 0)) {
            if (active) {
#pragma unroll
                for (int k = 0; k < UNIT; ++k) handed[k] = scan_value(sh.word[buf][found * a.row + q][k]);
                for (int j = found - 1; j >= 0; --j) {
#pragma unroll
                    for (int k = 0; k < UNIT; ++k)
                        handed[k] = scan_over_tile(a, handed[k], scan_value(sh.word[buf][j * a.row + q][k]));
                }
            }
            __syncthreads();
            return true;
        }
        if (look == 0) not_yet();
        else __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

// decay ^ (K * s)
__device__ __forceinline__ double scan_power(const ScanArgs& a, int s)
{
    double p = 1.0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        if ((s >> i) & 1) p *= a.decay_sub[i];
    return p;
}

// What the lane's slots of tile c, read one after another from memory, make of a state of 0, and
// whether they hold a boundary: the arithmetic of the kernels below, for the rare case that a
// workgroup computes tiles that are not its own.
template <typename ElemT, int UNIT, int K>
__device__ __forceinline__ uint32_t scan_slots_again(const ScanArgs& a, const ScanSpan& span, int s, int64_t feature,
                                                     bool active, float (&v)[UNIT])
{
    uint32_t closed = 0;
#pragma unroll
    for (int k = 0; k < UNIT; ++k) v[k] = 0.0f;
#pragma nounroll
    for (int t = s * K; active && t < min((s + 1) * K, span.n); ++t) {
        const int64_t g = span.g0 + t;
        const bool valid = a.valid[g] != 0;
        const bool first = span.rem0 + t == 0;                   // only blocks cut into tiles come here
        const bool starts = !valid || a.reset[g] != 0 || first || a.valid[g - (first ? 0 : 1)] == 0;
        closed |= starts ? 1u : 0u;
        const ElemT* x = reinterpret_cast<const ElemT*>(a.packed) + g * a.feat_dim + feature;
#pragma unroll
        for (int k = 0; k < UNIT; ++k)
            v[k] = __builtin_fmaf(a.decay, starts ? 0.0f : v[k], valid ? ScanElem<ElemT>::get(x[k]) : 0.0f);
    }
    return closed;
}

// The part both kernels share: from what the lane's slots make of a state of 0 (v), whether they
// hold a boundary (closed) and whether the tile's first slot is one (starts_closed, the same in
// all lanes), the state in front of the lane's first slot (h).  WALK: the state in front of the tile is `carried`,
// and the one behind it is left there.
template <typename ElemT, int UNIT, int K, bool WALK>
__device__ __forceinline__ void scan_carry_in(const ScanArgs& a, ScanShared<UNIT>& sh, const ScanTile& tile, int s,
                                              int q, int64_t feature, bool active, float (&v)[UNIT], uint32_t closed,
                                              bool starts_closed, double (&h)[UNIT], double (&carried)[UNIT])
{
    const int tid = (int)threadIdx.x;
    const int last = (a.subs - 1) * a.row + q;         // the lane that ends the tile at this place
    const bool open_front = tile.c > 0 && !starts_closed;
    const int buf = scan_groups(a, sh, s, v, closed);
    // what the groups in front make of a state of 0
    const bool front = s > 0 && s < a.subs;
    const bool front_closed = front && scan_mark(sh.word[buf][tid - a.row][0]) != 0;
#pragma unroll
    for (int k = 0; k < UNIT; ++k) h[k] = front ? scan_state(scan_value(sh.word[buf][tid - a.row][k])) : 0.0;
    if (a.chunks == 1) return;

    const bool publishes = tile.c + 1 < a.chunks && active && s == 0;
    const bool tile_closed = scan_mark(sh.word[buf][last][0]) != 0;
    double total[UNIT], handed[UNIT];
#pragma unroll
    for (int k = 0; k < UNIT; ++k) total[k] = scan_state(scan_value(sh.word[buf][last][k]));
    if constexpr (WALK) {
#pragma unroll
        for (int k = 0; k < UNIT; ++k) {
            handed[k] = carried[k];
            carried[k] = tile_closed ? total[k] : scan_over_tile(a, handed[k], total[k]);
        }
        if (open_front && !front_closed) {
            const double p = scan_power(a, s);
#pragma unroll
            for (int k = 0; k < UNIT; ++k) h[k] = scan_state(scan_join(p, false, handed[k], h[k]));
        }
        return;
    }
    unsigned long long* words = a.words + (tile.unit * (int64_t)(a.chunks - 1) + tile.c) * a.feat_dim + feature;
    if (publishes && tile_closed) {
#pragma unroll
        for (int k = 0; k < UNIT; ++k) scan_publish(words + k, total[k], kFinal);
    }
    if (!open_front) return;
    if (!scan_look_back<UNIT>(a, sh, buf ^ 1, words, s, q, min(a.subs, tile.c), active, handed, [&] {
            if (publishes && !tile_closed) {
#pragma unroll
                for (int k = 0; k < UNIT; ++k) scan_publish(words + k, total[k], kPartial);
            }
        })) {
        // not heard of in time: all tiles of the block in front of this one, one after another
#pragma unroll
        for (int k = 0; k < UNIT; ++k) handed[k] = 0.0;
#pragma nounroll
        for (int32_t c = 0; c < tile.c; ++c) {
            __syncthreads();
            const uint32_t any = scan_slots_again<ElemT, UNIT, K>(a, scan_span(a, tile.unit, c), s, feature, active, v);
            const int at = scan_groups(a, sh, s, v, any);
#pragma unroll
            for (int k = 0; k < UNIT; ++k) {
                const double t = scan_state(scan_value(sh.word[at][last][k]));
                handed[k] = scan_mark(sh.word[at][last][k]) ? t : scan_over_tile(a, handed[k], t);
            }
        }
    }
    if (publishes && !tile_closed) {
#pragma unroll
        for (int k = 0; k < UNIT; ++k) scan_publish(words + k, scan_over_tile(a, handed[k], total[k]), kFinal);
    }
    if (!front_closed) {
        const double p = scan_power(a, s);
#pragma unroll
        for (int k = 0; k < UNIT; ++k) h[k] = scan_state(scan_join(p, false, handed[k], h[k]));
    }
}

// Frames of 64 elements or more.  WALK, where there is no room for published states: a workgroup takes all tiles of
// its block, one after another with the state in registers: the same operations, the same bits.  (The loop's body is not indented;
// as a function of its own, with what it needs in LDS by reference, it came out 5 to 15 % slower for halfs.)
template <typename ElemT, int K, bool WALK, int TRAFFIC>
__global__ __launch_bounds__(kThreads, sizeof(ElemT) == 4 ? 2 : 3) void scan_direct_kernel(ScanArgs a)
{
    constexpr int UNIT = 4;
    constexpr int kMostSlots = kThreads / (kScanSmallFrame / 4) * K;     // groups of at least 16 lanes
    constexpr int kWords = (kMostSlots + 63) / 64;
    constexpr uint32_t ALL = K == 32 ? ~0u : (1u << (K & 31)) - 1u;
    static_assert(64 % K == 0, "the flags of a lane lie in one 64-bit word");
    __shared__ ScanShared<UNIT> sh;
    __shared__ unsigned long long s_valid[kWords], s_bound[kWords];
    ScanTile tile = scan_tile<WALK>(a);
    if (tile.unit >= a.n_units) return;
    const int tid = (int)threadIdx.x;
    const int s = (int)((uint32_t)tid / (uint32_t)a.row), q = tid - s * a.row;
    const int32_t unit = tile.slice * a.row + q;
    const bool active = s < a.subs && unit < a.frame_units;
    // a frame that is no whole number of quads: the last one lies over the end of the one before
    // (both lanes compute and store the same)
    const int64_t feature = active ? min((int64_t)unit * UNIT, (int64_t)a.feat_dim - UNIT) : 0;
    const int64_t D = a.feat_dim;
    const uint32_t lane_at = active ? (uint32_t)(s * K) * (uint32_t)a.feat_dim + (uint32_t)feature : 0u;

    double carried[UNIT] = {};         // WALK: the state in front of the tile
    do {
    ScanQuad<ElemT> x[K];
    uint32_t vm = 0, bm = 0;           // the lane's slots: valid, boundary
    const ScanSpan span = scan_span(a, tile.unit, tile.c);
    float v[UNIT], h[UNIT];
    double in[UNIT];                   // the state in front of the lane's first slot
    {
        for (int t0 = 0; t0 < a.chunk; t0 += kThreads) {
            const int t = t0 + tid;
            bool valid = false, bound = false;
            if (t < span.n) {
                const int64_t g = span.g0 + t;
                const uint32_t pos = a.chunks > 1 ? (uint32_t)(span.rem0 + t) : (uint32_t)t % (uint32_t)a.t_blk;
                const bool before = pos != 0 && a.valid[g - (pos != 0 ? 1 : 0)] != 0;
                valid = a.valid[g] != 0;
                bound = !valid || !before || a.reset[g] != 0;
            }
            const unsigned long long v64 = __ballot(valid), b64 = __ballot(bound);
            const int word = (t0 >> 6) + wave_id();
            if (lane_id() == 0 && word < kWords) { s_valid[word] = v64; s_bound[word] = b64; }
        }
        __syncthreads();
        vm = bm = 0;
        if (active) {
            vm = (uint32_t)(s_valid[(s * K) >> 6] >> ((s * K) & 63)) & ALL;
            bm = (uint32_t)(s_bound[(s * K) >> 6] >> ((s * K) & 63)) & ALL;
        }
        // wave-uniform frame addresses, 32-bit offsets of the lanes
        const int64_t frame_bytes = D * (int64_t)sizeof(ElemT);
        const uint8_t* from = a.packed + span.g0 * frame_bytes;
        const uint32_t at = lane_at * (uint32_t)sizeof(ElemT);
        typedef typename ScanBits<sizeof(ElemT) * 4>::T Bits;
        typedef typename ScanBits<sizeof(ElemT) * 4>::Any BitsAny;
        auto load = [](const uint8_t* place) -> Bits {
            const BitsAny* p = reinterpret_cast<const BitsAny*>(place);
            return TRAFFIC == kScanStream ? __builtin_nontemporal_load(p) : *p;
        };
        if (vm == ALL) {
#pragma unroll
            for (int u = 0; u < K; ++u)
                x[u].bits = load(from + u * frame_bytes + at);
        } else {
#pragma unroll
            for (int u = 0; u < K; ++u) {
                x[u].bits = Bits{};
                if ((vm >> u) & 1u)
                    x[u].bits = load(from + u * frame_bytes + at);
            }
        }
#pragma unroll
        for (int k = 0; k < UNIT; ++k) v[k] = 0.0f;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const bool starts = (bm >> u) & 1u;
#pragma unroll
            for (int k = 0; k < UNIT; ++k)
                v[k] = __builtin_fmaf(a.decay, starts ? 0.0f : v[k], ScanElem<ElemT>::get(x[u].e[k]));
        }
    }
    scan_carry_in<ElemT, UNIT, K, WALK>(a, sh, tile, s, q, feature, active, v, bm != 0u ? 1u : 0u, (s_bound[0] & 1ull) != 0, in,
                                        carried);
    if (!WALK && !active) return;
    // the payload stays packed until here: not the floats made of it above, four times as many registers
    if constexpr (sizeof(ElemT) < 4) {
#pragma unroll
        for (int u = 0; u < K; ++u) asm volatile("" : "+v"(x[u].bits));
    }

    uint8_t* to = reinterpret_cast<uint8_t*>(a.out + span.g0 * D);
    const uint32_t at = lane_at * 4u;
    const int left = active ? span.n - s * K : 0;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const bool starts = (bm >> u) & 1u;
#pragma unroll
        for (int k = 0; k < UNIT; ++k)
            h[k] = u == 0 ? scan_first(a.decay, starts ? 0.0 : in[k], ScanElem<ElemT>::get(x[u].e[k]))
                          : __builtin_fmaf(a.decay, starts ? 0.0f : h[k], ScanElem<ElemT>::get(x[u].e[k]));
        if (u < left) {
            const float4v o = {h[0], h[1], h[2], h[3]};
            float4v_any* place = reinterpret_cast<float4v_any*>(to + u * D * 4 + at);
            if (TRAFFIC == kScanPlain) *place = o;
            else __builtin_nontemporal_store(o, place);
        }
    }
    if constexpr (WALK) __syncthreads();
    } while (WALK && ++tile.c < a.chunks);
}

// The flags of the 16 slots from g on, of which `left` lie in the tile: one load that stays inside
// the plane of `total` slots (a plane of fewer than 16 is read byte by byte).
__device__ __forceinline__ uint32_t scan_flags16(const uint8_t* __restrict__ plane, int64_t g, int32_t left, int64_t total)
{
    if (left <= 0) return 0;
    const uint32_t in_tile = left >= 16 ? 0xffffu : (1u << left) - 1u;
    if (total >= 16) {
        const int64_t from = min(g, total - 16);
        return (nonzero_bytes16(*reinterpret_cast<const vec16_any*>(plane + from)) >> (int)(g - from)) & in_tile;
    }
    uint32_t m = 0;
    for (int j = 0; j < left && j < 16; ++j) m |= (uint32_t)(plane[g + j] != 0) << j;
    return m;
}

// Smaller frames.  K is odd, so that lanes K frames apart in LDS spread over the banks.
template <typename ElemT, int K, bool CACHED, bool WALK>
__global__ __launch_bounds__(kThreads, 4) void scan_staged_kernel(ScanArgs a)
{
    static_assert(K % 2 == 1 && K * kThreads <= kStagedElems && K < 34, "a lane's flags fit behind a 31-bit shift");
    constexpr int kGroups = kStagedElems / 16 + 4;     // groups of 16 flags, the last ones zero
    __shared__ ScanShared<1> sh;
    __shared__ alignas(16) float s_x[K * kThreads];
    __shared__ alignas(16) uint16_t s_valid[kGroups], s_reset[kGroups];
    ScanTile tile = scan_tile<WALK>(a);
    if (tile.unit >= a.n_units) return;
    const int tid = (int)threadIdx.x;
    const int D = a.feat_dim;
    const int s = (int)((uint32_t)tid / (uint32_t)D), q = tid - s * D;
    const bool active = s < a.subs;

    double carried[1] = {};            // WALK: the state in front of the tile
    do {
    float x[K];
    uint64_t bm = 0;                   // the lane's slots: boundary
    const ScanSpan span = scan_span(a, tile.unit, tile.c);
    float v[1], h;
    double in[1];
    bool starts_closed;
    {
        // the payload as whole vectors, all asked for before anything is waited for
        constexpr int EPV = 16 / (int)sizeof(ElemT);
        constexpr int NV = (K + EPV - 1) / EPV;
        const int elems = span.n * D, vecs = elems / EPV;
        const uint8_t* from = a.packed + span.g0 * D * (int64_t)sizeof(ElemT);
        vec16 in[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i = tid + k * kThreads;
            in[k] = vec16{0u, 0u, 0u, 0u};
            const vec16_any* at = reinterpret_cast<const vec16_any*>(from) + i;
            if (i < vecs) in[k] = CACHED ? *at : __builtin_nontemporal_load(at);
        }
        const int64_t total = a.num_blocks * (int64_t)a.t_blk;
        for (int i = tid; i < (a.chunk + 15) / 16 + 4; i += kThreads) {
            s_valid[i] = (uint16_t)scan_flags16(a.valid, span.g0 + 16 * i, span.n - 16 * i, total);
            s_reset[i] = (uint16_t)scan_flags16(a.reset, span.g0 + 16 * i, span.n - 16 * i, total);
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int i = tid + k * kThreads;
            union { vec16 v; ElemT e[EPV]; } u;
            u.v = in[k];
            if (i < vecs) {
#pragma unroll
                for (int j = 0; j < EPV; j += 4) {
                    const float4v o = {ScanElem<ElemT>::get(u.e[j]), ScanElem<ElemT>::get(u.e[j + 1]),
                                       ScanElem<ElemT>::get(u.e[j + 2]), ScanElem<ElemT>::get(u.e[j + 3])};
                    *reinterpret_cast<float4v*>(s_x + i * EPV + j) = o;
                }
            }
        }
        for (int i = vecs * EPV + tid; i < elems; i += kThreads)
            s_x[i] = ScanElem<ElemT>::get(reinterpret_cast<const ElemT*>(from)[i]);
        const bool before_tile = span.rem0 > 0 && a.valid[span.g0 - (span.rem0 > 0 ? 1 : 0)] != 0;
        __syncthreads();

        const int o = s * K, left = active ? min(K, span.n - o) : 0;
        uint64_t vm = 0;
        bm = 0;
        if (left > 0) {
            const uint32_t* v32 = reinterpret_cast<const uint32_t*>(s_valid) + (o >> 5);
            const uint32_t* r32 = reinterpret_cast<const uint32_t*>(s_reset) + (o >> 5);
            const uint64_t in_range = ~0ull >> (64 - left);
            vm = (((uint64_t)v32[1] << 32 | v32[0]) >> (o & 31)) & in_range;
            const uint64_t rm = ((uint64_t)r32[1] << 32 | r32[0]) >> (o & 31);
            const uint64_t before = o > 0 ? (s_valid[(o - 1) >> 4] >> ((o - 1) & 15)) & 1u : (uint32_t)before_tile;
            const uint32_t T = (uint32_t)a.t_blk, pos = (uint32_t)(span.rem0 + o) % T;
            uint64_t first = 0;
            for (uint32_t k = pos == 0 ? 0 : T - pos; k < (uint32_t)left; k += T) first |= 1ull << k;
            bm = (~vm | rm | first | ~(vm << 1 | before)) & in_range;
        }
#pragma unroll
        for (int u = 0; u < K; ++u) x[u] = (vm >> u) & 1u ? s_x[(o + u) * D + q] : 0.0f;
        float t = 0.0f;
#pragma unroll
        for (int u = 0; u < K; ++u) t = __builtin_fmaf(a.decay, (bm >> u) & 1u ? 0.0f : t, x[u]);
        v[0] = t;
        starts_closed = !before_tile || (s_reset[0] & 1u) || !(s_valid[0] & 1u);
    }
    scan_carry_in<ElemT, 1, K, WALK>(a, sh, tile, s, q, q, active, v, bm != 0 ? 1u : 0u, starts_closed, in, carried);

    const int left = active ? span.n - s * K : 0;
#pragma unroll
    for (int u = 0; u < K; ++u) {
        const bool starts = (bm >> u) & 1u;
        h = u == 0 ? scan_first(a.decay, starts ? 0.0 : in[0], x[u]) : __builtin_fmaf(a.decay, starts ? 0.0f : h, x[u]);
        if (u < left) s_x[(s * K + u) * D + q] = h;
    }
    __syncthreads();
    const int elems = span.n * D, quads = elems / 4;
    float* to = a.out + span.g0 * D;
    for (int i = tid; i < quads; i += kThreads)
        __builtin_nontemporal_store(*reinterpret_cast<const float4v*>(s_x + 4 * i), reinterpret_cast<float4v_any*>(to) + i);
    for (int i = quads * 4 + tid; i < elems; i += kThreads) __builtin_nontemporal_store(s_x[i], to + i);
    if constexpr (WALK) __syncthreads();
    } while (WALK && ++tile.c < a.chunks);
}

// No state is published yet.
__global__ __launch_bounds__(kThreads) void scan_clear_kernel(unsigned long long* words, int64_t n)
{
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) words[i] = 0;
}

struct ScanPlan {
    bool staged;
    bool cached;                       // staged: plain loads
    ScanTraffic traffic;               // direct
    int32_t k;                         // slots per lane
    int32_t row, subs, slices, frame_units;
    int32_t chunk, chunks, blocks_per_tile;
    int64_t n_units, grid;
    bool by_xcd;
    size_t bytes;                      // workspace: the published states
    bool walk;                         // no room for them: a workgroup per block
};

// The share of a tile's lanes that have slots, whether a tile holds whole blocks or a block is cut into tiles.
static double scan_tile_use(int64_t tile, int32_t t_blk)
{
    if (t_blk <= tile) return (double)(tile / t_blk * t_blk) / (double)tile;
    return (double)t_blk / (double)(ceil_div(t_blk, tile) * tile);
}

// Slots per lane of a staged tile: as many as leave the fewest lanes idle, unless it is a tenth or two that is
// gained (624 shapes; 101 slots x 37 halfs in tiles of 198 slots 92 us, of 102 slots 77; 72 x 63 floats, 132 and 84: 25
// and 22; 400 x 20 floats, two tiles of 396 and two of 204: 28.7 and 22; where all lengths fill alike they
// differ by as much to either side).
static int32_t scan_staged_slots(int32_t groups, int32_t t_blk)
{
    int32_t best = 0;
    double most = 0.0;
    for (int32_t k = kScanStagedLong; k >= kScanStagedHalf; k -= 4) {
        const double worth = scan_tile_use((int64_t)groups * k, t_blk) * (1.0 - 0.0125 * (kScanStagedLong - k));
        if (worth > most) { most = worth; best = k; }
    }
    return best;
}

// How direct tiles of 32 slots a lane read and write.
//   - Input that bload_pack leaves in the memory-side cache (256 MB of packed tensor, source and table) is read with plain loads
//     from there.  Scans behind a pack of the same tensor: 50 MB of 2048 halfs 43 -> 38 us, 94 MB of 320 bytes 67 -> 52, 640 bytes, 50 MB 78 -> 57; of
//     an input that lies in memory only 0 to 5 % slower (25 MB of 2048 halfs 21.8 us, 22.9).  Larger input is streamed: up to 256 MB plain
//     loads gained where the same tensor is scanned again and again (204 MB of 80 floats 89 -> 72 us), but behind a kernel that wrote a
//     gigabyte the input pushed its lines out: 300 MB of 2048 halfs 124 us streamed, 147; 200 MB of 256 floats 88 and 107.
//   - Where output lines are written by two workgroups (frames of several slices) or twice by one (frames that are no whole
//     half lines), in parts, streaming stores send both parts to memory; plain ones meet in the cache.  270 halfs, 1.2
//     GB: 1034 -> 820 us, 2415 of them 1710 -> 1504, 72 bytes 868 -> 736, 100 floats 504 -> 454; whole lines lose as much by it (256 floats 372
//     -> 418), and single slices from 192 elements on gain nothing (250 halfs 764 and 780).  Of single slices, input and output of 300 MB in
//     all stay in the cache, too (400 bytes, 51 MB 35 -> 28 us, 98 bytes, 57 MB 92 -> 74, also from memory 76 halfs, 74 MB 70 -> 61, but 400 bytes
//     31.4 and 33.1); below 40 MB the write-back at the call's end costs more than that (400 bytes, 26 MB from memory 17.2 us, 20.2).
//     Several slices are streamed there: 1273 halfs, 53 MB 51 us and 60 with plain stores, 3279, 76 MB 65 and 74, 2008 floats, 104 MB 53 and 56.
static ScanTraffic scan_traffic(int64_t elems, size_t elem, int64_t feat_dim, bool one_slice)
{
    const int64_t bytes = elems * (int64_t)elem;
    const bool kept = 2 * bytes + 10 * (elems / feat_dim) <= ((int64_t)256 << 20);
    const bool parts = one_slice ? feat_dim % (kScanLine / 2) != 0 && feat_dim < 192 : feat_dim % kScanLine != 0;
    if (parts && bytes > ((int64_t)256 << 20)) return kScanPlain;
    if (one_slice && parts && kept && bytes >= ((int64_t)40 << 20) && bytes + 4 * elems <= ((int64_t)300 << 20)) return kScanPlain;
    return kept ? kScanCached : kScanStream;
}

// `walk`: a block's tiles go to one workgroup, as long as there are.  `lines`: slices of whole cache lines.
static ScanPlan scan_plan(int64_t num_blocks, int32_t t_blk, int64_t feat_dim, size_t elem, bool walk = false, bool lines = true)
{
    ScanPlan p{};
    p.staged = feat_dim < kScanSmallFrame;
    // what was just written or read lies in the memory-side cache if it fits there, and plain loads fetch it
    // sooner (0.1 GB of 252-byte frames: 62 us with streaming loads, 49 plain); of small tensors they do not
    // (40 MB of 64-byte frames: 18 and 20)
    const int64_t elems = num_blocks * t_blk * feat_dim;
    p.cached = p.staged && !walk && elems > ((int64_t)16 << 20) && elems * (int64_t)elem <= ((int64_t)256 << 20);
    p.frame_units = (int32_t)(p.staged ? feat_dim : ceil_div(feat_dim, 4));
    // slices of equal width; a width of which the workgroup's 256 lanes hold a whole number
    p.slices = p.staged ? 1 : (int32_t)ceil_div(p.frame_units, kScanRow);
    p.row = (int32_t)ceil_div(p.frame_units, p.slices);
    // and of whole cache lines where frames are, or two workgroups would write the lines between them (1056 bytes, five
    // slices of 848 bytes of output: 289 -> 224 us, 800 floats 448 -> 383, 960 halfs 69 -> 64)
    if (lines && p.slices > 1 && feat_dim % kScanLine == 0) p.row = (int32_t)round_up((size_t)p.row, kScanLine / 4);
    p.traffic = scan_traffic(elems, elem, feat_dim, p.slices == 1);
    int32_t most_subs = kThreads / p.row;
    // slots per lane: 64 registers of payload; fewer where that leaves the chip without enough tiles
    p.k = !p.staged ? kScanLong : walk ? kScanStagedWalk : scan_staged_slots(most_subs, t_blk);
    const int32_t small_k = p.staged ? kScanStagedShort : kScanShort;
    // shorter tiles where the long ones are too few to fill the chip, but none that cut a block (a
    // chain of hand-overs costs more than idle CUs: 82 blocks of 109 slots x 874 bytes took 28 us in
    // four tiles per block, 20 us in one)
    if (!walk && t_blk <= most_subs * small_k && num_blocks / (most_subs * p.k / t_blk) * p.slices < 512) {
        // (staged: of two short lengths the one that fills; 30 slots x 37 halfs, 4 MB: 9 slots a lane 10.2 us, 17 7.4)
        const bool half = p.staged && scan_tile_use((int64_t)most_subs * kScanStagedHalf, t_blk) >= scan_tile_use((int64_t)most_subs * small_k, t_blk);
        p.k = half ? kScanStagedHalf : small_k;
    }
    // the lanes' places in a tile are 32-bit byte offsets from its first slot
    if (!p.staged) most_subs = (int32_t)std::min<int64_t>(most_subs, std::max<int64_t>(1, ((int64_t)1 << 32) / (4 * p.k * feat_dim)));
    const int64_t most = (int64_t)most_subs * p.k;
    if (t_blk > most) {
        p.chunks = (int32_t)ceil_div(t_blk, most);
        p.subs = (int32_t)ceil_div(ceil_div(t_blk, p.chunks), p.k);
        p.chunk = p.subs * p.k;
        p.chunks = (int32_t)ceil_div(t_blk, p.chunk);
        p.blocks_per_tile = 1;
        p.n_units = num_blocks;
    } else {
        p.chunks = 1;
        p.subs = most_subs;
        p.chunk = (int32_t)most;
        p.blocks_per_tile = (int32_t)(most / t_blk);
        p.n_units = ceil_div(num_blocks, p.blocks_per_tile);
    }
    p.walk = walk && p.chunks > 1;
    const int64_t per_unit = p.walk ? p.slices : (int64_t)p.chunks * p.slices;
    // every XCD gets whole blocks where there are enough of them for equal shares
    p.by_xcd = p.n_units >= 256;
    p.grid = p.by_xcd ? ceil_div(p.n_units, kXcds) * kXcds * per_unit : p.n_units * per_unit;
    p.bytes = p.walk ? 0 : round_up((size_t)num_blocks * (size_t)(p.chunks - 1) * (size_t)feat_dim * sizeof(unsigned long long), 16);
    return p;
}

// The least workspace that a scan is given: a boundary mark and float32 states for stretches of 64 slots and more,
// as many as fill the chip, and none where the blocks do that alone.
static size_t scan_least_bytes(int64_t num_blocks, int32_t t_blk, int64_t feat_dim, size_t elem)
{
    const bool vectors = feat_dim * (int64_t)elem % 16 == 0 && num_blocks * t_blk >= 8;
    const int64_t units = vectors ? feat_dim / 4 : feat_dim, per_lane = vectors ? 4 / (int64_t)elem : 1;
    int64_t lanes = 1;
    while (lanes < kWave && lanes * per_lane < units) lanes *= 2;
    const int64_t waves = 6144 * (kWave / lanes), rows = num_blocks * ceil_div(units, lanes * per_lane);
    const int64_t parts = std::min<int64_t>(ceil_div(waves, rows), std::max<int32_t>(1, t_blk / 64));
    const int64_t stretch = (int64_t)round_up((size_t)ceil_div(t_blk, parts), 8);
    const size_t borders = (size_t)num_blocks * (size_t)(ceil_div(t_blk, stretch) - 1);
    return round_up(borders * (size_t)feat_dim * sizeof(float), 16) + round_up(borders, 16);
}

static size_t scan_elem_bytes(bload_dtype dtype)
{
    return dtype == BLOAD_U8 ? 1 : (dtype == BLOAD_F16 ? 2 : 4);
}

template <typename ElemT, bool CACHED>
static void scan_launch_staged(const ScanArgs& a, const ScanPlan& p, hipStream_t stream)
{
    const dim3 grid((uint32_t)p.grid), block(kThreads);
    switch (p.k) {
        case 33: hipLaunchKernelGGL((scan_staged_kernel<ElemT, 33, CACHED, false>), grid, block, 0, stream, a); break;
        case 29: hipLaunchKernelGGL((scan_staged_kernel<ElemT, 29, CACHED, false>), grid, block, 0, stream, a); break;
        case 25: hipLaunchKernelGGL((scan_staged_kernel<ElemT, 25, CACHED, false>), grid, block, 0, stream, a); break;
        case 21: hipLaunchKernelGGL((scan_staged_kernel<ElemT, 21, CACHED, false>), grid, block, 0, stream, a); break;
        case 17: hipLaunchKernelGGL((scan_staged_kernel<ElemT, 17, CACHED, false>), grid, block, 0, stream, a); break;
        default: hipLaunchKernelGGL((scan_staged_kernel<ElemT, kScanStagedShort, false, false>), grid, block, 0, stream, a); break;
    }
}

template <typename ElemT>
static void scan_launch(const ScanArgs& a, const ScanPlan& p, hipStream_t stream)
{
    const dim3 grid((uint32_t)p.grid), block(kThreads);
    if (p.chunks > 1 && !p.walk) {
        const int64_t words = (int64_t)(p.bytes / sizeof(unsigned long long));
        const int64_t groups = ceil_div(words, kThreads);
        hipLaunchKernelGGL(scan_clear_kernel, dim3((uint32_t)(groups < 4096 ? groups : 4096)), block, 0, stream,
                           a.words, words);
    }
    if (p.walk) {
        if (p.staged) hipLaunchKernelGGL((scan_staged_kernel<ElemT, kScanStagedWalk, false, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((scan_direct_kernel<ElemT, kScanLong, true, kScanStream>), grid, block, 0, stream, a);
        return;
    }
    if (p.staged && p.cached) scan_launch_staged<ElemT, true>(a, p, stream);
    else if (p.staged) scan_launch_staged<ElemT, false>(a, p, stream);
    else if (p.k != kScanLong) hipLaunchKernelGGL((scan_direct_kernel<ElemT, kScanShort, false, kScanStream>), grid, block, 0, stream, a);
    else if (p.traffic == kScanStream) hipLaunchKernelGGL((scan_direct_kernel<ElemT, kScanLong, false, kScanStream>), grid, block, 0, stream, a);
    else if (p.traffic == kScanCached) hipLaunchKernelGGL((scan_direct_kernel<ElemT, kScanLong, false, kScanCached>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((scan_direct_kernel<ElemT, kScanLong, false, kScanPlain>), grid, block, 0, stream, a);
}

}  // namespace bload

using namespace bload;

extern "C" size_t bload_segment_scan_workspace_bytes(int64_t num_blocks, int32_t t_blk, int64_t feat_dim,
                                                     bload_dtype dtype)
{
    if (num_blocks < 0 || t_blk < 1 || feat_dim < 1 || feat_dim > (1 << 28)) return 0;
    if (dtype != BLOAD_U8 && dtype != BLOAD_F16 && dtype != BLOAD_F32) return 0;
    return scan_plan(num_blocks, t_blk, feat_dim, scan_elem_bytes(dtype)).bytes;
}

extern "C" bload_status bload_segment_scan(const void* d_packed, const uint8_t* d_reset,
                                           const uint8_t* d_valid, int64_t num_blocks, int32_t t_blk,
                                           int64_t feat_dim, bload_dtype dtype, float decay,
                                           float* d_out, void* d_workspace, size_t workspace_bytes,
                                           void* hip_stream)
{
    if (num_blocks < 0 || t_blk < 1 || feat_dim < 1 || feat_dim > (1 << 28)) return BLOAD_EINVAL;
    if (dtype != BLOAD_U8 && dtype != BLOAD_F16 && dtype != BLOAD_F32) return BLOAD_EINVAL;
    if (num_blocks == 0) return BLOAD_OK;
    if (!d_packed || !d_reset || !d_valid || !d_out) return BLOAD_EINVAL;
    if (!aligned_to(d_packed, 16) || !aligned_to(d_out, 16)) return BLOAD_EALIGN;
    if (num_blocks * (int64_t)t_blk >= ((int64_t)1 << 40)) return BLOAD_EOVERFLOW;
    ScanPlan p = scan_plan(num_blocks, t_blk, feat_dim, scan_elem_bytes(dtype));
    const size_t room = d_workspace && aligned_to(d_workspace, 16) ? workspace_bytes : 0;
    if (room < p.bytes) p = scan_plan(num_blocks, t_blk, feat_dim, scan_elem_bytes(dtype), false, false);
    if (room < p.bytes) {
        const size_t least = std::min(p.bytes, scan_least_bytes(num_blocks, t_blk, feat_dim, scan_elem_bytes(dtype)));
        if (least > 0) {
            if (!d_workspace) return BLOAD_EINVAL;
            if (!aligned_to(d_workspace, 16)) return BLOAD_EALIGN;
            if (workspace_bytes < least) return BLOAD_EWORKSPACE;
        }
        p = scan_plan(num_blocks, t_blk, feat_dim, scan_elem_bytes(dtype), true);
    }
    if (p.grid > 0x7fffffffLL) return BLOAD_EOVERFLOW;

    ScanArgs a{};
    a.packed = static_cast<const uint8_t*>(d_packed);
    a.reset = d_reset;
    a.valid = d_valid;
    a.out = d_out;
    a.words = static_cast<unsigned long long*>(d_workspace);
    a.num_blocks = num_blocks;
    a.n_units = p.n_units;
    a.t_blk = t_blk;
    a.feat_dim = (int32_t)feat_dim;
    a.chunk = p.chunk;
    a.chunks = p.chunks;
    a.blocks_per_tile = p.blocks_per_tile;
    a.row = p.row;
    a.subs = p.subs;
    a.slices = p.slices;
    a.frame_units = p.frame_units;
    a.by_xcd = p.by_xcd ? 1 : 0;
    a.group = p.chunks > 1 && !p.walk ? (int32_t)std::min<int64_t>(kScanGroup, p.n_units) : 1;
    a.polls = BLOAD_SCAN_POLLS;
    a.decay = decay;
    double power = pow((double)decay, (double)p.k);
    for (int i = 0; i < 8; ++i, power *= power) {
        a.decay_sub[i] = power;
        if (std::isfinite(power) && power != 0.0) a.plain |= 1u << i;
    }
    a.decay_chunk = pow((double)decay, (double)p.chunk);
    if (std::isfinite(a.decay_chunk) && a.decay_chunk != 0.0) a.plain |= 1u << 8;

    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (dtype == BLOAD_U8) scan_launch<uint8_t>(a, p, stream);
    else if (dtype == BLOAD_F16) scan_launch<scan_half>(a, p, stream);
    else scan_launch<float>(a, p, stream);
    return launch_status();
}
