// bload_segment_reduce: per-sequence sum / mean over the packed blocks, using
// only the packed tensor and the per-slot start table (BLoad, Methods section:
// the table of starting indices lets a consumer that carries state from frame
// to frame drop it where a new sequence begins).
//
// A segment is a maximal run of valid slots inside one block that begins at a
// start flag, at the block's first slot or behind a padding slot, and contains
// no other start flag.
// Time is cut into chunks; every chunk reduces the pieces of segments that lie
// in it.  A piece that is a whole segment goes straight to the output.  A
// piece cut by a chunk border goes to a partial buffer: "head" partial = the
// piece that continues a segment begun in an earlier chunk, "tail" partial =
// the piece that begins a segment continued in the next chunk.  A second
// small kernel adds tail + following heads in time order.  Fixed chunking and
// fixed order make the float32 result bit-reproducible.
//
// Four layouts of the work (reduce_plan and takes_flat draw the lines between them):
//   wide    frames of 64 bytes or more: a row of lanes (at most one wave) lies across the features of a frame, 16
//           bytes to a lane, or 4, or one element where frames are no whole vectors or workgroups too few;
//           each row walks one chunk of time (or two waves share it) serially with several loads in flight, restarting its
//           accumulators at every start flag.
//   staged  frames of 2 to 63 elements that are smaller, or of which wide rows would be too few workgroups: a tile of
//           slots goes through LDS as whole vectors, and each lane then sums 9 or 17 slots of one feature.
//   flat    frames of up to 512 bytes, whole multiples of which are at most a wave's 64 vectors, in pieces of some KB: a wave
//           takes the bytes of a piece as one stream, 16 to a lane, and adds the lanes' sums up by feature at its end.
//   narrow  frames of one element that are not wide: lanes across time, 16 consecutive slots per lane, segmented scan
//           over the workgroup with the segment breaks as heads and a carry between lanes and waves.
#include "bload_common.hpp"

#include <hip/hip_fp16.h>
#include <limits.h>

#include <algorithm>
#include <type_traits>

namespace bload {

constexpr int kHeadNone = 0, kHeadClosed = 1, kHeadThrough = 2;

struct ChunkDesc {
    int32_t head_state;   // kHead*: is there a piece continuing an earlier segment, and does
                          // it run through the whole chunk into the next one
    int32_t cnt_head;     // frames in that piece
    int32_t cnt_tail;     // frames in the piece that continues into the next chunk, 0 if none
    int32_t seq_tail;     // sequence id of that piece
};

struct ReduceArgs {
    const uint8_t* packed;
    const int32_t* seq_id;
    const uint8_t* reset;
    const uint8_t* valid;
    int64_t num_blocks;
    int64_t total_slots;
    int64_t total_chunks;
    int32_t t_blk;
    int32_t feat_dim;
    int32_t n_seq;
    int32_t mean;            // 1: divide by the frame count
    // narrow: a block is cut into `n_chunks` tiles (t_blk >= the tile), or a tile holds
    // `blocks_per_tile` whole blocks (t_blk < the tile); magic_t_blk = min(ceil(2^32 / t_blk),
    // 2^32 - 1) then divides positions inside a tile by t_blk (to within one, fixed up)
    int32_t blocks_per_tile;
    uint32_t magic_t_blk;
    void* out;               // [n_seq, feat_dim] float or int64
    // chunking
    int32_t chunk;           // slots per chunk
    int32_t split;           // wide, rows of one wave: 1 if two waves share a chunk
    int32_t reach;           // then: slots behind a chunk that a segment begun in it may end in and stay whole
    int32_t tile;            // staged, several tiles per workgroup: slots per tile
    int32_t n_chunks;        // wide: chunks per block
    int32_t row_lanes_log2;  // wide: lanes per row = 1 << this
    int32_t n_vec;           // wide: lanes needed to cover one frame
    int32_t feat_tiles;      // wide: workgroups side by side over one frame
    int32_t step_vec;        // flat: vectors that a wave takes in one step, a whole number of frames
    int32_t step_frames;     // and how many frames those are
    uint32_t step_magic;     // floor(2^32 / step_frames) + 1: divides counts of up to 2^16 frames
    // partial buffers (null when no chunk border can cut a segment)
    ChunkDesc* desc;         // [total_chunks]
    void* head_part;         // [total_chunks, feat_dim] accumulators; [total_chunks, 2, feat_dim] floats and
    void* tail_part;         // what they lack, where `pair_parts`
    int32_t pair_parts;
};

// ---- element access -----------------------------------------------------------

template <typename ElemT> struct Elem;
template <> struct Elem<uint8_t> {
    typedef float Acc;
    // a piece of a chunk holds fewer than 2^15 frames of at most 255: every float sum of
    // them is a whole number below 2^24, i.e. exact, and needs no compensation
    static constexpr bool kCompensate = false;
    __device__ static float get(uint8_t v) { return (float)v; }
};
struct half_bits { uint16_t bits; };           // IEEE binary16 storage
template <> struct Elem<half_bits> {
    typedef float Acc;
    static constexpr bool kCompensate = true;
    __device__ static float get(half_bits v) { return __half2float(__ushort_as_half(v.bits)); }
};
template <> struct Elem<float> {
    typedef float Acc;
    static constexpr bool kCompensate = true;
    __device__ static float get(float v) { return v; }
};
template <> struct Elem<int32_t> {
    typedef long long Acc;
    static constexpr bool kCompensate = false;
    __device__ static long long get(int32_t v) { return (long long)v; }
};

typedef vec16 __attribute__((aligned(1))) vec16_any;      // a 16-byte vector at any address

// The elements of one lane, 16 bytes or fewer, in one load at any address.
template <int BYTES> struct LaneBits;
template <> struct LaneBits<16> { typedef vec16 T; typedef vec16_any Any; };
template <> struct LaneBits<4> { typedef uint32_t T; typedef uint32_t __attribute__((aligned(1))) Any; };
template <> struct LaneBits<2> { typedef uint16_t T; typedef uint16_t __attribute__((aligned(1))) Any; };
template <> struct LaneBits<1> { typedef uint8_t T; typedef uint8_t Any; };

// STREAM: a streaming load, for tensors that do not fit the memory-side cache.  Rows of narrow lanes
// share cache lines with the rows beside them, which a streaming load would fetch again (78 slots x
// 271 int32: 174 us, 143 us with plain loads), and what fits the cache is worth keeping there (4300
// blocks of 30 slots x 113 bytes 108 us streamed, 89 plain; 800 MB of 320-byte frames 279 and 305).
template <typename ElemT, int VEC, bool STREAM>
struct LaneData {
    typedef LaneBits<VEC * (int)sizeof(ElemT)> Bits;
    union { typename Bits::T v; ElemT e[VEC]; } u;
    __device__ __forceinline__ void load(const uint8_t* p)
    {
        if (STREAM) u.v = __builtin_nontemporal_load(reinterpret_cast<const typename Bits::Any*>(p));
        else u.v = *reinterpret_cast<const typename Bits::Any*>(p);
    }
};
constexpr int64_t kMemorySideCache = (int64_t)256 << 20;

template <typename Acc> struct OutOf;
template <> struct OutOf<float> { typedef float T; };
template <> struct OutOf<long long> { typedef long long T; };

// A running sum that many terms are added to, one after the other.  Integers are
// exact.  A float sum (COMPENSATED) carries the rounding error of every addition
// along (Kahan's compensated summation), so that its error stays at about two
// units in the last place of the sum of the |terms| however many there are,
// instead of growing with their number.  Once the sum has left the finite range
// the compensation is dropped, so that infinities add up as in plain arithmetic.
template <typename Acc, bool COMPENSATED> struct Running {
    Acc sum;
    __device__ __forceinline__ void clear() { sum = 0; }
    __device__ __forceinline__ void add(Acc term) { sum += term; }
    __device__ __forceinline__ Acc missing() const { return 0; }
};
template <> struct Running<float, true> {
    float sum, lost;
    __device__ __forceinline__ void clear() { sum = 0.0f; lost = 0.0f; }
    __device__ __forceinline__ void add(float term)
    {
        const float y = term - lost;
        const float t = sum + y;
        const float l = (t - sum) - y;
        lost = __builtin_isfinite(t) ? l : 0.0f;
        sum = t;
    }
    __device__ __forceinline__ float missing() const { return -lost; }      // what `sum` lacks
};

template <typename Acc>
__device__ __forceinline__ Acc finish(Acc sum, int32_t cnt, int mean)
{
    return sum;
}
template <>
__device__ __forceinline__ float finish<float>(float sum, int32_t cnt, int mean)
{
    return mean ? sum / (float)cnt : sum;
}
template <>
__device__ __forceinline__ double finish<double>(double sum, int32_t cnt, int mean)
{
    return mean ? sum / (double)cnt : sum;
}

// ------------------------------------------------------------------- wide

constexpr int kWideUnroll = 8;
constexpr int64_t kShortPieces = 32;       // slots per row of the result
constexpr int32_t kReach = 32;             // longer ones gain no more, and leave waves with more slots than others
constexpr int kWideFlagBytes = 32768;      // LDS budget for the staged flags: also the longest chunk
static_assert((int64_t)kWideFlagBytes * 255 < ((int64_t)1 << 24), "uint8 pieces must sum exactly in float");

// First slot s in [t, len) whose staged flags say "valid" (WANT_VALID) or "not a
// plain continuation: padding or a start flag" (!WANT_VALID); len if none.  The
// lanes of a row (a whole wave, or an aligned part of one) test one slot
// each per step and vote; every lane of the row gets the same answer.  WAVE_ROW:
// the row is the whole wave, and everything here but the tested slot is wave-uniform.
template <bool WANT_VALID, bool WAVE_ROW>
__device__ __forceinline__ int32_t next_slot(const uint8_t* flags, int32_t t, int32_t len,
                                             int row_lanes_log2)
{
    const int width = WAVE_ROW ? kWave : (1 << row_lanes_log2);
    const int lane = lane_id();
    const int base = WAVE_ROW ? 0 : lane & ~(width - 1);
    const uint64_t row_mask = WAVE_ROW ? ~0ull : ((1ull << width) - 1ull) << base;
    for (; t < len; t += width) {
        const int32_t s = t + (lane - base);
        bool hit = false;
        if (s < len) {
            const uint8_t f = flags[s];
            hit = WANT_VALID ? (f & 1) != 0 : (f & 3) != 1;
        }
        const uint64_t vote = __ballot(hit) & row_mask;
        if (vote) return t + (__ffsll((unsigned long long)vote) - 1 - base);
    }
    return len;
}

// Elements of LDS scratch per lane for the transposed stores: the lane's VEC values plus
// padding against bank conflicts (a multiple of 4 for floats, which move 16 bytes at a time).
template <typename Acc, int VEC>
__host__ __device__ constexpr int kScratchStride() { return sizeof(Acc) == 4 ? VEC + 4 : VEC + 1; }

// Store the VEC accumulators of every lane of a row to dst[feat0 ...].  A lane
// holds VEC consecutive features, so storing straight from the registers
// writes 16-byte pieces 16 * VEC bytes apart; when a whole wave belongs to one
// row the values go through the wave's LDS scratch instead and leave as runs
// of 64 consecutive elements.  `scratch` is null for rows narrower than a wave.
// The last lane of a frame that is no whole number of vectors holds its last VEC
// features, some of them its neighbour's as well: it stores its own.
template <typename Acc, int VEC>
__device__ __forceinline__ void store_row(Acc* dst_row, int64_t feat0, const Acc (&v)[VEC],
                                          bool lane_stores, Acc* scratch, int64_t wave_feat0,
                                          int32_t feat_dim)
{
    const int32_t whole = feat_dim - feat_dim % VEC;      // features of whole vectors
    if (lane_stores && (VEC == 1 || scratch == nullptr || feat0 + VEC > whole)) {
#pragma unroll
        for (int k = 0; k < VEC; ++k) dst_row[feat0 + k] = v[k];
    }
    if (VEC == 1 || scratch == nullptr) return;
    const int lane = lane_id();
    constexpr int S = kScratchStride<Acc, VEC>();
    // element e of the wave's 64 * VEC span lives in lane e / VEC, register e % VEC
    if constexpr (sizeof(Acc) == 4 && VEC % 4 == 0) {
      if ((reinterpret_cast<uintptr_t>(dst_row) & 15) == 0) {
        // four floats at a time: VEC / 4 stores of 1 KiB per wave
        typedef float float4v __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int k = 0; k < VEC; k += 4) {
            const float4v q = {(float)v[k], (float)v[k + 1], (float)v[k + 2], (float)v[k + 3]};
            *reinterpret_cast<float4v*>(reinterpret_cast<float*>(scratch) + lane * S + k) = q;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < VEC / 4; ++j) {
            const int e = j * kWave * 4 + lane * 4;
            const float4v q = *reinterpret_cast<const float4v*>(reinterpret_cast<const float*>(scratch) +
                                                                (e / VEC) * S + (e % VEC));
            if (wave_feat0 + e < whole)
                *reinterpret_cast<float4v*>(reinterpret_cast<float*>(dst_row) + wave_feat0 + e) = q;
        }
        __builtin_amdgcn_wave_barrier();
        return;
      }
    }
#pragma unroll
    for (int k = 0; k < VEC; ++k) scratch[lane * S + k] = v[k];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
        const int e = j * kWave + lane;
        const Acc x = scratch[(e / VEC) * S + (e % VEC)];
        if (wave_feat0 + e < whole) dst_row[wave_feat0 + e] = x;
    }
    __builtin_amdgcn_wave_barrier();
}

// WAVE_ROW: a row of lanes is exactly one wave.  Its chunk, the pieces found in it and the
// addresses of the frames are then the same for all lanes of the wave, and saying so (the row
// index goes through readfirstlane) lets the compiler keep them in scalar registers and address
// the loads as scalar base + lane offset.
template <typename ElemT, int VEC, bool WAVE_ROW, bool STREAM>
__global__ __launch_bounds__(kThreads) void reduce_wide_kernel(ReduceArgs a)
{
    typedef typename Elem<ElemT>::Acc Acc;
    extern __shared__ uint8_t s_flags[];   // chunks x (chunk + reach + 2): bit0 valid, bit1 reset
    const int tid = (int)threadIdx.x;
    const int split = WAVE_ROW ? a.split : 0, reach = WAVE_ROW ? a.reach : 0;
    const int C = a.chunk, stride = C + reach + 2;
    const int chunks = (kThreads >> a.row_lanes_log2) >> split;       // of the workgroup
    // consecutive workgroups take the lane-slices of one frame range, so that
    // workgroups running side by side read neighbouring memory
    const int feat_tile = (int)(blockIdx.x % (uint32_t)a.feat_tiles);
    const int64_t q_base = (int64_t)(blockIdx.x / (uint32_t)a.feat_tiles) * chunks;
    const int64_t T = a.t_blk;

    // stage the flags of this workgroup's chunks, plus the slot before and the slots as far as a segment
    // is followed behind each chunk (0 outside the block): row r holds slots t0-1 .. t0+len+reach
    for (int r = 0; r < chunks; ++r) {
        const int64_t q = q_base + r;
        if (q >= a.total_chunks) break;
        const int64_t b = q / a.n_chunks;
        const int32_t t0 = (int32_t)(q - b * a.n_chunks) * C;
        const int32_t len = min(C, a.t_blk - t0);
        const int64_t g = b * T + t0;
        for (int t = tid - 1; t <= len + reach; t += kThreads) {
            uint8_t f = 0;
            if (t0 + t >= 0 && t0 + t < a.t_blk)
                f = (uint8_t)((a.valid[g + t] ? 1 : 0) | (a.reset[g + t] ? 2 : 0));
            s_flags[r * stride + 1 + t] = f;
        }
    }
    __syncthreads();

    const int row = WAVE_ROW ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> a.row_lanes_log2;
    const int col = WAVE_ROW ? lane_id() : tid & ((1 << a.row_lanes_log2) - 1);
    const int64_t q = q_base + (row >> split);
    if (q >= a.total_chunks) return;
    // which lane-slice of the frame; the surplus lanes of a row stay alive (they
    // take part in the votes of next_slot), read what the last lane reads, and store nothing
    const int fv_raw = feat_tile * (1 << a.row_lanes_log2) + col;
    const bool lane_stores = fv_raw < a.n_vec;
    const int fv = lane_stores ? fv_raw : a.n_vec - 1;

    const int64_t b = q / a.n_chunks;
    const int32_t t0 = (int32_t)(q - b * a.n_chunks) * C;
    const int64_t g = b * T + t0;
    const uint8_t* flags = s_flags + (row >> split) * stride + 1;      // flags[-1] = the slot before the chunk
    // Two waves to a chunk: they part where a segment begins or ends next to the middle, at the chunk's end if none does.  A
    // segment that runs out of the chunk and ends within `reach` slots stays whole as well; the next chunk sees the same
    // flags and leaves it out.  (`reach` is no longer than a chunk.)
    const int32_t chunk_len = min(C, a.t_blk - t0);
    int32_t len = chunk_len, begin = 0;
    bool has_end = true;                   // does this wave take the chunk's last slot
    if (split) {
        auto goes_on = [&](int32_t at) { return (flags[at] & 3) == 1 && (flags[at - 1] & 1); };
        int32_t cut = (chunk_len + 1) >> 1;
        if (cut < chunk_len && goes_on(cut)) {
            const int32_t end = next_slot<false, WAVE_ROW>(flags, cut + 1, chunk_len, a.row_lanes_log2);
            // the last slot in front of the middle that is padding or a start, if it is the nearer
            const int32_t least = max(2 * cut - end, 0);
            int32_t start = -1;
            for (int32_t hi = cut - 1; hi > least && start < 0; hi -= kWave) {
                const int32_t t = hi - lane_id();
                const uint64_t vote = __ballot(t > least && (flags[max(t, 0)] & 3) != 1);
                if (vote) start = hi - __builtin_ctzll(vote);
            }
            cut = start < 0 ? end : (flags[start] & 1) ? start : start + 1;
        }
        if (row & 1) {
            begin = cut;
            has_end = cut < chunk_len;
        } else {
            len = cut;
            has_end = cut == chunk_len;
            if (goes_on(0)) {
                const int32_t end = next_slot<false, WAVE_ROW>(flags, 1, reach + 1, a.row_lanes_log2);
                if (end <= reach) begin = end;
            }
        }
        if (has_end && goes_on(chunk_len)) {
            const int32_t end = next_slot<false, WAVE_ROW>(flags, chunk_len + 1, chunk_len + reach + 1, a.row_lanes_log2);
            if (end <= chunk_len + reach) len = end;
        }
    }
    const int64_t frame_bytes = (int64_t)a.feat_dim * (int64_t)sizeof(ElemT);
    const uint8_t* chunk_src = a.packed + g * frame_bytes;                 // the chunk's first frame
    // a frame that is no whole number of vectors: its last vector lies over the end of the one before
    // (both lanes compute the same)
    const int64_t feat0 = min((int64_t)fv * VEC, (int64_t)a.feat_dim - VEC);
    const uint32_t lane_off = (uint32_t)feat0 * (uint32_t)sizeof(ElemT);     // the lane's place in a frame
    const bool writes_desc = (col == 0 && feat_tile == 0 && a.desc != nullptr);
    typedef typename OutOf<Acc>::T Out;
    Out* out = static_cast<Out*>(a.out);
    Acc* head_part = static_cast<Acc*>(a.head_part);
    Acc* tail_part = static_cast<Acc*>(a.tail_part);

    // per-wave LDS scratch for the transposed stores (behind the flags), when a
    // wave lies inside one row
    Acc* scratch = nullptr;
    const int64_t wave_feat0 = (int64_t)(fv_raw - lane_id()) * VEC;   // first feature of the wave
    if (VEC > 1 && WAVE_ROW) {
        const size_t flag_bytes = ((size_t)chunks * stride + 15) & ~(size_t)15;
        scratch = reinterpret_cast<Acc*>(s_flags + flag_bytes) + (size_t)wave_id() * kWave * kScratchStride<Acc, VEC>();
    }

    Running<Acc, Elem<ElemT>::kCompensate> run[VEC];
    Acc acc[VEC];
    ChunkDesc desc{kHeadNone, 0, 0, -1};
    constexpr bool kPairs = Elem<ElemT>::kCompensate && VEC * sizeof(ElemT) < 16;     // (lanes of whole vectors never keep pairs)
    auto store_part = [&](Acc* parts) {
        parts += (kPairs && a.pair_parts ? 2 * q : q) * a.feat_dim;
        store_row<Acc, VEC>(parts, feat0, acc, lane_stores, scratch, wave_feat0, a.feat_dim);
        if constexpr (kPairs) {
            if (!a.pair_parts) return;
#pragma unroll
            for (int k = 0; k < VEC; ++k) acc[k] = run[k].missing();
            store_row<Acc, VEC>(parts + a.feat_dim, feat0, acc, lane_stores, scratch, wave_feat0, a.feat_dim);
        }
    };

    // The chunk is a sequence of pieces: maximal runs of valid slots that hold
    // no start flag after their first slot.  Find a piece [t, e) from the
    // staged flags, sum it with unconditional loads, hand the sum on.  The
    // frames of a piece are added eight at a time as a balanced tree, and the
    // sums of the eights go into a compensated running sum: the float32 result
    // is within a few units in the last place of sum |x| at any piece length.
    int32_t t = begin;
    for (;;) {
        t = next_slot<true, WAVE_ROW>(flags, t, len, a.row_lanes_log2);    // next valid slot
        if (t >= len) break;
        // a segment starts at a start flag, at the block's first slot, or behind padding;
        // a valid first slot of the chunk that does none of these continues the segment
        // of the chunk before
        const bool head_open = t == 0 && !(flags[0] & 2) && (flags[-1] & 1);
        const int32_t e = next_slot<false, WAVE_ROW>(flags, t + 1, len, a.row_lanes_log2);  // padding or a start
#pragma unroll
        for (int k = 0; k < VEC; ++k) run[k].clear();
        const uint8_t* p = chunk_src + (int64_t)t * frame_bytes;          // frame of slot s, lane 0
        int32_t s = t;
        static_assert(kWideUnroll == 8, "the tree below adds eight frames");
        for (; s + kWideUnroll <= e; s += kWideUnroll) {
            LaneData<ElemT, VEC, STREAM> x[kWideUnroll];
#pragma unroll
            for (int u = 0; u < kWideUnroll; ++u) x[u].load(p + (int64_t)u * frame_bytes + lane_off);
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                Acc v[kWideUnroll];
#pragma unroll
                for (int u = 0; u < kWideUnroll; ++u) v[u] = Elem<ElemT>::get(x[u].u.e[k]);
                run[k].add(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])));
            }
            p += (int64_t)kWideUnroll * frame_bytes;
        }
        if (s < e) {
            // the last, partial batch: all loads are issued at once as well (those
            // past the piece re-read its last slot and count as 0)
            const int32_t left = e - s;
            LaneData<ElemT, VEC, STREAM> x[kWideUnroll];
#pragma unroll
            for (int u = 0; u < kWideUnroll; ++u)
                x[u].load(p + (int64_t)min(u, left - 1) * frame_bytes + lane_off);
#pragma unroll
            for (int k = 0; k < VEC; ++k) {
                Acc v[kWideUnroll];
#pragma unroll
                for (int u = 0; u < kWideUnroll; ++u) v[u] = u < left ? Elem<ElemT>::get(x[u].u.e[k]) : (Acc)0;
                run[k].add(((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7])));
            }
        }
#pragma unroll
        for (int k = 0; k < VEC; ++k) acc[k] = run[k].sum;
        const int32_t cnt = e - t;
        // the segment ends here unless the piece runs to the chunk's end and the
        // slot after the chunk (flags[len], 0 past the block) continues it
        const bool closed = e < len || (flags[len] & 3) != 1;
        if (head_open) {
            if (head_part) store_part(head_part);
            desc.head_state = closed ? kHeadClosed : kHeadThrough;
            desc.cnt_head = cnt;
        } else {
            const int32_t seq = a.seq_id[g + t];
            if (closed) {
                if ((uint32_t)seq < (uint32_t)a.n_seq) {
#pragma unroll
                    for (int k = 0; k < VEC; ++k) acc[k] = finish<Acc>(acc[k], cnt, a.mean);
                    store_row<Acc, VEC>(out + (int64_t)seq * a.feat_dim, feat0, acc, lane_stores, scratch, wave_feat0, a.feat_dim);
                }
            } else {
                if (tail_part) store_part(tail_part);
                desc.cnt_tail = cnt;
                desc.seq_tail = seq;
            }
        }
        t = e;
    }
    if (!writes_desc) return;
    if (!split) {
        a.desc[q] = desc;
        return;
    }
    // what comes in is the first wave's
    if ((row & 1) == 0) {
        a.desc[q].head_state = desc.head_state;
        a.desc[q].cnt_head = desc.cnt_head;
    }
    if (has_end) {
        a.desc[q].cnt_tail = desc.cnt_tail;
        a.desc[q].seq_tail = desc.seq_tail;
    }
}

// ----------------------------------------------------------------- narrow
//
// Lanes across time: a workgroup takes 4096 consecutive slots (a "tile": a piece
// of one block, or several whole blocks), a lane 16 consecutive slots.  From the
// flags every lane builds two 16-bit masks: valid, and "break" (a slot that cannot
// continue the segment of the slot before it: padding, a start flag, a block's
// first slot, or a slot that follows padding).  Sums are a segmented scan with the
// breaks as heads: a lane contributes the sum of its slots from its last break
// on (`tail`: all its slots if it has none); the scan runs across the wave without
// LDS (DPP) and across the four waves through LDS, and gives every lane the sum of
// the segment that is open in front of it.  A lane keeps one more sum, of its
// slots in front of its first break (`head`), and not its 16 elements: a piece
// that ends in the lane is carry + head, or tail; only a piece between two breaks
// of one lane -- a segment of fewer than 16 slots -- is read again.  Frame counts
// need no scan: a segment's frames are consecutive, so its count is (end position
// - position of its break + 1).  Integer sums are exact, float sums add only the
// segment's own terms (no cancellation against neighbouring segments).

constexpr int kSlotsPerLane = 16;
constexpr int kNarrowTile = kThreads * kSlotsPerLane;      // 4096 slots per workgroup

// Running state of a segmented sum: `any` = a break was seen.
template <typename Acc>
struct SegState { Acc sum; uint32_t any; };

template <typename Acc>
struct SegCombine {
    __device__ __forceinline__ SegState<Acc> operator()(SegState<Acc> left, SegState<Acc> right) const
    {
        SegState<Acc> r;
        r.sum = right.any ? right.sum : left.sum + right.sum;
        r.any = left.any | right.any;
        return r;
    }
};

template <typename Acc>
struct PlainSum {
    __device__ __forceinline__ Acc operator()(Acc left, Acc right) const { return left + right; }
};
template <typename Acc>
struct PlainMove {
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ Acc at(Acc x) const { return dpp_move<CTRL, ROW_MASK>(x, (Acc)0); }
};

template <typename Acc>
struct SegMove {
    template <int CTRL, int ROW_MASK>
    __device__ __forceinline__ SegState<Acc> at(SegState<Acc> s) const
    {
        return SegState<Acc>{dpp_move<CTRL, ROW_MASK>(s.sum, (Acc)0), dpp_move<CTRL, ROW_MASK>(s.any, 0u)};
    }
};

// The flag bytes of 16 consecutive slots, asked for with loads that stay inside the planes of
// `total` slots wherever the slots lie (planes of fewer than 16 slots are read byte by byte).
struct FlagBytes {
    vec16 valid, reset;
    int64_t g, from;
    uint8_t before;                    // the valid flag of the slot in front (of the first slot: its own)

    __device__ __forceinline__ void load(const ReduceArgs& a, int64_t first, int32_t left)
    {
        g = first;
        from = max(min(g, a.total_slots - 16), (int64_t)0);
        valid = reset = vec16{0u, 0u, 0u, 0u};
        before = 0;
        if (left < 0) return;
        before = a.valid[max(min(g, a.total_slots) - 1, (int64_t)0)];
        if (a.total_slots >= 16) {
            valid = *reinterpret_cast<const vec16_any*>(a.valid + from);
            reset = *reinterpret_cast<const vec16_any*>(a.reset + from);
        }
    }
    // bit j: the flag of slot g + j is set, for the `left` slots that count
    __device__ __forceinline__ uint32_t mask(vec16 bytes, const uint8_t* plane, int32_t left, int64_t total) const
    {
        const uint32_t counts = left >= 16 ? 0xffffu : (1u << max(left, 0)) - 1u;
        if (total >= 16) return g - from < 16 ? (nonzero_bytes16(bytes) >> (int)(g - from)) & counts : 0u;
        uint32_t m = 0;
        for (int j = 0; j < left && j < 16; ++j) m |= (uint32_t)(plane[g + j] != 0) << j;
        return m;
    }
};

// Where a workgroup's tile lies.  Tiles never straddle a block: a tile is a piece of one block
// (blocks of at least a tile's length) or a whole number of blocks.
struct NarrowTile {
    int64_t g0;            // first slot
    int32_t n;             // slots in the tile
    int32_t rem0;          // position of the tile's first slot inside its block
};

__device__ __forceinline__ NarrowTile narrow_tile(const ReduceArgs& a, int64_t q)
{
    NarrowTile t;
    if (a.t_blk >= kNarrowTile) {
        const int64_t b = a.n_chunks == 1 ? q : (int64_t)((uint32_t)q / (uint32_t)a.n_chunks);
        const int32_t c = (int32_t)(q - b * a.n_chunks);
        t.rem0 = c * kNarrowTile;
        t.g0 = b * (int64_t)a.t_blk + t.rem0;
        t.n = min(kNarrowTile, a.t_blk - t.rem0);
    } else {
        const int64_t b0 = q * a.blocks_per_tile;
        t.rem0 = 0;
        t.g0 = b0 * (int64_t)a.t_blk;
        t.n = (int32_t)min((int64_t)a.blocks_per_tile, a.num_blocks - b0) * a.t_blk;
    }
    return t;
}

// What a lane knows about its 16 slots after reading the flags.
struct LaneFlags {
    uint32_t vmask;        // bit j: slot j is valid
    uint32_t bmask;        // bit j: slot j is a break
    uint32_t ends;         // bit j: a segment ends at slot j
    int32_t j_last;        // index of the tile's last slot in this lane (may lie outside 0..15)
    bool tail_open;        // the tile's last slot is here and its segment goes on into the next tile
};

// The flag bytes of a lane as they come from memory, and what the whole wave is, as far as a
// look at whole words can tell.
struct LaneFlagBytes {
    vec16 valid, reset;    // zero where the lane has not all its 16 slots in the tile
    bool wave_blank;       // the wave holds nothing but padding
    bool wave_plain;       // the wave holds nothing but valid slots without a start flag
};

__device__ __forceinline__ LaneFlagBytes narrow_flag_bytes(const ReduceArgs& a, const NarrowTile& tile)
{
    constexpr int SPL = kSlotsPerLane;
    static_assert(SPL == 16, "the flags of a lane are one 16-byte vector per plane");
    const int pos0 = (int)threadIdx.x * SPL;
    const int32_t left = tile.n - pos0;
    LaneFlagBytes b;
    b.valid = vec16{0u, 0u, 0u, 0u};
    b.reset = vec16{0u, 0u, 0u, 0u};
    if (left >= SPL) {
        b.valid = __builtin_nontemporal_load(reinterpret_cast<const vec16_any*>(a.valid + tile.g0 + pos0));
        b.reset = __builtin_nontemporal_load(reinterpret_cast<const vec16_any*>(a.reset + tile.g0 + pos0));
    }
    // Two kinds of waves are common in packed blocks and need no byte-by-byte look at their
    // flags: nothing but padding (block tails), and nothing but valid slots without a start flag
    // (the inside of long sequences).  Both tests are wave-uniform.
    const uint32_t v_any = b.valid[0] | b.valid[1] | b.valid[2] | b.valid[3];
    const uint32_t v_all = b.valid[0] & b.valid[1] & b.valid[2] & b.valid[3];
    const uint32_t r_any = b.reset[0] | b.reset[1] | b.reset[2] | b.reset[3];
    const bool lane_blank = left >= SPL ? v_any == 0u : left <= 0;
    // (a non-zero byte in the AND of the four words means four non-zero bytes)
    const bool lane_plain = left >= SPL && r_any == 0u &&
                            ((((v_all & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v_all) & 0x80808080u) == 0x80808080u;
    b.wave_blank = __ballot(lane_blank) == ~0ull;
    b.wave_plain = __ballot(lane_plain) == ~0ull;
    return b;
}

// Derives the masks of the lane's slots from its flag bytes and those of its neighbours.
// Called by every thread of the workgroup (the lanes of a wave exchange their border slots).
__device__ __forceinline__ LaneFlags narrow_lane_flags(const ReduceArgs& a, const NarrowTile& tile,
                                                       const LaneFlagBytes& bytes)
{
    constexpr int SPL = kSlotsPerLane;
    constexpr uint32_t ALL = (1u << SPL) - 1u;
    const int tid = (int)threadIdx.x;
    const int lane = lane_id();
    const uint32_t T = (uint32_t)a.t_blk;
    const int pos0 = tid * SPL;
    const int32_t left = tile.n - pos0;                  // slots from this lane's first one to the tile's end
    const int64_t s0 = tile.g0 + pos0;
    LaneFlags r;

    // position of the lane's first slot inside its block, and of the slot behind its last one
    uint32_t rem0 = (uint32_t)tile.rem0 + (uint32_t)pos0;
    if (T < (uint32_t)kNarrowTile) {
        rem0 -= __umulhi((uint32_t)pos0, a.magic_t_blk) * T;        // pos0 mod T, possibly one T too many
        if (rem0 >= T) rem0 -= T;
    }
    uint32_t rem_next = rem0 + (uint32_t)SPL;
    while (rem_next >= T) rem_next -= T;                 // at most once unless t_blk < 16

    // the slots in front of and behind the lanes of this wave, where they belong to the same block
    uint8_t before_valid = 0, after_valid = 0, after_reset = 0;
    if (lane == 0 && rem0 != 0 && left > 0) before_valid = a.valid[s0 - 1];
    if (lane == kWave - 1 && rem_next != 0 && left >= SPL) { after_valid = a.valid[s0 + SPL]; after_reset = a.reset[s0 + SPL]; }

    uint32_t vmask = 0, rmask = 0;
    if (bytes.wave_blank) {
        // vmask = rmask = 0
    } else if (bytes.wave_plain) {
        vmask = ALL;
    } else if (left >= SPL) {
        vmask = nonzero_bytes16(bytes.valid);
        rmask = nonzero_bytes16(bytes.reset);
    } else if (left > 0) {
        // the tile ends inside this lane: slot by slot (those past the end re-read its last slot)
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            vmask |= (uint32_t)(a.valid[s0 + min(j, left - 1)] != 0) << j;
            rmask |= (uint32_t)(a.reset[s0 + min(j, left - 1)] != 0) << j;
        }
        vmask &= (1u << left) - 1u;
        rmask &= (1u << left) - 1u;
    }
    // first slots of blocks among the lane's slots: `gap` = slots to the next block start
    uint32_t smask = 0;
    for (uint32_t gap = rem0 == 0 ? 0u : T - rem0; gap < (uint32_t)SPL; gap += T) smask |= 1u << gap;
    // validity of the slot before this lane's first one
    uint32_t prev_valid = dpp_move<kDppWaveShr1>((vmask >> (SPL - 1)) & 1u, 0u);
    if (lane == 0) prev_valid = (uint32_t)(before_valid != 0);
    const uint32_t after_pad = ~((vmask << 1) | prev_valid);          // bit j: slot j-1 is not valid
    const uint32_t bmask = (~vmask | rmask | smask | after_pad) & ALL;
    // is the slot after this lane's last one a break
    uint32_t next_first = dpp_move<kDppWaveShl1>(bmask & 1u, 0u);
    if (lane == kWave - 1) {
        next_first = 1u;
        if (rem_next != 0 && left >= SPL)
            next_first = (!after_valid || after_reset || !((vmask >> (SPL - 1)) & 1u)) ? 1u : 0u;
    }
    const uint32_t next_brk = (bmask >> 1) | (next_first << (SPL - 1));
    r.vmask = vmask;
    r.bmask = bmask;
    r.ends = vmask & next_brk;
    r.j_last = left - 1;
    r.tail_open = r.j_last >= 0 && r.j_last < SPL && ((vmask >> r.j_last) & 1u) &&
                  !((next_brk >> r.j_last) & 1u);
    return r;
}

// LDS staging of the payload of one workgroup: the NV 16-byte vectors of a lane lie together,
// vector k of lane l in place k ^ (l / (16 / NV)) of the lane's NV, so that the 16 lanes which
// one pass of a 16-byte LDS access serves touch every bank once, both when a lane writes vector
// l of a row and when it reads its own vectors.
template <typename ElemT>
struct NarrowStage {
    static constexpr int NV = kSlotsPerLane * (int)sizeof(ElemT) / 16;     // vectors per lane
    static_assert(NV == 1 || NV == 2 || NV == 4, "the bank swizzle below is written for 1, 2 or 4 vectors");
    static constexpr int kVectors = NV > 1 ? kThreads * NV : 1;
    // place of vector k of lane l (l counted within the wave) in the wave's part of the stage
    __device__ static __forceinline__ int at(int l, int k) { return l * NV + (k ^ ((l / (16 / NV)) & (NV - 1))); }
};

// The payload of a wave whose 1024 elements are contiguous (a frame is one element, every lane
// has all its slots): read as whole 1 KiB rows, lane l taking vector l of each row, because 64
// lanes that each read their own 64 bytes would touch four times as many cache lines per load.
// `issue` only starts the loads (so that the work on the flags runs while they are in flight),
// `finish` hands every vector to the lane it belongs to, through LDS.
template <typename ElemT>
struct NarrowRows {
    static constexpr int NV = NarrowStage<ElemT>::NV;
    vec16 v[NV > 0 ? NV : 1];

    __device__ __forceinline__ void issue(const ReduceArgs& a, int64_t wave_s0)
    {
        const vec16_any* row = reinterpret_cast<const vec16_any*>(a.packed + wave_s0 * (int64_t)sizeof(ElemT));
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = __builtin_nontemporal_load(row + k * kWave + lane_id());
    }
    __device__ __forceinline__ void finish(vec16* stage, ElemT (&raw)[kSlotsPerLane])
    {
        const int lane = lane_id();
        vec16* mine = stage + (int)(threadIdx.x - lane) * NV;                // the wave's part
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int row_at = k * kWave + lane;             // vector `row_at` of the wave belongs to lane row_at / NV
            mine[NarrowStage<ElemT>::at(row_at / NV, row_at % NV)] = v[k];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        union { vec16 q[NV > 0 ? NV : 1]; ElemT e[kSlotsPerLane]; } u;
#pragma unroll
        for (int k = 0; k < NV; ++k) u.q[k] = mine[NarrowStage<ElemT>::at(lane, k)];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < kSlotsPerLane; ++j) raw[j] = u.e[j];
    }
    // Element j of the lane once more, from the stage (which keeps the wave's rows until the
    // workgroup ends): for the few lanes that need single elements again.
    __device__ __forceinline__ static ElemT again(const vec16* stage, int j)
    {
        constexpr int EPV = 16 / (int)sizeof(ElemT);
        const int lane = lane_id();
        const vec16* mine = stage + (int)(threadIdx.x - lane) * NV;
        return reinterpret_cast<const ElemT*>(mine + NarrowStage<ElemT>::at(lane, j / EPV))[j % EPV];
    }
};

// The lane's 16 elements where they do not come as rows; only those of valid slots mean anything.
// `left` = slots from the lane's first one to the tile's end.
template <typename ElemT>
__device__ __forceinline__ void narrow_load(const ReduceArgs& a, int64_t s0, int32_t left, ElemT (&raw)[kSlotsPerLane])
{
    constexpr int SPL = kSlotsPerLane;
    constexpr int NV = NarrowStage<ElemT>::NV;
    const uint8_t* from = a.packed + s0 * (int64_t)sizeof(ElemT);
    if (left >= SPL) {
        union { vec16 v[NV > 0 ? NV : 1]; ElemT e[SPL]; } u;
#pragma unroll
        for (int k = 0; k < NV; ++k) u.v[k] = __builtin_nontemporal_load(reinterpret_cast<const vec16_any*>(from) + k);
#pragma unroll
        for (int j = 0; j < SPL; ++j) raw[j] = u.e[j];
    } else if (left > 0) {
        // slots past the tile's end re-read its last slot (their valid bits are 0)
#pragma unroll
        for (int j = 0; j < SPL; ++j) raw[j] = reinterpret_cast<const ElemT*>(from)[min(j, left - 1)];
    } else {
#pragma unroll
        for (int j = 0; j < SPL; ++j) raw[j] = ElemT{};
    }
}

// x where bit j of `mask` is set, 0 (of the accumulator's type) elsewhere
__device__ __forceinline__ float masked(float x, uint32_t mask, int j)
{
    return __int_as_float(__float_as_int(x) & (int32_t)__builtin_amdgcn_sbfe(mask, j, 1));
}
// The same, kept from becoming a comparison and a select (more instructions, with waits between them).
__device__ __forceinline__ float masked_by_and(float x, uint32_t mask, int j)
{
    int32_t all = (int32_t)__builtin_amdgcn_sbfe(mask, j, 1);
    asm("" : "+v"(all));
    return __int_as_float(__float_as_int(x) & all);
}
__device__ __forceinline__ long long masked_by_and(long long x, uint32_t mask, int j)
{
    return (long long)((int32_t)x & (int32_t)__builtin_amdgcn_sbfe(mask, j, 1));     // x holds an int32 here
}
__device__ __forceinline__ long long masked(long long x, uint32_t mask, int j)
{
    return (long long)((int32_t)x & (int32_t)__builtin_amdgcn_sbfe(mask, j, 1));     // x holds an int32 here
}

// Hand one finished piece on: to the output row of its sequence, or to the partial buffers when the
// tile border cuts its segment.  `seq` is the sequence id at the first slot of the piece when the
// segment starts in this tile (`started`), as in the wide layout; `value` is finished (a mean is
// divided) where the piece is a whole segment.  A partial sum in double is kept as a float and
// what that lacks.
template <typename Part>
__device__ __forceinline__ void put_part(void* parts, int64_t q, int d, int32_t D, Part v)
{
    static_cast<Part*>(parts)[q * D + d] = v;
}
template <>
__device__ __forceinline__ void put_part<double>(void* parts, int64_t q, int d, int32_t D, double v)
{
    const float hi = (float)v;
    float* row = static_cast<float*>(parts) + 2 * q * D + d;
    row[0] = hi;
    row[D] = __builtin_isfinite(hi) ? (float)(v - (double)hi) : 0.0f;
}

template <typename Acc, typename Part>
__device__ __forceinline__ void emit_piece(const ReduceArgs& a, int64_t q, int d, int32_t seq,
                                           bool is_end, bool started, Part value, int32_t cnt,
                                           ChunkDesc* s_desc)
{
    typedef typename OutOf<Acc>::T Out;
    const int D = a.feat_dim;
    if (is_end && started) {
        if ((uint32_t)seq < (uint32_t)a.n_seq) static_cast<Out*>(a.out)[(int64_t)seq * D + d] = (Out)value;
    } else if (!started) {
        // continues a segment of the previous tile; closed here or running through
        if (a.head_part) put_part<Part>(a.head_part, q, d, D, value);
        if (d == 0) {
            s_desc->head_state = is_end ? kHeadClosed : kHeadThrough;
            s_desc->cnt_head = cnt;
        }
    } else {
        if (a.tail_part) put_part<Part>(a.tail_part, q, d, D, value);
        if (d == 0) {
            s_desc->cnt_tail = cnt;
            s_desc->seq_tail = seq;
        }
    }
}

template <typename ElemT>
__global__ __launch_bounds__(kThreads) void reduce_narrow_kernel(ReduceArgs a)
{
    typedef typename Elem<ElemT>::Acc Acc;
    constexpr int NW = kThreads / kWave;
    constexpr int SPL = kSlotsPerLane;
    __shared__ Acc s_wave_sum[NW];                     // the wave's sum behind its last break (all of it if none)
    __shared__ uint32_t s_wave_any[NW];                // the wave holds a break
    __shared__ unsigned long long s_wave_breaks[NW];   // which lanes of the wave hold a break
    __shared__ int32_t s_last_break[kThreads];         // position of a lane's last break (lanes that have one)
    __shared__ int32_t s_break_seq[kThreads];          // and the sequence id found there
    __shared__ vec16 s_stage[NarrowStage<ElemT>::kVectors];
    __shared__ ChunkDesc s_desc;

    const int tid = (int)threadIdx.x;
    const int lane = lane_id(), wave = wave_id();
    const int64_t q = blockIdx.x;
    const NarrowTile tile = narrow_tile(a, q);
    const int64_t g0 = tile.g0;
    const int pos0 = tid * SPL;
    const int64_t s0 = g0 + pos0;
    if (tid == 0) s_desc = ChunkDesc{kHeadNone, 0, 0, -1};
    const LaneFlagBytes bytes = narrow_flag_bytes(a, tile);
    // a wave without a valid slot reads no payload; a wave that lies whole in the tile asks for
    // its rows now, before the flags are looked at
    const bool wave_valid = !bytes.wave_blank;
    const int32_t left = tile.n - pos0;
    const bool by_rows = NarrowStage<ElemT>::NV > 1 && left - (kWave - 1 - lane) * SPL >= SPL;
    NarrowRows<ElemT> rows;
    if (wave_valid && by_rows) rows.issue(a, s0 - lane * SPL);
    const LaneFlags f = narrow_lane_flags(a, tile, bytes);
    const uint32_t bmask = f.bmask;
    const unsigned long long wave_breaks = __ballot(bmask != 0);
    const int last_break = bmask ? 31 - __clz((int)bmask) : 0;
    const int first_break = bmask ? __ffs((int)bmask) - 1 : SPL;
    // the sequence that starts at the lane's last break: asked for now, so that the answer is
    // there when a lane further on (or this one) closes that segment
    int32_t own_seq = -1;
    if (bmask && ((f.vmask >> last_break) & 1u)) own_seq = a.seq_id[s0 + last_break];
    if (lane == 0) s_wave_breaks[wave] = wave_breaks;
    const uint32_t from_last_break = f.vmask & (~0u << last_break);   // the lane's part of the open segment
    const uint32_t to_first_break = f.vmask & ((1u << first_break) - 1u);   // its part of the segment it inherits
    const bool finishes = f.ends != 0 || f.tail_open;                 // a piece ends in this lane
    int32_t prev_start = -1;           // position of the last break in front of this lane, -1: none in the tile
    int32_t prev_seq = -1;             // and the sequence id found there

    SegState<Acc> scan, carry;
    Acc tail = 0;                      // the lane's slots from its last break on (all of them if it has none)
    Acc head = 0;                      // the lane's slots in front of its first break
    if (!wave_valid) {
        // nothing but padding: every slot is a break, nothing to add
        scan = SegState<Acc>{0, 1u};
        carry = SegState<Acc>{0, lane == 0 ? 0u : 1u};
    } else {
        ElemT raw[SPL];
        if (by_rows) rows.finish(s_stage, raw);
        else narrow_load<ElemT>(a, s0, left, raw);
        if (wave_breaks == 0) {
            // no break in the whole wave (so every slot is valid): plain sums
#pragma unroll
            for (int j = 0; j < SPL; ++j) tail += Elem<ElemT>::get(raw[j]);
            scan = SegState<Acc>{wave_scan(tail, PlainSum<Acc>(), PlainMove<Acc>()), 0u};
            carry = SegState<Acc>{dpp_move<kDppWaveShr1>(scan.sum, (Acc)0), 0u};
        } else {
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                tail += masked((Acc)Elem<ElemT>::get(raw[j]), from_last_break, j);
                head += masked((Acc)Elem<ElemT>::get(raw[j]), to_first_break, j);
            }
            scan = wave_scan(SegState<Acc>{tail, bmask != 0 ? 1u : 0u}, SegCombine<Acc>(), SegMove<Acc>());
            carry = SegMove<Acc>().template at<kDppWaveShr1, 0xF>(scan);      // the lanes before this one
        }
    }
    if (lane == kWave - 1) { s_wave_sum[wave] = scan.sum; s_wave_any[wave] = scan.any; }
    if (bmask) { s_last_break[tid] = pos0 + last_break; s_break_seq[tid] = own_seq; }
    __syncthreads();
    if (finishes) {
        // the segments that end in this lane, and the open tail of the tile
        SegState<Acc> before{0, 0};
        for (int w = 0; w < wave; ++w)
            before = SegCombine<Acc>()(before, SegState<Acc>{s_wave_sum[w], s_wave_any[w]});
        carry = SegCombine<Acc>()(before, carry);
        const unsigned long long lower = wave_breaks & ((1ull << lane) - 1ull);
        int holder = lower ? wave * kWave + 63 - __clzll((long long)lower) : -1;
        for (int w = wave - 1; w >= 0 && holder < 0; --w) {
            const unsigned long long b = s_wave_breaks[w];
            if (b) holder = w * kWave + 63 - __clzll((long long)b);
        }
        if (holder >= 0) { prev_start = s_last_break[holder]; prev_seq = s_break_seq[holder]; }
        // One piece per end (usually one per lane).  The piece that closes what the lanes before
        // left open ends in front of the lane's first break: carry + head.  The piece that the
        // lane's last break opened ends at its last slot: tail (plus the carry if the lane has no
        // break at all).  A piece between two breaks of the lane is read again, slot by slot: from
        // the LDS stage where the wave's rows went through it (workload of 10^6 token sequences:
        // 1.24 -> 1.15 ms against reading them from memory), else from memory.
        uint32_t todo = f.ends | (f.tail_open ? 1u << f.j_last : 0u);
        while (todo) {
            const int j = 31 - __clz((int)todo);                          // last one first
            todo &= ~(1u << j);
            const uint32_t upto = bmask & ((2u << j) - 1u);               // breaks at or before j
            const int lb = upto ? 31 - __clz((int)upto) : -1;
            Acc sum;
            if (lb < 0) {
                sum = carry.sum + (bmask ? head : tail);
            } else if (lb == last_break) {
                sum = tail;
            } else {
                sum = 0;
                if (by_rows) {
                    for (int k = lb; k <= j; ++k) sum += Elem<ElemT>::get(NarrowRows<ElemT>::again(s_stage, k));
                } else {
                    const ElemT* from = reinterpret_cast<const ElemT*>(a.packed) + s0;
                    for (int k = lb; k <= j; ++k) sum += Elem<ElemT>::get(from[k]);
                }
            }
            const int32_t start = lb >= 0 ? pos0 + lb : prev_start;
            const int32_t cnt = start >= 0 ? pos0 + j - start + 1 : pos0 + j + 1;
            const int32_t seq = lb < 0 ? prev_seq : (lb == last_break ? own_seq : a.seq_id[s0 + lb]);
            const bool is_end = (f.ends >> j) & 1u;
            emit_piece<Acc, Acc>(a, q, 0, seq, is_end, start >= 0, finish<Acc>(sum, is_end && start >= 0 ? cnt : 1, a.mean), cnt, &s_desc);
        }
    }
    __syncthreads();
    if (tid == 0 && a.desc) a.desc[q] = s_desc;
}

// ----------------------------------------------------------------- staged
//
// Frames of 2 to 63 elements.  A tile of whole frames (a piece of one block, or several whole
// blocks) comes into LDS as whole 16-byte vectors, because rows this short read lane by lane
// would touch a cache line per lane; then lanes take one feature each and kStagedSlots
// consecutive slots, D lanes side by side and 256 / D groups of them one behind the other in
// time.  As in the narrow layout a lane contributes the sum of its slots from its last break on
// to a segmented scan over the groups, and then hands on the pieces that end in its slots.
// A lane adds its frames as trees of eight, like the rows of lanes above; the trees and the lanes are added in
// 64 bits, which is no less exact than the compensated sums there.  The sequence ids are read at the starts only, all at once, and wait in
// LDS.  Bound by HBM where the sequences are long, by the pieces of the lanes where they are of
// a few frames.
// Measured against a loop over the features of lanes across time (the narrow layout before): 39
// features of a byte, 115427 sequences, 0.46 GB: 4.20 -> 0.25 ms.

constexpr int kStagedSlots = 17;       // odd, so that the groups' places in LDS spread over the banks
constexpr int kStagedSlotsShort = 9;   // where long lanes would leave the chip without enough tiles
constexpr int kStagedFrame = 64;       // frames of fewer elements are staged
constexpr int32_t kLeanRun = 3 * kNarrowTile;     // lean cut: the longest chunk of tiles

template <typename Acc> struct WideSum { typedef double T; };
template <> struct WideSum<long long> { typedef long long T; };

// What sums of a tile's frames are kept in: whole numbers are exact in the accumulator.
template <typename ElemT> struct TileSum {
    typedef typename std::conditional<Elem<ElemT>::kCompensate, double, typename Elem<ElemT>::Acc>::type T;
};

// The sum of the elements of x whose bit in `mask` is set.
template <typename ElemT, int K>
__device__ __forceinline__ typename TileSum<ElemT>::T masked_sum(const ElemT (&x)[K], uint32_t mask)
{
    typedef typename Elem<ElemT>::Acc Acc;
    if constexpr (!Elem<ElemT>::kCompensate) {       // whole numbers, exact in any order
        Acc even = 0, odd = 0;
#pragma unroll
        for (int u = 0; u < K; ++u) {
            const Acc v = masked_by_and((Acc)Elem<ElemT>::get(x[u]), mask, u);
            if (u & 1) odd += v; else even += v;
        }
        return even + odd;
    }
    typename TileSum<ElemT>::T sum = 0;
#pragma unroll
    for (int u0 = 0; u0 < K; u0 += 8) {
        Acc v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = u0 + u < K ? masked_by_and((Acc)Elem<ElemT>::get(x[u0 + u < K ? u0 + u : 0]), mask, u0 + u) : (Acc)0;
        sum += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
    return sum;
}

// RUN: the workgroup takes the tiles of a whole chunk one after another and carries the open segment from
// one to the next.  No border inside the chunk, so fewer partial sums or none.
template <typename ElemT, int K, bool RUN>
__global__ __launch_bounds__(kThreads) void reduce_staged_kernel(ReduceArgs a)
{
    typedef typename Elem<ElemT>::Acc Acc;
    typedef typename WideSum<Acc>::T Sum;
    typedef typename TileSum<ElemT>::T Part;
    static_assert(K % 2 == 1 && K < 32, "a lane's flags fit a word");
    constexpr int kElems = K * kThreads;
    constexpr int kMostSlots = kElems / 2;
    constexpr int kGroups = (kMostSlots + 15) / 16 + 6;      // groups of 16 flags, the last ones zero
    constexpr int EPV = 16 / (int)sizeof(ElemT);
    constexpr int NV = (K + EPV - 1) / EPV;
    __shared__ alignas(16) ElemT s_x[kElems];
    __shared__ int32_t s_seq[kMostSlots];                    // at starts: the sequence id
    __shared__ alignas(16) uint16_t s_valid[kGroups], s_break[kGroups];
    __shared__ Sum s_sum[2][kThreads];
    __shared__ int32_t s_pos[2][kThreads];                   // last break up to there, -1: none in the tile
    __shared__ ChunkDesc s_desc;
    __shared__ int32_t s_carry_seq;                          // RUN: sequence id of the segment carried from the tile before

    const int tid = (int)threadIdx.x;
    const int D = a.feat_dim;
    const int s = (int)((uint32_t)tid / (uint32_t)D), d = tid - s * D;
    const int subs = (RUN ? a.tile : a.chunk) / K;
    const bool active = s < subs;
    const int64_t q = blockIdx.x;
    // the tile (RUN: the chunk, of which `tile` slots at a time): a piece of one block, or blocks_per_tile whole ones
    int64_t g0;
    int32_t n, rem0;
    if (a.n_chunks > 1) {
        const int64_t b = (int64_t)((uint32_t)q / (uint32_t)a.n_chunks);
        rem0 = (int32_t)(q - b * a.n_chunks) * a.chunk;
        g0 = b * (int64_t)a.t_blk + rem0;
        n = min(a.chunk, a.t_blk - rem0);
    } else {
        const int64_t b0 = q * a.blocks_per_tile;
        rem0 = 0;
        g0 = b0 * (int64_t)a.t_blk;
        n = (int32_t)min((int64_t)a.blocks_per_tile, a.num_blocks - b0) * a.t_blk;
    }
    if (tid == 0) s_desc = ChunkDesc{kHeadNone, 0, 0, -1};
    const int32_t run_n = n;
    int32_t base = 0;                  // the tile's first slot in the chunk
    Sum carry = 0;                     // lanes of the first group: the open segment in front of the tile,
    int32_t carry_pos = -1;            // and where it starts in the chunk, -1: in front of it
    for (;; __syncthreads()) {
    if (RUN) n = min(a.tile, run_n - base);

    // payload: all vectors asked for before anything is waited for
    const int elems = n * D, vecs = elems / EPV;
    const uint8_t* from = a.packed + g0 * D * (int64_t)sizeof(ElemT);
    vec16 in[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = tid + k * kThreads;
        in[k] = vec16{0u, 0u, 0u, 0u};
        if (i < vecs) in[k] = __builtin_nontemporal_load(reinterpret_cast<const vec16_any*>(from) + i);
    }
    // flags, 16 slots to a lane: which slots are valid, and which cannot continue the segment of the slot
    // in front (padding, a start flag, a block's first slot, a slot behind padding)
    const uint32_t T = (uint32_t)a.t_blk;
    // (every load unconditional, at an address inside the planes, so that none waits for another)
    constexpr int kRounds = (kGroups + kThreads - 1) / kThreads;
    FlagBytes fb[kRounds];
    const bool more_behind = rem0 + n < a.t_blk && (RUN || a.n_chunks > 1);
    const int64_t behind = min(g0 + n, a.total_slots - 1);
    const uint8_t behind_valid = a.valid[behind], behind_reset = a.reset[behind];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) fb[r].load(a, g0 + 16 * (tid + r * kThreads), n - 16 * (tid + r * kThreads));
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int i = tid + r * kThreads;
        if (i >= kGroups) break;
        uint32_t vm16 = 0, brk = 0xffffu;                    // behind the tile: breaks
        const int32_t left16 = n - 16 * i;
        if (left16 >= 0) {
            const uint32_t pos = (uint32_t)(rem0 + 16 * i) % T;
            const uint32_t before = pos != 0 && fb[r].before != 0 ? 1u : 0u;
            vm16 = fb[r].mask(fb[r].valid, a.valid, left16, a.total_slots);
            const uint32_t rm16 = fb[r].mask(fb[r].reset, a.reset, left16, a.total_slots);
            uint32_t first = 0;
            for (uint32_t k = pos == 0 ? 0 : T - pos; k < 16; k += T) first |= 1u << k;
            brk = (~vm16 | rm16 | first | ~(vm16 << 1 | before)) & 0xffffu;
            if (left16 < 16) {                               // the slot behind the tile
                const bool goes_on = more_behind && behind_valid != 0 && behind_reset == 0 &&
                                     ((left16 == 0 ? before : vm16 >> (left16 - 1)) & 1u);
                brk = goes_on ? brk & ~(1u << left16) : brk | 1u << left16;
            }
        }
        s_valid[i] = (uint16_t)vm16;
        s_break[i] = (uint16_t)brk;
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int i = tid + k * kThreads;
        if (i < vecs) *reinterpret_cast<vec16*>(s_x + i * EPV) = in[k];
    }
    for (int i = vecs * EPV + tid; i < elems; i += kThreads) s_x[i] = reinterpret_cast<const ElemT*>(from)[i];
    __syncthreads();
    // the sequence ids at the starts: the first two per lane are on their way while the lane adds up
    auto starts_at = [&](int t) { return t < n && ((s_valid[t >> 4] & s_break[t >> 4]) >> (t & 15)) & 1u; };
    const bool start0 = starts_at(tid), start1 = starts_at(tid + kThreads);
    int32_t seq0 = -1, seq1 = -1;
    if (start0) seq0 = a.seq_id[g0 + tid];
    if (start1) seq1 = a.seq_id[g0 + tid + kThreads];

    const int o = s * K, left = active ? min(K, n - o) : 0;
    uint32_t vm = 0, bm = 0, next_brk = 0;
    Part tail = 0, head = 0;           // the slots from the last break on, and those in front of the first one
    if (left > 0) {
        const uint32_t* v32 = reinterpret_cast<const uint32_t*>(s_valid) + (o >> 5);
        const uint32_t* b32 = reinterpret_cast<const uint32_t*>(s_break) + (o >> 5);
        const uint32_t in_lane = (1u << left) - 1u;
        vm = (uint32_t)(((uint64_t)v32[1] << 32 | v32[0]) >> (o & 31)) & in_lane;
        const uint32_t brk = (uint32_t)(((uint64_t)b32[1] << 32 | b32[0]) >> (o & 31));
        bm = brk & in_lane;
        next_brk = brk >> 1;                                 // also of the slot behind the lane's last
        ElemT x[K];
#pragma unroll
        for (int u = 0; u < K; ++u) x[u] = s_x[(o + u) * D + d];             // only valid slots count below
        const uint32_t open = bm ? vm & (~0u << (31 - __clz((int)bm))) : vm;
        const uint32_t front = bm ? vm & ((bm & -bm) - 1u) : vm;
        head = tail = masked_sum(x, open);
        if (bm) head = masked_sum(x, front);
    }
    if (start0) s_seq[tid] = seq0;
    if (start1) s_seq[tid + kThreads] = seq1;
    for (int t = tid + 2 * kThreads; t < n; t += kThreads)
        if (starts_at(t)) s_seq[t] = a.seq_id[g0 + t];
    // segmented scan over the groups
    Sum sum = (Sum)tail;
    int32_t pos = bm ? base + o + 31 - __clz((int)bm) : -1;
    if (RUN && s == 0 && base > 0 && pos < 0) {
        sum = carry + sum;
        pos = carry_pos;
    }
    int buf = 0;
    for (int step = 1; step < subs; step <<= 1) {
        s_sum[buf][tid] = sum;
        s_pos[buf][tid] = pos;
        __syncthreads();
        if (active && s >= step && pos < 0) {
            sum = s_sum[buf][tid - step * D] + sum;
            pos = s_pos[buf][tid - step * D];
        }
        buf ^= 1;
    }
    s_sum[buf][tid] = sum;
    s_pos[buf][tid] = pos;
    __syncthreads();

    // One piece per end in the lane's slots, and the open one at the tile's end
    const uint32_t ends = vm & next_brk;
    uint32_t todo = ends;
    if (left > 0 && base + o + left == run_n) todo |= vm & (1u << (left - 1));
    while (todo) {
        const int j = __ffs((int)todo) - 1;
        todo &= todo - 1u;
        const uint32_t upto = bm & ((2u << j) - 1u);
        int32_t start = -1;
        Sum piece;
        if (upto == 0) {
            // it closes what the groups in front left open
            piece = (Sum)head;
            if (s > 0) {
                piece = s_sum[buf][tid - D] + piece;
                start = s_pos[buf][tid - D];
            } else if (RUN && base > 0) {
                piece = carry + piece;
                start = carry_pos;
            }
        } else {
            const int from = 31 - __clz((int)upto);
            start = base + o + from;
            if (upto == bm) {
                piece = (Sum)tail;
            } else {                   // a segment between two breaks of the lane is read again
                Part again = 0;
                for (int k = from; k <= j; ++k) again += Elem<ElemT>::get(s_x[(o + k) * D + d]);
                piece = (Sum)again;
            }
        }
        const bool started = start >= 0, is_end = (ends >> j) & 1u;
        const int32_t cnt = base + o + j - (started ? start : 0) + 1;
        if (started && is_end && a.mean) piece = piece / (Sum)cnt;
        int32_t seq = -1;
        if (started) seq = RUN && start < base ? s_carry_seq : s_seq[start - base];
        emit_piece<Acc, Part>(a, q, d, seq, is_end, started, (Part)piece, cnt, &s_desc);
    }
    __syncthreads();
    if (!RUN || base + n >= run_n) break;
    if (s == 0) {
        carry = s_sum[buf][(subs - 1) * D + d];
        carry_pos = s_pos[buf][(subs - 1) * D + d];
        if (d == 0 && carry_pos >= base) s_carry_seq = s_seq[carry_pos - base];
    }
    base += n;
    g0 += n;
    rem0 += n;
    }
    if (tid == 0 && a.desc) a.desc[q] = s_desc;
}

// ------------------------------------------------------------------- flat
//
// Frames of few bytes in pieces that are long beside them: a wave takes the bytes of a piece as one flat stream, 16 to a
// lane, whatever a frame is.  The least common multiple of a frame and a vector is `P` vectors (of 74 bytes: 37, eight
// frames), and a step is as many whole multiples of that as the wave's lanes hold, a vector to each, so that a lane
// finds the same features of the same frames in every step and adds them up in registers.  Only where a piece ends are
// the lanes' sums brought together by feature, through LDS.
// A workgroup takes a piece of one block, or several whole ones, and each of its four waves a quarter of the slots, wherever
// that cuts a segment: what the waves leave open is put together in LDS, so that only borders between workgroups inside a
// block cost partial sums.

constexpr int kFlatSlots = 8000;           // of a workgroup, at most: a wave's quarter and its neighbours' flags are 64 words
constexpr int kFlatGroups = 512;           // of 16 slots' flags
constexpr int kFlatLoads = 4;              // steps asked for at a time (8 take registers from half the waves: 5 to 40 % slower)
// int32, whose sums take two registers each, looks at its flags in LDS again for every piece: with two words of them in registers,
// as the others have them, it needs 66 of the 64 that eight waves per SIMD leave, and kept them in memory instead (364 MB of
// 36-byte frames in pieces of 620 frames 72.2 us, 64.1 like this; with seven waves 64.4, but 254 MB of 80-byte frames, whose 1977
// workgroups are more than are at work at once then, 59.7 -> 66.7, 59.3 like this).  (All keep some 15 scalar registers in lanes
// of a vector one; with seven waves, where none need to, bytes, halfs and floats take 0.97 to 1.03 of the time.)
template <typename ElemT> constexpr bool kFlatLooksAgain = std::is_same<ElemT, int32_t>::value;
constexpr int kWaves = kThreads / kWave;
static_assert(kFlatSlots / kWaves + 1 + 32 <= kWave * 32, "a wave's slots: a word of flags per lane");
static_assert((kFlatSlots / kWaves * (kWaves - 1)) / 32 + kWave <= kFlatGroups / 2, "the words that the last wave reads");

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename ElemT>
constexpr int kFlatScratch = kWave * (16 / (int)sizeof(ElemT));      // sums of a wave's lanes

// What a lane adds up of a piece: element k of its vector in every step.  Trees of the steps taken at a time, and those
// in 64 bits.
template <typename ElemT>
struct FlatSums {
    typedef typename Elem<ElemT>::Acc Acc;
    typedef typename TileSum<ElemT>::T Part;
    static constexpr int EPV = 16 / (int)sizeof(ElemT);
    Part sum[EPV];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < EPV; ++k) sum[k] = 0;
    }
    template <int C>
    __device__ __forceinline__ void add(const vec16 (&x)[C])
    {
#pragma unroll
        for (int k = 0; k < EPV; ++k) {
            Acc s[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                union { vec16 v; ElemT e[EPV]; } w;
                w.v = x[u];
                s[u] = Elem<ElemT>::get(w.e[k]);
            }
#pragma unroll
            for (int w = 1; w < C; w *= 2)
#pragma unroll
                for (int u = 0; u + w < C; u += 2 * w) s[u] += s[u + w];
            sum[k] += (Part)s[0];
        }
    }
    __device__ __forceinline__ Part get(int k) const { return sum[k]; }
};
// Bytes: whole numbers, two to a word, the even and the odd ones of each.
template <>
struct FlatSums<uint8_t> {
    uint32_t even[4], odd[4];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j < 4; ++j) even[j] = odd[j] = 0;
    }
    template <int C>
    __device__ __forceinline__ void add(const vec16 (&x)[C])
    {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int u = 0; u < C; ++u) {
                even[j] += x[u][j] & 0x00ff00ffu;
                odd[j] += (x[u][j] >> 8) & 0x00ff00ffu;
            }
    }
    __device__ __forceinline__ float get(int k) const
    {
        const uint32_t w = (k & 1) ? odd[k / 4] : even[k / 4];
        return (float)((k & 2) ? w >> 16 : w & 0xffffu);
    }
};
constexpr int kFlatByteFrames = 8;         // of bytes, a step holds so many frames or more:
static_assert((kFlatSlots / kWaves + 1 + kFlatByteFrames - 1) / kFlatByteFrames * 255 < 1 << 16, "a piece's bytes add up in 16 bits");

template <typename ElemT, bool STREAM>
__global__ __launch_bounds__(kThreads, 8) void reduce_flat_kernel(ReduceArgs a)
{
    typedef typename Elem<ElemT>::Acc Acc;
    typedef typename TileSum<ElemT>::T Part;
    typedef typename OutOf<Acc>::T Out;
    constexpr int EPV = 16 / (int)sizeof(ElemT);
    constexpr int N = kFlatLoads;
    extern __shared__ vec16 s_flat[];          // sums of the waves' lanes, then heads and tails of the waves
    __shared__ alignas(16) uint16_t s_valid[kFlatGroups], s_break[kFlatGroups];
    __shared__ ChunkDesc s_piece[kWaves];
    const int tid = (int)threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(wave_id());
    const int32_t D = a.feat_dim;
    Part* const scratch = reinterpret_cast<Part*>(s_flat) + wave * kFlatScratch<ElemT>;
    Part* const s_head = reinterpret_cast<Part*>(s_flat) + kWaves * kFlatScratch<ElemT>;       // [kWaves][D]
    Part* const s_tail = s_head + kWaves * D;

    const int64_t q = blockIdx.x;
    int64_t g0;
    int32_t n, rem0;
    if (a.n_chunks > 1) {
        const int64_t b = (int64_t)((uint32_t)q / (uint32_t)a.n_chunks);
        rem0 = (int32_t)(q - b * a.n_chunks) * a.chunk;
        g0 = b * (int64_t)a.t_blk + rem0;
        n = min(a.chunk, a.t_blk - rem0);
    } else {
        const int64_t b0 = q * a.blocks_per_tile;
        rem0 = 0;
        g0 = b0 * (int64_t)a.t_blk;
        n = (int32_t)min((int64_t)a.blocks_per_tile, a.num_blocks - b0) * a.t_blk;
    }
    // flags, 16 slots to a lane: which slots are valid, and which cannot continue the segment of the slot in front (padding, a
    // start flag, a block's first slot, a slot behind padding); breaks behind the tile but for the slot next to it
    {
        const uint32_t T = (uint32_t)a.t_blk;
        constexpr int kRounds = kFlatGroups / kThreads;
        FlagBytes fb[kRounds];
        const bool more_behind = a.n_chunks > 1 && rem0 + n < a.t_blk;
        const int64_t behind = min(g0 + n, a.total_slots - 1);
        const uint8_t behind_valid = a.valid[behind], behind_reset = a.reset[behind];
#pragma unroll
        for (int r = 0; r < kRounds; ++r) fb[r].load(a, g0 + 16 * (tid + r * kThreads), n - 16 * (tid + r * kThreads));
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int i = tid + r * kThreads;
            uint32_t vm16 = 0, brk = 0xffffu;
            const int32_t left16 = n - 16 * i;
            if (left16 >= 0) {
                const uint32_t pos = (uint32_t)(rem0 + 16 * i) % T;
                const uint32_t before = pos != 0 && fb[r].before != 0 ? 1u : 0u;
                vm16 = fb[r].mask(fb[r].valid, a.valid, left16, a.total_slots);
                const uint32_t rm16 = fb[r].mask(fb[r].reset, a.reset, left16, a.total_slots);
                uint32_t first = 0;
                for (uint32_t k = pos == 0 ? 0 : T - pos; k < 16; k += T) first |= 1u << k;
                brk = (~vm16 | rm16 | first | ~(vm16 << 1 | before)) & 0xffffu;
                if (left16 < 16) {
                    const bool goes_on = more_behind && behind_valid != 0 && behind_reset == 0 &&
                                         ((left16 == 0 ? before : vm16 >> (left16 - 1)) & 1u);
                    brk = goes_on ? brk & ~(1u << left16) : brk | 1u << left16;
                }
            }
            s_valid[i] = (uint16_t)vm16;
            s_break[i] = (uint16_t)brk;
        }
    }
    __syncthreads();

    // the wave's slots [lo, hi); a lane holds the flags of 32 of them
    const int32_t lo = n * wave / kWaves, hi = n * (wave + 1) / kWaves;
    const int32_t base = lo & ~31, mine = base + 32 * lane;
    auto below = [&](int32_t slot) { const int32_t k = slot - mine; return k <= 0 ? 0u : k >= 32 ? ~0u : (1u << k) - 1u; };
    auto breaks = [&]() { return reinterpret_cast<const uint32_t*>(s_break)[(base >> 5) + lane] | ~below(hi + 1); };
    auto valids = [&]() { return reinterpret_cast<const uint32_t*>(s_valid)[(base >> 5) + lane] & below(hi); };
    constexpr bool kAgain = kFlatLooksAgain<ElemT>;
    const uint32_t kept_breaks = kAgain ? 0u : breaks(), kept_valids = kAgain ? 0u : valids();
    // the first slot from `t` on whose bit is set, INT32_MAX if there is none
    auto find = [&](uint32_t bits, int32_t t) {
        const uint32_t m = bits & ~below(t);
        const uint64_t vote = __ballot(m != 0);
        if (vote == 0) return INT32_MAX;
        const int l = __builtin_ctzll(vote);
        return base + 32 * l + (int32_t)__builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)m, l));
    };

    const int64_t frame_bytes = (int64_t)D * (int64_t)sizeof(ElemT);
    const uint8_t* const end_of_all = a.packed + a.total_slots * frame_bytes;
    const uint32_t step_bytes = (uint32_t)a.step_vec * 16u;
    const uint32_t lane_off = 16u * (uint32_t)min(lane, a.step_vec - 1);      // (what idle lanes add up is not looked at)
    ChunkDesc piece{kHeadNone, 0, 0, -1};
    FlatSums<ElemT> run;
    auto load = [](const uint8_t* at) {
        const vec16_any* from = reinterpret_cast<const vec16_any*>(at);
        return STREAM ? __builtin_nontemporal_load(from) : *from;
    };

    for (int32_t t = lo; t < hi;) {
        t = find(kAgain ? valids() : kept_valids, t);
        if (t >= hi) break;
        const uint32_t brk = kAgain ? breaks() : kept_breaks;
        const int32_t stop = find(brk, t + 1), e = min(stop, hi);
        const bool closed = stop <= hi;
        const bool head_open = t == lo && find(brk, t) != t;
        const int32_t seq = head_open ? -1 : a.seq_id[g0 + t];
        const int32_t frames = e - t;
        // whole steps, and frames of one more
        const int32_t steps = (int32_t)__umulhi((uint32_t)frames, a.step_magic), rest = frames - steps * a.step_frames;
        const uint8_t* p = a.packed + (g0 + t) * frame_bytes;
        run.clear();
        int32_t at = 0;
        for (; at + N <= steps; at += N) {
            vec16 x[N];
#pragma unroll
            for (int u = 0; u < N; ++u) x[u] = load(p + (uint32_t)u * step_bytes + lane_off);
            run.add(x);
            p += (int64_t)N * step_bytes;
        }
        const int32_t left = steps - at + (rest ? 1 : 0);          // the last ones, `rest` frames in the very last
        auto last_steps = [&](auto count) {
            constexpr int C = decltype(count)::value;
            // in the very last step: how many of a lane's bytes count, and vectors up to the last that holds one
            const int32_t bytes = rest ? rest * (int32_t)frame_bytes : (int32_t)step_bytes;
            const uint32_t last_vec = (uint32_t)(bytes + 15) / 16u - 1u;
            const bool careful = p + (int64_t)(left - 1) * step_bytes + 16 * ((int64_t)last_vec + 1) > end_of_all;
            vec16 x[C];
#pragma unroll
            for (int u = 0; u < C; ++u) {
                const uint32_t off = u < left - 1 ? lane_off : min(lane_off, 16u * last_vec);
                const uint8_t* from = p + (int64_t)min(u, left - 1) * step_bytes + off;
                // (the tensor's last vector, where it is no whole one, is put together below)
                x[u] = load(careful && from > end_of_all - 16 ? end_of_all - 16 : from);
            }
            const int32_t counts = bytes - 16 * lane;
            vec16 keep;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int32_t bits = 8 * counts - 32 * j;
                keep[j] = bits >= 32 ? ~0u : (1u << max(bits, 0)) - 1u;
            }
            if (careful && lane == (int)last_vec) {
                const uint8_t* from = p + (int64_t)(left - 1) * step_bytes + 16u * last_vec;
                union { vec16 v; ElemT e[EPV]; } own;
                own.v = vec16{0u, 0u, 0u, 0u};
#pragma unroll
                for (int k = 0; k < EPV; ++k)
                    if (k * (int)sizeof(ElemT) < counts) own.e[k] = reinterpret_cast<const ElemT*>(from)[k];
#pragma unroll
                for (int u = 0; u < C; ++u)
                    if (u == left - 1) x[u] = own.v;
            }
#pragma unroll
            for (int u = 0; u < C; ++u) {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[u][j] &= u < left - 1 ? ~0u : u == left - 1 ? keep[j] : 0u;
            }
            run.add(x);
        };
        if (left > N / 2) last_steps(std::integral_constant<int, N>());
        else if (left > 0) last_steps(std::integral_constant<int, N / 2>());

        // the lanes' sums by feature: element i of a step is feature i % D
        wave_sync();
#pragma unroll
        for (int k = 0; k < EPV; ++k) scratch[lane * EPV + k] = run.get(k);
        wave_sync();
        const int32_t side = D <= kWave / 2 ? kWave / D : 1;          // lanes that share a feature
        for (int32_t d0 = 0; d0 < D; d0 += kWave) {
            const int32_t j0 = side > 1 ? lane / D : 0;
            const int32_t d = side > 1 ? lane - j0 * D : d0 + lane;
            Part sum = 0;
            if (j0 < side && d < D) {
                for (int32_t j = j0; j < a.step_frames; j += 4 * side) {      // (four look-ups at a time)
                    Part part[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) part[i] = scratch[min(j + i * side, a.step_frames - 1) * D + d];
#pragma unroll
                    for (int i = 0; i < 4; ++i) sum += j + i * side < a.step_frames ? part[i] : (Part)0;
                }
            }
            if (side > 1) {
                wave_sync();
                scratch[lane] = sum;
                wave_sync();
                if (lane < D) {
                    sum = 0;
                    for (int32_t j = 0; j < side; j += 4) {
                        Part part[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) part[i] = scratch[min(j + i, side - 1) * D + lane];
#pragma unroll
                        for (int i = 0; i < 4; ++i) sum += j + i < side ? part[i] : (Part)0;
                    }
                }
            }
            if (j0 != 0 || d >= D) continue;
            if (head_open) s_head[wave * D + d] = sum;
            else if (!closed) s_tail[wave * D + d] = sum;
            else if ((uint32_t)seq < (uint32_t)a.n_seq)
                static_cast<Out*>(a.out)[(int64_t)seq * D + d] = (Out)finish<Part>(sum, frames, a.mean);
        }
        if (head_open) {
            piece.head_state = closed ? kHeadClosed : kHeadThrough;
            piece.cnt_head = frames;
        } else if (!closed) {
            piece.cnt_tail = frames;
            piece.seq_tail = seq;
        }
        t = e;
    }
    if (lane == 0) s_piece[wave] = piece;
    __syncthreads();

    // what the waves left open, in time order
    ChunkDesc desc{kHeadNone, 0, 0, -1};
    for (int32_t d = tid; d == tid || d < D; d += kThreads) {
        Part sum = 0;
        int32_t cnt = 0, seq = -1;
        bool live = false, started = false;
        for (int w = 0; w < kWaves; ++w) {
            const ChunkDesc part = s_piece[w];
            if (part.head_state != kHeadNone) {
                if (!live) { sum = 0; cnt = 0; started = false; }     // it comes from the tile in front
                live = part.head_state == kHeadThrough;
                cnt += part.cnt_head;
                if (d < D) sum += s_head[w * D + d];
                if (!live && started) {
                    if (d < D && (uint32_t)seq < (uint32_t)a.n_seq)
                        static_cast<Out*>(a.out)[(int64_t)seq * D + d] = (Out)finish<Part>(sum, cnt, a.mean);
                } else if (!live) {
                    if (d < D && a.head_part) put_part<Part>(a.head_part, q, d, D, sum);
                    desc.head_state = kHeadClosed;
                    desc.cnt_head = cnt;
                }
            }
            if (part.cnt_tail > 0) {
                live = started = true;
                cnt = part.cnt_tail;
                seq = part.seq_tail;
                if (d < D) sum = s_tail[w * D + d];
            }
        }
        if (live && started) {
            if (d < D && a.tail_part) put_part<Part>(a.tail_part, q, d, D, sum);
            desc.cnt_tail = cnt;
            desc.seq_tail = seq;
        } else if (live) {
            if (d < D && a.head_part) put_part<Part>(a.head_part, q, d, D, sum);
            desc.head_state = kHeadThrough;
            desc.cnt_head = cnt;
        }
    }
    if (tid == 0 && a.desc) a.desc[q] = desc;
}

// ----------------------------------------------------------------- stitch

// Segments cut by chunk borders: tail piece + the head pieces of the following
// chunks, added in time order.  One thread per (chunk, feature): a workgroup
// takes 256 features of one chunk, or, for frames of fewer than 256 features,
// all features of `chunks_per_wg` consecutive chunks.  Nothing but latency: the next
// chunk's piece is asked for together with this chunk's description (most segments end there), and
// of those behind it kStitchAhead at once; what a segment that ends earlier asked for too much is in
// the workspace but not looked at.  One sequence in 74 chunks of 347 int32: 38 us with one piece after
// the other, 8 like this; 16 or 32 ahead gain nothing more and cost the others registers (100000
// sequences of 16 floats, whole call: 267 us with one, 269 with 8, 275 with 16, 296 with 32).
constexpr int kStitchAhead = 8;
template <typename Acc, typename Part>
__global__ __launch_bounds__(kThreads) void reduce_stitch_kernel(ReduceArgs a, int32_t feat_tiles,
                                                                 int32_t chunks_per_wg)
{
    typedef typename OutOf<Acc>::T Out;
    int64_t q, d;
    if (chunks_per_wg > 1) {
        const int32_t r = (int32_t)threadIdx.x / a.feat_dim;
        if (r >= chunks_per_wg) return;
        q = (int64_t)blockIdx.x * chunks_per_wg + r;
        d = (int32_t)threadIdx.x - r * a.feat_dim;
        if (q >= a.total_chunks) return;
    } else {
        q = (int64_t)blockIdx.x / feat_tiles;
        d = ((int64_t)blockIdx.x % feat_tiles) * kThreads + threadIdx.x;
    }
    const int64_t last = a.total_chunks - 1;
    const int64_t q1 = q < last ? q + 1 : last;
    const ChunkDesc first = a.desc[q], next = a.desc[q1];
    if (first.cnt_tail <= 0 || d >= a.feat_dim) return;
    auto part_of = [&](const void* parts, int64_t chunk) -> Part {
        if constexpr (sizeof(Part) != sizeof(Acc)) {
            const float* row = static_cast<const float*>(parts) + 2 * chunk * a.feat_dim + d;
            return (Part)row[0] + (Part)row[a.feat_dim];
        } else {
            return static_cast<const Part*>(parts)[chunk * a.feat_dim + d];
        }
    };
    const Part tail = part_of(a.tail_part, q), head = part_of(a.head_part, q1);
    Running<Part, sizeof(Part) == 4> sum;
    sum.clear();
    sum.add(tail);
    int64_t cnt = first.cnt_tail;
    bool goes_on = q < last && next.head_state != kHeadNone;
    if (goes_on) {
        sum.add(head);
        cnt += next.cnt_head;
        goes_on = next.head_state == kHeadThrough;
    }
    for (int64_t from = q + 2; goes_on && from <= last; from += kStitchAhead) {
        int32_t state[kStitchAhead], frames[kStitchAhead];
        Part part[kStitchAhead];
#pragma unroll
        for (int k = 0; k < kStitchAhead; ++k) {
            const int64_t q2 = from + k < last ? from + k : last;
            state[k] = a.desc[q2].head_state;
            frames[k] = a.desc[q2].cnt_head;
            part[k] = part_of(a.head_part, q2);
        }
#pragma unroll
        for (int k = 0; k < kStitchAhead; ++k) {
            // no branch: the loads above would move into it
            const bool here = goes_on && from + k <= last && state[k] != kHeadNone;
            auto added = sum;
            added.add(part[k]);
            sum = here ? added : sum;
            cnt += here ? frames[k] : 0;
            goes_on = here && state[k] == kHeadThrough;
        }
    }
    if ((uint32_t)first.seq_tail < (uint32_t)a.n_seq)
        static_cast<Out*>(a.out)[(int64_t)first.seq_tail * a.feat_dim + d] =
            (Out)finish<Part>(sum.sum, (int32_t)cnt, a.mean);
}

// ------------------------------------------------------------------- host

struct ReducePlan {
    bool wide, staged;
    bool run;                // staged: a workgroup takes the tiles of a whole chunk one after another
    int32_t tile;            // of this many slots
    bool flat;
    int step_vec, step_frames;   // flat: see ReduceArgs
    bool split;              // wide: two waves to a chunk, and see ReduceArgs
    int32_t reach;
    int vec;                 // wide: elements per lane (16 bytes, 4 bytes or one element)
    int row_lanes_log2;
    int n_vec;
    int32_t chunk, n_chunks;
    int32_t blocks_per_tile;  // narrow and staged, t_blk < the tile: whole blocks per tile
    int32_t slots;           // staged: slots per lane
    int64_t total_chunks;
    bool partials;           // can a chunk border cut a segment
    bool pair_parts;         // partial sums are floats and what those lack
    size_t desc_off, head_off, tail_off, bytes;
};

static int elem_size(bload_dtype dtype) { return dtype == BLOAD_U8 ? 1 : dtype == BLOAD_F16 ? 2 : 4; }

// Which of two cuts is the faster hangs, for some frames, on the length of the pieces as well.  The guess at hand
// is `mean`, the slots per row of the result (too short for a worker's share, whose rows are those of all
// workers; either cut is right).
//
// Lanes of one element, for frames that are no whole vectors:
//   - floats and int32 over more than one wave, pieces of a few frames (24 frames: 1.3-8 KB a frame up to
//     12 % slower with 16-byte lanes, 1550 frames: 2-30 % faster; equal at 53 frames and four fifths of the
//     lanes at work), unless blocks are short (34 slots x 5012 bytes: 40 us, one float a lane 49)
//   - bytes and halfs of which a row of 4-byte lanes holds few, none of them at a whole word, long
//     pieces (2 GB, 1550 frames: 101 bytes 670 us, 4 bytes a lane 770; 0.8 GB, 32 frames: 447 and 266)
static bool takes_one_element(int32_t t_blk, int64_t feat_dim, int es, int64_t mean)
{
    const int64_t frame_bytes = feat_dim * es, vectors = ceil_div(frame_bytes, 16);
    if (frame_bytes < 64 || feat_dim < 33 || frame_bytes % 16 == 0) return false;
    if (es == 4) return vectors > kWave && t_blk >= 128 && mean * vectors < 40 * (int64_t)round_up((size_t)vectors, kWave);
    return frame_bytes % 4 != 0 && feat_dim < (es == 1 ? 128 : 96) && mean >= 512;
}

// Staged tiles of frames of 2 to 5 elements, a block in two or three of them: one workgroup takes them one after
// another, which spares the stitching kernel (2 us), where pieces are long.  255 blocks of 2828 slots x 2 floats:
// 10.2 -> 8.5 us; two halfs in pieces of 24 frames, 17 blocks of 4243 slots: 10.4 -> 13.  With many tiles
// only where elements are 4 bytes, of which a tile is many loads (444 blocks of 3757 x 3 floats: 17.8 -> 13.4 us;
// 33985 sequences in blocks of 2828 x 2 bytes: 131 -> 195).
static bool takes_run(int64_t tiles, bool few, int64_t feat_dim, int es, int64_t mean)
{
    return feat_dim <= 5 && mean >= 64 && (few ? tiles <= 2 : es == 4 && tiles <= 3);
}

// The flat cut, if the frames allow it: a step holds two frames or more, and of bytes eight.
constexpr int64_t kFlatLeast = (int64_t)12 << 20, kFlatMiddle = (int64_t)50 << 20, kFlatLarge = (int64_t)200 << 20;
static bool flat_cut(ReducePlan& p, int64_t num_blocks, int32_t t_blk, int64_t feat_dim, int es)
{
    const int64_t frame_bytes = feat_dim * es;
    if (feat_dim < 2 || frame_bytes > kWave * 16 / 2 || num_blocks * t_blk * frame_bytes < kFlatLeast) return false;
    int64_t common = 16;                   // of a frame and a vector
    while (frame_bytes % common) common /= 2;
    const int64_t period = frame_bytes / common;
    if (period > kWave) return false;
    p.step_vec = (int)(kWave / period * period);
    p.step_frames = (int)(p.step_vec * 16 / frame_bytes);
    if (es == 1 && p.step_frames < kFlatByteFrames) return false;
    p.flat = true;
    // A thousand workgroups are enough (four times as many: 7 to 25 % slower where that cuts blocks), none smaller than 16
    // KiB, and several short blocks to one up to 128 KiB (600 MB of 384 bytes, blocks of 60 slots, pieces of 40: 182 us with
    // 32 KiB, 123 like this).
    int64_t cuts = std::min<int64_t>(ceil_div((int64_t)1024, num_blocks), t_blk * frame_bytes >> 14);
    cuts = std::max<int64_t>(std::max<int64_t>(cuts, 1), ceil_div(t_blk, kFlatSlots));
    p.chunk = (int32_t)ceil_div(t_blk, cuts);
    p.n_chunks = (int32_t)ceil_div(t_blk, p.chunk);
    p.blocks_per_tile = 1;
    p.total_chunks = num_blocks * p.n_chunks;
    if (p.n_chunks == 1) {
        const int64_t blocks = std::min(std::min<int64_t>(kFlatSlots / t_blk, ((int64_t)128 << 10) / (t_blk * frame_bytes)), num_blocks / 1024);
        p.blocks_per_tile = (int32_t)std::max<int64_t>(1, blocks);
        p.total_chunks = ceil_div(num_blocks, p.blocks_per_tile);
    }
    p.partials = p.n_chunks > 1;
    return true;
}

// Whether pieces are long enough for it.  A piece costs a wave some 5 us whatever it holds, with 8192 waves at work, so
// that its bytes have to make up for that against
//   - staged tiles, which take their time by elements: 250 MB, 58 bytes in pieces of 80 frames 173 -> 69 us, 14 bytes x 80 211
//     -> 147, 16 bytes x 80 even, 17 bytes x 20 0.4 times as fast; 28 halfs x 130 189 -> 77; 8 bytes of floats x 400 107 -> 76, x 80 123 and 266
//     (frames of few floats end in many lanes).  Tensors of 16 to 50 MB, less in flight: 64 bytes of floats x 59 33.7 -> 21.5, 80 x 43 32.5
//     -> 20.9, but 22 bytes of halfs x 40 20 and 30, 84 of floats x 37 17 and 20, 24 x 116 18 and 22; 16 MB of 80-byte frames in blocks
//     of 3000, which both cut, x 160 12 and 14; and not where a tile takes several blocks that would be a workgroup each (1949 blocks
//     of 8 KB 9.7 us, 12.7)
//   - wide rows of 4-byte lanes or single elements: 600 MB, 86 bytes of halfs x 40 197 -> 148; 100 bytes of int32 x 80 153 ->
//     127; but 140 bytes of floats, half the lanes idle here, x 60 43 and 52.  Frames of up to 128 bytes of bytes and halfs
//     in short blocks, which a row walks whole: 72 bytes x 71, 91 MB 32 and 39, 122 x 57, 81 MB 19 and 23, 118 x 27, 240 MB 75 and 85, but 108 x
//     76, 141 MB 38 -> 32; in blocks that rows cut, 120 x 41, 194 MB 74 -> 57.  Longer ones, whose rows have all their lanes at
//     work, below 200 MB: 172 bytes x 24, 83 MB 25 and 30, 220 x 39, 94 MB 22 and 25; in blocks that rows cut 236 x 22, 81 MB 34 -> 32, 184 x 22, 164 MB 57 and 63
//   - wide rows of whole vectors, whose rows wait for each other: 600 MB, 64 bytes x 80 184 -> 117, 208 x 10 176 -> 152, 480 x 20 159 ->
//     135; 60 MB, 336 bytes x 40 24.5 -> 18, 144 x 20 23 and 30; 16 MB, 384 x 400 12 and 14.  (More than 192 halfs take 30 KB of
//     LDS here, four or five workgroups to a compute unit: 480 bytes x 28, 56 MB in 1387 workgroups 17 and 23.)
static bool takes_flat(const ReducePlan& flat, const ReducePlan& other, int64_t total_bytes, int64_t frame_bytes, int es, int64_t mean)
{
    const int64_t piece = mean * frame_bytes;
    const bool large = total_bytes >= kFlatLarge, middle = total_bytes >= kFlatMiddle;
    if (!other.wide) {
        if (!middle && (flat.n_chunks > 1 ? frame_bytes >= 32 : flat.total_chunks > other.total_chunks)) return false;
        const int64_t least = es == 1 ? 1100 : es == 2 ? 2000 : frame_bytes < 20 ? 3200 : 1600;
        return piece >= (large ? least : middle || (es != 4 && frame_bytes <= 64) ? least * 8 / 5 : least * 2);
    }
    if (frame_bytes % 16 == 0)
        return large ? piece >= 2000 : middle && flat.n_chunks == 1 && piece >= 12000 && (es != 2 || frame_bytes <= 384);
    if (es == 4) return frame_bytes <= 128 && piece >= 5000;
    const bool short_blocks = other.n_chunks == 1;
    if (large) return piece >= 3800;
    if (frame_bytes > 128) return middle && !short_blocks && piece >= 5000;
    return piece >= (short_blocks ? 8000 : 3800);
}

// Where the workspace holds what borders cut.
static void add_partials(ReducePlan& p, int64_t feat_dim, bload_dtype dtype, bool lean)
{
    const int es = elem_size(dtype);
    if (!p.partials) return;
    {
        // Rows of whole vectors keep their partial sums of halfs and floats in 32 bits.  Tiles, and narrower lanes
        // of frames that are no whole vectors, make more of them, and rounding each would cost accuracy (sequences
        // of 388 frames of 66 halfs in chunks of 70 slots: root mean square error against 64 bits 2.7e-8, 2.3e-8 in
        // half as many chunks)
        p.pair_parts = (dtype == BLOAD_F16 || dtype == BLOAD_F32) &&
                       (p.staged || p.flat || (p.wide && p.vec * es < 16 && feat_dim * es % 16 != 0 && !lean));
        const size_t acc = dtype == BLOAD_I32 || p.pair_parts ? 8 : 4;
        size_t off = 0;
        p.desc_off = off; off += round_up((size_t)p.total_chunks * sizeof(ChunkDesc), 16);
        p.head_off = off; off += round_up((size_t)p.total_chunks * (size_t)feat_dim * acc, 16);
        p.tail_off = off; off += round_up((size_t)p.total_chunks * (size_t)feat_dim * acc, 16);
        p.bytes = off;
    }
}

// `lean`: a cut that makes do with little workspace, or none, at the price of workgroups: tiles of a whole chunk
// one after another by one workgroup, chunks as long as whole blocks and 12288 slots; lanes of one element (the
// most workgroups per chunk) and plain partial sums for wide frames that are no whole vectors.
static ReducePlan reduce_plan(int64_t num_blocks, int32_t t_blk, int64_t feat_dim, bload_dtype dtype, int64_t mean,
                              bool lean = false)
{
    ReducePlan p{};
    const int es = elem_size(dtype);
    const int64_t frame_bytes = feat_dim * es;
    p.wide = frame_bytes >= 64;
    const bool one_element = takes_one_element(t_blk, feat_dim, es, mean) ||
                             (lean && feat_dim >= kStagedFrame && frame_bytes % 16 != 0);
    // Lanes of 16 bytes, unless that leaves fewer than two workgroups per compute unit (four where the
    // vectors are not aligned): then lanes of 4 bytes, then of one element, which spread a frame over
    // more waves (15 blocks of 830 slots x 342 bytes: 23 us with 16 bytes a lane, 14 with one).
    // Frames that are no whole vectors also take the narrower lanes where
    //   - a row would be 16 lanes or fewer (up to 256 bytes): four rows and more to a wave wait for each
    //     other's pieces, and no vector is aligned (2 GB, sequences of 1550 frames, 16 / 4 bytes a lane:
    //     132 bytes of halfs 611 / 416 us, 140 of bytes 650 / 425; of 24 frames, 1 GB: 115 bytes 577 / 385)
    //   - a frame is some waves of vectors and a bit, a third of the lanes idle (1028 bytes of floats in
    //     pieces of 24 frames, 1 GB: 300 us, 240 with one a lane; of halfs 350, 262 with 4 bytes); a row
    //     of 32 or 64 lanes in one wave keeps the vectors, half idle or not (260 bytes of floats: 266 us,
    //     342 with one a lane)
    // Whole vectors stay 16 bytes a lane whatever is idle (272 bytes, 2.5 GB: 484 us, one float a lane 722).
    const bool whole = frame_bytes % 16 == 0;
    const int widths[3] = {16, 4, es};
    for (int w = 0; p.wide && w < 3; ++w) {
        p.vec = widths[w] / es;
        p.n_vec = (int)ceil_div(feat_dim, p.vec);
        // a row is at most one wave wide: the last lane-slice of a frame then idles at most 63
        // lanes, and the four waves of a workgroup walk four different chunks, or two
        p.row_lanes_log2 = 0;
        while ((1 << p.row_lanes_log2) < p.n_vec && p.row_lanes_log2 < 6) ++p.row_lanes_log2;
        const int rows = kThreads >> p.row_lanes_log2;
        const int64_t feat_tiles = ceil_div(p.n_vec, 1 << p.row_lanes_log2);
        // Enough chunks per block for ~1024 workgroups (four per compute unit, as many as are
        // resident at once), each at least 64 slots long.  No more: reads at full rate need few
        // waves in flight, while every chunk border costs partial sums, and writes mixed into the
        // read stream cost far more than their bytes.
        int64_t want = ceil_div((int64_t)1024 * rows, num_blocks * feat_tiles);
        const int64_t most = t_blk / 64 > 0 ? t_blk / 64 : 1;
        if (want > most) want = most;
        if (want < 1) want = 1;
        // Whole blocks that already make more workgroups than are resident at once (2048) run in
        // a few long rounds, and the last one leaves the chip half empty for a long time: then
        // chunks of at least 512 slots towards 12288 workgroups (34576 blocks of 3000 slots x 320
        // bytes: 3.98 ms in whole blocks, 3.89 in two chunks per block, 3.85 in three, 3.87 in
        // four, 3.91 in five).
        const int64_t whole_block_groups = num_blocks * feat_tiles / rows;
        if (want == 1 && whole_block_groups >= 2048 && whole_block_groups < 12288) {
            want = ceil_div((int64_t)12288, whole_block_groups);
            const int64_t most_long = t_blk / 512 > 0 ? t_blk / 512 : 1;
            if (want > most_long) want = most_long;
        }
        int64_t chunk = ceil_div(t_blk, want);
        // Rows of one wave and sequences of a few frames: the waves' chunks hold very different numbers of pieces, and
        // all are at work at once, so that the call lasts as long as the slowest.  Two waves to a chunk even that out.  Neither
        // cuts a segment, and one that ends within 32 slots behind the chunk stays whole, so that hardly any partial sums
        // are left (10000 sequences of 23 frames of 4096 bytes: 220 -> 197 us, 203 where the chunks' borders cut; 330 of them
        // 21.0 -> 15.9; 8900 of 3072 bytes 156 -> 136).  Chunks half as long would even out as much, but where pieces are
        // long, as they may be in a worker's share whatever `mean` says, those cost partial sums (an eighth of the rows, 128
        // frames of 1024 bytes in blocks of 300: 99 us, 136 in half chunks, 82 like this; 250 of 4096 bytes 64, 77, 67).
        // (Not where the chunks above are cut for more workgroups than are at work at once.)
        p.split = !lean && whole && p.row_lanes_log2 == 6 && want > 1 && whole_block_groups < 2048 && mean <= kShortPieces;
        const int64_t lds_cap = kWideFlagBytes / rows - 2;
        if (chunk > lds_cap) chunk = lds_cap;
        p.chunk = (int32_t)chunk;
        p.reach = p.split ? std::min(kReach, p.chunk) : 0;
        p.n_chunks = (int32_t)ceil_div(t_blk, chunk);
        p.total_chunks = num_blocks * p.n_chunks;
        p.partials = p.n_chunks > 1;
        const int64_t groups = ceil_div(p.total_chunks << p.split, rows) * feat_tiles;
        // Small frames in rows of a few lanes: a workgroup walks many chunks, and where that leaves too
        // few workgroups the staged tiles are the more.  The line lies at some 24 KiB of lanes' vectors at a time,
        // at half of that for blocks of less than two chunks (13 blocks of 1580 slots x 128 bytes: 33 -> 15 us;
        // 857 of 777 x 64: 70 us in wide rows of 16 or 4 bytes a lane 34, in tiles 16; 571 of 777 x 96: 51, 29, 24;
        // 428 of 777 x 192: 45, 23, 31; 2500 of 110 x 192: 32, 13, 20).
        if (w == 0 && feat_dim < kStagedFrame && (lean || groups * p.n_vec < (t_blk < 128 ? 760 : 1550))) p.wide = false;
        const bool suits = w > 0 || whole ||
                           (frame_bytes > 256 && (feat_tiles == 1 || p.n_vec * 3 >= (feat_tiles << p.row_lanes_log2) * 2));
        if (groups >= (whole ? 512 : 1024) && suits && !one_element) break;
    }
    if (!p.wide) {
        p.staged = feat_dim > 1;
        // tiles never straddle a block: pieces of one block, or several whole blocks
        p.chunk = kNarrowTile;
        if (p.staged) {
            const int32_t groups = kThreads / (int32_t)feat_dim;
            const int32_t longest = groups * kStagedSlots;
            // shorter lanes where tiles are few, unless only the longer ones hold a whole block (a border costs the
            // stitching kernel: 10 blocks of 1305 slots x 2 floats 11 -> 8.5 us)
            const bool few = num_blocks * t_blk / longest < 512;
            p.slots = few && (t_blk <= groups * kStagedSlotsShort || t_blk > longest) ? kStagedSlotsShort : kStagedSlots;
            p.chunk = groups * p.slots;
            if (t_blk > longest && (lean || takes_run(ceil_div(t_blk, longest), few, feat_dim, es, mean))) {
                p.run = true;
                p.slots = kStagedSlots;
                p.tile = longest;
                p.chunk = lean ? std::min(t_blk, kLeanRun) : t_blk;
            } else if (t_blk > p.chunk) {  // equal pieces
                const int32_t pieces = (int32_t)ceil_div(t_blk, p.chunk);
                p.chunk = (int32_t)ceil_div(ceil_div(t_blk, pieces), p.slots) * p.slots;
            }
        }
        if (t_blk >= p.chunk) {
            p.n_chunks = (int32_t)ceil_div(t_blk, p.chunk);
            p.blocks_per_tile = 1;
            p.total_chunks = num_blocks * p.n_chunks;
        } else {
            p.n_chunks = 1;
            p.blocks_per_tile = p.chunk / t_blk;
            p.total_chunks = ceil_div(num_blocks, p.blocks_per_tile);
        }
        // only a block cut into several tiles can have a segment across a tile border
        p.partials = p.n_chunks > 1;
    }
    add_partials(p, feat_dim, dtype, lean);
    return p;
}

static ReducePlan flat_plan(int64_t num_blocks, int32_t t_blk, int64_t feat_dim, bload_dtype dtype)
{
    ReducePlan p{};
    if (flat_cut(p, num_blocks, t_blk, feat_dim, elem_size(dtype))) add_partials(p, feat_dim, dtype, false);
    return p;
}

// The cut of a call with `room` bytes of workspace, aligned or not.
static ReducePlan chosen_plan(int64_t num_blocks, int32_t t_blk, int64_t feat_dim, bload_dtype dtype, int64_t n_seq, size_t room,
                              bool aligned)
{
    const int64_t slots = num_blocks * (int64_t)t_blk, mean = slots / n_seq;
    const int es = elem_size(dtype);
    ReducePlan p = reduce_plan(num_blocks, t_blk, feat_dim, dtype, mean);
    // (the flat cut takes a workspace only where it is aligned: cuts that need none leave it alone)
    const ReducePlan flat = flat_plan(num_blocks, t_blk, feat_dim, dtype);
    if (flat.flat && flat.bytes <= (aligned ? room : 0) && takes_flat(flat, p, slots * feat_dim * es, feat_dim * es, es, mean)) p = flat;
    // a workspace that is smaller than the query's answer but holds what another cut needs, in the end the leanest
    if (room < p.bytes) {
        const ReducePlan lean = reduce_plan(num_blocks, t_blk, feat_dim, dtype, mean, true);
        if (lean.bytes <= room) p = lean;
    }
    return p;
}

template <typename ElemT, int VEC, bool STREAM>
static void launch_wide(const ReducePlan& p, const ReduceArgs& a, hipStream_t stream)
{
    typedef typename Elem<ElemT>::Acc Acc;
    const int chunks = (kThreads >> p.row_lanes_log2) >> p.split;      // of a workgroup
    const dim3 grid((uint32_t)(ceil_div(p.total_chunks, chunks) * a.feat_tiles));
    size_t lds = (size_t)chunks * (size_t)(p.chunk + p.reach + 2);
    if (VEC > 1 && p.row_lanes_log2 >= 6)     // + the per-wave scratch of the transposed stores
        lds = round_up(lds, 16) + (size_t)(kThreads / kWave) * kWave * kScratchStride<Acc, VEC>() * sizeof(Acc);
    if (p.row_lanes_log2 == 6)
        hipLaunchKernelGGL((reduce_wide_kernel<ElemT, VEC, true, STREAM>), grid, dim3(kThreads), lds, stream, a);
    else
        hipLaunchKernelGGL((reduce_wide_kernel<ElemT, VEC, false, STREAM>), grid, dim3(kThreads), lds, stream, a);
}

template <typename ElemT, bool STREAM>
static void launch_flat(const ReducePlan& p, const ReduceArgs& a, hipStream_t stream)
{
    const size_t lds = (size_t)kWaves * (size_t)(kFlatScratch<ElemT> + 2 * a.feat_dim) * sizeof(typename TileSum<ElemT>::T);
    hipLaunchKernelGGL((reduce_flat_kernel<ElemT, STREAM>), dim3((uint32_t)p.total_chunks), dim3(kThreads), lds, stream, a);
}

template <typename ElemT>
static void launch_reduce(const ReducePlan& p, const ReduceArgs& a, hipStream_t stream)
{
    typedef typename Elem<ElemT>::Acc Acc;
    const bool fits_cache = a.total_slots * a.feat_dim * (int64_t)sizeof(ElemT) <= kMemorySideCache;
    if (p.flat) {
        if (fits_cache) launch_flat<ElemT, false>(p, a, stream);
        else launch_flat<ElemT, true>(p, a, stream);
    } else if (p.wide) {
        constexpr int kVec = 16 / (int)sizeof(ElemT), kSmallVec = 4 / (int)sizeof(ElemT);
        if (p.vec == kVec && fits_cache) launch_wide<ElemT, kVec, false>(p, a, stream);
        else if (p.vec == kVec) launch_wide<ElemT, kVec, true>(p, a, stream);
        else if (p.vec == kSmallVec) launch_wide<ElemT, kSmallVec, false>(p, a, stream);
        else launch_wide<ElemT, 1, false>(p, a, stream);
    } else {
        const dim3 grid((uint32_t)p.total_chunks), block(kThreads);
        // (One element a frame: streaming loads at any size.  A pack leaves no such tensor in the cache, so plain loads find only
        // what a reduction before left there (60 MB of halfs 61 -> 48 us), and behind a kernel that wrote a gigabyte they push its
        // lines out: 64 MB of halfs 68 us, 84, 29 MB of bytes 56 and 66.)
        if (!p.staged)
            hipLaunchKernelGGL(reduce_narrow_kernel<ElemT>, grid, block, 0, stream, a);
        else if (p.run)
            hipLaunchKernelGGL((reduce_staged_kernel<ElemT, kStagedSlots, true>), grid, block, 0, stream, a);
        else if (p.slots == kStagedSlots)
            hipLaunchKernelGGL((reduce_staged_kernel<ElemT, kStagedSlots, false>), grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL((reduce_staged_kernel<ElemT, kStagedSlotsShort, false>), grid, block, 0, stream, a);
    }
    if (p.partials) {
        const int32_t feat_tiles = (int32_t)ceil_div(a.feat_dim, kThreads);
        const int32_t chunks_per_wg = a.feat_dim >= kThreads ? 1 : kThreads / a.feat_dim;
        const int64_t groups = chunks_per_wg > 1 ? ceil_div(p.total_chunks, chunks_per_wg)
                                                 : p.total_chunks * feat_tiles;
        const dim3 grid((uint32_t)groups), block(kThreads);
        if (p.pair_parts)
            hipLaunchKernelGGL((reduce_stitch_kernel<Acc, typename WideSum<Acc>::T>), grid, block, 0, stream, a, feat_tiles, chunks_per_wg);
        else
            hipLaunchKernelGGL((reduce_stitch_kernel<Acc, Acc>), grid, block, 0, stream, a, feat_tiles, chunks_per_wg);
    }
}

}  // namespace bload

using namespace bload;

extern "C" size_t bload_segment_reduce_workspace_bytes(int64_t num_blocks, int32_t t_blk,
                                                       int64_t feat_dim, bload_dtype dtype)
{
    if (num_blocks <= 0 || t_blk < 1 || feat_dim < 1 || (int)dtype < 0 || (int)dtype > 3) return 0;
    // either end of the guess at the pieces' length, and the flat cut
    return std::max(flat_plan(num_blocks, t_blk, feat_dim, dtype).bytes,
                    std::max(reduce_plan(num_blocks, t_blk, feat_dim, dtype, 0).bytes,
                             reduce_plan(num_blocks, t_blk, feat_dim, dtype, (int64_t)1 << 40).bytes));
}

extern "C" int32_t bload_segment_reduce_layout(int64_t num_blocks, int32_t t_blk, int64_t feat_dim, bload_dtype dtype, int64_t n_seq,
                                               size_t workspace_bytes, int64_t* h_chunks)
{
    if (h_chunks) *h_chunks = 0;
    if (num_blocks <= 0 || t_blk < 1 || feat_dim < 1 || feat_dim >= ((int64_t)1 << 28) || n_seq < 1 || n_seq > BLOAD_MAX_SEQ ||
        (int)dtype < 0 || (int)dtype > 3 || num_blocks >= ((int64_t)1 << 40) / t_blk)
        return BLOAD_REDUCE_NONE;
    const ReducePlan p = chosen_plan(num_blocks, t_blk, feat_dim, dtype, n_seq, workspace_bytes, true);
    if (h_chunks) *h_chunks = p.total_chunks;
    return p.flat ? BLOAD_REDUCE_FLAT : p.wide ? BLOAD_REDUCE_WIDE : p.staged ? BLOAD_REDUCE_STAGED : BLOAD_REDUCE_NARROW;
}

extern "C" bload_status bload_segment_reduce(const void* d_packed, const int32_t* d_seq_id,
                                             const uint8_t* d_reset, const uint8_t* d_valid,
                                             int64_t num_blocks, int32_t t_blk, int64_t feat_dim,
                                             bload_dtype dtype, bload_op op, int64_t n_seq,
                                             void* d_out, void* d_workspace, size_t workspace_bytes,
                                             void* hip_stream)
{
    if (num_blocks < 0 || t_blk < 1 || feat_dim < 1 || n_seq < 0) return BLOAD_EINVAL;
    if ((int)dtype < 0 || (int)dtype > 3 || (int)op < 0 || (int)op > 1) return BLOAD_EINVAL;
    if (dtype == BLOAD_I32 && op == BLOAD_MEAN) return BLOAD_EINVAL;
    if (n_seq > BLOAD_MAX_SEQ || feat_dim >= ((int64_t)1 << 28)) return BLOAD_EOVERFLOW;
    if (num_blocks == 0 || n_seq == 0) return BLOAD_OK;
    if (!d_packed || !d_seq_id || !d_reset || !d_valid || !d_out) return BLOAD_EINVAL;
    const int64_t total_slots = num_blocks * (int64_t)t_blk;
    if (total_slots >= ((int64_t)1 << 40)) return BLOAD_EOVERFLOW;
    if (!aligned_to(d_packed, 16) || !aligned_to(d_seq_id, 4) || !aligned_to(d_reset, 16) ||
        !aligned_to(d_valid, 16) || !aligned_to(d_out, 8))
        return BLOAD_EALIGN;

    const ReducePlan p = chosen_plan(num_blocks, t_blk, feat_dim, dtype, n_seq, d_workspace ? workspace_bytes : 0, aligned_to(d_workspace, 16));
    if (p.total_chunks * ceil_div(feat_dim, kThreads) > INT32_MAX) return BLOAD_EOVERFLOW;
    if (p.wide && ceil_div(p.total_chunks, (kThreads >> p.row_lanes_log2) >> p.split) *
                      ceil_div(p.n_vec, 1 << p.row_lanes_log2) > INT32_MAX)
        return BLOAD_EOVERFLOW;
    if (p.partials) {
        if (!d_workspace) return BLOAD_EINVAL;
        if (!aligned_to(d_workspace, 16)) return BLOAD_EALIGN;
        if (workspace_bytes < p.bytes) return BLOAD_EWORKSPACE;
    }

    ReduceArgs a{};
    a.packed = static_cast<const uint8_t*>(d_packed);
    a.seq_id = d_seq_id;
    a.reset = d_reset;
    a.valid = d_valid;
    a.num_blocks = num_blocks;
    a.total_slots = total_slots;
    a.total_chunks = p.total_chunks;
    a.t_blk = t_blk;
    a.feat_dim = (int32_t)feat_dim;
    a.n_seq = (int32_t)n_seq;
    a.mean = op == BLOAD_MEAN ? 1 : 0;
    a.blocks_per_tile = p.blocks_per_tile;
    a.magic_t_blk = (uint32_t)std::min<uint64_t>((((uint64_t)1 << 32) + (uint64_t)t_blk - 1) / (uint64_t)t_blk, 0xFFFFFFFFull);
    a.out = d_out;
    a.chunk = p.chunk;
    a.tile = p.tile;
    a.split = p.wide && p.split ? 1 : 0;
    a.reach = a.split ? p.reach : 0;
    a.n_chunks = p.n_chunks;
    a.row_lanes_log2 = p.row_lanes_log2;
    a.n_vec = p.n_vec;
    a.step_vec = p.step_vec;
    a.step_frames = p.step_frames;
    a.step_magic = p.flat ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)p.step_frames + 1) : 0u;
    a.feat_tiles = p.wide ? (int32_t)ceil_div(p.n_vec, 1 << p.row_lanes_log2) : 1;
    if (p.partials) {
        uint8_t* ws = static_cast<uint8_t*>(d_workspace);
        a.desc = reinterpret_cast<ChunkDesc*>(ws + p.desc_off);
        a.head_part = ws + p.head_off;
        a.tail_part = ws + p.tail_off;
        a.pair_parts = p.pair_parts ? 1 : 0;
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    switch (dtype) {
        case BLOAD_U8: launch_reduce<uint8_t>(p, a, stream); break;
        case BLOAD_F16: launch_reduce<half_bits>(p, a, stream); break;
        case BLOAD_F32: launch_reduce<float>(p, a, stream); break;
        case BLOAD_I32: launch_reduce<int32_t>(p, a, stream); break;
    }
    return launch_status();
}
