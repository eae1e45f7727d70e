// bload_pack: gather the frames of every sequence into the dense
// [num_blocks, T_blk, frame] tensor, fill the rest with 0's, and write the
// per-slot form of the start table (BLoad, Methods section).
//
// The kernels are destination driven: a workgroup owns a contiguous piece of
// the packed tensor (a "tile"), looks up which sequences land in it, and
// streams 16-byte vectors from the ragged source to the tile.  Every output
// byte is written by exactly one thread, so no memset pass and no atomics are
// needed.  A first pass (pack_prepare_kernel) turns the plan into a table of
// "runs" in shuffled order -- one 32-byte record per sequence saying where it
// lands and where it comes from, so that the copy kernels need one contiguous
// read per sequence instead of a chain of look-ups through five tables -- and
// finds, for every tile, where in that table its runs begin.
//
// Calls of few tiles do without that pass: their workgroups look the runs up by themselves (pack_direct_kernel).
//
// Two tile shapes (takes_wide_tiles chooses, from the frame size and the bytes
// per sequence):
//   wide   a tile is 4 KiB of the packed tensor, one 16-byte vector per thread;
//          best where runs (a sequence's bytes) are long: a tile inside one run
//          is a plain copy with wave-uniform scalar look-ups.  Frames of at
//          least 64 bytes.
//   narrow a tile is 1024 consecutive slots; a tile inside one run or inside a
//          block's padding is written straight away, for any other the runs go
//          into an LDS table, lanes take consecutive 16-byte destination vectors
//          and assemble them from source elements of the widest type that
//          divides the frame.  Small frames, and middle-sized frames of short
//          sequences.  Without its payload part the same kernel writes the start
//          table of large tensors of wide frames, whose 4 KiB tiles then only
//          copy.
// Large outputs leave through streaming stores (see store_slot), small ones stay in the memory-side cache (pack_traffic).
#include "bload_common.hpp"

#include <limits.h>

#include <mutex>
#include <type_traits>

namespace bload {

// Where one sequence goes: the record the copy kernels work from.  Position p of the
// table belongs to shuffled position p; slots are numbered globally (block * T_blk +
// slot in block).  A position that holds no sequence (a worker's share lists only its
// own) has dst = INT64_MAX, which also ends the list.
struct __attribute__((aligned(32))) Run {
    int64_t dst;       // first slot
    int64_t src;       // first source frame
    int32_t len;       // frames
    int32_t seq;       // original sequence index
    int32_t block;     // dst / T_blk
    int32_t pad_;
};
static_assert(sizeof(Run) == 32, "a run is two 16-byte vectors");
constexpr int64_t kNoRun = INT64_MAX;

struct PackArgs {
    const uint8_t* src;
    int32_t n_seq;
    int32_t t_blk;
    int64_t frame_bytes;
    int64_t total_slots;      // num_blocks * t_blk
    uint8_t* packed;
    int32_t* seq_id;
    int32_t* frame_idx;
    uint8_t* reset;
    uint8_t* valid;
};

// The plan as the entry points get it.
struct PlanTables {
    const int64_t* src_offsets;
    const int32_t* lengths;
    const int32_t* order;
    const int32_t* block_of_seq;
    const int32_t* offset_of_seq;
    const int32_t* block_first;
};

// The run of shuffled position p, from the plan's tables.
__device__ __forceinline__ Run run_at_position(const PlanTables& t, int64_t p, int32_t n_seq, int64_t num_blocks, int64_t t_blk)
{
    Run r{kNoRun, 0, 0, -1, -1, 0};
    const uint32_t i = (uint32_t)t.order[p];
    if (i < (uint32_t)n_seq) {
        const int64_t b = t.block_of_seq[i];
        if (b >= 0 && b < num_blocks) {
            r.dst = b * t_blk + t.offset_of_seq[i];
            r.src = t.src_offsets[i];
            r.len = t.lengths[i];
            r.seq = (int32_t)i;
            r.block = (int32_t)b;
        }
    }
    return r;
}

// The sequences ("runs") that overlap one tile, in shuffled order.  Slots are
// numbered globally (block * T_blk + slot in block); dst is relative to the
// tile's first slot and is negative for a run that starts before the tile.
template <int MAXRUNS>
struct RunTable {
    int64_t src[MAXRUNS];      // first source frame of the run
    int32_t dst[MAXRUNS + 1];  // first slot, tile relative; [n] = INT_MAX sentinel
    int16_t end[MAXRUNS];      // one past its last slot, tile relative, cut to [0, MAXRUNS]: 18 bytes per
                               // run keep the table of a 1024-slot tile under an eighth of a CU's LDS
    int32_t seq[MAXRUNS];      // original sequence index
};

// Fill `tab` with the runs that can overlap global slots [gs_lo, gs_hi): the shuffled positions
// first .. last, where `first` is the tile's entry of the prepare pass (the last position of the
// tile's first block that starts at or before gs_lo) and `last` that of the tile behind it (no
// run that starts before gs_hi has a later position).  Runs are sorted by destination, so the
// runs to keep are a prefix of these candidates; candidate k becomes table entry k, and a
// candidate that starts at or behind gs_hi becomes an end mark (as does the entry behind the
// last candidate), so that a search over all candidates finds only runs of the tile.  Called by
// the whole workgroup, all look-ups in flight together; ends with a barrier.  Returns the
// number of candidates.
template <int MAXRUNS>
__device__ __forceinline__ int gather_runs(const Run* __restrict__ runs, int32_t n_seq, int32_t first,
                                           int32_t last, int64_t gs_lo, int64_t gs_hi, RunTable<MAXRUNS>& tab)
{
    const int tid = (int)threadIdx.x;
    const int n_cand = max(0, min(min(last, n_seq - 1) - first + 1, MAXRUNS));
    constexpr int PER = (MAXRUNS + kThreads - 1) / kThreads;
    Run r[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int k = tid + i * kThreads;
        if (k < n_cand) r[i] = runs[(int64_t)first + k];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int k = tid + i * kThreads;
        if (k < n_cand) {
            const bool take = r[i].dst < gs_hi;
            tab.src[k] = r[i].src;
            tab.dst[k] = take ? (int32_t)(r[i].dst - gs_lo) : INT_MAX;
            tab.end[k] = (int16_t)min(max(r[i].dst - gs_lo + r[i].len, (int64_t)0), (int64_t)MAXRUNS);
            tab.seq[k] = r[i].seq;
        }
    }
    if (tid == 0) tab.dst[n_cand] = INT_MAX;
    __syncthreads();
    return n_cand;
}

// Index of the last run whose first slot is <= slot (tile relative), -1 if none.
template <int MAXRUNS>
__device__ __forceinline__ int run_of_slot(const RunTable<MAXRUNS>& tab, int n, int32_t slot)
{
    int lo = 0, hi = n;                 // first run with dst > slot
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tab.dst[mid] <= slot) lo = mid + 1; else hi = mid;
    }
    return lo - 1;
}

// ------------------------------------------------------------------- wide
//
// One workgroup writes one small flat piece of the packed tensor and ends:
// workgroups that run at the same time then touch a few compact windows of the
// destination (one per XCD, see xcd_contiguous) and a handful of source
// streams, which is what HBM wants; a workgroup that loops over a large private
// tile does measurably worse.
// To keep so short a workgroup cheap there is no LDS and no barrier here, and
// the lookup of the tile's runs is wave-uniform (a binary search over the
// block's positions followed by a walk over consecutive positions), so it
// runs on the scalar unit with a handful of dependent scalar loads.

constexpr int kWideMinFrame = 64;                   // smallest frame the wide kernel takes
constexpr int kWideTile = 4096;                     // tile used: one 16-byte vector per thread
constexpr int kWideWalkRuns = 2;                    // up to this many runs in a tile are walked one by one
constexpr int kWideRuns = 128;                      // shuffled positions looked up per tile; a power of two
static_assert(kWideTile / kWideMinFrame + 2 <= kWideRuns, "a tile's runs must fit the look-up window");

typedef vec16 __attribute__((aligned(1))) vec16_unaligned;

// How the payload passes the caches (pack_traffic).
enum PackTraffic : int {
    kPackStream = 0,     // streaming loads and stores
    kPackCached = 1,     // plain loads (slot tiles)
    kPackThrough = 2,    // stores go through the XCD's cache at once and stay in the memory-side cache (4 KiB tiles)
};

// A 16-byte buffer store of device scope (sc1 of its cache policy) writes whole lines through at once, where plain stores leave
// them as modified lines in the XCD's cache, whose write-back the call's end waits for: 67 MB of 80 floats from a source in
// memory 32.8 us streamed, 35.0 with plain stores and loads, 32.6 like this.
constexpr int kDeviceScope = 16;
constexpr int kRawBuffer = 0x00027000;              // a buffer's fourth word: untyped, addressed in bytes

template <int TRAFFIC>
__device__ __forceinline__ vec16 load_source(const uint8_t* p)
{
    const vec16_unaligned* v = reinterpret_cast<const vec16_unaligned*>(p);
    return TRAFFIC == kPackCached ? *v : __builtin_nontemporal_load(v);
}
// Vector `at` of the 4 KiB tile that begins at `tile` (the same for the whole wave).
template <int TRAFFIC>
__device__ __forceinline__ void store_packed(vec16* tile, int at, vec16 v)
{
    if (TRAFFIC != kPackThrough) {
        store_stream(tile + at, v);
        return;
    }
    const __amdgpu_buffer_rsrc_t lines = __builtin_amdgcn_make_buffer_rsrc(tile, 0, kWideTile, kRawBuffer);
    __builtin_amdgcn_raw_buffer_store_b128(v, lines, 16 * at, 0, kDeviceScope);
}
// A vector of a tile that is written in parts, byte by byte where they meet.  Lines in parts do not go through: plain
// stores let them meet in the XCD's cache first (40 MB of 74-byte frames 37 us with parts written through, 29).
template <int TRAFFIC>
__device__ __forceinline__ void store_part(vec16* p, vec16 v)
{
    if (TRAFFIC == kPackThrough) *p = v;
    else store_stream(p, v);
}

// floor(x / d) for 0 <= x < 2^52, d >= 1, with inv_d = 1.0 / d: the double
// quotient is within one of the answer, fixed up exactly in integers.
__device__ __forceinline__ int64_t floor_div(int64_t x, int64_t d, double inv_d)
{
    int64_t q = (int64_t)((double)x * inv_d);
    if (q * d > x) --q;
    else if ((q + 1) * d <= x) ++q;
    return q;
}

// Write packed bytes [lo, hi): copies of src[0 ..) (any alignment) or zeros.
// Destination vectors are 16-byte aligned; the ragged ends of the range are
// written byte by byte.  Called by all threads of the workgroup.
template <bool ZERO, int TRAFFIC>
__device__ __forceinline__ void write_range(uint8_t* packed, int64_t lo, int64_t hi,
                                            const uint8_t* src)
{
    const int tid = (int)threadIdx.x;
    int64_t lo_al = (lo + 15) & ~(int64_t)15;
    if (lo_al > hi) lo_al = hi;
    int64_t hi_al = hi & ~(int64_t)15;
    if (hi_al < lo_al) hi_al = lo_al;
    const int head = (int)(lo_al - lo);
    const int tail = (int)(hi - hi_al);
    if (tid < head) packed[lo + tid] = ZERO ? (uint8_t)0 : src[tid];
    if (tid >= kWave && tid - kWave < tail)
        packed[hi_al + (tid - kWave)] = ZERO ? (uint8_t)0 : src[(hi_al - lo) + (tid - kWave)];

    const int nv = (int)((hi_al - lo_al) >> 4);
    vec16* d = reinterpret_cast<vec16*>(packed + lo_al);
    const uint8_t* s = src + (lo_al - lo);
    int v = tid;
    if (ZERO) {
        const vec16 z = {0u, 0u, 0u, 0u};
        for (; v < nv; v += kThreads) store_part<TRAFFIC>(d + v, z);
    } else {
        for (; v + 3 * kThreads < nv; v += 4 * kThreads) {
            const vec16 x0 = load_source<TRAFFIC>(s + 16 * (int64_t)v);
            const vec16 x1 = load_source<TRAFFIC>(s + 16 * (int64_t)(v + kThreads));
            const vec16 x2 = load_source<TRAFFIC>(s + 16 * (int64_t)(v + 2 * kThreads));
            const vec16 x3 = load_source<TRAFFIC>(s + 16 * (int64_t)(v + 3 * kThreads));
            store_part<TRAFFIC>(d + v, x0);
            store_part<TRAFFIC>(d + v + kThreads, x1);
            store_part<TRAFFIC>(d + v + 2 * kThreads, x2);
            store_part<TRAFFIC>(d + v + 3 * kThreads, x3);
        }
        for (; v < nv; v += kThreads) store_part<TRAFFIC>(d + v, load_source<TRAFFIC>(s + 16 * (int64_t)v));
    }
}

// The start-table entry of one slot (frame index -1: padding).  Streamed like the payload of large tensors: plain
// stores leave these planes (a gigabyte at 10^8 slots) as modified lines in the memory-side
// cache, and a consumer that streams the packed tensor right afterwards then reads about a tenth
// slower (measured: the reduction of 3000 x 320-byte blocks takes 3.98 ms alone and 4.45 ms
// behind a pack that wrote them with plain stores).
template <int TRAFFIC = kPackStream>
__device__ __forceinline__ void store_slot(const PackArgs& a, int64_t slot, int32_t seq, int32_t fid)
{
    if (TRAFFIC == kPackThrough) {
        a.seq_id[slot] = seq;
        a.frame_idx[slot] = fid;
        a.reset[slot] = (uint8_t)(fid == 0);
        a.valid[slot] = (uint8_t)(fid >= 0);
        return;
    }
    __builtin_nontemporal_store(seq, a.seq_id + slot);
    __builtin_nontemporal_store(fid, a.frame_idx + slot);
    __builtin_nontemporal_store((uint8_t)(fid == 0), a.reset + slot);
    __builtin_nontemporal_store((uint8_t)(fid >= 0), a.valid + slot);
}

// Start-table entries of global slots [lo, hi): lane k of the calling wave writes the slots
// lo + k, lo + k + 64, ...  frame0 = frame index of slot lo, or -1 for padding.
template <int TRAFFIC>
__device__ __forceinline__ void write_slots(const PackArgs& a, int64_t lo, int64_t hi, int32_t seq,
                                            int64_t frame0)
{
    for (int64_t k = lane_id(); lo + k < hi; k += kWave) {
        const int64_t g = lo + k;
        const int32_t fid = frame0 < 0 ? -1 : (int32_t)(frame0 + k);
        store_slot<TRAFFIC>(a, g, frame0 < 0 ? -1 : seq, fid);
    }
}

constexpr int kTableSlots = 1024;                   // slots per workgroup of the slot-tile kernel

// Pass 1 (used by both tile shapes, which come after it in this file's launch
// order).  Thread p < n_seq writes the run of shuffled position p.  Thread t < n_tiles
// finds, for tile t, the last shuffled position of the tile's first block whose
// sequence starts at or before the tile's first slot (the block's first sequence
// starts at slot 0, so there is one); it searches the plan's own tables, so the two
// halves do not depend on each other.
__global__ __launch_bounds__(kThreads) void pack_prepare_kernel(
    PlanTables t, int32_t n_seq, int64_t num_blocks, int64_t t_blk, int64_t frame_bytes, int64_t n_tiles,
    int32_t tile_bytes, double inv_frame_bytes, double inv_t_blk, Run* __restrict__ runs,
    int32_t* __restrict__ first_pos, int64_t n_table_tiles, int32_t* __restrict__ first_pos_table)
{
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (idx < n_seq) runs[idx] = run_at_position(t, idx, n_seq, num_blocks, t_blk);
    // the last shuffled position of slot gs_lo's block whose sequence starts at or before gs_lo
    auto entry_of = [&](int64_t gs_lo) {
        const int64_t b0 = floor_div(gs_lo, t_blk, inv_t_blk);
        const int32_t rel = (int32_t)(gs_lo - b0 * t_blk);
        int32_t p = min(max(t.block_first[b0], 0), n_seq);
        int32_t above = min(max(t.block_first[b0 + 1], p), n_seq);
        while (above - p > 1) {
            const int32_t mid = p + ((above - p) >> 1);
            const uint32_t i = (uint32_t)t.order[mid];
            if (i < (uint32_t)n_seq && t.offset_of_seq[i] <= rel) p = mid; else above = mid;
        }
        return p;
    };
    if (idx < n_tiles) first_pos[idx] = entry_of(floor_div(idx * tile_bytes, frame_bytes, inv_frame_bytes));
    // tiles of kTableSlots slots, for the pass that writes the start table of wide frames
    if (idx < n_table_tiles) first_pos_table[idx] = entry_of(idx * kTableSlots);
}

// The runs of some 4 KiB tiles in a row, looked up side by side.
template <int TILES>
struct WideRuns {
    static constexpr int kMost = TILES * kWideRuns;
    int64_t lo[kMost + 1];         // first packed byte of the run; INT64_MAX: no run
    int64_t hi[kMost];             // one past its last packed byte
    int64_t src[kMost];            // source byte that goes to `lo`
    int32_t seq[kMost];
};

// Packed bytes [D0, D1) of tiles whose runs, `n` at most and in destination order, are known, and the start-table entries of
// slots [m_lo, m_hi) if `table_wave`.  Every thread finds the run of its own 16 bytes of each tile.
template <int TRAFFIC, int TILES>
__device__ __forceinline__ void write_wide_tiles(const PackArgs& a, const WideRuns<TILES>& r, int32_t n, int64_t D0, int64_t D1,
                                                 int64_t m_lo, int64_t m_hi, bool table_wave, double inv_frame_bytes)
{
    const int64_t F = a.frame_bytes;
    const int tid = (int)threadIdx.x;
    // last gathered run that starts at or before packed byte x, -1 if none
    // (a binary search over the first `span` entries, span = a power of two that covers them)
    int span = 1;
    while (span < min(n, WideRuns<TILES>::kMost)) span <<= 1;
    auto run_at = [&](int64_t x) {
        int k = -1;
        for (int step = span >> 1; step >= 1; step >>= 1)
            if (r.lo[k + step] <= x) k += step;
        if (r.lo[k + 1] <= x) ++k;
        return k;
    };

    vec16 out[TILES];
    bool whole[TILES];
#pragma unroll
    for (int u = 0; u < TILES; ++u) {
        const int64_t x0 = D0 + 16 * (int64_t)(u * kThreads + tid);
        out[u] = vec16{0u, 0u, 0u, 0u};
        whole[u] = x0 + 16 <= D1;
        if (x0 >= D1) continue;
        int k = run_at(x0);
        const int64_t next_lo = r.lo[k + 1];
        const int64_t lo = k >= 0 ? r.lo[k] : 0, hi = k >= 0 ? r.hi[k] : 0;
        if (whole[u] && x0 + 16 <= hi) {                                // inside one run
            out[u] = load_source<TRAFFIC>(a.src + r.src[k] + (x0 - lo));
        } else if (!(whole[u] && x0 >= hi && x0 + 16 <= next_lo)) {     // not inside a block's zero tail
            // a border inside: byte by byte, all of them asked for before the first is stored
            uint32_t bytes[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int64_t x = x0 + j;
                while (r.lo[k + 1] <= x) ++k;
                bytes[j] = 0;
                if (k >= 0 && x < r.hi[k] && x < D1) bytes[j] = a.src[r.src[k] + (x - r.lo[k])];
            }
#pragma unroll
            for (int w = 0; w < 4; ++w) out[u][w] = bytes[4 * w] | bytes[4 * w + 1] << 8 | bytes[4 * w + 2] << 16 | bytes[4 * w + 3] << 24;
            if (!whole[u]) {
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    if (x0 + j < D1) a.packed[x0 + j] = (uint8_t)bytes[j];
            }
        }
    }
    // (one store for whatever a lane's vector is, so that a wave's goes out as whole lines)
#pragma unroll
    for (int u = 0; u < TILES; ++u)
        if (whole[u]) store_packed<TRAFFIC>(reinterpret_cast<vec16*>(a.packed + D0) + u * kThreads, tid, out[u]);
    if (table_wave) {
        for (int64_t slot = m_lo + lane_id(); slot < m_hi; slot += kWave) {
            const int64_t x = slot * F;
            const int k = run_at(x);
            int32_t seq = -1, fid = -1;
            if (k >= 0 && x < r.hi[k]) {
                seq = r.seq[k];
                fid = (int32_t)(slot - floor_div(r.lo[k], F, inv_frame_bytes));
            }
            store_slot<TRAFFIC>(a, slot, seq, fid);
        }
    }
}

// Pass 2: the copy.  The run table and the tiles' entries come as separate
// __restrict__ pointers so that the compiler knows nothing this kernel stores
// can alias them and keeps their loads on the scalar unit.
template <int TRAFFIC>
__global__ __launch_bounds__(kThreads) void pack_wide_kernel(
    PackArgs a, const Run* __restrict__ runs, const int32_t* __restrict__ first_pos,
    int32_t tile_bytes, double inv_frame_bytes, int32_t writes_table)
{
    const int64_t F = a.frame_bytes;
    const int64_t T = a.t_blk;
    const int32_t n_seq = a.n_seq;
    const int64_t total_bytes = a.total_slots * F;
    const uint32_t tile = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t D0 = (int64_t)tile * tile_bytes;
    const int64_t D1 = min(D0 + (int64_t)tile_bytes, total_bytes);
    const bool table_wave = writes_table != 0 && wave_id() == 0;
    int32_t p = min(max(first_pos[tile], 0), n_seq);

    // the common case first: the tile lies inside one run -- one load and one
    // store per thread, plus the start-table entries of the few frames that
    // begin in the tile
    if (p < n_seq && tile_bytes == kThreads * 16) {
        const Run r = runs[p];
        if (r.dst != kNoRun) {
            const int64_t g = r.dst;
            const int64_t len = r.len;
            const int64_t run_lo = g * F;
            if (run_lo <= D0 && run_lo + len * F >= D0 + tile_bytes && D0 + tile_bytes <= total_bytes) {
                const uint8_t* s = a.src + r.src * F + (D0 - run_lo) + 16 * (int64_t)threadIdx.x;
                store_packed<TRAFFIC>(reinterpret_cast<vec16*>(a.packed + D0), (int)threadIdx.x, load_source<TRAFFIC>(s));
                if (table_wave) {
                    // frames t of this run with D0 <= run_lo + t * F < D1
                    for (int64_t t = floor_div(D0 - run_lo + F - 1, F, inv_frame_bytes) + lane_id();
                         run_lo + t * F < D1 && t < len; t += kWave) {
                        store_slot<TRAFFIC>(a, g + t, r.seq, (int32_t)t);
                    }
                }
                return;
            }
            // next most common: the tile lies in the zero tail of the run's block
            if (run_lo + len * F <= D0 && ((int64_t)r.block + 1) * T * F >= D0 + tile_bytes) {
                const vec16 z = {0u, 0u, 0u, 0u};
                store_packed<TRAFFIC>(reinterpret_cast<vec16*>(a.packed + D0), (int)threadIdx.x, z);
                if (table_wave) {
                    for (int64_t slot = floor_div(D0 + F - 1, F, inv_frame_bytes) + lane_id(); slot * F < D1;
                         slot += kWave) {
                        store_slot<TRAFFIC>(a, slot, -1, -1);
                    }
                }
                return;
            }
        }
    }

    const int64_t gs_lo = floor_div(D0, F, inv_frame_bytes);              // first slot touched
    const int64_t gs_hi = floor_div(D1 + F - 1, F, inv_frame_bytes);      // one past the last
    // slots whose first byte lies in this tile get their start-table entry here
    const int64_t m_lo = gs_lo + ((gs_lo * F < D0) ? 1 : 0);
    const int64_t m_hi = min(gs_hi, a.total_slots);

    // A tile that few runs touch walks them one after the other (their look-ups are scalar
    // loads, the whole workgroup copies each run's part).  The shuffled position in front of
    // the next tile bounds the number of runs from above.
    const int32_t p_next = (tile + 1 < gridDim.x) ? min(max(first_pos[tile + 1], 0), n_seq) : n_seq - 1;
    if (p_next - p + 1 <= kWideWalkRuns) {
        // runs in destination order from there on, zeros in the gaps (block tails)
        int64_t cursor = D0;          // payload bytes written so far
        int64_t mcursor = m_lo;       // start-table slots written so far
        for (; p < n_seq; ++p) {
            const Run r = runs[p];
            const int64_t g = r.dst;
            if (g >= gs_hi) break;                    // also the end of the list (kNoRun)
            const int64_t len = r.len;
            if (g + len <= gs_lo) continue;           // ends before the tile: the tile starts in padding
            const int64_t run_lo = g * F;
            const int64_t lo = max(max(run_lo, D0), cursor);
            const int64_t hi = min(run_lo + len * F, D1);
            if (hi > lo) {
                if (lo > cursor) write_range<true, TRAFFIC>(a.packed, cursor, lo, nullptr);
                write_range<false, TRAFFIC>(a.packed, lo, hi, a.src + r.src * F + (lo - run_lo));
                cursor = hi;
            }
            if (table_wave) {
                const int64_t s_lo = max(g, mcursor), s_hi = min(g + len, m_hi);
                if (s_lo > mcursor) write_slots<TRAFFIC>(a, mcursor, s_lo, -1, -1);
                if (s_hi > s_lo) { write_slots<TRAFFIC>(a, s_lo, s_hi, r.seq, s_lo - g); mcursor = s_hi; }
            }
        }
        if (cursor < D1) write_range<true, TRAFFIC>(a.packed, cursor, D1, nullptr);
        if (table_wave && mcursor < m_hi) write_slots<TRAFFIC>(a, mcursor, m_hi, -1, -1);
        return;
    }

    // Every other tile: the runs that touch it are looked up side by side (thread k takes the
    // k-th shuffled position from p on), so that the cost does not grow with their number, and
    // every thread then finds the run of its own 16 bytes.  A frame of kWideMinFrame bytes or
    // more puts at most kWideTile / kWideMinFrame + 2 runs into a tile.
    __shared__ WideRuns<1> runs_here;
    const int tid = (int)threadIdx.x;
    if (tid <= kWideRuns) {
        int64_t lo = INT64_MAX, hi = 0, from = 0;
        int32_t seq = -1;
        const int64_t pos = (int64_t)p + tid;
        if (tid < kWideRuns && pos < n_seq) {
            const Run r = runs[pos];
            if (r.dst < gs_hi) {
                lo = r.dst * F;
                hi = lo + (int64_t)r.len * F;
                from = r.src * F;
                seq = r.seq;
            }
        }
        runs_here.lo[tid] = lo;
        if (tid < kWideRuns) {
            runs_here.hi[tid] = hi;
            runs_here.src[tid] = from;
            runs_here.seq[tid] = seq;
        }
    }
    __syncthreads();
    write_wide_tiles<TRAFFIC>(a, runs_here, p_next - p + 2, D0, D1, m_lo, m_hi, table_wave, inv_frame_bytes);
}

// The runs that overlap slots [gs_lo, gs_hi), the last of which that there is lies at or before `slot_hi` - 1, from the plan's tables, a
// thread to a shuffled position of the blocks that the slots touch: put(index, run), in destination order.  Returns how many there
// are.  Called by the whole workgroup; what it put is there for all behind a barrier.
// Of more positions than threads, the one that the slots begin in is searched first, every wave for itself, and only as many
// are looked at from there on as the slots can hold: a look is five scattered loads, and thousands of workgroups make
// them (30000 sequences of one 512-byte frame in a block 17.7 us with a run table, 30.7 where 256 positions were tried and 256
// looked at, 14.4 like this; with 16 or 64 ways 15.4 and 14.8).
constexpr int kFindWays = 32;
template <typename Put>
__device__ __forceinline__ int32_t find_runs(const PackArgs& a, const PlanTables& t, int64_t num_blocks, double inv_t_blk, int64_t gs_lo,
                                             int64_t slot_hi, int64_t gs_hi, Put put)
{
    __shared__ int32_t s_found[kThreads / kWave];
    const int64_t T = a.t_blk;
    const int tid = (int)threadIdx.x;
    const int64_t b0 = floor_div(gs_lo, T, inv_t_blk), b1 = floor_div(slot_hi - 1, T, inv_t_blk);
    int32_t first = min(max(t.block_first[b0], 0), a.n_seq);
    const int32_t last = min(max(t.block_first[b1 + 1], first), a.n_seq);
    int32_t looks = kThreads;
    if (last - first > kThreads) {
        const int32_t rel = (int32_t)(gs_lo - b0 * T);
        int32_t above = min(max(t.block_first[b0 + 1], first), last);
        while (above - first > 1) {
            const int32_t step = (above - first + kFindWays - 1) / kFindWays, at = lane_id() * step;
            bool in_front = false;
            if (lane_id() < kFindWays && at < above - first) {
                const uint32_t i = (uint32_t)t.order[first + at];
                in_front = i < (uint32_t)a.n_seq && t.offset_of_seq[i] <= rel;
            }
            first += max((int32_t)__popcll(__ballot(in_front)) - 1, 0) * step;
            above = min(above, first + step);
        }
        looks = (int32_t)min((int64_t)kThreads, gs_hi - gs_lo + 1);
    }
    int32_t n = 0;
    for (int32_t p0 = first; p0 < last; p0 += looks) {
        Run r{kNoRun, 0, 0, -1, -1, 0};
        if (tid < looks && p0 + tid < last) r = run_at_position(t, p0 + tid, a.n_seq, num_blocks, T);
        const bool here = r.dst < gs_hi && r.dst + r.len > gs_lo;
        const uint64_t vote = __ballot(here);
        const int behind = __syncthreads_or(tid < looks && r.dst >= gs_hi);      // (also a barrier behind the counts of the round before)
        if (lane_id() == 0) s_found[wave_id()] = (int32_t)__popcll(vote);
        __syncthreads();
        int32_t at = n + (int32_t)__popcll(vote & ((1ull << lane_id()) - 1ull));
#pragma unroll
        for (int w = 0; w < kThreads / kWave; ++w) {
            at += w < wave_id() ? s_found[w] : 0;
            n += s_found[w];
        }
        if (here) put(at, r);
        if (behind) break;
    }
    return n;
}

// The same in one launch, for calls of few tiles: every workgroup looks up the runs of its tile, or of two in a row, in the plan's tables
// by itself, a thread to a shuffled position of the blocks that it touches.  Bound by latency: four look-ups one after the other here,
// against three and a launch there.
template <int TILES>
__global__ __launch_bounds__(kThreads) void pack_direct_kernel(PackArgs a, PlanTables t, int64_t num_blocks, double inv_frame_bytes,
                                                               double inv_t_blk)
{
    constexpr int kMost = WideRuns<TILES>::kMost;
    static_assert(TILES * kWideTile / kWideMinFrame + 2 <= kMost, "the tiles' runs must fit their table");
    const int64_t F = a.frame_bytes, total_bytes = a.total_slots * F;
    const uint32_t tile = xcd_contiguous(blockIdx.x, gridDim.x);
    const int64_t D0 = (int64_t)tile * (TILES * kWideTile), D1 = min(D0 + TILES * kWideTile, total_bytes);
    const int64_t gs_lo = floor_div(D0, F, inv_frame_bytes);              // first slot touched
    const int64_t gs_hi = floor_div(D1 + F - 1, F, inv_frame_bytes);      // one past the last
    const int64_t m_lo = gs_lo + ((gs_lo * F < D0) ? 1 : 0), m_hi = min(gs_hi, a.total_slots);
    __shared__ WideRuns<TILES> runs_here;
    const int tid = (int)threadIdx.x;
    for (int k = tid; k <= kMost; k += kThreads) runs_here.lo[k] = INT64_MAX;
    const int32_t n = find_runs(a, t, num_blocks, inv_t_blk, gs_lo, m_hi, gs_hi, [&](int32_t at, const Run& r) {
        if (at < kMost) {
            runs_here.lo[at] = r.dst * F;
            runs_here.hi[at] = (r.dst + r.len) * F;
            runs_here.src[at] = r.src * F;
            runs_here.seq[at] = r.seq;
        }
    });
    __syncthreads();
    write_wide_tiles<kPackThrough>(a, runs_here, n + 1, D0, D1, m_lo, m_hi, wave_id() == 0, inv_frame_bytes);      // (16 MB at most)
}

// ----------------------------------------------------------------- narrow

constexpr int kNarrowSlots = kTableSlots;            // slots per workgroup
constexpr int kNarrowMaxRuns = kNarrowSlots + 2;

// The run a lane is currently reading from, kept in registers and advanced
// as the lane walks over consecutive slots.
template <int MAXRUNS>
struct RunCursor {
    const RunTable<MAXRUNS>& tab;
    int r;
    int32_t dst, end, next, seq;
    int64_t src;

    __device__ __forceinline__ RunCursor(const RunTable<MAXRUNS>& t, int n, int32_t slot)
        : tab(t)
    {
        r = run_of_slot(t, n, slot);
        load();
    }
    __device__ __forceinline__ void load()
    {
        next = tab.dst[r + 1];
        if (r >= 0) { dst = tab.dst[r]; end = tab.end[r]; seq = tab.seq[r]; src = tab.src[r]; }
        else        { dst = 0; end = 0; seq = -1; src = 0; }
    }
    // frame index of `slot` inside the current run, or -1 on padding
    __device__ __forceinline__ int32_t seek(int32_t slot)
    {
        while (slot >= next) { ++r; load(); }
        return (r >= 0 && slot < end) ? slot - dst : -1;
    }
};

// What a tile of kNarrowSlots slots is, as far as the run its entry names can tell.
enum NarrowKind : int { kTileGeneral = 0, kTileOneRun = 1, kTilePadding = 2, kTileAbsent = 3 };

// The start-table entries of a whole tile that lies inside one run (`r`), or inside the padding
// behind a block's last run (`r` null): four slots per lane, without a look at any table.
__device__ __forceinline__ void narrow_uniform_table(const PackArgs& a, int64_t g0, const Run* r)
{
    const int64_t g = g0 + 4 * (int)threadIdx.x;
    vec16 vs = {~0u, ~0u, ~0u, ~0u}, vf = vs;
    uint32_t rs = 0, vl = 0;
    if (r) {
        const uint32_t fid = (uint32_t)(g - r->dst);           // >= 0: the run begins at or before the tile
        vs = vec16{(uint32_t)r->seq, (uint32_t)r->seq, (uint32_t)r->seq, (uint32_t)r->seq};
        vf = vec16{fid, fid + 1u, fid + 2u, fid + 3u};
        rs = fid == 0u ? 1u : 0u;
        vl = 0x01010101u;
    }
    store_stream(reinterpret_cast<vec16*>(a.seq_id + g), vs);
    store_stream(reinterpret_cast<vec16*>(a.frame_idx + g), vf);
    __builtin_nontemporal_store(rs, reinterpret_cast<uint32_t*>(a.reset + g));
    __builtin_nontemporal_store(vl, reinterpret_cast<uint32_t*>(a.valid + g));
}

// The payload of such a tile: per step one 16-byte vector per lane.
template <int TRAFFIC>
__device__ __forceinline__ void narrow_uniform_payload(const PackArgs& a, int64_t g0, const Run* r,
                                                       int32_t part, int32_t parts)
{
    const int first = part * kThreads + (int)threadIdx.x, step = parts * kThreads;
    const int64_t F = a.frame_bytes;
    vec16* dst = reinterpret_cast<vec16*>(a.packed + g0 * F);      // 16-byte aligned: g0 is a multiple of 1024
    const int32_t nvec = (int32_t)(kNarrowSlots * F / 16);
    if (r) {
        const uint8_t* from = a.src + (r->src + (g0 - r->dst)) * F;
        for (int32_t v = first; v < nvec; v += step)
            store_stream(dst + v, load_source<TRAFFIC>(from + 16 * (int64_t)v));
    } else {
        const vec16 z = {0u, 0u, 0u, 0u};
        for (int32_t v = first; v < nvec; v += step) store_stream(dst + v, z);
    }
}

// A 16-byte vector put together from elements of type E (1, 2, 4 or 16 bytes).  Element numbers
// are compile-time constants where it is used, so the vector stays in registers.
template <typename E>
struct Assembled {
    vec16 vec = {0u, 0u, 0u, 0u};
    __device__ __forceinline__ void set(int e, E v)
    {
        vec[e * (int)sizeof(E) / 4] |= (uint32_t)v << (8 * (e * (int)sizeof(E) % 4));
    }
    __device__ __forceinline__ E get(int e) const
    {
        return (E)(vec[e * (int)sizeof(E) / 4] >> (8 * (e * (int)sizeof(E) % 4)));
    }
};
template <>
struct Assembled<vec16> {
    vec16 vec = {0u, 0u, 0u, 0u};
    __device__ __forceinline__ void set(int, vec16 v) { vec = v; }
    __device__ __forceinline__ vec16 get(int) const { return vec; }
};

// One tile of kNarrowSlots slots (or the shorter last one) whose `n` runs are in `tab`.  Called by the whole workgroup.
template <typename E, bool FUSED, bool PAYLOAD, bool TABLE, int TRAFFIC>
__device__ __forceinline__ void narrow_write_tile(const PackArgs& a, const RunTable<kNarrowMaxRuns>& tab, int n, int64_t g0, int64_t g1,
                                                  int32_t part, int32_t parts)
{
    const int tid = (int)threadIdx.x;
    const int nslot = (int)(g1 - g0);
    const bool long_runs = (int64_t)(n - 1) * 4096 <= nslot * a.frame_bytes;      // borders four waves of vectors apart
    // start table (and, FUSED, the payload): 4 consecutive slots per lane -> 16-byte / 4-byte stores
    for (int q = tid; (TABLE || FUSED) && part == 0 && 4 * q < nslot; q += kThreads) {
        const int32_t s0 = 4 * q;
        RunCursor<kNarrowMaxRuns> cur(tab, n, s0);
        int32_t sid[4], fid[4];
        int64_t from[4];                 // source frame of each slot (FUSED only)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            fid[j] = (s0 + j < nslot) ? cur.seek(s0 + j) : -1;
            sid[j] = fid[j] >= 0 ? cur.seq : -1;
            from[j] = cur.src + fid[j];
        }
        if (FUSED && s0 + 4 <= nslot) {
            const uint32_t* src32 = reinterpret_cast<const uint32_t*>(a.src);
            vec16 pv;
            if (fid[0] >= 0 && sid[3] == sid[0] && fid[3] == fid[0] + 3) {
                // one run: 16 contiguous source bytes (4-byte aligned)
                pv = load_source<TRAFFIC>(reinterpret_cast<const uint8_t*>(src32 + from[0]));
            } else {
                uint32_t e0 = 0u, e1 = 0u, e2 = 0u, e3 = 0u;
                if (fid[0] >= 0) e0 = src32[from[0]];
                if (fid[1] >= 0) e1 = src32[from[1]];
                if (fid[2] >= 0) e2 = src32[from[2]];
                if (fid[3] >= 0) e3 = src32[from[3]];
                pv = vec16{e0, e1, e2, e3};
            }
            store_stream(reinterpret_cast<vec16*>(a.packed + (g0 + s0) * 4), pv);
        }
        if (!TABLE) continue;
        const int64_t g = g0 + s0;
        if (s0 + 4 <= nslot) {
            const vec16 vs = {(uint32_t)sid[0], (uint32_t)sid[1], (uint32_t)sid[2], (uint32_t)sid[3]};
            const vec16 vf = {(uint32_t)fid[0], (uint32_t)fid[1], (uint32_t)fid[2], (uint32_t)fid[3]};
            store_stream(reinterpret_cast<vec16*>(a.seq_id + g), vs);
            store_stream(reinterpret_cast<vec16*>(a.frame_idx + g), vf);
            uint32_t rs = 0, vl = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                rs |= (uint32_t)(fid[j] == 0) << (8 * j);
                vl |= (uint32_t)(fid[j] >= 0) << (8 * j);
            }
            __builtin_nontemporal_store(rs, reinterpret_cast<uint32_t*>(a.reset + g));
            __builtin_nontemporal_store(vl, reinterpret_cast<uint32_t*>(a.valid + g));
        } else {
            for (int j = 0; s0 + j < nslot; ++j) {
                store_slot(a, g + j, sid[j], fid[j]);
            }
        }
    }

    if (!PAYLOAD) return;
    // payload: one 16-byte destination vector per lane and step, assembled
    // from elements of type E (k elements per frame)
    constexpr int EPV = 16 / (int)sizeof(E);
    const int done_slots = FUSED ? (nslot & ~3) : 0;            // already written above
    const int32_t k = (int32_t)(a.frame_bytes / (int64_t)sizeof(E));
    const int32_t tile_elems = nslot * k;                       // < 1024 * 512
    const int32_t nvec = (tile_elems + EPV - 1) / EPV;
    const E* src = reinterpret_cast<const E*>(a.src);
    uint8_t* dst_tile = a.packed + g0 * a.frame_bytes;          // 16-byte aligned
    for (int32_t v = (FUSED ? done_slots / 4 : 0) + part * kThreads + tid; v < nvec; v += parts * kThreads) {
        const int32_t w = v * EPV;
        int32_t slot = w / k;
        int32_t j = w - slot * k;
        RunCursor<kNarrowMaxRuns> cur(tab, n, slot);
        const int nvalid = min(EPV, tile_elems - w);
        if (EPV > 1 && !FUSED && long_runs) {
            // where every vector of the wave lies inside one run or one stretch of padding: 16 contiguous
            // source bytes, at any alignment, instead of one load per element (9-byte frames of 500-slot
            // sequences 1.13 -> 0.79 ms for 1.4 GB, 62-byte frames of 75-slot sequences 1.67 -> 1.09 ms, 56
            // bytes 1.01 -> 0.97).  By the whole wave only, and only where runs are several waves long (the
            // host's rule): a wave with a vector across a border does both (60-byte frames of 27-slot
            // sequences 70 -> 90 us, 20-byte frames of 75 slots 91 -> 104).  By the tile's own runs: the call's
            // sequences would tell too little of a worker's share, whose tables keep the numbers of all.  A plain load, as the elements':
            // a streaming one loses to them where the source is in the memory-side cache (60-byte frames,
            // 0.2 GB: 84 us by elements, 111 streaming, 86 plain).
            const int32_t t = cur.seek(slot);
            const bool inside = nvalid == EPV && w + EPV <= (t >= 0 ? cur.end : min(cur.next, nslot)) * k;
            if (__ballot(!inside) == 0) {
                vec16 x = {0u, 0u, 0u, 0u};
                if (t >= 0)
                    x = *reinterpret_cast<const vec16_unaligned*>(src + (cur.src + t) * k + j);
                store_stream(reinterpret_cast<vec16*>(dst_tile) + v, x);
                continue;
            }
        }
        Assembled<E> u;
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            E val{};
            if (e < nvalid) {
                const int32_t t = cur.seek(slot);
                if (t >= 0) val = src[(cur.src + t) * k + j];
                if (++j == k) { j = 0; ++slot; }
            }
            u.set(e, val);
        }
        if (nvalid == EPV) {
            store_stream(reinterpret_cast<vec16*>(dst_tile) + v, u.vec);
        } else {
#pragma unroll
            for (int e = 0; e < EPV; ++e)
                if (e < nvalid) reinterpret_cast<E*>(dst_tile)[w + e] = u.get(e);
        }
    }
}

// FUSED (4-byte frames, e.g. tokens): the four slots of a lane's start-table
// quad are also exactly one 16-byte vector of payload, so both are written in
// the same pass and the payload pass is skipped.
//
// PAYLOAD false: only the start table is written; TABLE false: only the payload.  Large tensors
// of 4-byte frames are packed in two such passes, and the start table of large tensors of wide
// frames, whose payload the 4 KiB tiles copy, by the first of them: five output streams written
// at once reach 5.1-5.2 TB/s on this GPU, the payload alone 6.0 and the four planes of the table
// alone 6.2 (plain streaming kernels with this traffic, 2^30 tokens: 3.46 ms in one pass, 1.17 +
// 1.73 ms in two).
//
// GROUP consecutive tiles per workgroup.  What decides a tile's kind hangs on two look-ups, one
// after the other (the tile's entry, then the run it names), and the payload on a third: with
// several tiles per workgroup the look-ups of a stage are asked for together, and so is the
// payload of all tiles that lie inside one run, so that a wave has GROUP times the bytes in
// flight per wait.  Tiles that need their runs gathered follow one by one.
template <typename E, bool FUSED, int TRAFFIC, bool PAYLOAD = true, bool TABLE = true, int GROUP = 1>
__global__ __launch_bounds__(kThreads) void pack_narrow_kernel(PackArgs a, const Run* __restrict__ runs,
                                                               const int32_t* __restrict__ first_pos,
                                                               uint32_t n_tiles, int32_t parts)
{
    static_assert(PAYLOAD || !FUSED, "the fused form is about the payload");
    static_assert(PAYLOAD || TABLE, "a pass writes something");
    __shared__ RunTable<kNarrowMaxRuns> tab;
    const int tid = (int)threadIdx.x;
    constexpr bool kSplit = PAYLOAD && TABLE && !FUSED && GROUP == 1;     // else parts is 1
    const uint32_t unit = xcd_contiguous(blockIdx.x, gridDim.x);
    const uint32_t tile0 = !kSplit ? unit * (uint32_t)GROUP : parts == 1 ? unit : unit / (uint32_t)parts;
    const int32_t part = kSplit ? (int32_t)(unit - tile0 * (uint32_t)parts) : 0;
    if (!kSplit) parts = 1;

    // entry[u]: where tile tile0 + u starts in the run table; behind the last tile: the last run
    int32_t entry[GROUP + 1];
#pragma unroll
    for (int u = 0; u <= GROUP; ++u) {
        const uint32_t t = tile0 + (uint32_t)u;
        entry[u] = first_pos[min(t, n_tiles - 1u)];
    }
#pragma unroll
    for (int u = 0; u <= GROUP; ++u)
        entry[u] = tile0 + (uint32_t)u < n_tiles ? min(max(entry[u], 0), a.n_seq) : a.n_seq - 1;

    // The two most common tiles where sequences are long need no table: a tile inside one run,
    // and a tile inside the padding behind its block's last run.  The tile's entry names the
    // last run of the tile's first block that begins at or before the tile; that record alone
    // tells (runs of a block follow each other without a gap).  Wave-uniform look-ups, no LDS,
    // no barrier: every wave decides alone and all decide alike.
    Run r[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) r[u] = runs[min(entry[u], a.n_seq - 1)];
    int kind[GROUP];
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
        const uint32_t t = tile0 + (uint32_t)u;
        const int64_t g0 = (int64_t)t * kNarrowSlots, g1 = g0 + kNarrowSlots;
        kind[u] = kTileGeneral;
        if (t >= n_tiles) {
            kind[u] = kTileAbsent;
        } else if (g1 <= a.total_slots && entry[u] < a.n_seq && r[u].dst != kNoRun) {
            if (r[u].dst <= g0 && r[u].dst + r[u].len >= g1) kind[u] = kTileOneRun;
            else if (r[u].dst + r[u].len <= g0 && ((int64_t)r[u].block + 1) * a.t_blk >= g1) kind[u] = kTilePadding;
        }
    }

    if (PAYLOAD && FUSED) {
        // 4-byte frames: a tile's payload is one 16-byte vector per lane
        vec16 pv[GROUP];
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            pv[u] = vec16{0u, 0u, 0u, 0u};
            if (kind[u] == kTileOneRun) {
                const int64_t g0 = (int64_t)(tile0 + (uint32_t)u) * kNarrowSlots;
                const uint8_t* from = a.src + (r[u].src + (g0 - r[u].dst)) * 4;
                pv[u] = load_source<TRAFFIC>(from + 16 * tid);
            }
        }
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            if (kind[u] == kTileOneRun || kind[u] == kTilePadding) {
                const int64_t g0 = (int64_t)(tile0 + (uint32_t)u) * kNarrowSlots;
                store_stream(reinterpret_cast<vec16*>(a.packed + g0 * 4) + tid, pv[u]);
            }
        }
    } else if (PAYLOAD) {
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            const int64_t g0 = (int64_t)(tile0 + (uint32_t)u) * kNarrowSlots;
            if (kind[u] == kTileOneRun) narrow_uniform_payload<TRAFFIC>(a, g0, &r[u], part, parts);
            else if (kind[u] == kTilePadding) narrow_uniform_payload<TRAFFIC>(a, g0, nullptr, part, parts);
        }
    }
    if (TABLE && part == 0) {
#pragma unroll
        for (int u = 0; u < GROUP; ++u) {
            const int64_t g0 = (int64_t)(tile0 + (uint32_t)u) * kNarrowSlots;
            if (kind[u] == kTileOneRun) narrow_uniform_table(a, g0, &r[u]);
            else if (kind[u] == kTilePadding) narrow_uniform_table(a, g0, nullptr);
        }
    }

    bool table_in_use = false;
#pragma unroll
    for (int u = 0; u < GROUP; ++u) {
        if (kind[u] != kTileGeneral) continue;
        const int64_t g0 = (int64_t)(tile0 + (uint32_t)u) * kNarrowSlots;
        if (table_in_use) __syncthreads();           // the tile before is done with the gathered runs
        const int64_t g1 = min(g0 + kNarrowSlots, a.total_slots);
        const int n = gather_runs(runs, a.n_seq, entry[u], entry[u + 1], g0, g1, tab);
        narrow_write_tile<E, FUSED, PAYLOAD, TABLE, TRAFFIC>(a, tab, n, g0, g1, part, parts);
        table_in_use = true;
    }
}

// Slot tiles in one launch, like pack_direct_kernel.
template <typename E, bool FUSED>
__global__ __launch_bounds__(kThreads) void pack_narrow_direct_kernel(PackArgs a, PlanTables t, int64_t num_blocks, double inv_t_blk,
                                                                      int32_t parts)
{
    __shared__ RunTable<kNarrowMaxRuns> tab;
    const uint32_t unit = xcd_contiguous(blockIdx.x, gridDim.x), tile = unit / (uint32_t)parts;
    const int64_t g0 = (int64_t)tile * kNarrowSlots, g1 = min(g0 + kNarrowSlots, a.total_slots);
    const int32_t n = find_runs(a, t, num_blocks, inv_t_blk, g0, g1, g1, [&](int32_t at, const Run& r) {
        if (at < kNarrowMaxRuns) {
            tab.src[at] = r.src;
            tab.dst[at] = (int32_t)(r.dst - g0);
            tab.end[at] = (int16_t)min(max(r.dst - g0 + r.len, (int64_t)0), (int64_t)kNarrowMaxRuns);
            tab.seq[at] = r.seq;
        }
    });
    const int kept = min(n, kNarrowMaxRuns);
    if (threadIdx.x == 0) tab.dst[kept] = INT_MAX;
    __syncthreads();
    narrow_write_tile<E, FUSED, true, true, kPackCached>(a, tab, kept, g0, g1, (int32_t)(unit - tile * (uint32_t)parts), parts);
}

// ------------------------------------------------------------------ check
//
// Are the tables a plan: every rule is local to one shuffled position (or one block), so
// one thread tests one of each; the smallest failing index is kept with an atomic minimum.
__global__ __launch_bounds__(kThreads) void pack_check_kernel(
    const int64_t* __restrict__ src_offsets, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ order, const int32_t* __restrict__ block_of_seq,
    const int32_t* __restrict__ offset_of_seq, const int32_t* __restrict__ block_first,
    int32_t n_seq, int32_t num_blocks, int32_t t_blk, int64_t total_frames,
    unsigned long long* __restrict__ first_bad)
{
    const int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    bool bad = false;
    // block idx: its range of positions
    if (idx < num_blocks) {
        const int64_t lo = block_first[idx], hi = block_first[idx + 1];
        bad |= lo < 0 || hi < lo || hi > n_seq || (idx == 0 && lo != 0);
    }
    // position idx: its sequence
    const int64_t listed = min(max((int64_t)block_first[num_blocks], (int64_t)0), (int64_t)n_seq);
    if (idx < listed) {
        const uint32_t i = (uint32_t)order[idx];
        if (i >= (uint32_t)n_seq) {
            bad = true;
        } else {
            const int64_t b = block_of_seq[i], off = offset_of_seq[i], len = lengths[i];
            const int64_t from = src_offsets[i];
            bad |= len < 1 || off < 0 || off + len > t_blk;
            bad |= from < 0 || from + len > total_frames || src_offsets[i + 1] - from != len;
            if (b < 0 || b >= num_blocks) {
                bad = true;
            } else {
                const int64_t lo = block_first[b], hi = block_first[b + 1];
                if (lo < 0 || idx < lo || idx >= hi) {
                    bad = true;
                } else if (idx == lo) {
                    bad |= off != 0;
                } else {
                    const uint32_t before = (uint32_t)order[idx - 1];
                    bad |= before >= (uint32_t)n_seq ||
                           (before < (uint32_t)n_seq &&
                            off != (int64_t)offset_of_seq[before] + (int64_t)lengths[before]);
                }
            }
        }
    }
    if (bad) atomicMin(first_bad, (unsigned long long)idx);
}

__global__ void pack_check_clear_kernel(unsigned long long* first_bad) { *first_bad = ~0ull; }

}  // namespace bload

using namespace bload;

// Which tile shape packs faster, from what the host knows.  The 4 KiB tiles win where runs
// (a sequence's bytes) are long: a tile inside one run is a plain copy.  The 1024-slot tiles
// amortise their run table better where many short runs meet, and copy 16 bytes per lane when
// frames are multiples of 16 bytes and the source is aligned.  Measured crossovers, in bytes
// per run (bounded from above here by packed bytes / sequences).
static bool takes_wide_tiles(int64_t frame_bytes, int64_t total_bytes, int64_t n_seq, bool src_aligned16)
{
    if (frame_bytes < kWideMinFrame) return false;
    if (frame_bytes >= 512) return true;
    const int64_t run_bytes = total_bytes / (n_seq > 0 ? n_seq : 1);
    const bool narrow_copies_vectors = frame_bytes % 16 == 0 && src_aligned16;
    return run_bytes >= (narrow_copies_vectors ? 24 * 1024 : 4 * 1024);
}

extern "C" int32_t bload_pack_tile_bytes(int64_t n_seq, int64_t num_blocks, int32_t t_blk,
                                         int64_t frame_bytes, int32_t src_aligned_16)
{
    if (n_seq < 0 || num_blocks <= 0 || t_blk < 1 || frame_bytes < 1) return 0;
    const int64_t total_slots = num_blocks * (int64_t)t_blk;
    if (total_slots >= ((int64_t)1 << 40) || total_slots > (((int64_t)1 << 52) - 1) / frame_bytes) return 0;
    return takes_wide_tiles(frame_bytes, total_slots * frame_bytes, n_seq, src_aligned_16 != 0) ? kWideTile : 0;
}

namespace {

// Workspace: the run table, then one int32 per tile.
struct PackLayout {
    bool wide;
    int64_t tiles;
    int64_t table_tiles;       // slot tiles of the separate start-table pass (wide frames, large tensors), else 0
    size_t runs_off, first_off, table_off, bytes;
};

// From this many slots on, the start table of wide frames is written by a pass of its own, in
// slot tiles with full-width stores: the few entries per 4 KiB tile, written by that tile's first
// wave, are 2 % of the bytes and cost 5 % of the time (10^8 slots of 320 bytes: 9.64 ms, 9.11 ms
// without them, 9.36 ms with the pass).  About 3 ns per 1000 slots: below a couple of million
// slots the pass saves less than its launch costs, and the one pass stays.
constexpr int64_t kTablePassFromSlots = (int64_t)1 << 21;
// Tiles per workgroup in the passes that large tensors get (pack_narrow_kernel's GROUP).  Measured on
// 0.8-1.3 * 10^9 token slots of four length mixes: two tiles 1-3.5 % faster than one, four between 3 %
// slower and 2 % faster, eight 40 % slower.
constexpr int kPassGroup = 2;
// Up to so many tiles, every workgroup looks up its runs itself, in one launch.  4 KiB tiles (pack_direct_kernel): 64 clips of 3 KB frames
// 11.4 -> 8.2 us, 3000 sequences of two 700-byte frames 13.4 -> 9.2; 8192 tiles: 19.4 -> 20.4.  Beyond kDirectAtOnce tiles, as many as
// are at work at once, a workgroup takes two: those of a second round would wait for their look-ups alone (16 MB in one
// sequence 12.6 us in two launches, 14.6 with a tile each, 12.3 like this; 13 MB in ten 12.4, 12.7, 10.7; 9 MB in three 12.4, 12.0, 9.7).  Slot tiles:
// 300 sequences of tokens 10.7 -> 8.0, 400 of 63-byte frames 22.5 -> 16.2, 4 MB of 40-byte frames 14.8 -> 11.9, 3000 full ones of 60
// bytes 64 -> 62.  Every workgroup of a slot tile looks up all of its runs, five scattered loads each: with one to a tile 500000 sequences
// are fine (of one byte each 46 -> 38 us, of two tokens in blocks of 10^6 slots 45.5 -> 42), 600000 are not (of two tokens
// 48.6 and 52, 900000 75 and 84); where several share a tile, not more than 2^18 looks (20000 sequences of ten 64-byte frames, 21 to a
// tile, 14.6 us and 17.7, 6000 of ten 250-byte frames, 63, 18.9 and 21.1; 2000 of ten 400-byte frames, 100 to a tile, 11.7 -> 9.3), and
// no tiles of more than 256 sequences (20000 of one 40-byte frame 13.0 us, 13.5).
constexpr int64_t kDirectAtOnce = 2048, kDirectTiles = 4096, kDirectMost = (int64_t)1 << 19, kDirectLooks = (int64_t)1 << 18;

// Sizes the caller cannot know in advance (which tile shape the lengths will choose) are
// taken at their larger value when `for_query`.
bool pack_layout(int64_t n_seq, int64_t num_blocks, int32_t t_blk, int64_t frame_bytes,
                 bool src_aligned16, bool for_query, PackLayout* l)
{
    const int64_t total_slots = num_blocks * (int64_t)t_blk;
    if (total_slots >= ((int64_t)1 << 40) || total_slots > (((int64_t)1 << 52) - 1) / frame_bytes) return false;
    const int64_t total_bytes = total_slots * frame_bytes;
    const int64_t wide_tiles = ceil_div(total_bytes, kWideTile), narrow_tiles = ceil_div(total_slots, kNarrowSlots);
    if (for_query) {
        // frames that may take either shape get room for the 4 KiB tiles, which are more
        l->wide = frame_bytes >= kWideMinFrame;
        l->tiles = l->wide ? (wide_tiles > narrow_tiles ? wide_tiles : narrow_tiles) : narrow_tiles;
    } else {
        l->wide = takes_wide_tiles(frame_bytes, total_bytes, n_seq, src_aligned16);
        l->tiles = l->wide ? wide_tiles : narrow_tiles;
    }
    l->table_tiles = l->wide && total_slots >= kTablePassFromSlots ? narrow_tiles : 0;
    l->runs_off = 0;
    l->first_off = round_up((size_t)n_seq * sizeof(Run), 32);
    l->table_off = l->first_off + round_up((size_t)l->tiles * sizeof(int32_t), 16);
    l->bytes = l->table_off + round_up((size_t)l->table_tiles * sizeof(int32_t), 16);
    return true;
}

// Argument checks shared by the entry points that pack.
bload_status pack_check_args(const void* d_src, const int64_t* d_src_offsets, const int32_t* d_lengths,
                             const int32_t* d_order, const int32_t* d_block_of_seq,
                             const int32_t* d_offset_of_seq, const int32_t* d_block_first, int64_t n_seq,
                             int64_t num_blocks, int32_t t_blk, int64_t frame_bytes, void* d_packed,
                             int32_t* d_seq_id, int32_t* d_frame_idx, uint8_t* d_reset, uint8_t* d_valid)
{
    if (!d_src || !d_src_offsets || !d_lengths || !d_order || !d_block_of_seq ||
        !d_offset_of_seq || !d_block_first || !d_packed || !d_seq_id || !d_frame_idx ||
        !d_reset || !d_valid)
        return BLOAD_EINVAL;
    const int64_t total_slots = num_blocks * (int64_t)t_blk;
    if (total_slots >= ((int64_t)1 << 40) || frame_bytes >= ((int64_t)1 << 31) ||
        total_slots > INT64_MAX / frame_bytes / 2 || total_slots * frame_bytes >= ((int64_t)1 << 52))
        return BLOAD_EOVERFLOW;
    if (!aligned_to(d_packed, 16) || !aligned_to(d_seq_id, 16) || !aligned_to(d_frame_idx, 16) ||
        !aligned_to(d_reset, 16) || !aligned_to(d_valid, 16) || !aligned_to(d_src_offsets, 8) ||
        !aligned_to(d_lengths, 4) || !aligned_to(d_order, 4) || !aligned_to(d_block_of_seq, 4) ||
        !aligned_to(d_offset_of_seq, 4) || !aligned_to(d_block_first, 4))
        return BLOAD_EALIGN;
    return BLOAD_OK;
}

// How a call reads its source and writes its payload.
//   - 4 KiB tiles, packed tensor, source and table of 256 MB in all (the source taken as long as the packed tensor: what the host
//     knows): the payload is written through and the table plainly, so that a consumer finds both in the memory-side cache.  Pack
//     and reduction, each pack from another source, before and after: 1000 sequences of 37 halfs, 28 MB, 49 -> 49 us, 3001 of them 92 -> 74, 20 of
//     video, 65 MB, 52 -> 46, 312 of 128 floats, 76 MB, 61 -> 53.5; with the scan 59 -> 52, 149 -> 124, 100 -> 86, 81 -> 69.
//   - Their sources are streamed, at any size.  With plain loads the same source again and again comes from the cache (86 MB 48
//     -> 41 us), but one that is read once pushes out what others left there: behind a kernel that wrote a gigabyte the same
//     pack takes 67 us, 53 like this, 94 MB of 80 floats 63 and 46, 220 MB 156 and 117.  Larger tensors stream their payload,
//     too: it would not stay.
//   - Slot tiles of up to 128 MB of payload: plain loads, since their lanes look for elements here and there: 40 MB of halfs one a
//     frame 94 -> 66 us where the source is in the cache, 45 MB of 9-byte frames 53 -> 41; where it is not, even; behind a kernel
//     that wrote a gigabyte 118 and 118, 63 and 64.5, 40 MB of tokens 59 and 63 (160 MB 194 and 216: hence the line).  They stream their stores:
//     five streams of parts of lines (20-byte frames 47 us, 60 with plain stores).
static PackTraffic pack_traffic(int64_t total_slots, int64_t total_bytes, bool wide)
{
    if (wide) return 2 * total_bytes + 10 * total_slots <= ((int64_t)256 << 20) ? kPackThrough : kPackStream;
    return total_bytes <= ((int64_t)128 << 20) ? kPackCached : kPackStream;
}

template <int TRAFFIC>
static void pack_launch_wide(const PackArgs& a, const Run* runs, const int32_t* first_pos, uint32_t n_tiles, double inv_frame,
                             int32_t writes_table, hipStream_t stream)
{
    hipLaunchKernelGGL(pack_wide_kernel<TRAFFIC>, dim3(n_tiles), dim3(kThreads), 0, stream, a, runs, first_pos, kWideTile, inv_frame,
                       writes_table);
}

// The widest elements that divide the frame and that the source is aligned to: f(element, whether payload and table share a loop).
template <typename F>
static void with_element(const PackArgs& a, F f)
{
    if (a.frame_bytes % 16 == 0 && aligned_to(a.src, 16)) f(vec16{}, std::false_type());
    else if (a.frame_bytes == 4 && aligned_to(a.src, 4)) f(uint32_t{}, std::true_type());
    else if (a.frame_bytes % 4 == 0 && aligned_to(a.src, 4)) f(uint32_t{}, std::false_type());
    else if (a.frame_bytes % 2 == 0 && aligned_to(a.src, 2)) f(uint16_t{}, std::false_type());
    else f(uint8_t{}, std::false_type());
}

// One pass over slot tiles.
template <int TRAFFIC>
static void pack_launch_slots(const PackArgs& a, const Run* runs, const int32_t* first_pos, uint32_t n_tiles, int32_t parts,
                              hipStream_t stream)
{
    with_element(a, [&](auto element, auto fused) {
        hipLaunchKernelGGL((pack_narrow_kernel<decltype(element), decltype(fused)::value, TRAFFIC>), dim3(n_tiles * (uint32_t)parts),
                           dim3(kThreads), 0, stream, a, runs, first_pos, n_tiles, parts);
    });
}

// Enqueue the two passes.  `ws` holds l.bytes bytes, 32-byte aligned or better.
bload_status pack_enqueue(const PackLayout& l, const void* d_src, const int64_t* d_src_offsets,
                          const int32_t* d_lengths, const int32_t* d_order, const int32_t* d_block_of_seq,
                          const int32_t* d_offset_of_seq, const int32_t* d_block_first, int64_t n_seq,
                          int64_t num_blocks, int32_t t_blk, int64_t frame_bytes, void* d_packed,
                          int32_t* d_seq_id, int32_t* d_frame_idx, uint8_t* d_reset, uint8_t* d_valid,
                          uint8_t* ws, hipStream_t stream)
{
    if (l.tiles > INT32_MAX || l.table_tiles > INT32_MAX) return BLOAD_EOVERFLOW;
    Run* runs = reinterpret_cast<Run*>(ws + l.runs_off);
    int32_t* first_pos = reinterpret_cast<int32_t*>(ws + l.first_off);
    int32_t* first_pos_table = reinterpret_cast<int32_t*>(ws + l.table_off);
    PackArgs a;
    a.src = static_cast<const uint8_t*>(d_src);
    a.n_seq = (int32_t)n_seq;
    a.t_blk = t_blk;
    a.frame_bytes = frame_bytes;
    a.total_slots = num_blocks * (int64_t)t_blk;
    a.packed = static_cast<uint8_t*>(d_packed);
    a.seq_id = d_seq_id;
    a.frame_idx = d_frame_idx;
    a.reset = d_reset;
    a.valid = d_valid;

    // A tile is 1024 frames, one workgroup's work: where that leaves compute units idle, several workgroups share
    // a tile, towards 1024 of them, or 4096 from 64 bytes on, where a tile is 64 KiB and more; never more than
    // one per vector of a lane.  Short sequences, before and after: 8 tiles of 62 bytes 37 -> 12 us, 59 tiles
    // of 104 bytes 38 -> 12, 209 of 68 bytes 27 -> 14, 209 of 400 bytes 90 -> 30, 859 of 400 bytes 135 -> 101.
    // Towards 2048 under 64 bytes: 1055 tiles of 10 bytes 19 -> 21 us, of 48 bytes 25 -> 29.  1024 to 2047 tiles
    // of the large frames fill the card once by themselves, and a share each would be a second look at every tile's
    // runs for nothing: whole and in shares, 1059 of 64 bytes 27.5 and 29.7 us, of 128 bytes 45.3 and 46.9, 1399
    // of 400 bytes 220 and 234, 1199 of 68 bytes 36.0 and 38.5.  From 2048 on some tiles would run alone after the
    // others: 2099 of 64 bytes 54 and 49, of 128 bytes 95 and 85, of 256 bytes 245 and 226 with two shares.
    // Frames from 96 bytes on that are put together from elements, a load each, gain there too: 1556 tiles of
    // 104 bytes 52 and 47 us, of 200 bytes 88 and 75.
    const int64_t vectors = ceil_div(frame_bytes, 4);               // 1024 slots / 256 lanes / 16 bytes
    const bool vectors_copied = frame_bytes % 16 == 0 && aligned_to(d_src, 16);
    const bool once = l.tiles >= 1024 && l.tiles < 2048 && (vectors_copied || frame_bytes < 96);
    const int64_t wanted = once ? 1 : ceil_div(frame_bytes < 64 ? 1024 : 4096, l.tiles);
    const int32_t parts = (int32_t)(frame_bytes == 4 && aligned_to(d_src, 4) ? 1 : wanted < vectors ? wanted : vectors);
    const bool two_passes = frame_bytes == 4 && aligned_to(d_src, 4) && a.total_slots >= kTablePassFromSlots;

    const PlanTables t{d_src_offsets, d_lengths, d_order, d_block_of_seq, d_offset_of_seq, d_block_first};
    if (l.wide && l.tiles <= kDirectTiles) {
        const bool pairs = l.tiles > kDirectAtOnce;
        hipLaunchKernelGGL(pairs ? pack_direct_kernel<2> : pack_direct_kernel<1>, dim3((uint32_t)ceil_div(l.tiles, pairs ? 2 : 1)), dim3(kThreads),
                           0, stream, a, t, num_blocks, 1.0 / (double)frame_bytes, 1.0 / (double)t_blk);
        return launch_status();
    }
    const bool looks_pay = parts == 1 ? n_seq <= kDirectMost : n_seq * parts <= kDirectLooks && n_seq * 4 <= a.total_slots;
    if (!l.wide && !two_passes && l.tiles * parts <= kDirectTiles && looks_pay) {
        with_element(a, [&](auto element, auto fused) {
            hipLaunchKernelGGL((pack_narrow_direct_kernel<decltype(element), decltype(fused)::value>), dim3((uint32_t)(l.tiles * parts)),
                               dim3(kThreads), 0, stream, a, t, num_blocks, 1.0 / (double)t_blk, parts);
        });
        return launch_status();
    }
    // pass 1 (both tile shapes): the run table, and where each tile starts in it.  The
    // narrow tiles are 1024 slots, which the kernel takes as "1024 bytes of 1-byte frames".
    const int64_t unit_bytes = l.wide ? frame_bytes : 1;
    const int32_t tile_units = l.wide ? kWideTile : kNarrowSlots;
    const double inv_unit = 1.0 / (double)unit_bytes, inv_t = 1.0 / (double)t_blk;
    const int64_t prepare_threads = l.tiles > n_seq ? l.tiles : n_seq;       // table_tiles <= tiles
    hipLaunchKernelGGL(pack_prepare_kernel, dim3((uint32_t)ceil_div(prepare_threads, kThreads)),
                       dim3(kThreads), 0, stream, t, (int32_t)n_seq, num_blocks, (int64_t)t_blk, unit_bytes,
                       l.tiles, tile_units, inv_unit, inv_t, runs, first_pos, l.table_tiles, first_pos_table);
    const dim3 block(kThreads);
    const uint32_t n_tiles = (uint32_t)l.tiles;
    const PackTraffic traffic = pack_traffic(a.total_slots, a.total_slots * frame_bytes, l.wide);
    if (l.wide) {
        const auto launch = traffic == kPackThrough ? pack_launch_wide<kPackThrough> : pack_launch_wide<kPackStream>;
        launch(a, runs, first_pos, n_tiles, inv_unit, l.table_tiles == 0 ? 1 : 0, stream);
        if (l.table_tiles > 0)
            hipLaunchKernelGGL((pack_narrow_kernel<uint8_t, false, kPackStream, false, true, kPassGroup>),
                               dim3((uint32_t)ceil_div(l.table_tiles, kPassGroup)), block, 0, stream, a, runs,
                               first_pos_table, (uint32_t)l.table_tiles, 1);
        return launch_status();
    }
    // slot tiles: one pass; 4-byte frames (whose payload and table share a loop, so that one kernel writes
    // five streams at once) from kTablePassFromSlots slots on: the payload and the start table in a pass
    // each over the same tiles.  Measured on 1.3 * 10^9 token slots: 3.98 -> 3.72 ms; frames of 6 and 8
    // bytes, whose one pass already writes the table first and the payload after it, lose 5-7 % to the
    // second pass's look-ups and keep the one pass.
    if (two_passes) {
        const dim3 groups((uint32_t)ceil_div(l.tiles, kPassGroup));
        if (traffic == kPackCached)
            hipLaunchKernelGGL((pack_narrow_kernel<uint32_t, true, kPackCached, true, false, kPassGroup>), groups, block, 0, stream, a,
                               runs, first_pos, n_tiles, parts);
        else
            hipLaunchKernelGGL((pack_narrow_kernel<uint32_t, true, kPackStream, true, false, kPassGroup>), groups, block, 0, stream, a,
                               runs, first_pos, n_tiles, parts);
        hipLaunchKernelGGL((pack_narrow_kernel<uint8_t, false, kPackStream, false, true, kPassGroup>), groups, block, 0, stream, a,
                           runs, first_pos, n_tiles, parts);
    } else if (traffic == kPackCached) {
        pack_launch_slots<kPackCached>(a, runs, first_pos, n_tiles, parts, stream);
    } else {
        pack_launch_slots<kPackStream>(a, runs, first_pos, n_tiles, parts, stream);
    }
    return launch_status();
}

}  // namespace

extern "C" size_t bload_pack_workspace_bytes(int64_t n_seq, int64_t num_blocks, int32_t t_blk,
                                             int64_t frame_bytes)
{
    if (n_seq <= 0 || n_seq > BLOAD_MAX_SEQ || num_blocks <= 0 || t_blk < 1 || frame_bytes < 1) return 0;
    PackLayout l;
    if (!pack_layout(n_seq, num_blocks, t_blk, frame_bytes, true, true, &l)) return 0;
    return l.bytes;
}

extern "C" bload_status bload_pack(const void* d_src, const int64_t* d_src_offsets,
                                   const int32_t* d_lengths, const int32_t* d_order,
                                   const int32_t* d_block_of_seq, const int32_t* d_offset_of_seq,
                                   const int32_t* d_block_first, int64_t n_seq, int64_t num_blocks,
                                   int32_t t_blk, int64_t frame_bytes, void* d_packed,
                                   int32_t* d_seq_id, int32_t* d_frame_idx, uint8_t* d_reset,
                                   uint8_t* d_valid, void* d_workspace, size_t workspace_bytes,
                                   void* hip_stream)
{
    if (n_seq < 0 || num_blocks < 0 || t_blk < 1 || frame_bytes < 1) return BLOAD_EINVAL;
    if (n_seq > BLOAD_MAX_SEQ || num_blocks > n_seq) return n_seq > BLOAD_MAX_SEQ ? BLOAD_EOVERFLOW
                                                                                 : BLOAD_EINVAL;
    if (n_seq == 0 || num_blocks == 0) return BLOAD_OK;
    const bload_status st = pack_check_args(d_src, d_src_offsets, d_lengths, d_order, d_block_of_seq,
                                            d_offset_of_seq, d_block_first, n_seq, num_blocks, t_blk,
                                            frame_bytes, d_packed, d_seq_id, d_frame_idx, d_reset, d_valid);
    if (st != BLOAD_OK) return st;
    PackLayout l;
    if (!pack_layout(n_seq, num_blocks, t_blk, frame_bytes, aligned_to(d_src, 16), false, &l))
        return BLOAD_EOVERFLOW;
    if (!d_workspace) return BLOAD_EINVAL;
    if (!aligned_to(d_workspace, 32)) return BLOAD_EALIGN;
    if (workspace_bytes < l.bytes) return BLOAD_EWORKSPACE;
    return pack_enqueue(l, d_src, d_src_offsets, d_lengths, d_order, d_block_of_seq, d_offset_of_seq,
                        d_block_first, n_seq, num_blocks, t_blk, frame_bytes, d_packed, d_seq_id,
                        d_frame_idx, d_reset, d_valid, static_cast<uint8_t*>(d_workspace),
                        static_cast<hipStream_t>(hip_stream));
}

// ---------------------------------------------------- bload_pack_noalloc
//
// bload_pack for callers that cannot bring a workspace: the run table and the tiles'
// entries live in a fixed array in device memory that is part of the loaded library.
// Every GPU the library runs on holds its own copy of the array, at its own address,
// until the process ends; the address is asked for once per device.

constexpr size_t kStaticRunBytes = (size_t)BLOAD_PACK_NOALLOC_MAX_SEQ * sizeof(Run);
constexpr size_t kStaticBytes = kStaticRunBytes + (size_t)BLOAD_PACK_NOALLOC_MAX_TILES * sizeof(int32_t);
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_of_device[kMaxDevices] = {};

// Device address of `scratch` on the current device.
bload_status static_scratch(uint8_t** out)
{
    int dev = -1;
    if (!hip_ok(hipGetDevice(&dev))) return BLOAD_EHIP;
    if (dev < 0 || dev >= kMaxDevices) return BLOAD_EINVAL;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_of_device[dev]) {
        void* ptr = nullptr;
        if (!hip_ok(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch))) || !ptr) return BLOAD_EHIP;
        g_scratch_of_device[dev] = ptr;
    }
    *out = static_cast<uint8_t*>(g_scratch_of_device[dev]);
    return BLOAD_OK;
}

}  // namespace

extern "C" bload_status bload_pack_noalloc(const void* d_src, const int64_t* d_src_offsets,
                                           const int32_t* d_lengths, const int32_t* d_order,
                                           const int32_t* d_block_of_seq, const int32_t* d_offset_of_seq,
                                           const int32_t* d_block_first, int64_t n_seq,
                                           int64_t num_blocks, int32_t t_blk, int64_t frame_bytes,
                                           void* d_packed, int32_t* d_seq_id, int32_t* d_frame_idx,
                                           uint8_t* d_reset, uint8_t* d_valid, void* hip_stream)
{
    if (n_seq < 0 || num_blocks < 0 || t_blk < 1 || frame_bytes < 1) return BLOAD_EINVAL;
    if (n_seq > BLOAD_MAX_SEQ || num_blocks > n_seq) return n_seq > BLOAD_MAX_SEQ ? BLOAD_EOVERFLOW
                                                                                 : BLOAD_EINVAL;
    if (n_seq == 0 || num_blocks == 0) return BLOAD_OK;
    const bload_status st = pack_check_args(d_src, d_src_offsets, d_lengths, d_order, d_block_of_seq,
                                            d_offset_of_seq, d_block_first, n_seq, num_blocks, t_blk,
                                            frame_bytes, d_packed, d_seq_id, d_frame_idx, d_reset, d_valid);
    if (st != BLOAD_OK) return st;
    PackLayout l;
    if (!pack_layout(n_seq, num_blocks, t_blk, frame_bytes, aligned_to(d_src, 16), false, &l))
        return BLOAD_EOVERFLOW;
    // the fixed array holds this many runs and tiles, no more
    if (n_seq > BLOAD_PACK_NOALLOC_MAX_SEQ || l.tiles + l.table_tiles + 4 > BLOAD_PACK_NOALLOC_MAX_TILES)
        return BLOAD_EOVERFLOW;
    l.first_off = kStaticRunBytes;
    l.table_off = l.first_off + round_up((size_t)l.tiles * sizeof(int32_t), 16);
    uint8_t* ws = nullptr;
    const bload_status got = static_scratch(&ws);
    if (got != BLOAD_OK) return got;
    return pack_enqueue(l, d_src, d_src_offsets, d_lengths, d_order, d_block_of_seq, d_offset_of_seq,
                        d_block_first, n_seq, num_blocks, t_blk, frame_bytes, d_packed, d_seq_id,
                        d_frame_idx, d_reset, d_valid, ws, static_cast<hipStream_t>(hip_stream));
}

extern "C" bload_status bload_pack_check(const int64_t* d_src_offsets, const int32_t* d_lengths,
                                         const int32_t* d_order, const int32_t* d_block_of_seq,
                                         const int32_t* d_offset_of_seq, const int32_t* d_block_first,
                                         int64_t n_seq, int64_t num_blocks, int32_t t_blk,
                                         int64_t total_frames, int64_t* h_first_bad, void* d_workspace,
                                         size_t workspace_bytes, void* hip_stream)
{
    if (h_first_bad) *h_first_bad = -1;
    if (n_seq < 0 || num_blocks < 0 || t_blk < 1 || total_frames < 0) return BLOAD_EINVAL;
    if (n_seq > BLOAD_MAX_SEQ) return BLOAD_EOVERFLOW;
    if (num_blocks > n_seq) return BLOAD_EINVAL;
    if (n_seq == 0 || num_blocks == 0) return BLOAD_OK;
    if (!d_src_offsets || !d_lengths || !d_order || !d_block_of_seq || !d_offset_of_seq ||
        !d_block_first || !d_workspace)
        return BLOAD_EINVAL;
    if (!aligned_to(d_src_offsets, 8) || !aligned_to(d_lengths, 4) || !aligned_to(d_order, 4) ||
        !aligned_to(d_block_of_seq, 4) || !aligned_to(d_offset_of_seq, 4) ||
        !aligned_to(d_block_first, 4) || !aligned_to(d_workspace, 16))
        return BLOAD_EALIGN;
    if (workspace_bytes < 16) return BLOAD_EWORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    unsigned long long* first_bad = static_cast<unsigned long long*>(d_workspace);
    hipLaunchKernelGGL(pack_check_clear_kernel, dim3(1), dim3(1), 0, stream, first_bad);
    hipLaunchKernelGGL(pack_check_kernel, dim3((uint32_t)ceil_div(n_seq, kThreads)), dim3(kThreads), 0,
                       stream, d_src_offsets, d_lengths, d_order, d_block_of_seq, d_offset_of_seq,
                       d_block_first, (int32_t)n_seq, (int32_t)num_blocks, t_blk, total_frames, first_bad);
    if (launch_status() != BLOAD_OK) return BLOAD_EHIP;
    unsigned long long host = 0;
    if (!hip_ok(hipMemcpyAsync(&host, first_bad, sizeof(host), hipMemcpyDeviceToHost, stream)))
        return BLOAD_EHIP;
    if (!hip_ok(hipStreamSynchronize(stream))) return BLOAD_EHIP;
    if (host == ~0ull) return BLOAD_OK;
    if (h_first_bad) *h_first_bad = (int64_t)host;
    return BLOAD_EINVAL;
}
