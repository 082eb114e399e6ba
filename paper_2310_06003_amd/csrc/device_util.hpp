// Device-side building blocks of libparo (gfx950): launch-shape and cache-policy knobs, vector
// types, dtype conversions, streaming loads and stores, the wave-wide fp64 sum.  Included by
// kernels.hip only; everything lives in that translation unit's anonymous namespace.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "plan.hpp"

namespace {

// Cache-policy and occupancy knobs (the defaults are the measured best on MI355X).
// Nearly everything is touched once: loads are streaming (nt) loads.  Cache policy of the stores, as the
// instruction's bits: 1 = sc0, 2 = nt, 16 = sc1 (0 = default policy): streaming at system scope
// (nt sc1), which the large mixed read/write sweeps like 2 % better than nt alone - and without the
// streaming hint (sc1) for what the 256 MB memory-side cache holds until it is read again, see the
// PARO_KEEP_ limits.
#ifndef PARO_POL_STREAM_ST
#define PARO_POL_STREAM_ST 18
#endif
#ifndef PARO_POL_KEEP_ST
#define PARO_POL_KEEP_ST 16
#endif
// Largest results that are stored without the streaming hint.
// The reduced gradient, which sweep 2 reads again (in the fused step with plain loads: a streaming load gives the line up), where the
// contributions that pass through the cache meanwhile are no more than it holds.  Whole clipped steps, bf16, on the same buffers, streaming
// and kept: P = 2, 12 M elements 75.7 and 71.5 us; P = 4, 16 M 111.0 and 103.9; P = 8, 3 M 29.9 and 28.9, 8 M 71.1 and 67.0, 16 M 129.9 and
// 121.8; P = 16, 6 M 70.7 and 67.6.  With other work on the GPU between the steps:
//   contributions just written, or copied in: up to 200 MB of them P = 2 to 16 are ahead by 1 to 5 %, up to 13 %.  Copied ones of 205 to 260 MB
//   fill the cache by themselves and are behind by 3 to 13 % in places (P = 15, 8 M elements 77.5 and 89.0 us, P = 16, 7 M 71.7 and 80.7, P = 12,
//   10 M 90.2 and 98.8, P = 8, 13 M 100.3 and 105.5), ahead by as much in others (P = 8, 16 M 131.6 and 120.0); written ones there are 2 to 4 %
//   ahead, from 256 MB on 1 to 5 % behind (P = 16, 8 M 87.7 and 89.4; P = 8, 16 M 123.0 and 125.4).  Hence the limit on the contributions, and
//   a lower one for arrays in shard coordinates of more than 8 ranks, for which what is lost there weighs more than what is won.  Lists of
//   tensors do not mind (GPT-2, P = 16, 249 MB: 3 to 5 % ahead in all but one)
//   512 MB of something else: P = 2 to 8 ahead by 1 to 4 %, P = 12 by 1 % to behind by 1, P = 16 behind by 0 to 3; P = 32 and 64 were behind by
//   2 to 4 % from 2 M on, so more than 16 ranks keep only what is small enough to keep its state as well.
// Beyond these limits the last PARO_KEEP_G_TAIL_ELEMS are kept, 224 MB, and sweep 2 begins at the end (not with a mask, see k_adam4).
#ifndef PARO_KEEP_G_ELEMS
#define PARO_KEEP_G_ELEMS (16 << 20)
#endif
#ifndef PARO_KEEP_G_READ_BYTES
#define PARO_KEEP_G_READ_BYTES (256 << 20)
#endif
#ifndef PARO_KEEP_G_FEW_RANKS
#define PARO_KEEP_G_FEW_RANKS 8
#endif
#ifndef PARO_KEEP_G_WIDE_READ_BYTES
#define PARO_KEEP_G_WIDE_READ_BYTES (192 << 20)   // ... chunk layout, more ranks than that
#endif
// Of a larger gradient the end, which sweep 2, begun there, reads before anything else has passed through the cache (streaming loads and
// plain ones are alike then).  Whole clipped steps, bf16, same buffers, without and with 128 and 224 MB of it:
//   P = 2, 40 M elements 236 us, -3.1 %, -2.7 %, 60 M 343, -1.4, -3.3, 150 M 853, -0.5, -1.1; P = 4, 17 M 113, -6.2, -6.4, 100 M 632, -1.1, -2.1; P = 6, 70 M
//   491, -2.0, -4.4; P = 8, 17 M 135, -4.7, -4.7, 60 M 457, -0.9, -1.3, 200 M 1502, -0.4, -0.1; fp16, 124 M 953, -1.5, -2.3; P = 16, 9 M 100.6, -4.5, -5.2, 30 M
//   300, -3.7, -3.6, 100 M 998, -0.8, -1.6, 420 M 4141, -0.3, -0.5; P = 32, 8 M 135, -1.5, -1.5, 20 M 304, -2.7, -2.8; P = 64, 5 M 143, -1.7, -1.9, 105 M 2583, 0, -0.3;
//   fp32, P = 4, 30 M 238, -6.7, -5.9, P = 16, 20 M 311, -3.8, -3.9.  256 MB: as 224; more: P = 2, 60 M -4.0, but P = 8, 200 M up to +1.5, P = 16, 200 M up to +1.9
//   contributions just written, or copied in: -1 to -7 % in all of these; after 512 MB of something else -2 to -12 %
//   the split calls: P = 8, 20 M -4.6 %, 60 M -1.2, P = 16, 12 M -5.4; fp32, 2 chunks of 62.5 M, P = 16, 1875 us -1.2 to -1.7
// Kept whole and read from the start, what is below the limits above is as fast (P = 8, 10 M 77.8 and 77.9 us) or up to 1 % faster (4 M and less).
#ifndef PARO_KEEP_G_TAIL_ELEMS
#define PARO_KEEP_G_TAIL_ELEMS ((int64_t)56 << 20)
#endif
// p, m, v and the packed parameters, which the next step reads: with 1 M elements (18 MB with the gradient)
// 15.3 -> 14.1 us (P = 8, clipped) and 9.6 -> 8.5 (one sweep), on ten states as on three; 4 M on ten states 37.5 -> 40.0.  With contributions
// just written 16.8 -> 15.9 (clipped) and 11.8 -> 10.4; after 512 MB of something else 0 to 3 % behind (17.1 and 17.6; 12.0 and 12.1).
#ifndef PARO_KEEP_STATE_ELEMS
#define PARO_KEEP_STATE_ELEMS (1 << 20)
#endif
// The result of a hop, which the next one reads: 8 M elements 13.6 -> 12.9 us, 30 M 45.1 -> 45.6; with its addend just written 15.7
// -> 14.2, after 512 MB of something else 15.9 -> 16.2.
#ifndef PARO_KEEP_MESSAGE_BYTES
#define PARO_KEEP_MESSAGE_BYTES (48 << 20)
#endif
// The messages of one step of an all-gather, over all its ranks: the next step reads them, and of each as much is kept, from its start, as
// the cache holds of all.  Streamed, messages up to 48 MB whole, and these: 8 ranks, 16 MB 361, 313, 313 us, 31 MB 631, 594, 590, 62 MB 1112, 1112,
// 1070, 125 MB 2247, 2247, 2215; 16 ranks, 31 MB 2558, 2545, 2520; 4 ranks, 62 MB 236.5, 236.5, 232.9, 120 MB 438, 438, 425; 3 ranks, 60 MB 114.9, 114.9, 109.7; 2
// ranks, 100 MB 61.1, 61.1, 57.7; but 6 ranks, 40 MB 400, 376.5, 378.
#ifndef PARO_KEEP_MESSAGES_BYTES
#define PARO_KEEP_MESSAGES_BYTES (224 << 20)
#endif
#ifndef PARO_KEEP_OF_MESSAGE_BYTES
#define PARO_KEEP_OF_MESSAGE_BYTES (64 << 20)
#endif
#ifndef PARO_BATCH
#define PARO_BATCH 16               // contributions loaded before the first is consumed
#endif
#ifndef PARO_LANE_BATCH
#define PARO_LANE_BATCH 2          // ... in a block that a wave takes element by element (each has its own pointer: registers)
#endif
// One-wave blocks in flight per compute unit (0 = as many as fit).  The mixed read/write sweeps
// run faster with fewer requests outstanding than the registers would allow.  For the fold the
// budget is in loads: a wave has min(P, PARO_BATCH) of them in flight, so with P = 16 the numbers
// below mean 14 waves per compute unit for sweep 1 and 10 for the single sweep (whose waves also
// load 3 state vectors); with fewer contributions per wave, more waves.  Where other numbers hold: fold_budget, fused_waves.
// Wave counts here and there are counts asked for; throttle_lds says what fits.
#ifndef PARO_FOLD_LOADS_PER_CU
#define PARO_FOLD_LOADS_PER_CU 224
#endif
#ifndef PARO_FOLD_WIDE_LOADS_PER_CU
#define PARO_FOLD_WIDE_LOADS_PER_CU 192   // many contributions (see fold_budget)
#endif
#ifndef PARO_FOLD_F32_LIST_LOADS_PER_CU
#define PARO_FOLD_F32_LIST_LOADS_PER_CU 160   // sweep 1 over large chunks of fp32 gradients, tensor layout
#endif
#ifndef PARO_FUSED_LOADS_PER_CU
#define PARO_FUSED_LOADS_PER_CU 190
#endif
#ifndef PARO_FUSED_MIN_BLOCKS
#define PARO_FUSED_MIN_BLOCKS 8192  // blocks of a single sweep from which on fused_waves thins out its waves
#endif
// Blocks of a single sweep up to which it runs all waves that fit (see runs_at_once): over a range of two-byte contributions, other, over one chunk
// of 17 to 31 two-byte ones, of up to 16 of them this many blocks times ranks.
#ifndef PARO_AT_ONCE_RANGE_BLOCKS
#define PARO_AT_ONCE_RANGE_BLOCKS 8192
#endif
#ifndef PARO_AT_ONCE_BLOCKS
#define PARO_AT_ONCE_BLOCKS 4096
#endif
#ifndef PARO_AT_ONCE_SHORT_BATCH_BLOCKS
#define PARO_AT_ONCE_SHORT_BATCH_BLOCKS 3840
#endif
#ifndef PARO_AT_ONCE_READS
#define PARO_AT_ONCE_READS 49152
#endif
#ifndef PARO_FUSED_RANGE_MIN_READS
#define PARO_FUSED_RANGE_MIN_READS 81920   // ... and blocks times ranks of one over several chunks of two-byte contributions
#endif
#ifndef PARO_ADAM_WAVES_PER_CU
#define PARO_ADAM_WAVES_PER_CU 12
#endif
// A large sweep 2, from PARO_LARGE_TILES blocks on, wants one wave less since its waves start at once (whole clipped steps, same buffers, 12,
// 11 and 10 waves: fp16, P = 8, 124 M elements 955, 946 and 948 us; P = 16, 421 M 4244, 4227 and 4242; P = 8, 62 M 481, 476 and 477; P = 2, 80 M
// 462, 462 and 467; but 16 M 121.4 and 122.1.  12 and 11 on another GPU: 949 and 943; 4288 and 4273; 474 and 470; 459 and 457; P = 8, 40 M 304.6 and
// 304.2).
#ifndef PARO_ADAM_LARGE_WAVES_PER_CU
#define PARO_ADAM_LARGE_WAVES_PER_CU 11
#endif
// A small sweep 2 runs in as many waves as the masked one where all of it fits the chip at once, and not beyond (whole clipped steps, same
// buffers, 12 and 16 waves: 1 M elements, P = 2, 11.0 and 10.1 us, P = 16 14.3 and 13.8; 1.5 M, P = 8, 16.8 and 17.0; 2 M, P = 2, 17.0 and 17.2;
// 3 M, P = 8, 28.1 and 28.4; 4 M, P = 16, 46.5 and 47.0; 0.4 M no difference).
#ifndef PARO_ADAM_SMALL_ELEMS
#define PARO_ADAM_SMALL_ELEMS (1 << 20)
#endif
#ifndef PARO_ADAM_MASK_WAVES_PER_CU
#define PARO_ADAM_MASK_WAVES_PER_CU 16   // with a decay mask: a table look-up per wave to hide as well
#endif
// The tensor layout.  What decides is the list: a chunk made of a few large tensors ("large": at least
// PARO_DENSE_BLOCKS_PER_TENSOR blocks per tensor piece in the chunk, on average) behaves like the chunk
// layout - its look-ups hit the scalar cache - and keeps the chunk layout's budget.  A chunk cut into
// many small pieces has waves that spend part of their life on look-ups with no data in flight: it is
// launched without the throttle (the single sweep, whose waves load their state as well, only in
// chunks of fewer than PARO_LARGE_TILES blocks).  With at most PARO_PAIR_MAX_RANKS contributions and at
// least PARO_PAIR_MIN_BLOCKS blocks, and with at most PARO_PAIR_SMALL_MAX_RANKS in a large chunk of many
// small pieces that are not mostly fp32, a wave takes two consecutive blocks (see k_reduce4t).
#ifndef PARO_PAIR_MAX_RANKS
#define PARO_PAIR_MAX_RANKS 4
#endif
#ifndef PARO_PAIR_SMALL_MAX_RANKS
#define PARO_PAIR_SMALL_MAX_RANKS 6
#endif
#ifndef PARO_PAIR_MIN_BLOCKS
#define PARO_PAIR_MIN_BLOCKS 16384
#endif
#ifndef PARO_DENSE_BLOCKS_PER_TENSOR
#define PARO_DENSE_BLOCKS_PER_TENSOR 1024
#endif
#ifndef PARO_FOLD_TM_LOADS_PER_CU
#define PARO_FOLD_TM_LOADS_PER_CU 100000
#endif
#ifndef PARO_FUSED_TL_WAVES_PER_CU
#define PARO_FUSED_TL_WAVES_PER_CU 20    // the single sweep over a large chunk of many small tensors, more than 8 ranks
#endif
#ifndef PARO_LARGE_TILES
#define PARO_LARGE_TILES 131072
#endif
#ifndef PARO_MIN_WAVES_PER_CU
#define PARO_MIN_WAVES_PER_CU 8     // the throttle never goes below this
#endif
#ifndef PARO_PACE_SLEEP
#define PARO_PACE_SLEEP 4           // units of 64 clocks between two loads of a paced fold
#endif
#ifndef PARO_PACE_WIDE_SLEEP
#define PARO_PACE_WIDE_SLEEP 10     // ... in sweep 1 over one chunk with more than 16 ranks
#endif
#ifndef PARO_PACE_WIDE_F32_SLEEP
#define PARO_PACE_WIDE_F32_SLEEP 6  // ... of fp32 gradients
#endif
#ifndef PARO_PACE_MIN_BLOCKS
#define PARO_PACE_MIN_BLOCKS 65536  // blocks of a launch over one chunk from which on it is paced (32 ranks: half)
#endif
// Write windows of sweep 1: which launches have them (see holds_back), and their times in ticks of 10 ns.
#ifndef PARO_WINDOW_MIN_RANKS
#define PARO_WINDOW_MIN_RANKS 12
#endif
#ifndef PARO_WINDOW_MANY_RANKS
#define PARO_WINDOW_MANY_RANKS 48
#endif
#ifndef PARO_WINDOW_MIN_BLOCKS
#define PARO_WINDOW_MIN_BLOCKS 98304     // two-byte contributions; 24 to 47 ranks: half
#endif
#ifndef PARO_WINDOW_F32_MIN_BLOCKS
#define PARO_WINDOW_F32_MIN_BLOCKS 16384
#endif
#ifndef PARO_WINDOW_TICKS
#define PARO_WINDOW_TICKS 50             // how long a window is open to waves that arrive
#endif
#ifndef PARO_WINDOW_REST_TICKS
#define PARO_WINDOW_REST_TICKS 60        // how long new waves leave the memory to it
#endif
#ifndef PARO_WINDOW_TICKS_PER_RANK
#define PARO_WINDOW_TICKS_PER_RANK 36    // from one window to the next
#endif
#ifndef PARO_WINDOW_MAX_PERIOD
#define PARO_WINDOW_MAX_PERIOD 1600
#endif
#ifndef PARO_ALL_WAVES_MIN_BLOCKS
#define PARO_ALL_WAVES_MIN_BLOCKS 16384          // tensor layout, 48 ranks and more: from here on sweep 1 runs all waves that fit
#endif
#ifndef PARO_ALL_WAVES_F32_LARGE_RANKS
#define PARO_ALL_WAVES_F32_LARGE_RANKS 56        // ... over a large chunk of fp32 gradients
#endif
// ... over a range of several chunks (see range_holds_back).
#ifndef PARO_RANGE_WINDOW_MIN_BLOCKS
#define PARO_RANGE_WINDOW_MIN_BLOCKS 16384       // two-byte contributions of up to 16 ranks: four times as many
#endif
#ifndef PARO_RANGE_WINDOW_TICKS_PER_RANK
#define PARO_RANGE_WINDOW_TICKS_PER_RANK 24      // two-byte contributions: from one window to the next
#endif
#ifndef PARO_RANGE_WINDOW_MAX_PERIOD
#define PARO_RANGE_WINDOW_MAX_PERIOD 1300
#endif
#ifndef PARO_RANGE_ALWAYS_RANKS
#define PARO_RANGE_ALWAYS_RANKS 100              // two-byte contributions, from here on one launch whatever the chunks' size
#endif
#ifndef PARO_WINDOW_PACE_SLEEP
#define PARO_WINDOW_PACE_SLEEP 5         // pause between two loads of a launch with windows
#endif
#ifndef PARO_WINDOW_F32_WAVES_PER_CU
#define PARO_WINDOW_F32_WAVES_PER_CU 18  // of a launch with windows over fp32 contributions
#endif
// ... and of the single sweep (see fused_holds_back).
#ifndef PARO_FUSED_WINDOW_RANK_BYTES
#define PARO_FUSED_WINDOW_RANK_BYTES 64          // bytes of contributions for an element from which on it has windows ...
#endif
#ifndef PARO_FUSED_WINDOW_MIN_BYTES
#define PARO_FUSED_WINDOW_MIN_BYTES (512 << 20)  // ... and of all; more than 64 ranks: for each 64
#endif
#ifndef PARO_FUSED_WINDOW_MANY_BYTES
#define PARO_FUSED_WINDOW_MANY_BYTES 80          // with fewer bytes for an element half as many again of all
#endif
#ifndef PARO_FUSED_WINDOW_TWO_BATCHES_BYTES
#define PARO_FUSED_WINDOW_TWO_BATCHES_BYTES ((int64_t)1664 << 20)   // 32 two-byte ranks: of all
#endif
#ifndef PARO_FUSED_WINDOW_TICKS_PER_BYTE
#define PARO_FUSED_WINDOW_TICKS_PER_BYTE 26      // from one window to the next, for each of the element's bytes
#endif
#ifndef PARO_FUSED_WINDOW_MAX_PERIOD
#define PARO_FUSED_WINDOW_MAX_PERIOD 2800
#endif
#ifndef PARO_FUSED_WINDOW_F32_MAX_PERIOD
#define PARO_FUSED_WINDOW_F32_MAX_PERIOD 2300
#endif
// ... over a range of several chunks of two-byte contributions (see fused_range_holds_back).
#ifndef PARO_FUSED_RANGE_WINDOW_MIN_RANKS
#define PARO_FUSED_RANGE_WINDOW_MIN_RANKS 28
#endif
#ifndef PARO_FUSED_RANGE_UNPACED_RANKS
#define PARO_FUSED_RANGE_UNPACED_RANKS 96
#endif
#ifndef PARO_FUSED_RANGE_WINDOW_MAX_PERIOD
#define PARO_FUSED_RANGE_WINDOW_MAX_PERIOD 1800
#endif
#ifndef PARO_FUSED_WINDOW_PACE_SLEEP
#define PARO_FUSED_WINDOW_PACE_SLEEP 3
#endif
#ifndef PARO_FUSED_WINDOW_F32_WAVES_PER_CU
#define PARO_FUSED_WINDOW_F32_WAVES_PER_CU 21    // the registers let 20 run
#endif
// A small single sweep whose waves pause (see pauses_single, pauses_range): how long, and the bytes that the launch reads.
#ifndef PARO_PAUSE_SLEEP
#define PARO_PAUSE_SLEEP 26         // units of 64 clocks (20 and 40: 3 to 7 % slower at 25 to 27 MB with P = 1, and with P = 3 or 2)
#endif
#ifndef PARO_PAUSE_MAX_RANKS
#define PARO_PAUSE_MAX_RANKS 3
#endif
#ifndef PARO_PAUSE_MIN_BYTES
#define PARO_PAUSE_MIN_BYTES 21000000       // P = 3, 20.5 MB: 7 % ahead without
#endif
#ifndef PARO_PAUSE_MIN_BYTES_ONE
#define PARO_PAUSE_MIN_BYTES_ONE 20000000   // one rank
#endif
#ifndef PARO_PAUSE_MAX_BYTES
#define PARO_PAUSE_MAX_BYTES 30500000
#endif
#ifndef PARO_PAUSE_RANGE_MIN_BYTES
#define PARO_PAUSE_RANGE_MIN_BYTES 19500000   // over a range of several chunks
#endif
#ifndef PARO_PAUSE_RANGE_MAX_BYTES
#define PARO_PAUSE_RANGE_MAX_BYTES 31000000
#endif
#ifndef PARO_PAUSE_RANGE_MAX_BYTES_TWO
#define PARO_PAUSE_RANGE_MAX_BYTES_TWO 27000000   // ... of two ranks
#endif
#ifndef PARO_SPLIT_MAX
#define PARO_SPLIT_MAX 16           // a tile with up to so many tensors inside is cut into pieces
#endif
#ifndef PARO_RANGE_MAX_BLOCKS
#define PARO_RANGE_MAX_BLOCKS 65536   // chunks of so many blocks are launched one by one (see chunk_by_chunk)
#endif
#ifndef PARO_HOP_WAVES_PER_CU
#define PARO_HOP_WAVES_PER_CU 0
#endif
#ifndef PARO_COPY_WAVES_PER_CU
#define PARO_COPY_WAVES_PER_CU 0
#endif

constexpr int WAVE = 64;              // threads of a block: every sweep kernel runs in one-wave blocks
constexpr int EPT = 4;                // elements per thread
constexpr int COMPUTE_UNITS = 256;
constexpr int MAX_WAVES_PER_CU = 32;
constexpr int PIECE = WAVE * EPT;     // elements per block
constexpr int TILE = PARO_TILE;       // granularity of the plan's per-block table
constexpr int FINALIZE_TPB = 1024;    // threads of the kernel that adds the partial sums
constexpr int FINALIZE_CHUNK = 8192;  // partials per block in its first level: eight per thread, all in flight
constexpr int NORM_DIRECT_PARTIALS = 2048;      // partials that every wave of sweep 2 adds up itself
constexpr int NORM_SLICES = 8;                  // else: slice sums that it does (one scalar load) ...
constexpr int NORM_SLICES_PARTIALS = 131072;    // ... up to so many partials (33.5 M elements)
constexpr int NORM_ONE_BLOCK_PARTIALS = 2 * FINALIZE_TPB * NORM_SLICES;     // slices and total by one block up to here
constexpr unsigned NORM_GROUP = PARO_STATIC_MAX_CHUNK / PIECE;              // blocks of a range whose partials are added up together
static_assert(TILE == PIECE, "the per-tile tables have one entry per block");

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// P device pointers in fold order (or in rank order, see RangeMap).  Lives in the kernel-argument
// segment and is only ever indexed with wave-uniform indices, i.e. read with scalar loads.  Kernels
// come with room for 16 pointers and for PARO_MAX_RANKS: 2 KB of arguments cost the host 0.2-0.3 us a
// launch (a small step of one launch: 6.20 -> 5.99 us; of two: 10.2 -> 9.6).
template <int N, bool HELD = false>
struct SrcTableOf {
    const void *p[N];
    int paced;               // the chunk layout's loads go out one by one, with a pause in between
    unsigned keep_from;      // block of the update range from which on the reduced gradient is stored to stay in the memory-side cache
};
using SrcTable = SrcTableOf<PARO_MAX_RANKS>;
constexpr int FEW_SRC = 16;

// Write windows of a launch that holds its results back (see holds_back), in ticks of the constant 100 MHz clock that the whole chip shares: one begins at every
// multiple of `period`.  inverse: 2^32 / period, rounded down.  The launch's last blocks, `waves` for each compute unit, do not wait: at least as many as run at
// once.  Where the registers let fewer run than were asked for - 20 for 21 in single sweeps over fp32 contributions, 28 for 32 in launches over a range of several
// chunks of two-byte ones and in single sweeps that look up exempt tensors - that is up to 1024 of them more than have nobody behind them.  Waves that arrive within
// `open` of a window's start store at once, and new ones begin to read after `rest`.
struct WriteWindow {
    unsigned inverse;
    unsigned short period, waves, open, rest;
};
// It comes with the pointers of such a launch: as an argument of its own it would be there, if empty, for the others as well.
template <int N>
struct SrcTableOf<N, true> : SrcTableOf<N, false> {
    WriteWindow window;
};
template <int N>
__device__ __forceinline__ WriteWindow window_of(const SrcTableOf<N, true> &src) { return src.window; }
template <int N>
__device__ __forceinline__ WriteWindow window_of(const SrcTableOf<N, false> &) { return WriteWindow(); }

struct AdamConsts {
    float beta1, beta2, omb1, omb2, eps, step_size, sqrt_bc2, decay, wd, grad_scale, max_norm;
    int adamw, skip_nonfinite, pack_dtype;
    int keep_state;     // p, m, v and the packed parameters are stored to stay in the memory-side cache
};

// What a launch needs to map its elements to tensors.
struct TensorMap {
    const int64_t *nz_off;      // [n_nz + 1] flat start of every non-empty tensor, then Psi
    const int32_t *nz_tensor;   // [n_nz]
    const uint8_t *nz_dtype;    // [n_nz] gradient dtype of that tensor
    const uint8_t *dtype;       // [T]
    const uint8_t *no_decay;    // [T]
    int n_nz;
    int64_t total;              // Psi
    int64_t begin;              // flat index of the launch's element 0
    const uint32_t *decay_tab;        // the weight-decay table of the launch's chunk, or null
    const paro_piece_info *pieces;    // [n_pieces] the chunk's pieces, or null
    unsigned n_pieces;
};

// Lane of the thread in its wave (the sweep kernels run in one-wave blocks).
__device__ __forceinline__ unsigned lane_id() { return threadIdx.x & (WAVE - 1); }

// ---------------------------------------------------------------- small helpers
__device__ __forceinline__ float bf16_lo(unsigned int w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned int w) { return __uint_as_float(w & 0xFFFF0000u); }

// fp16 <-> fp32: the hardware conversions (exact upwards, round-to-nearest-even downwards)
__device__ __forceinline__ float f16_bits_to_f32(unsigned int h16) {
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h16);
}
__device__ __forceinline__ unsigned int f32_to_f16_bits(float f) {
    return (unsigned int)__builtin_bit_cast(unsigned short, (_Float16)f);
}
// the two 16-bit values of a word, as fp32, for a 2-byte gradient dtype
template <int DT>
__device__ __forceinline__ float cvt_lo(unsigned int w) {
    return DT == PARO_F16 ? f16_bits_to_f32(w & 0xFFFFu) : bf16_lo(w);
}
template <int DT>
__device__ __forceinline__ float cvt_hi(unsigned int w) {
    return DT == PARO_F16 ? f16_bits_to_f32(w >> 16) : bf16_hi(w);
}
__device__ __forceinline__ float cvt16(unsigned int h16, int dt) {
    return dt == PARO_F16 ? f16_bits_to_f32(h16) : __uint_as_float(h16 << 16);
}

__device__ __forceinline__ unsigned int f32_to_bf16_rne(float f) {
    unsigned int u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (u >> 16) | 0x0040u;      // NaN stays NaN
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// two parameters rounded to the low-precision format, packed into one word
__device__ __forceinline__ unsigned int pack2_lowp(float a, float b, int pack_dtype) {
    if (pack_dtype == PARO_F16) return f32_to_f16_bits(a) | (f32_to_f16_bits(b) << 16);
    return f32_to_bf16_rne(a) | (f32_to_bf16_rne(b) << 16);
}

// Pointers that were themselves loaded from memory carry no address space; these are device
// (global) addresses by contract, so say so and get global rather than flat loads.
template <class V>
__device__ __forceinline__ const __attribute__((address_space(1))) V *global_ptr(uintptr_t a) {
    return reinterpret_cast<const __attribute__((address_space(1))) V *>(a);
}
// Streaming (non-temporal) load of something read once.
template <class V>
__device__ __forceinline__ V ld_nt(const V *p) { return __builtin_nontemporal_load(p); }
template <class V>
__device__ __forceinline__ V ld_nt(const __attribute__((address_space(1))) V *p) { return __builtin_nontemporal_load(p); }

// Vector load of 4 elements at any address that suits one element (2 bytes of the 2-byte dtypes, 4 of
// fp32); NT: streaming.  The alignment is part of the type of the pointer that is dereferenced, so the type is
// named here and not handed in as a template argument, which would drop it.
template <class V, bool NT>
__device__ __forceinline__ V ld_any(uintptr_t a) {
    typedef u32x2 u32x2_at2 __attribute__((aligned(2)));
    typedef u32x4 u32x4_at4 __attribute__((aligned(4)));
    if constexpr (std::is_same_v<V, u32x2>) {
        const auto *p = reinterpret_cast<const __attribute__((address_space(1))) u32x2_at2 *>(a);
        if constexpr (NT) return __builtin_nontemporal_load(p);
        else return *p;
    } else {
        const auto *p = reinterpret_cast<const __attribute__((address_space(1))) u32x4_at4 *>(a);
        if constexpr (NT) return __builtin_nontemporal_load(p);
        else return *p;
    }
}

// ---- stores through per-wave buffer descriptors.  A block's stores to one array go through a
// descriptor that covers exactly the block's piece of it (a wave-uniform base address and a byte
// count): the instruction then carries its cache policy as an immediate - which a plain store
// cannot express beyond "non-temporal" - and the hardware drops whatever falls outside the piece.
// (Loads stay plain streaming loads: building a descriptor per contribution cost the fold 5 %.)
typedef __amdgpu_buffer_rsrc_t wave_buf;
__device__ __forceinline__ wave_buf wave_buffer(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
template <int POL>
__device__ __forceinline__ void buf_store8(u32x2 v, wave_buf b, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b64(v, b, (int)off, 0, POL);
}
template <int POL>
__device__ __forceinline__ void buf_store16(u32x4 v, wave_buf b, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b128(v, b, (int)off, 0, POL);
}
// ... with the streaming hint or, where the memory-side cache is to keep the data, without.
__device__ __forceinline__ void buf_store16_as(bool keep, u32x4 v, wave_buf b, unsigned off) {
    if (keep) buf_store16<PARO_POL_KEEP_ST>(v, b, off);
    else buf_store16<PARO_POL_STREAM_ST>(v, b, off);
}
__device__ __forceinline__ u32x4 as_u32x4(float a, float b, float c, float d) {
    return u32x4{__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)};
}

// A value that is the same in every lane, marked as such for the compiler (scalar registers,
// scalar branches, scalar loads of what it indexes).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// One lane's value, for the whole wave.
__device__ __forceinline__ double of_lane(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// The value of another lane of the same row of 16, picked by a DPP control.
template <int CTRL>
__device__ __forceinline__ double from_lane(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false));
}
// Ticks since the last write window began.
__device__ __forceinline__ unsigned window_phase(const WriteWindow &w) {
    const unsigned now = (unsigned)__builtin_amdgcn_s_memrealtime();
    const unsigned phase = now - __umulhi(now, w.inverse) * w.period;       // the quotient may be one too small
    return phase >= w.period ? phase - w.period : phase;
}
// What a wave does before its first load: while a window is open it leaves the memory to the stores.
__device__ __forceinline__ void leave_window(const WriteWindow &w) {
    for (int i = 0; i < 128 && window_phase(w) < w.rest; ++i) __builtin_amdgcn_s_sleep(2);
}
// Whether a block has others behind it that wait for its place (of the last ones see WriteWindow).
__device__ __forceinline__ bool has_followers(const WriteWindow &w) {
    return blockIdx.x + (unsigned)w.waves * COMPUTE_UNITS < gridDim.x;
}
// ... and before its stores, with everything in registers that they need: is_formed() says so, of each four values.  Both waits are
// bounded by counts: the clock decides when data go out and never whether.
__device__ __forceinline__ void is_formed(const float X[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" ::"v"(X[i]));
}
__device__ __forceinline__ void wait_for_window(const WriteWindow &w) {
    for (int i = 0; i < 512 && window_phase(w) >= w.open; ++i) __builtin_amdgcn_s_sleep(3);
}

// Sum over the wave, in every lane; all 64 take part.  Fixed shape: lanes 32 apart, then 16, 8, 4, 2, 1 - after each step they
// hold the same sums, so a rotation by 8 or 4 within a row brings the partner's value.  Swaps of half-waves and rows and DPP
// moves stay in the vector unit; as shuffles the six steps were twelve trips to the LDS unit in a row, some 800 clocks at
// the end of every wave of sweep 1 with nothing in flight (whole clipped steps, same buffers: P = 16, 1 M elements 14.7 -> 14.3 us; P
// = 8, 1.5 M 18.1 -> 17.8, 3 M 29.1 -> 28.8; ragged tensors, P = 16, 26.8 -> 26.3; from 10 M elements on as before).
__device__ __forceinline__ double wave_sum(double v) {
    {   // the halves of the wave
        const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
    {   // rows of 16 lanes
        const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
        v = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
    }
    v += from_lane<0x128>(v);       // rotated by 8 within the row
    v += from_lane<0x124>(v);       // by 4
    v += from_lane<0x4E>(v);        // lanes 2 3 0 1 of every four
    v += from_lane<0xB1>(v);        // lanes 1 0 3 2
    return v;
}

// Sum over a block of FINALIZE_TPB threads, valid in thread 0: the lanes of each wave, then the waves in order.
__device__ __forceinline__ double block_sum(double v) {
    __shared__ double s_wave[FINALIZE_TPB / 64];
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) s_wave[wave] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0) {
        r = s_wave[0];
        for (int w = 1; w < FINALIZE_TPB / 64; ++w) r += s_wave[w];
    }
    return r;
}

// Compile-time loop: the body sees its index as a constant, so arrays indexed by it stay in
// registers whatever the size of the body.
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

}  // namespace
