// Internal definition of the plan object (host side) shared by plan.cpp and the
// device entry points.  Not part of the public interface.
#pragma once
#include <algorithm>
#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "paro.h"

#ifndef PARO_TILE_ELEMS
#define PARO_TILE_ELEMS 256
#endif
constexpr int PARO_TILE = PARO_TILE_ELEMS;      // elements per tile of the per-tile tables: a block's

// A piece of a chunk: elements [lo, hi) of a tile (hi == PARO_TILE: to its end), which lie in one
// tensor.  Pieces are listed in address order (those of cut tiles first, in a small chunk); a tile is
// one piece, or, where it is cut, one for each tensor in it (and one for the padding at its end).
struct paro_piece_info {
    int64_t where;      // offset in the tensor of the tile's first element (< 0 where the tensor starts
                        // later) << 19 | gradient dtype << 17 | hi << 8 | lo
    int32_t tensor;     // -2: padding; -1: a whole tile that holds too many tensors to be cut (or no room for
                        // more pieces), and the offset is the index of its first non-empty tensor
    uint32_t tile;
};

// An entry of a chunk's weight-decay table: all elements of the tile take weight decay, none does, or DECAY_BITS + the index,
// in the table, of the first of eight words with a bit for each element (set: it does).
constexpr uint32_t DECAY_ALL = 0, DECAY_NONE = 1, DECAY_BITS = 2;

struct paro_device_tables {
    int device = -1;
    int lds_per_cu = 0;             // bytes of LDS a compute unit has (for the occupancy throttle)
    int64_t *nz_off = nullptr;      // [n_nz + 1] flat start of every non-empty tensor, then Psi
    int32_t *nz_tensor = nullptr;   // [n_nz]     index of that tensor in the caller's list
    uint8_t *nz_dtype = nullptr;    // [n_nz]     its gradient dtype
    uint8_t *dtype = nullptr;       // [T]
    uint8_t *no_decay = nullptr;    // [T]
    // per chunk, each built at the first call that needs it:
    std::vector<uint32_t *> decay_tab;        // [P] the chunk's weight-decay table (see list_decays), or null
    std::vector<uint8_t> decay_tab_tried;     // [P] the decision for the chunk has been made
    std::vector<paro_piece_info *> piece_tab; // [P] the chunk's list of pieces, or null (tensor layout)
    std::vector<uint32_t> n_pieces;           // [P]
    std::vector<uint8_t> on_lines;            // [P] on_cache_lines() of the chunk
    std::vector<uint8_t> f32;                 // [P] mostly_f32() of the chunk
    std::vector<uint8_t> piece_tab_tried;     // [P]
    int64_t tiles_per_chunk = 0;
    int64_t max_pieces = 0;         // of a chunk: what the partial sums have room for
    double *partials = nullptr;     // per-block partial sums of squares, then the second-level sums
    int64_t n_partials = 0;         // capacity of the first level
};

struct paro_plan_s {
    int P = 0, G = 0, g = 0;
    char letters[4] = {0, 0, 0, 0};     // parameter, gradient, optimizer state
    int sched = PARO_RING;
    int pack_dtype = PARO_BF16;         // dtype of the packed low-precision parameters
    int64_t align = 8;
    int64_t T = 0;
    std::vector<int64_t> sizes;         // [T]
    std::vector<int64_t> off;           // [T + 1]
    std::vector<uint8_t> dtype;         // [T]
    std::vector<uint8_t> no_decay;      // [T]
    bool uniform_dtype = true;
    bool any_no_decay = false;
    int64_t total = 0;                  // Psi
    int64_t L = 0;                      // chunk length
    std::vector<int64_t> nz_off;        // non-empty tensors only (see paro_device_tables)
    std::vector<int32_t> nz_tensor;

    std::mutex dev_mutex;
    paro_device_tables dev;             // filled on the first device call
};

enum { PARO_MIN_PARTIALS = 4096 };   // smallest partial-sum scratch

namespace paro {
int fail(int code, const std::string &msg);     // records the thread's last error, returns code
inline int group_of(const paro_plan_t *pl, int rank) { return rank / pl->G; }
inline int local_of(const paro_plan_t *pl, int rank) { return rank % pl->G; }
inline int chunk_of_rank(const paro_plan_t *pl, int rank) {
    return local_of(pl, rank) * pl->g + group_of(pl, rank);
}
inline int owner_of_chunk(const paro_plan_t *pl, int chunk) {
    return (chunk % pl->g) * pl->G + chunk / pl->g;
}
// [begin, begin+len) of a rank's range for a sharding letter
void letter_range(const paro_plan_t *pl, int rank, char letter, int64_t *begin, int64_t *len);
// Whether nearly every piece of a chunk (the part of a block that lies in one tensor) belongs to a block
// that starts on a multiple of 64 elements of its tensor: on a cache line, if the tensor does.
bool on_cache_lines(const paro_plan_t *pl, int64_t chunk);
// Whether more than half of a chunk's gradient elements are fp32.
bool mostly_f32(const paro_plan_t *pl, int64_t chunk);
// Walks the tiles of a chunk in address order: fn(i, f0, f1, k), tile i holding the flat indices
// [f0, f1) and k the segment (non-empty tensor) that f0 lies in, or their number where f0 is padding.
template <class F>
void for_each_tile(const paro_plan_t *pl, int64_t chunk, F fn) {
    const int64_t c0 = chunk * pl->L, c1 = c0 + pl->L, n_nz = (int64_t)pl->nz_tensor.size();
    int64_t k = std::upper_bound(pl->nz_off.begin(), pl->nz_off.end(), c0) - pl->nz_off.begin() - 1;
    for (int64_t f0 = c0, i = 0; f0 < c1; f0 += PARO_TILE, ++i) {
        while (k < n_nz && pl->nz_off[(size_t)k + 1] <= f0) ++k;
        fn(i, f0, std::min(f0 + PARO_TILE, c1), k);
    }
}
// The weight-decay table of a chunk: one entry per tile, then the words of the tiles in which some elements take weight
// decay and some do not (padding does, and stays 0).
void list_decays(const paro_plan_t *pl, int64_t chunk, std::vector<uint32_t> *tab);
// One rank's messages of a collective, in the order of the public table: all of them, or those of one
// (phase, ring, step).
struct MessageId {
    int phase, ring, step;
};
int schedule_messages(const paro_plan_t *pl, int rank, int sched, int collective, const MessageId *only,
                      std::vector<paro_msg_t> *out);
// ranks in fold order for a chunk, and the run length of the first-level sums
void fold_order(const paro_plan_t *pl, int chunk, int32_t *ranks, int32_t *group_len);
}  // namespace paro
