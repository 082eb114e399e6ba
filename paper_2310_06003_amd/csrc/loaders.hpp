// How the fold gets its operands - the chunk layout (arrays in shard coordinates) and the tensor
// layout (per-tensor gradients, found through the plan's list of pieces or by searching its offset
// table) - and the ordered fold itself.  Every sweep kernel runs in one-wave blocks of 256
// elements, 4 per thread.  Included by kernels.hip only.
#pragma once

#include "device_util.hpp"

namespace {

// ------------------------------------------------------------------- loaders
// A loader hands the fold the 4 values that a contribution (entry k of the pointer table) holds for
// the thread's 4 elements: source() finds where they lie, load() issues the memory operations,
// unpack() turns what came back into fp32.  kBatch contributions are loaded before the first is
// consumed, and all their sources are found before the first load: found one by one, each would wait
// for its own scalar loads.

// Contributions are arrays in shard coordinates, all of one dtype: an 8-byte load per
// contribution for the 2-byte dtypes (a wave instruction covers 512 consecutive bytes), a
// 16-byte load for fp32.
// PACE: the pause between two loads of a paced launch, see load_batch.
template <int DT, int PACE = PARO_PACE_SLEEP>
struct Chunk4Loader {
    static constexpr int kBatch = PARO_BATCH;
    static constexpr int kElems = 4;
    static constexpr int kPace = PACE;
    static constexpr int ESIZE = DT == PARO_F32 ? 4 : 2;
    using Raw = std::conditional_t<DT == PARO_F32, u32x4, u32x2>;
    using At = const void *;
    int64_t e;                                   // first of the thread's 4 elements
    template <class Src>
    __device__ __forceinline__ At source(const Src &src, int k) const { return src.p[k]; }
    __device__ __forceinline__ void load(At at, Raw &r) const {
        r = ld_nt(reinterpret_cast<const Raw *>(static_cast<const char *>(at) + e * ESIZE));
    }
    static __device__ __forceinline__ void to_f32(const Raw &r, float x[4]) {
        if constexpr (DT != PARO_F32) {
            x[0] = cvt_lo<DT>(r.x); x[1] = cvt_hi<DT>(r.x); x[2] = cvt_lo<DT>(r.y); x[3] = cvt_hi<DT>(r.y);
        } else {
            x[0] = __uint_as_float(r.x); x[1] = __uint_as_float(r.y);
            x[2] = __uint_as_float(r.z); x[3] = __uint_as_float(r.w);
        }
    }
    __device__ __forceinline__ void unpack(const Raw &r, float x[4]) const { to_f32(r, x); }
};

// Largest k in [0, n_entries) with tab[k] <= f, for a sorted table with
// tab[0] <= f; the 64 lanes of the wave probe 64 places per round.
__device__ __forceinline__ int wave_search(const int64_t *tab, int n_entries, int64_t f, int lane) {
    int lo = 0, hi = n_entries;
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64;
        const int idx = lo + lane * step;
        const bool le = idx < hi && tab[idx] <= f;
        const int cnt = __popcll(__ballot(le));        // the lanes that hold form a prefix
        lo = lo + (cnt - 1) * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

// What a block knows about its 256 elements.
struct Piece {
    int tensor;        // >= 0: all of them lie in this tensor; -1: a tensor boundary (or the end of the
                       // data) falls inside; -2: all padding
    int dt;            // tensor >= 0: its gradient dtype
    int64_t toff;      // tensor >= 0: offset of the block's first element inside the tensor
    int seg;           // tensor == -1: index, in the table of non-empty tensors, of the one that
                       // holds the block's first element
};

// e0: the block's first element (< n, the launch's length).  The wave searches the offset table; where the
// plan has made a list or a table, nobody comes here.  Everything returned is wave-uniform.
__device__ __forceinline__ Piece piece_of(const TensorMap &tm, int64_t e0, int64_t n) {
    Piece pc;
    pc.tensor = -2;
    pc.dt = PARO_BF16;
    pc.toff = 0;
    pc.seg = 0;
    const int64_t f0 = tm.begin + e0;
    if (f0 >= tm.total) return pc;                                    // padding
    const int k = uniform(wave_search(tm.nz_off, tm.n_nz + 1, f0, (int)lane_id()));
    const int64_t piece_end = tm.begin + min(e0 + (int64_t)PIECE, n);
    if (tm.nz_off[k + 1] >= piece_end) {
        pc.tensor = tm.nz_tensor[k];
        pc.dt = tm.dtype[pc.tensor];
        pc.toff = f0 - tm.nz_off[k];
    } else {
        pc.tensor = -1;
        pc.seg = k;
    }
    return pc;
}

// For a block with a boundary inside: tensor (-1 = padding), gradient dtype and offset inside the
// tensor of each of the thread's 4 elements.  EVERY lane of the wave must call this (lanes past the
// end of the launch included): the search runs across the lanes' registers.
//   f0: flat index of the block's first element, which lies in segment seg (nz_off[seg] <= f0);
//   x0: position of the thread's first element inside the block (4 * lane).
// Lane l fetches the l-th segment start after seg, as a position relative to the block (PIECE or
// more = beyond the block): one load per lane instead of a binary search through memory per lane.
// An element's segment is seg + the number of those starts at or before it, found by a binary
// search over the 64 lanes' values with shuffles.  Only a block with more than 64 starts inside
// (tensors of 1-3 elements in a row) walks the table in memory instead.
struct Located {
    int tens[4];
    int dt[4];
    int64_t toff[4];
};
__device__ __forceinline__ void locate4(const TensorMap &tm, int seg, int64_t f0, int x0, Located &loc) {
    const int lane = (int)lane_id();
    const int idx = seg + 1 + lane;                                    // nz_off[n_nz] = Psi: where padding starts
    int R = PIECE;
    if (idx <= tm.n_nz) R = (int)min(tm.nz_off[idx] - f0, (int64_t)PIECE);
    const int64_t first_start = tm.nz_off[seg];                        // wave-uniform: a scalar load
    if (uniform(__shfl(R, WAVE - 1, WAVE)) >= PIECE) {                 // the 64 starts cover the block
        int lo = 0, hi = WAVE - 1;                                     // starts at or before x0: a number in [lo, hi]
#pragma unroll                                                         // (not 64: lane 63's start lies beyond the block)
        for (int it = 0; it < 6; ++it) {                               // 64 candidates -> 1
            const int mid = (lo + hi) >> 1;
            const int r = __shfl(R, mid, WAVE);
            if (r <= x0) lo = mid + 1; else hi = mid;
        }
        int c = lo;                                                    // < 64: the last start lies beyond the block
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i > 0 && __shfl(R, c, WAVE) <= x0 + i) ++c;            // starts are distinct: at most one step
            const int before = __shfl(R, max(c - 1, 0), WAVE);         // start of the element's segment, if c > 0
            const int s = seg + c;
            loc.toff[i] = c == 0 ? f0 + x0 + i - first_start : (int64_t)(x0 + i - before);
            if (s < tm.n_nz) {
                loc.tens[i] = tm.nz_tensor[s];
                loc.dt[i] = tm.nz_dtype[s];
            } else {
                loc.tens[i] = -1;
                loc.dt[i] = PARO_BF16;
                loc.toff[i] = 0;
            }
        }
        return;
    }
    // more than 64 segment starts inside the block: per-lane search through the table
    const int64_t f = f0 + x0;
    int lo = seg, hi = min(seg + PIECE + 1, tm.n_nz + 1);             // nz_off[lo] <= f; nz_off[n_nz] = Psi
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tm.nz_off[mid] <= f) lo = mid; else hi = mid;
    }
    int c = lo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (c < tm.n_nz && tm.nz_off[c + 1] <= f + i) ++c;            // at most one step per element
        if (c < tm.n_nz) {
            loc.tens[i] = tm.nz_tensor[c];
            loc.dt[i] = tm.nz_dtype[c];
            loc.toff[i] = f + i - tm.nz_off[c];
        } else {
            loc.tens[i] = -1;
            loc.dt[i] = PARO_BF16;
            loc.toff[i] = 0;
        }
    }
}

// Contributions are per-tensor gradients (source k is a device array of T pointers) and the
// block's elements lie in one tensor: one vector load fetches the thread's 4 values, as in the chunk
// layout, wherever the tensor's data start (the hardware takes vector loads at any address; a branch
// on the alignment, source by source, costs more than the misaligned load does).

// Address of the tensor's data in contribution k (wave-uniform).
template <class Src>
__device__ __forceinline__ uintptr_t tensor_base(const Src &src, int k, int tensor) {
    return global_ptr<uintptr_t>(reinterpret_cast<uintptr_t>(src.p[k]))[tensor];
}

// NT: streaming loads, for blocks that start on a cache line (a Llama-like list, P = 16, 26 M elements: 313
// us a clipped step against 325 with plain loads); a line shared with the next block is better kept (160 000
// ragged tensors, P = 8, single sweep: 922 us against 1055).
template <int DT, bool NT, int KB = PARO_BATCH>
struct Tensor4Loader {
    static constexpr int kBatch = (DT == PARO_F32 && KB > 8) ? KB / 2 : KB;     // 32 registers of loads in flight at most
    static constexpr int kElems = 4;
    static constexpr int kPace = 0;
    static constexpr int ESIZE = DT == PARO_F32 ? 4 : 2;
    using Raw = typename Chunk4Loader<DT>::Raw;
    using At = uintptr_t;
    int tensor;
    int64_t piece_byte_off;    // of the block's first element inside the tensor
    template <class Src>
    __device__ __forceinline__ At source(const Src &src, int k) const { return tensor_base(src, k, tensor); }
    __device__ __forceinline__ void load(At at, Raw &r) const {
        const uintptr_t mine = at + (uintptr_t)piece_byte_off + (uintptr_t)lane_id() * (4 * ESIZE);
        r = ld_any<Raw, NT>(mine);
    }
    __device__ __forceinline__ void unpack(const Raw &r, float x[4]) const { Chunk4Loader<DT>::to_f32(r, x); }
};

// A part of a block: the elements of [lo, hi) lie in one tensor, found like a whole block's; a thread
// with all of its 4 elements inside loads them as above, at the part's ends element by element.
template <int DT>
struct Part4Loader {
    static constexpr int kBatch = 4;              // more costs every wave of the kernel registers
    static constexpr int kElems = 4;
    static constexpr int kPace = 0;
    static constexpr int ESIZE = DT == PARO_F32 ? 4 : 2;
    struct Raw { unsigned int w[4]; };
    using At = uintptr_t;
    int tensor;
    int64_t piece_byte_off;    // of the block's first element inside the tensor (may be negative: it is not loaded)
    int a, b;                  // the thread's elements [a, b) of its 4 belong to the part
    template <class Src>
    __device__ __forceinline__ At source(const Src &src, int k) const { return tensor_base(src, k, tensor); }
    __device__ __forceinline__ bool whole() const { return a == 0 && b == 4; }
    __device__ __forceinline__ void load(At at, Raw &r) const {
        const uintptr_t mine = at + (uintptr_t)piece_byte_off + (uintptr_t)lane_id() * (4 * ESIZE);
        if (whole()) {
            using V = typename Chunk4Loader<DT>::Raw;
            const V v = ld_any<V, false>(mine);
            r.w[0] = v.x; r.w[1] = v.y;
            if constexpr (DT == PARO_F32) { r.w[2] = v.z; r.w[3] = v.w; }
        } else {
            using E = std::conditional_t<DT == PARO_F32, unsigned int, uint16_t>;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (i >= a && i < b) r.w[i] = global_ptr<E>(mine)[i];
        }
    }
    __device__ __forceinline__ void unpack(const Raw &r, float x[4]) const {
        if constexpr (DT == PARO_F32) {
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(r.w[i]);
        } else {
            const bool pairs = whole();
            x[0] = cvt_lo<DT>(r.w[0]);
            x[1] = pairs ? cvt_hi<DT>(r.w[0]) : cvt_lo<DT>(r.w[1]);
            x[2] = pairs ? cvt_lo<DT>(r.w[1]) : cvt_lo<DT>(r.w[2]);
            x[3] = pairs ? cvt_hi<DT>(r.w[1]) : cvt_lo<DT>(r.w[3]);
        }
    }
};

// Two consecutive blocks inside one tensor, folded by one wave (sweep 1 with few contributions: the wave
// then has twice the loads in flight, and one look-up serves 512 elements).
// The thread's elements 0-3 lie in the first block, 4-7 in the second, 256 elements further on.
template <int DT, bool NT, int KB>
struct Tensor8Loader {
    static constexpr int kBatch = KB;
    static constexpr int kElems = 8;
    static constexpr int kPace = 0;
    static constexpr int ESIZE = DT == PARO_F32 ? 4 : 2;
    using Raw4 = typename Chunk4Loader<DT>::Raw;
    struct Raw { Raw4 a, b; };
    using At = uintptr_t;
    int tensor;
    int64_t piece_byte_off;    // of the first block's first element inside the tensor
    template <class Src>
    __device__ __forceinline__ At source(const Src &src, int k) const { return tensor_base(src, k, tensor); }
    __device__ __forceinline__ void load(At at, Raw &r) const {
        const uintptr_t mine = at + (uintptr_t)piece_byte_off + (uintptr_t)lane_id() * (4 * ESIZE);
        r.a = ld_any<Raw4, NT>(mine);
        r.b = ld_any<Raw4, NT>(mine + (uintptr_t)PIECE * ESIZE);
    }
    __device__ __forceinline__ void unpack(const Raw &r, float x[8]) const {
        Chunk4Loader<DT>::to_f32(r.a, x);
        Chunk4Loader<DT>::to_f32(r.b, x + 4);
    }
};

// ... and a tensor boundary (or the end of the data) falls inside the block: every element has
// its own tensor, dtype and offset; element loads.  Padding contributes +0.
struct Lane4Loader {
    static constexpr int kBatch = PARO_LANE_BATCH;
    static constexpr int kElems = 4;
    static constexpr int kPace = 0;
    struct Raw { unsigned int bits[4]; };
    struct At { uintptr_t base[4]; };
    Located at;
    template <class Src>
    __device__ __forceinline__ At source(const Src &src, int k) const {
        const auto *ptrs = global_ptr<uintptr_t>(reinterpret_cast<uintptr_t>(src.p[k]));
        At a;
#pragma unroll
        for (int i = 0; i < 4; ++i) a.base[i] = ptrs[max(at.tens[i], 0)];      // padding: any entry, never followed
        return a;
    }
    __device__ __forceinline__ void load(const At &a, Raw &r) const {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r.bits[i] = 0u;
            if (at.tens[i] >= 0) {
                if (at.dt[i] != PARO_F32)
                    r.bits[i] = global_ptr<uint16_t>(a.base[i])[at.toff[i]];
                else
                    r.bits[i] = global_ptr<unsigned int>(a.base[i])[at.toff[i]];
            }
        }
    }
    __device__ __forceinline__ void unpack(const Raw &r, float x[4]) const {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            x[i] = at.tens[i] < 0 ? 0.0f
                                  : at.dt[i] != PARO_F32 ? cvt16(r.bits[i], at.dt[i]) : __uint_as_float(r.bits[i]);
    }
};

// ---------------------------------------------------------------------- fold
// X[i] = contributions added in table order: runs of group_len into a partial A
// (left to right), partials into X (left to right).  The first value of a run
// and the first partial are copied, not added to zero (that would lose -0).
// A thread folds Ld::kElems elements (4, or 8 when the wave takes two blocks).
// ord: which pointer of the table the k-th contribution is (InOrder: the k-th).
struct InOrder {
    __device__ __forceinline__ int next(int k) { return k; }
};

template <class Ld>
struct Folding {
    static constexpr int NE = Ld::kElems;
    float A[NE];
    int pos = 0;
    bool first_group = true;
};

// N contributions, from the k-th on: all sources, then all loads - straight-line code.  A large launch
// over the chunk layout is paced: with all its loads issued at once a wave touches P DRAM pages in one go;
// with a pause after each, waves that start together read the same contribution together.  Whole clipped
// steps unpaced -> paced, on the same buffers: P = 64, 90 M elements 2446 -> 2373 us, P = 16, 150 M 1544 -> 1521,
// P = 4, 150 M as they were; single sweep, P = 64, 16 M 418 -> 409, P = 16, 24 M 224 -> 223, P = 8, 16 M 109 -> 109.  A
// small launch is bound by latency (P = 16, 2 M 26.5 -> 28.5; P = 32, 2 M, single sweep 29 -> 32) and is not paced.
// How long a pause goes with how many waves is in fold_budget.  The pause is a constant of the kernel and the branch is
// taken load by load: a pause that the launch chooses (a loop of short ones, two or three tests, copies of the code behind one
// branch) costs the scalar work of choosing after every load and was 2 to 12 % slower at the same length.
template <int N, class Ld, class Src, class Order>
__device__ __forceinline__ void load_batch(const Ld &ld, const Src &src, int k, Order &ord, typename Ld::Raw *raw) {
    typename Ld::At at[N];
    static_for<0, N>([&](auto b) { at[b] = ld.source(src, ord.next(k + b)); });
    static_for<0, N>([&](auto b) {
        ld.load(at[b], raw[b]);
        if constexpr (Ld::kPace > 0) {
            if (src.paced) __builtin_amdgcn_s_sleep(Ld::kPace);
        }
    });
}
template <int N, class Ld>
__device__ __forceinline__ void add_batch(const Ld &ld, const typename Ld::Raw *raw, int group_len, Folding<Ld> &f, float *X) {
    constexpr int NE = Ld::kElems;
    static_for<0, N>([&](auto b) {
        float x[NE];
        ld.unpack(raw[b], x);
        if (f.pos == 0) {
#pragma unroll
            for (int i = 0; i < NE; ++i) f.A[i] = x[i];
        } else {
#pragma unroll
            for (int i = 0; i < NE; ++i) f.A[i] = f.A[i] + x[i];
        }
        if (++f.pos == group_len) {
            f.pos = 0;
            if (f.first_group) {
#pragma unroll
                for (int i = 0; i < NE; ++i) X[i] = f.A[i];
                f.first_group = false;
            } else {
#pragma unroll
                for (int i = 0; i < NE; ++i) X[i] = X[i] + f.A[i];
            }
        }
    });
}

// Whole batches, then what is left as batches of 8, 4, 2 and 1 (their loads are all issued before the
// first is consumed).
template <class Ld, class Src, class Order = InOrder>
__device__ __forceinline__ void fold4(const Ld &ld, const Src &src, int P, int group_len, float *X,
                                      Order ord = Order()) {
    constexpr int B = Ld::kBatch;
    static_assert(B == 16 || B == 8 || B == 4 || B == 2, "the rest is split into powers of two");
    Folding<Ld> f;
    int k = 0;
    for (; k + B <= P; k += B) {
        typename Ld::Raw raw[B];
        load_batch<B>(ld, src, k, ord, raw);
        add_batch<B>(ld, raw, group_len, f, X);
    }
    const int rest = P - k;
    if (rest == 0) return;
    typename Ld::Raw r8[8], r4[4], r2[2], r1[1];
    if constexpr (B > 8) {
        if (rest & 8) load_batch<8>(ld, src, k, ord, r8), k += 8;
    }
    if constexpr (B > 4) {
        if (rest & 4) load_batch<4>(ld, src, k, ord, r4), k += 4;
    }
    if constexpr (B > 2) {
        if (rest & 2) load_batch<2>(ld, src, k, ord, r2), k += 2;
    }
    if (rest & 1) load_batch<1>(ld, src, k, ord, r1);
    if constexpr (B > 8) {
        if (rest & 8) add_batch<8>(ld, r8, group_len, f, X);
    }
    if constexpr (B > 4) {
        if (rest & 4) add_batch<4>(ld, r4, group_len, f, X);
    }
    if constexpr (B > 2) {
        if (rest & 2) add_batch<2>(ld, r2, group_len, f, X);
    }
    if (rest & 1) add_batch<1>(ld, r1, group_len, f, X);
}

// Fold order of a chunk, walked inside the kernel: the pointer table is in rank order, and the
// walk starts at the successor of the chunk's owner - the next local index of the next group -
// goes round the group, then on to the next group (a plain ring: one group of P ranks).
struct RingWalk {
    int G, g, grp, loc, left;          // ranks per group, groups, current group, local index, ranks left in the group
    __device__ __forceinline__ int next(int) {
        const int r = grp * G + loc;
        if (++loc == G) loc = 0;
        if (--left == 0) {
            left = G;
            if (++grp == g) grp = 0;
        }
        return r;
    }
};

// What a launch over several chunks of an update range needs to find an element's chunk and the
// chunk's fold order.
struct RangeMap {
    int64_t L;            // elements of a chunk (a multiple of 8: a thread's 4 elements share their chunk)
    double inv_L;
    int first_chunk;      // the chunk that the range starts with
    int G, g;             // the plan's groups; chunk c belongs to rank (group c % g, local index c / g)
    int walk_G, walk_g;   // the fold's groups: the plan's, or one group of P ranks (ring)
    int own;              // the chunk, counted from first_chunk, whose squares are added up; -1: every chunk
};

// Chunk (counted from the range's first) that element e of the range lies in.  One product in
// fp64 is off by at most one from the quotient below 2^53.
__device__ __forceinline__ int chunk_at(const RangeMap &rm, int64_t e) {
    int c = (int)((double)e * rm.inv_L);
    if ((int64_t)c * rm.L > e) --c;
    if ((int64_t)(c + 1) * rm.L <= e) ++c;
    return uniform(c);
}

__device__ __forceinline__ RingWalk walk_of(const RangeMap &rm, int c) {
    c += rm.first_chunk;
    const int oi = c / rm.g, oj = c - oi * rm.g;                     // the owner's local index and group
    RingWalk w{rm.walk_G, rm.walk_g, 0, 0, rm.walk_G};
    if (rm.walk_g == 1) {
        w.loc = oj * rm.G + oi + 1;
    } else {
        w.loc = oi + 1;
        w.grp = oj + 1 == rm.g ? 0 : oj + 1;
    }
    if (w.loc == w.G) w.loc = 0;
    return w;
}

// The ordered fold of the thread's 4 elements of an update range of several chunks (arrays in shard
// coordinates): e0 the block's first element, n the range's length.  Nearly every block lies inside
// one chunk; where chunks meet inside a block, its lanes take turns, chunk by chunk.  Returns
// whether the thread's elements count for the sum of squares.
template <int DT, int PACE = PARO_PACE_SLEEP, class Src>
__device__ __forceinline__ bool fold_range(const RangeMap &rm, const Src &src, int P, int64_t e0, int64_t n, float X[4]) {
    Chunk4Loader<DT, PACE> ld{e0 + lane_id() * EPT};
    const int64_t end = min(e0 + (int64_t)PIECE, n);
    bool counts = false;
    int c = chunk_at(rm, e0);
#pragma unroll 1
    for (;; ++c) {
        const int64_t c_lo = (int64_t)c * rm.L, c_hi = c_lo + rm.L;
        if (ld.e >= c_lo && ld.e < min(c_hi, n)) {
            fold4(ld, src, P, rm.walk_G, X, walk_of(rm, c));
            counts = rm.own < 0 || rm.own == c;
        }
        if (c_hi >= end) return counts;
    }
}

// The ordered fold of the thread's 4 elements out of per-tensor gradients, for a block that is
// not all padding.  loc: from locate4 when the block holds a boundary (pc.tensor == -1).
// KB: contributions loaded before the first is consumed (a kernel that is only launched for few
// contributions says so, and saves the registers).
template <bool NT, int KB = PARO_BATCH, class Src>
__device__ __forceinline__ void fold_tensors(const Piece &pc, const Located &loc, const Src &src, int P,
                                             int group_len, float X[4]) {
    if (pc.tensor >= 0) {
        if (pc.dt == PARO_BF16) {
            Tensor4Loader<PARO_BF16, NT, KB> ld{pc.tensor, pc.toff * 2};
            fold4(ld, src, P, group_len, X);
        } else if (pc.dt == PARO_F16) {
            Tensor4Loader<PARO_F16, NT, KB> ld{pc.tensor, pc.toff * 2};
            fold4(ld, src, P, group_len, X);
        } else {
            Tensor4Loader<PARO_F32, NT, KB> ld{pc.tensor, pc.toff * 4};
            fold4(ld, src, P, group_len, X);
        }
    } else {
        Lane4Loader ld{loc};
        fold4(ld, src, P, group_len, X);
    }
}

// ... of the thread's 8 elements in two consecutive blocks that lie in one tensor (pc: the first).
template <bool NT, int KB, class Src>
__device__ __forceinline__ void fold_tensor_pair(const Piece &pc, const Src &src, int P, int group_len, float X[8]) {
    if (pc.dt == PARO_BF16) {
        Tensor8Loader<PARO_BF16, NT, KB> ld{pc.tensor, pc.toff * 2};
        fold4(ld, src, P, group_len, X);
    } else if (pc.dt == PARO_F16) {
        Tensor8Loader<PARO_F16, NT, KB> ld{pc.tensor, pc.toff * 2};
        fold4(ld, src, P, group_len, X);
    } else {
        Tensor8Loader<PARO_F32, NT, KB> ld{pc.tensor, pc.toff * 4};
        fold4(ld, src, P, group_len, X);
    }
}

// One piece of a launch's list, as the wave that takes it sees it.
struct Cut {
    Piece pc;
    int64_t e0;        // first element of the piece's block, in the launch (n or more: nothing to do)
    int a, b;          // the thread's elements [a, b) of its 4 belong to the piece (ends of the launch apart)
    bool whole;        // the piece is its whole block
};

// The i-th piece; without a list the i-th block.  Everything but a and b is wave-uniform.
__device__ __forceinline__ Cut cut_of(const TensorMap &tm, int64_t i, int64_t n) {
    Cut c;
    c.a = 0;
    c.b = EPT;
    c.whole = true;
    c.e0 = i * PIECE;
    if (!tm.pieces) {
        if (c.e0 < n) c.pc = piece_of(tm, c.e0, n);
        return c;
    }
    c.e0 = n;
    if (i >= tm.n_pieces) return c;
    const paro_piece_info info = tm.pieces[i];                                // one address for the whole wave
    const int64_t w = uniform(info.where);
    const int lo = (int)(w & 255), hi = (int)(w >> 8 & 511), x0 = (int)lane_id() * EPT;
    c.e0 = (int64_t)(unsigned)uniform((int)info.tile) * TILE;
    c.pc.tensor = uniform(info.tensor);
    c.pc.dt = (int)(w >> 17 & 3);
    c.pc.toff = w >> 19;
    c.pc.seg = (int)(w >> 19);
    c.whole = lo == 0 && hi == PIECE;
    if (!c.whole) {
        c.a = max(lo - x0, 0);
        c.b = min(hi - x0, EPT);
    }
    return c;
}

// Whether the i-th and the next piece (without a list: block) are whole consecutive blocks inside one tensor;
// *pc: the first.  A piece that ends before its block does says so: two whole ones lie inside the launch but
// for the last block of the chunk, which n tells apart.
__device__ __forceinline__ bool pair_of(const TensorMap &tm, int64_t i, int64_t n, Piece *pc, int64_t *e0) {
    if (!tm.pieces) {
        *e0 = i * PIECE;
        if (*e0 + 2 * PIECE > n) return false;
        *pc = piece_of(tm, *e0, n);
        return pc->tensor >= 0 && piece_of(tm, *e0 + PIECE, n).tensor == pc->tensor;
    }
    if (i + 1 >= tm.n_pieces) return false;
    const paro_piece_info x = tm.pieces[i], y = tm.pieces[i + 1];
    const int64_t w = uniform(x.where);
    const unsigned tile = (unsigned)uniform((int)x.tile);
    constexpr unsigned WHOLE = (unsigned)TILE << 8, ENDS = 0x1FFFF;
    pc->tensor = uniform(x.tensor);
    pc->dt = (int)(w >> 17 & 3);
    pc->toff = w >> 19;
    *e0 = (int64_t)tile * TILE;
    return pc->tensor >= 0 && uniform(y.tensor) == pc->tensor && (unsigned)uniform((int)y.tile) == tile + 1 &&
           ((unsigned)w & ENDS) == WHOLE && ((unsigned)uniform((int)y.where) & ENDS) == WHOLE && *e0 + 2 * PIECE <= n;
}

// The ordered fold of the thread's elements [a, b) of a piece that is part of its block.
template <class Src>
__device__ __forceinline__ void fold_part(const Cut &c, const Src &src, int P, int group_len, float X[4]) {
    if (c.pc.dt == PARO_BF16) {
        Part4Loader<PARO_BF16> ld{c.pc.tensor, c.pc.toff * 2, c.a, c.b};
        fold4(ld, src, P, group_len, X);
    } else if (c.pc.dt == PARO_F16) {
        Part4Loader<PARO_F16> ld{c.pc.tensor, c.pc.toff * 2, c.a, c.b};
        fold4(ld, src, P, group_len, X);
    } else {
        Part4Loader<PARO_F32> ld{c.pc.tensor, c.pc.toff * 4, c.a, c.b};
        fold4(ld, src, P, group_len, X);
    }
}

}  // namespace
