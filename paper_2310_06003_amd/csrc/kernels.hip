// Device side of libparo for gfx950 (MI355X): the streaming kernels of the
// Update stage (paper Sec. 3.2) and the entry points that launch them.
//
// Everything here is bound by HBM bandwidth: per shard parameter the method
// moves 2P bytes of bf16 contributions and 26-34 bytes of fp32 state, against
// P adds and ~20 flops.  So the kernels are plain sweeps with many independent
// loads in flight per thread; there is no dense contraction and hence no MFMA.
//
//   shape     every sweep runs in one-wave blocks (64 threads) of 256 consecutive
//             elements, 4 per thread: each load or store instruction of a wave
//             covers 512 B - 1 KB of consecutive addresses (whole cache lines), and
//             the many short-lived waves, dealt round-robin to the 8 XCDs in
//             address order, interleave reads and writes finely.  On MI355X this
//             beat 256-thread blocks of 8-element threads by 8-11 %, and those had
//             beaten persistent grid-stride blocks by 8-15 %.
//   occupancy the heavy sweeps ask for unused dynamic LDS so that only 8 to 25 waves
//             run per compute unit, by kernel and number of ranks: fewer requests
//             outstanding fight less over DRAM pages (another 3-6 %).  The tensor layout over many small
//             tensors wants the opposite - its waves wait on look-ups with no
//             data in flight - and gets every wave the registers allow.
//   caches    nearly everything is touched once: streaming (non-temporal) loads; stores
//             through per-wave buffer descriptors, which let the instruction say
//             "streaming, system scope" (nt sc1: 2 % better than nt alone).
//   fold      the P contributions of an element are added in a fixed order
//             (never re-associated, never contracted into FMAs) so the result
//             is bit-identical to a reduce-scatter ring run in that order
//   norm      squares are exact in fp64; per-thread fp64 sums -> sum over the
//             wave -> one partial per block -> added in a fixed order, by a small
//             kernel, by sweep 2's waves, or both.  No atomics: run-to-run identical.
//   tensors   the tensor layout needs the tensor an element belongs to: a list of
//             pieces (built once per chunk), each inside one tensor, answers with
//             a single look-up; a block of very many tensors finds its elements'
//             tensors with one load per lane and a search across the lanes'
//             registers.  The weight-decay mask has a per-block table.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <cstdlib>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "plan.hpp"

#include "device_util.hpp"
#include "loaders.hpp"

namespace {

// ---------------------------------------------------------------------- Adam
// sums[k0] + sums[k0 + STRIDE] + ... up to sums[n - 1], in that order; U loads in flight at a time.
template <int STRIDE, int U>
__device__ __forceinline__ double strided_sum(const double *__restrict__ sums, int k0, int n) {
    double acc = 0.0;
    for (; k0 < n; k0 += U * STRIDE) {
        double x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) x[u] = (k0 + u * STRIDE < n) ? sums[k0 + u * STRIDE] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) acc += x[u];
    }
    return acc;
}

// The global sum of squares as sweep 2 gets it: n sums to be added up in a fixed order, the same in every wave.
// Lanes hold the result.  MANY: more than NORM_SLICES, up to NORM_DIRECT_PARTIALS of them.  fetch() issues the vector loads of
// many: before a wave's state, because loads return in the order of their issue, and sums behind the state would be waited for
// together with it, with their adds to come (whole clipped steps, same buffers: P = 8, 0.5 M elements 10.0 -> 9.4 us, 0.375 M 8.4 -> 8.1;
// P = 4, 0.5 M 9.5 -> 9.0).  Their registers (82 against 32) cost a sweep 2 with few 1 to 2 %: a kernel of its own.  Few are one scalar load, on
// a way of its own (there is room for as many).  One kernel for both took 39; why GPT-2's tensors at P = 16, which leave few sums,
// went from 85.8 to 82.0 us when it was parted is not known.
template <bool MANY>
struct NormTotal {
    static constexpr int U = MANY ? NORM_DIRECT_PARTIALS / WAVE : 1, ROUND = 8;
    double x[U];
    __device__ __forceinline__ void fetch(const double *__restrict__ sums, int n) {
        if constexpr (MANY) {
#pragma unroll
            for (int u0 = 0; u0 < U; u0 += ROUND) {
                if (u0 * WAVE >= n) break;
#pragma unroll
                for (int u = u0; u < u0 + ROUND; ++u) {
                    const int k = (int)lane_id() + u * WAVE;
                    x[u] = k < n ? sums[k] : 0.0;
                }
            }
        }
    }
    __device__ __forceinline__ double total(const double *__restrict__ sums, int n) const {
        if constexpr (MANY) {
            double acc = 0.0;
#pragma unroll
            for (int u0 = 0; u0 < U; u0 += ROUND) {
                if (u0 * WAVE >= n) break;
#pragma unroll
                for (int u = u0; u < u0 + ROUND; ++u) acc += x[u];
            }
            return wave_sum(acc);
        }
        if (n == 1) return sums[0];
        double y[NORM_SLICES];
#pragma unroll
        for (int k = 0; k < NORM_SLICES; ++k) y[k] = sums[k];
        double s = y[0];
        if (n == NORM_SLICES) {
#pragma unroll
            for (int k = 1; k < NORM_SLICES; ++k) s += y[k];
        } else {
#pragma unroll
            for (int k = 1; k < NORM_SLICES; ++k) s += k < n ? y[k] : 0.0;
        }
        return s;
    }
};

// sc = grad_scale * clip coefficient, from the global sum of squares.
__device__ __forceinline__ float scale_from_norm(const AdamConsts &a, double total_sumsq) {
    double coef = 1.0;
    if (a.max_norm > 0.0f) {
        const double norm = (double)a.grad_scale * sqrt(total_sumsq);
        const double c = (double)a.max_norm / (norm + 1e-6);
        coef = c < 1.0 ? c : 1.0;
    }
    return (float)((double)a.grad_scale * coef);
}

// One element.  Every operation is a separate fp32 rounding, in this order
// (the library is compiled without FMA contraction).
__device__ __forceinline__ void adam1(const AdamConsts &a, float sc, bool decays, float g, float &p, float &m,
                                      float &v) {
    float gh = sc * g;
    if (!a.adamw && decays) gh = gh + a.wd * p;
    const float t1 = a.beta1 * m, t2 = a.omb1 * gh;
    m = t1 + t2;
    const float t3 = a.beta2 * v, t4 = gh * gh;
    const float t5 = a.omb2 * t4;
    v = t3 + t5;
    float den = sqrtf(v) / a.sqrt_bc2;
    den = den + a.eps;
    const float q = m / den;
    const float upd = a.step_size * q;
    if (a.adamw && decays) {
        const float pd = p * a.decay;
        p = pd - upd;
    } else {
        p = p - upd;
    }
}

struct State4 { u32x4 p, m, v; };

// elements of the block at e0 that lie inside a launch of n elements
__device__ __forceinline__ unsigned piece_elems(int64_t e0, int64_t n) {
    return (unsigned)min((int64_t)PIECE, n - e0);
}

__device__ __forceinline__ State4 load_state4(const float *p, const float *m, const float *v, int64_t e) {
    State4 s;
    s.p = ld_nt(reinterpret_cast<const u32x4 *>(p + e));
    s.m = ld_nt(reinterpret_cast<const u32x4 *>(m + e));
    s.v = ld_nt(reinterpret_cast<const u32x4 *>(v + e));
    return s;
}

// Adam on the thread's 4 elements; state and (optionally) the low-precision copy written back.
// PART: only elements [lo, hi) of the 4 are the thread's (the others are some other wave's).
// HELD: the results wait for the chip's next write window (see holds_back).
template <bool PACK, bool PART = false, bool HELD = false>
__device__ __forceinline__ void update4(const AdamConsts &a, float sc, const bool decays[4], const float gg[4],
                                        const State4 &s, float *p, float *m, float *v, uint16_t *dst, int64_t e0,
                                        unsigned elems, int lo = 0, int hi = EPT, const WriteWindow &window = WriteWindow()) {
    float pp[4] = {__uint_as_float(s.p.x), __uint_as_float(s.p.y), __uint_as_float(s.p.z), __uint_as_float(s.p.w)},
          mm[4] = {__uint_as_float(s.m.x), __uint_as_float(s.m.y), __uint_as_float(s.m.z), __uint_as_float(s.m.w)},
          vv[4] = {__uint_as_float(s.v.x), __uint_as_float(s.v.y), __uint_as_float(s.v.z), __uint_as_float(s.v.w)};
#pragma unroll
    for (int i = 0; i < 4; ++i) adam1(a, sc, decays[i], gg[i], pp[i], mm[i], vv[i]);
    if constexpr (HELD) {
        is_formed(pp);
        is_formed(mm);
        is_formed(vv);
        if (has_followers(window)) wait_for_window(window);
    }
    if (PART && (lo > 0 || hi < 4)) {
        const int64_t e = e0 + lane_id() * EPT;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i >= lo && i < hi) {
                p[e + i] = pp[i];
                m[e + i] = mm[i];
                v[e + i] = vv[i];
                if (PACK) dst[e + i] = (uint16_t)pack2_lowp(pp[i], 0.0f, a.pack_dtype);
            }
        }
        return;
    }
    const auto store = [&](auto pol) {
        constexpr int ST = decltype(pol)::value;
        buf_store16<ST>(as_u32x4(pp[0], pp[1], pp[2], pp[3]), wave_buffer(p + e0, elems * 4), lane_id() * 16);
        buf_store16<ST>(as_u32x4(mm[0], mm[1], mm[2], mm[3]), wave_buffer(m + e0, elems * 4), lane_id() * 16);
        buf_store16<ST>(as_u32x4(vv[0], vv[1], vv[2], vv[3]), wave_buffer(v + e0, elems * 4), lane_id() * 16);
        if (PACK) {
            const u32x2 w = {pack2_lowp(pp[0], pp[1], a.pack_dtype), pack2_lowp(pp[2], pp[3], a.pack_dtype)};
            buf_store8<ST>(w, wave_buffer(dst + e0, elems * 2), lane_id() * 8);
        }
    };
    if (a.keep_state) store(std::integral_constant<int, PARO_POL_KEEP_ST>{});
    else store(std::integral_constant<int, PARO_POL_STREAM_ST>{});
}

// How a kernel knows which elements are exempt from weight decay: none are; from the chunk's weight-decay table; from
// the tensors that the elements lie in.
enum { MASK_NONE = 0, MASK_TABLE = 1, MASK_TENSORS = 2 };

// Which of the thread's 4 elements take weight decay, by the block's entry of the table.
__device__ __forceinline__ void decay_flags(const uint32_t *tab, uint32_t entry, bool decays[4]) {
    uint32_t bits = entry == DECAY_ALL ? 15u : 0u;
    if (entry >= DECAY_BITS) bits = tab[entry - DECAY_BITS + lane_id() / 8] >> lane_id() % 8 * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) decays[i] = bits >> i & 1;
}

// ... by their tensors (padding does, and stays 0).  loc: from locate4 when the block holds a boundary.
__device__ __forceinline__ void decay_flags(const TensorMap &tm, const Piece &pc, const Located &loc, bool decays[4]) {
    if (pc.tensor != -1) {
        const bool d = pc.tensor < 0 || tm.no_decay[pc.tensor] == 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) decays[i] = d;
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) decays[i] = loc.tens[i] < 0 || tm.no_decay[loc.tens[i]] == 0;
    }
}

// The thread's first element; n (the launch's length) is a multiple of 8, so a thread's 4
// elements are all inside the range or all outside.
__device__ __forceinline__ int64_t block_first() { return (int64_t)blockIdx.x * PIECE; }

// Where a block of sweep 1 puts its partial sum.  Blocks are dealt round-robin to the 8 XCDs, each
// with an L2 of its own: giving every XCD its own run of slots lets each L2 collect whole lines of
// partials before writing them back (slot = blockIdx would make every line a patchwork of 8-byte
// writes from 8 caches).  The grid of such a launch is a multiple of 8.
__device__ __forceinline__ unsigned partial_slot() { return (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3); }

__device__ __forceinline__ double sumsq4(const float X[4]) {
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc += (double)X[i] * (double)X[i];
    return acc;
}

// --------------------------------------------------------------------- kernels
// Order of their arguments: the first 14 words are in scalar registers when a wave starts (a flag of the build), as long
// as they are plain values and pointers; a structure ends the row.  So what the first loads need comes first, tables and constants
// behind it.  A wave used to begin with two or three trips to the scalar cache, one after the other, with no data in flight:
// whole steps on the same buffers, P = 8, clipped, 0.5 M elements 9.2 -> 8.9 us, 1.5 M 17.7 -> 17.0, 7.5 M 61.4 -> 60.4; 10 000 ragged
// tensors 68.0 -> 67.1; GPT-2 tensors, P = 64, 64.8 -> 63.8; all-gather of GPT-2 608 -> 592; from 100 M elements on as before.

__device__ __forceinline__ void store_g4(bool keep, float *g, int64_t e0, unsigned elems, const float X[4]) {
    buf_store16_as(keep, as_u32x4(X[0], X[1], X[2], X[3]), wave_buffer(g + e0, elems * 4), lane_id() * 16);
}

// Sweep 1, chunk layout: g = fold of the contributions; optional per-block partial of sum g^2.  The chunk is
// elements [lo, hi) of the update range; blocks are counted from the start of the range (see k_reduce4r), and
// one that two chunks share is launched for both.  HELD: results wait for the chip's next write window (see holds_back).
template <int DT, bool SUMSQ, int NSRC, bool HELD>
__global__ __launch_bounds__(WAVE) void k_reduce4(int64_t lo, int64_t hi, int P, int group_len, float *__restrict__ g,
                                                  double *__restrict__ partials, const SrcTableOf<NSRC, HELD> src) {
    const int64_t e0 = (lo & ~(int64_t)(PIECE - 1)) + block_first(), e = e0 + lane_id() * EPT;
    const bool inside = e >= lo && e < hi;
    float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    double acc = 0.0;
    if constexpr (HELD) leave_window(src.window);
    if (inside) {
        constexpr int WIDE = DT == PARO_F32 ? PARO_PACE_WIDE_F32_SLEEP : PARO_PACE_WIDE_SLEEP;
        Chunk4Loader<DT, (HELD ? PARO_WINDOW_PACE_SLEEP : NSRC > FEW_SRC ? WIDE : PARO_PACE_SLEEP)> ld{e};
        fold4(ld, src, P, group_len, X);
        if (!HELD) store_g4((unsigned)(e0 / PIECE) >= src.keep_from, g, e0, piece_elems(e0, hi), X);
        if (SUMSQ) acc = sumsq4(X);
    }
    if (SUMSQ) acc = wave_sum(acc);
    if constexpr (HELD) {
        is_formed(X);
        if (has_followers(src.window)) wait_for_window(src.window);
        if (inside) store_g4((unsigned)(e0 / PIECE) >= src.keep_from, g, e0, piece_elems(e0, hi), X);
    }
    if (SUMSQ && lane_id() == 0) partials[partial_slot()] = acc;
}

// Sweep 1, chunk layout, over blocks [block0, block0 + gridDim) of an update range of several chunks
// (optimizer state sharded inside the group only, or not at all): one launch, each chunk in its own
// fold order.  Blocks are cut from the start of the range, not of the chunk: a chunk is only a
// multiple of 8 elements, and blocks counted from its start would straddle cache lines in every array
// (MI355X, P = 16 fp32, chunks of 62.5 M elements: 5.1 TB/s there against 6.1).  Partial sums of blocks
// [part0, part0 + part_n) only (both multiples of 8, block0 too); the others hold no element that counts.
// The partials are laid out group by group (NORM_GROUP blocks), each like a launch of its own.
template <int DT, bool SUMSQ, int NSRC, bool HELD>
__global__ __launch_bounds__(WAVE) void k_reduce4r(int64_t block0, int64_t n, int P, unsigned part0, unsigned part_n,
                                                   float *__restrict__ g, double *__restrict__ partials, const RangeMap rm,
                                                   const SrcTableOf<NSRC, HELD> src) {
    const int64_t e0 = (block0 + blockIdx.x) * PIECE, e = e0 + lane_id() * EPT;
    if constexpr (HELD) leave_window(src.window);
    double acc = 0.0;
    if (e0 < n) {
        float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        const bool counts = fold_range<DT, HELD ? PARO_WINDOW_PACE_SLEEP : PARO_PACE_SLEEP>(rm, src, P, e0, n, X);
        if constexpr (HELD) {
            is_formed(X);
            if (has_followers(src.window)) wait_for_window(src.window);
        }
        if (e < n) {
            store_g4((unsigned)(e0 / PIECE) >= src.keep_from, g, e0, piece_elems(e0, n), X);
            if (SUMSQ && counts) acc = sumsq4(X);
        }
    }
    if (SUMSQ) {
        const unsigned b = blockIdx.x - part0;
        if (b < part_n) {
            const double s = wave_sum(acc);
            const unsigned group = b & ~(NORM_GROUP - 1), in_group = min(part_n - group, NORM_GROUP), k = b - group;
            if (lane_id() == 0) partials[group + (k & 7u) * (in_group >> 3) + (k >> 3)] = s;     // see partial_slot()
        }
    }
}

// Sweep 1, tensor layout: one piece of the launch.  Every lane of the wave takes part.
template <bool SUMSQ, int KB, bool NT, bool KEEP, class Src>
__device__ __forceinline__ void reduce_cut(const TensorMap &tm, const Cut &c, const Src &src, int P, int group_len,
                                           int64_t n, float *g, double &acc) {
    const int64_t e = c.e0 + lane_id() * EPT;
    float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};               // padding: the sum of zeros
    if (c.whole) {
        Located loc;
        if (c.pc.tensor == -1) locate4(tm, c.pc.seg, tm.begin + c.e0, lane_id() * EPT, loc);     // the whole wave
        if (e >= n) return;
        if (c.pc.tensor != -2) fold_tensors<NT, KB>(c.pc, loc, src, P, group_len, X);
        store_g4(KEEP, g, c.e0, piece_elems(c.e0, n), X);
        if (SUMSQ) acc += sumsq4(X);
    } else if (c.a < c.b) {
        if (c.pc.tensor != -2) fold_part(c, src, P, group_len, X);
        if (c.a == 0 && c.b == EPT) {
            store_g4(KEEP, g, c.e0, piece_elems(c.e0, n), X);
            if (SUMSQ) acc += sumsq4(X);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i >= c.a && i < c.b) {
                    g[e + i] = X[i];
                    if (SUMSQ) acc += (double)X[i] * (double)X[i];
                }
            }
        }
    }
}

// A wave takes PPW consecutive pieces.  PPW = 2 is for few contributions (P <= 4; P <= 6 over large chunks of
// many small tensors): where both are whole blocks that lie inside one tensor - the usual case - the wave folds
// them as one stream of 512 elements per contribution: one look-up and twice the bytes in flight per wave.
// Whole clipped steps, one and two blocks per wave: P = 2, 31 M elements of tensors of 1 to 65536: 216 and 205
// us; P = 4, 10 M elements of a Llama-like list 73.4 and 70.0 us; P = 5, 115 M of tensors of 1 to 65536 878 and
// 835, P = 6, 80 M 641 and 611, P = 7, 80 M with a quarter fp32 699 and 696; at P = 8 the other way round (69 M
// elements: 457 and 476 us).  The list must leave its blocks whole: cut ones part the pairs (P = 5, 115 M: 884).
// KB: contributions loaded before the first is consumed (8 when launched for P <= 8 only: fewer
// registers, more waves).  NT: the list's blocks start on cache lines.  KEEP: g is stored to stay in the memory-side
// cache (a branch on it in the kernel cost 12 scalar registers and, in a launch that streams or not, 2 % of a step).
// What bounds it: HBM, behind two dependent look-ups per wave (the piece, then the P pointers).  Taken one
// by one - pointer of the table, pointer of the tensor, a branch on its alignment, the load - the second
// was P round trips to the scalar cache in a row; now all pointers of a batch are fetched together and the
// loads are straight-line code.  Sweep 1 over 10 000 tensors of 1 to 65536 elements (P = 8, 174 MB): 49.8
// -> 35 us; GPT-2's 100 tensors (P = 8, 310 MB) 70 -> 57 us; the single sweep over 5 tensors at P = 32
// (290 MB): 113 -> 86 us.
template <bool SUMSQ, int PPW, int KB, bool NT, int NSRC, bool KEEP>
__global__ __launch_bounds__(WAVE) void k_reduce4t(int64_t n, const paro_piece_info *pieces, unsigned n_pieces, int P, int group_len,
                                                   float *__restrict__ g, double *__restrict__ partials,
                                                   const SrcTableOf<NSRC> src, TensorMap tm) {
    tm.pieces = pieces;
    tm.n_pieces = n_pieces;
    const int64_t i0 = (int64_t)blockIdx.x * PPW;
    double acc = 0.0;
    bool done = false;
    if constexpr (PPW == 2) {
        Piece pc;
        int64_t e0;
        if (pair_of(tm, i0, n, &pc, &e0)) {                  // two whole blocks inside one tensor
            float X[8];
            fold_tensor_pair<NT, KB>(pc, src, P, group_len, X);
            const wave_buf out = wave_buffer(g + e0, 2 * PIECE * 4);
            buf_store16_as(KEEP, as_u32x4(X[0], X[1], X[2], X[3]), out, lane_id() * 16);
            buf_store16_as(KEEP, as_u32x4(X[4], X[5], X[6], X[7]), out, PIECE * 4 + lane_id() * 16);
            if (SUMSQ) acc = sumsq4(X) + sumsq4(X + 4);
            done = true;
        }
    }
    if (!done) {                                             // piece by piece (one copy of the code: no unrolling)
#pragma unroll 1
        for (int j = 0; j < PPW; ++j) {
            const Cut c = cut_of(tm, i0 + j, n);
            if (c.e0 < n) reduce_cut<SUMSQ, KB, NT, KEEP>(tm, c, src, P, group_len, n, g, acc);
        }
    }
    if (SUMSQ) {
        const double s = wave_sum(acc);
        if (lane_id() == 0) partials[partial_slot()] = s;
    }
}

// Adds partials in a fixed order: block b takes the slice [b*chunk, b*chunk + chunk) of the n
// values; thread t adds its slice's elements t, t+T, t+2T, ... (eight loads in flight at a time,
// added in index order); then the fixed block tree.
__global__ __launch_bounds__(FINALIZE_TPB) void k_finalize(const double *__restrict__ partials, int n, int chunk,
                                                           double *out) {
    const int lo = blockIdx.x * chunk, hi = min(n, lo + chunk);
    const double s = block_sum(strided_sum<FINALIZE_TPB, 8>(partials, lo + threadIdx.x, hi));
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// What sweep 2's waves do with n sums, for the call that leaves the total itself: the same adds in the
// same order, so the same value to the last bit.
template <bool MANY>
__global__ __launch_bounds__(WAVE) void k_norm_total(const double *__restrict__ sums, int n, double *out) {
    NormTotal<MANY> norm;
    norm.fetch(sums, n);
    const double total = norm.total(sums, n);
    if (lane_id() == 0) *out = total;
}

// The NORM_SLICES slice sums of k_finalize and their total in one small launch: block_sum() of every slice -
// the same pairs of lanes at every step, the same order of waves - then the slices in order.  Eight separate
// sums across the lanes would be 48 steps a wave, 16 waves on one compute unit, and eight loops as many round
// trips to memory (together 4 us); here each of the first three steps also halves the slices that a lane carries: ten.
__global__ __launch_bounds__(FINALIZE_TPB) void k_norm_slices_total(const double *__restrict__ partials, int n, int chunk,
                                                                    double *out) {
    static_assert(NORM_SLICES == 8, "three halvings leave one slice to a lane");
    __shared__ double s_wave[NORM_SLICES][FINALIZE_TPB / WAVE + 1];     // + 1: the slices' rows start in different banks
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    constexpr int U = NORM_ONE_BLOCK_PARTIALS / NORM_SLICES / FINALIZE_TPB;
    double x[NORM_SLICES][U], acc[NORM_SLICES];
#pragma unroll
    for (int b = 0; b < NORM_SLICES; ++b)                   // all in flight
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (int)threadIdx.x + u * FINALIZE_TPB;
            x[b][u] = k < chunk && b * chunk + k < n ? partials[b * chunk + k] : 0.0;
        }
#pragma unroll
    for (int b = 0; b < NORM_SLICES; ++b) {
        acc[b] = x[b][0];
#pragma unroll
        for (int u = 1; u < U; ++u) acc[b] += x[b][u];
    }
    static_for<0, 3>([&](auto step) {
        constexpr int HALF = NORM_SLICES >> (step + 1), FAR = WAVE / 2 >> step;
        const bool upper = lane & FAR;                      // keeps the upper half of the slices, hands over the lower
#pragma unroll
        for (int b = 0; b < HALF; ++b) {
            const double keep = upper ? acc[b + HALF] : acc[b], give = upper ? acc[b] : acc[b + HALF];
            acc[b] = keep + __shfl_xor(give, FAR, WAVE);
        }
    });
    double s = acc[0];                                      // of slice lane / 8
    for (int d = WAVE / 16; d >= 1; d >>= 1) s += __shfl_xor(s, d, WAVE);
    if (lane % 8 == 0) s_wave[lane / 8][wave] = s;
    __syncthreads();
    if (wave == 0) {
        const double *of_slice = s_wave[lane & (NORM_SLICES - 1)];
        double r = of_slice[0];
#pragma unroll
        for (int w = 1; w < FINALIZE_TPB / WAVE; ++w) r += of_slice[w];
        double total = of_lane(r, 0);
#pragma unroll
        for (int b = 1; b < NORM_SLICES; ++b) total += of_lane(r, b);
        if (lane == 0) *out = total;
    }
}

// Sweep 2: Adam on the stored gradient, optionally packing the low-precision parameters.
// MASK: how it finds the elements exempt from weight decay.  The global sum of squares comes as n_sums sums
// (0: nobody needs it), which every wave adds up while its state is on its way; the first block writes
// the total to sumsq_out unless that is null.
// KEPT: the launch before this one stored all of the gradient to stay in the memory-side cache (see PARO_KEEP_G_ELEMS): plain loads.
// Otherwise the last blocks come first: it is the end of the gradient that the cache may hold (see PARO_KEEP_G_TAIL_ELEMS).  Not with a mask, where that costs
// paro_adam_shard alone up to 3 % and brings a whole step nothing (from the end and from the start: the call alone after its gradient was scaled in place and copied
// in, 6 M elements 31.9, 33.1 and 31.2, 32.4 us, on another GPU 33.6, 35.0 and 32.4, 34.2; 9 M 44.3, 44.6 and 43.6, 43.8; 30 M 134, 142 and 135, 141, there 137, 143
// and 135, 141; 200 M 906, 911 and 910, 915; clipped steps, P = 4, GPT-2's list 199 and 198, its tensors 198 and 197, P = 2 384 and 382; 8 chunks, P = 8, 973 and
// 977; Llama-like lists, P = 8, 42 M 312 and 312, P = 16, 84 M 830 and 828, 421 M 4200 and 4200).
template <bool PACK, int MASK, bool KEPT, bool MANY>
__global__ __launch_bounds__(WAVE) void k_adam4(int64_t n, const float *__restrict__ g, float *__restrict__ p, float *__restrict__ m,
                                                float *__restrict__ v, const double *__restrict__ sums, int n_sums, const AdamConsts a,
                                                uint16_t *__restrict__ dst, double *__restrict__ sumsq_out, const TensorMap tm) {
    const unsigned block = KEPT || MASK != MASK_NONE ? blockIdx.x : (unsigned)((n - 1) / PIECE) - blockIdx.x;
    const int64_t e0 = (int64_t)block * PIECE, e = e0 + lane_id() * EPT;
    bool decays[4] = {true, true, true, true};
    Piece pc;
    Located loc;
    uint32_t entry = DECAY_ALL;
    if (MASK == MASK_TABLE) entry = tm.decay_tab[block];
    if (MASK == MASK_TENSORS) {
        pc = piece_of(tm, e0, n);
        if (pc.tensor == -1) locate4(tm, pc.seg, tm.begin + e0, lane_id() * EPT, loc);     // the whole wave
    }
    NormTotal<MANY> norm;
    norm.fetch(sums, n_sums);
    u32x4 G;
    State4 s;
    if (e < n) {
        G = KEPT ? *reinterpret_cast<const u32x4 *>(g + e) : ld_nt(reinterpret_cast<const u32x4 *>(g + e));
        s = load_state4(p, m, v, e);
    }
    if (MASK == MASK_TABLE) decay_flags(tm.decay_tab, (uint32_t)uniform((int)entry), decays);
    float sc = a.grad_scale;
    if (n_sums > 0) {                                                                      // the whole wave
        const double total = norm.total(sums, n_sums);
        if (sumsq_out && blockIdx.x == 0 && lane_id() == 0) *sumsq_out = total;
        // an overflowed (non-finite) gradient makes its sum of squares non-finite: the whole step is skipped
        if (a.skip_nonfinite && !isfinite(total)) return;
        sc = scale_from_norm(a, total);
    }
    if (e >= n) return;
    if (MASK == MASK_TENSORS) decay_flags(tm, pc, loc, decays);
    const float gg[4] = {__uint_as_float(G.x), __uint_as_float(G.y), __uint_as_float(G.z), __uint_as_float(G.w)};
    update4<PACK>(a, sc, decays, gg, s, p, m, v, dst, e0, piece_elems(e0, n));
}

// Single sweep when nothing has to wait for the norm (no clipping): fold, Adam and pack; the
// reduced gradient never goes to memory.  TENSORS: contributions are per-tensor gradients; else
// arrays in shard coordinates of dtype DT.  NT: as for k_reduce4t.
template <bool TENSORS, int DT, int MASK, bool NT, int NSRC, int PAUSE, bool HELD>
__global__ __launch_bounds__(WAVE) void k_fused4(int64_t n, float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                                                 const paro_piece_info *pieces, unsigned n_pieces, int P, int group_len,
                                                 const SrcTableOf<NSRC, HELD> src, const AdamConsts a, uint16_t *__restrict__ dst,
                                                 TensorMap tm) {
    tm.pieces = pieces;
    tm.n_pieces = n_pieces;
    Piece pc;
    Located loc;
    int64_t e0 = block_first();
    if constexpr (HELD) leave_window(src.window);
    if constexpr (TENSORS) {
        const Cut c = cut_of(tm, blockIdx.x, n);
        if (c.e0 >= n) return;
        if (!c.whole) {
            if (c.a >= c.b) return;
            const State4 s = load_state4(p, m, v, c.e0 + lane_id() * EPT);
            float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (c.pc.tensor != -2) fold_part(c, src, P, group_len, X);
            const bool d = MASK == MASK_NONE || c.pc.tensor < 0 || tm.no_decay[c.pc.tensor] == 0;
            const bool decays[4] = {d, d, d, d};
            update4<true, true>(a, a.grad_scale, decays, X, s, p, m, v, dst, c.e0, piece_elems(c.e0, n), c.a, c.b);
            return;
        }
        e0 = c.e0;
        pc = c.pc;
    } else {
        if (e0 >= n) return;
        if (MASK == MASK_TENSORS) pc = piece_of(tm, e0, n);
    }
    uint32_t entry = DECAY_ALL;
    if (MASK == MASK_TABLE) entry = tm.decay_tab[e0 / TILE];
    const int64_t e = e0 + lane_id() * EPT;
    if ((TENSORS || MASK == MASK_TENSORS) && pc.tensor == -1) locate4(tm, pc.seg, tm.begin + e0, lane_id() * EPT, loc);     // the whole wave
    if (e >= n) return;
    const unsigned elems = piece_elems(e0, n);
    const State4 s = load_state4(p, m, v, e);
    float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (TENSORS) {
        if (pc.tensor != -2) fold_tensors<NT>(pc, loc, src, P, group_len, X);
    } else {
        if (PAUSE > 0) __builtin_amdgcn_s_sleep(PAUSE);         // see pauses_single
        Chunk4Loader<DT, PAUSE ? 0 : HELD ? PARO_FUSED_WINDOW_PACE_SLEEP : PARO_PACE_SLEEP> ld{e};
        fold4(ld, src, P, group_len, X);
    }
    bool decays[4] = {true, true, true, true};
    if (MASK == MASK_TABLE) decay_flags(tm.decay_tab, (uint32_t)uniform((int)entry), decays);
    if (MASK == MASK_TENSORS) decay_flags(tm, pc, loc, decays);
    update4<true, false, HELD>(a, a.grad_scale, decays, X, s, p, m, v, dst, e0, elems, 0, EPT, window_of(src));
}

// The same for blocks from block0 on of an update range of several chunks (chunk layout, no mask).
template <int DT, int NSRC, int PAUSE, bool HELD>
__global__ __launch_bounds__(WAVE) void k_fused4r(int64_t block0, int64_t n, float *__restrict__ p, float *__restrict__ m,
                                                  float *__restrict__ v, int P, const RangeMap rm, const SrcTableOf<NSRC, HELD> src,
                                                  const AdamConsts a, uint16_t *__restrict__ dst) {
    const int64_t e0 = (block0 + blockIdx.x) * PIECE, e = e0 + lane_id() * EPT;
    if constexpr (HELD) leave_window(src.window);
    if (e0 >= n) return;
    State4 s;
    if (e < n) s = load_state4(p, m, v, e);
    float X[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (PAUSE > 0) __builtin_amdgcn_s_sleep(PAUSE);             // see pauses_range
    fold_range<DT, PAUSE ? 0 : HELD ? PARO_FUSED_WINDOW_PACE_SLEEP : PARO_PACE_SLEEP>(rm, src, P, e0, n, X);
    if (e >= n) return;
    const bool decays[4] = {true, true, true, true};
    update4<true, false, HELD>(a, a.grad_scale, decays, X, s, p, m, v, dst, e0, piece_elems(e0, n), 0, EPT, window_of(src));
}

// Low-precision pack alone.
__global__ __launch_bounds__(WAVE) void k_pack(const float *__restrict__ p, uint16_t *__restrict__ dst, int64_t n,
                                               int pack_dtype) {
    const int64_t e0 = block_first(), e = e0 + lane_id() * EPT;
    if (e >= n) return;
    const unsigned elems = piece_elems(e0, n);
    const u32x4 P = ld_nt(reinterpret_cast<const u32x4 *>(p + e));
    const u32x2 w = {pack2_lowp(__uint_as_float(P.x), __uint_as_float(P.y), pack_dtype),
                     pack2_lowp(__uint_as_float(P.z), __uint_as_float(P.w), pack_dtype)};
    buf_store8<PARO_POL_STREAM_ST>(w, wave_buffer(dst + e0, elems * 2), lane_id() * 8);
}

// One ring hop / one accumulation: out = a + b, element by element in fp32.  n may be any
// length: the descriptors cover the block's whole groups of 4 elements, the thread that holds
// the last, partial group takes it element by element.
template <int DT>
__device__ __forceinline__ void hop_load4(const void *a, int64_t e, float x[4]) {
    constexpr int ESIZE = DT == PARO_F32 ? 4 : 2;
    using Raw = typename Chunk4Loader<DT>::Raw;
    Chunk4Loader<DT>::to_f32(ld_nt(reinterpret_cast<const Raw *>(static_cast<const char *>(a) + e * ESIZE)), x);
}
template <int DT>
__device__ __forceinline__ float hop_load1(const void *a, int64_t i) {
    return DT != PARO_F32 ? cvt16(static_cast<const uint16_t *>(a)[i], DT) : static_cast<const float *>(a)[i];
}

template <int DA, int DB>
__global__ __launch_bounds__(WAVE) void k_hop(const void *a, const void *b, float *out, int64_t n, int keep) {
    const int64_t e0 = block_first(), e = e0 + lane_id() * EPT;
    const unsigned whole = piece_elems(e0, n) & ~3u;       // elements of the block in whole groups of 4
    if (e + EPT <= n) {
        float x[4], y[4];
        hop_load4<DA>(a, e, x);
        hop_load4<DB>(b, e, y);
        buf_store16_as(keep, as_u32x4(x[0] + y[0], x[1] + y[1], x[2] + y[2], x[3] + y[3]), wave_buffer(out + e0, whole * 4),
                       lane_id() * 16);
    } else {
        for (int64_t i = e; i < n; ++i) out[i] = hop_load1<DA>(a, i) + hop_load1<DB>(b, i);
    }
}

// Plain copy of n 16-byte units (an all-gather message landing in the parameter buffer); the first `keep` blocks are
// stored to stay in the memory-side cache.
__global__ __launch_bounds__(WAVE) void k_copy16(const u32x4 *__restrict__ src, u32x4 *__restrict__ dst, int64_t n, unsigned keep) {
    const int64_t i0 = (int64_t)blockIdx.x * WAVE;
    if (i0 + threadIdx.x >= n) return;
    const unsigned bytes = (unsigned)min((int64_t)WAVE, n - i0) * 16;
    const u32x4 v = ld_nt(src + i0 + threadIdx.x);
    buf_store16_as(blockIdx.x < keep, v, wave_buffer(dst + i0, bytes), lane_id() * 16);
}

}  // namespace

// =========================================================================
// host side: validation and launches
// =========================================================================
namespace {

using paro::fail;

#define PARO_HIP(expr)                                                                             \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) return fail(PARO_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

int check_ptr(const void *p, const char *what) {
    if (!p) return fail(PARO_EINVAL, std::string(what) + " is NULL");
    if (reinterpret_cast<uintptr_t>(p) & 15) return fail(PARO_EALIGN, std::string(what) + " is not 16-byte aligned");
    return PARO_OK;
}

// One-wave blocks of a sweep over n elements, ppw pieces per wave.
int64_t piece_count(int64_t n, int ppw = 1) {
    const int64_t nb = (n + (int64_t)PIECE * ppw - 1) / ((int64_t)PIECE * ppw);
    return nb < 1 ? 1 : nb;
}
unsigned piece_grid(int64_t n, int ppw = 1) { return (unsigned)piece_count(n, ppw); }
// Largest grid of a launch that can be cut into several (2^31 threads; the runtime takes fewer than 2^32).
constexpr int64_t MAX_GRID = (int64_t)1 << 25;

// Occupancy throttle for the one-wave-block sweeps: on this part the mixed read/write sweeps run
// faster with 8 to 25 waves per compute unit in flight than with the 32 the registers would allow
// (fewer requests fighting over DRAM pages).  The launch asks for dynamic LDS it never touches,
// a share of the compute unit's 160 KB for each of `waves_per_cu` blocks.
// That is the count asked for, and so are all wave counts in knobs, rules and comments here: LDS is handed out in units of 1280 bytes,
// to which the share is not rounded down, so that one or two waves fewer may fit (counted by the time that blocks of sleeping waves take;
// the occupancy query answers with the count asked for):
//   asked 8 or 9: 8   10: 9   11: 10   12: 11   13: 12   14, 15: 14   16, 17: 16   18 to 20: 18   21 to 24: 21   25 to 30: 25
// The rules were measured as they stand, with what fits; rounding the share would change launches and not only names.
unsigned throttle_lds(int lds_per_cu, int waves_per_cu) {
    if (waves_per_cu <= 0) return 0;
    unsigned bytes = (unsigned)(lds_per_cu / waves_per_cu) / 256u * 256u;
    return bytes > 65536u ? 65536u : bytes;
}

// Waves per compute unit that keep about `loads_per_cu` loads in flight when a wave issues
// `per_wave` loads at a time; 0 (no limit) when that is all that fit anyway.
int fold_waves(int per_wave, int loads_per_cu) {
    const int waves = loads_per_cu / per_wave;
    return waves >= 32 ? 0 : std::max(waves, PARO_MIN_WAVES_PER_CU);
}
// Loads a wave of the fold has in flight: a batch of contributions.
int fold_loads(int P) { return std::min(P, PARO_BATCH); }
// The budget of sweep 1 over the chunk layout; paced: a large launch over one chunk (see paces).
// More contributions than one batch are more DRAM pages than the wave's loads in flight say: 12 waves instead of 14, but
// where a large part of a wave's life belongs to a short last batch of two-byte contributions, with few bytes in flight.
// A paced launch is told apart further - whole clipped steps on the same buffers, with the numbers of the line before
// (224 loads, 192 for more than 16 ranks, a pause of 4) and with these:
//   more than 16 ranks, a pause of 10 and more waves, so that waves side by side read the same page for longer: P = 64, 105 M
//     elements 2794 -> 2787 us, 40 M 1069 -> 1034; P = 48, 40 M 856 -> 829; P = 32, 30 M 474 -> 464; P = 31, 60 M 924 -> 917; P = 24
//     776 -> 775; P = 20 685 -> 683; P = 17 648 -> 639
//   fp32, whose loads are twice as wide, half as many waves: P = 64, 20 M 954 -> 920; P = 16, 100 M 1572 -> 1528; P = 12, 60 M
//     787 -> 760; P = 11 749 -> 718; P = 9 673 -> 646; P = 8, 150 M 1603 -> 1527; P = 6, 100 M 909 -> 884; P = 4 771 -> 766; P = 3 702
//     -> 703; P = 2 637 -> 636
//   5 to 10 ranks, 20 waves instead of 28 (P = 8): P = 8, 200 M 1523 -> 1500; P = 5, 80 M 533 -> 532; P = 7 589 -> 581; P = 10, 60 M
//     500 -> 496
int fold_budget(const paro_plan_t *pl, bool paced) {
    const bool f32 = pl->dtype[0] == PARO_F32;
    if (paced && f32) return pl->P <= 8 ? 80 : 112;
    if (paced && pl->P > PARO_BATCH) return pl->P >= 2 * PARO_BATCH ? 288 : 352;
    if (paced && pl->P > PARO_PAIR_MAX_RANKS && pl->P <= 10) return 160;
    const bool short_batch = !f32 && pl->P % PARO_BATCH != 0 && pl->P < 5 * PARO_BATCH / 2;
    return pl->P > PARO_BATCH && !short_batch ? PARO_FOLD_WIDE_LOADS_PER_CU : PARO_FOLD_LOADS_PER_CU;
}

// Whether a single sweep is so small that a budget would only keep waves from starting, of which the chip holds all at once: with 10 or 11 per compute unit it takes
// two or three rounds.  Whole steps, by the budget and with all waves: over a range of two-byte contributions (up to 8192 blocks), whose waves walk to their
// pointers first, P = 14, 2 x 0.9 M elements 17.4 -> 17.0 us; P = 16, 2 x 0.3 M 8.1 -> 7.0, 2 x 0.5 M 11.3 -> 10.4, 2 x 1 M 20.2 -> 19.2; P = 24, 2 x 0.5 M 15.1 ->
// 13.0, 2 x 1 M 26.5 -> 24.4; P = 32, 2 x 1 M 31.2 -> 29.3; P = 64, 2 x 0.5 M 29.8 -> 25.1, 2 x 1 M 53.6 -> 52.7; P = 128, 2 x 0.4 M 45.3 -> 42.7, 2 x 1 M 98.5 ->
// 99.4 and 98.5 -> 97.4; but beyond that P = 16, 2 x 2 M 38.8 -> 41.9, P = 32, 2 x 1.5 M 45.2 -> 47.2; P = 8, 2 x 0.8 M 11.2 -> 12.5, P = 12, 2 x 0.9 M 15.8 ->
// 16.1.  Otherwise up to 64 ranks: fp32 (up to 4096 blocks), P = 16, 0.7 M 10.3 -> 10.0, P = 64, 1 M 46.6 -> 45.4, a range, P = 16, 2 x 0.5 M 15.0 -> 14.6, P = 32
// 24.9 -> 24.4; but P = 128, 1 M 43.6 -> 45.0; one chunk of two bytes, P = 32, 0.8 M 12.7 -> 12.5, 1 M 15.1 -> 14.8; P = 64, 0.6 M 17.9 -> 15.7, 1 M 24.6 -> 24.4;
// but P = 32, 2 M 28.9 -> 29.4.  With up to 16 of them each wave asks for all it reads in one go, and beyond 25 MB for the launch that is too much at once: P = 12,
// 0.75 M 7.2 -> 5.7, 0.9 M 7.8 -> 7.4, 1.045 M 8.8 -> 8.7; P = 14, 0.75 M 7.7 -> 6.2, 0.85 M 8.0 -> 7.7, but 0.95 M 8.6 -> 8.8, 1.045 M 9.3 -> 9.9; P = 15, 0.75 M
// 7.9 -> 6.5, but 0.95 M 9.2 -> 9.5; P = 16, 0.65 M 7.0 -> 6.7, 0.75 M 7.3 -> 7.3, but 0.85 M 8.0 -> 8.5, 0.9 M 8.5 -> 9.1.  17 to 31: P = 17, 0.7 M 8.2 -> 7.2,
// 0.98 M 10.8 -> 10.6; P = 24, 0.7 M 9.9 -> 9.4, 0.98 M 12.8 -> 12.7, but 1.02 M 12.8 -> 13.2; P = 26 13.5 -> 13.9; P = 28 14.7 -> 14.8.
bool runs_at_once(int P, bool f32, bool range, int64_t blocks) {
    if (range && !f32) return P > 12 && blocks <= PARO_AT_ONCE_RANGE_BLOCKS;
    if (P < 12 || P > 64) return false;
    if (f32 || P >= 2 * PARO_BATCH) return blocks <= PARO_AT_ONCE_BLOCKS;
    return P > PARO_BATCH ? blocks <= PARO_AT_ONCE_SHORT_BATCH_BLOCKS : blocks * P <= PARO_AT_ONCE_READS;
}

// Waves per compute unit of a single sweep over `blocks` blocks.  The budget, which was found at P = 16, lets too many waves
// with few loads each run beside one another: a wave also loads and stores its state, and what counts is the bytes that a
// compute unit has in flight: 50 KB (P = 2) to 100 (P = 12) with two-byte contributions, 60 to 150 with fp32 ones.  So no
// more than 13 waves of two-byte contributions with up to 7 ranks, 12 beyond, and 13 (P = 2) to 8 (P >= 8) of fp32.  Whole
// steps on the same buffers, by the budget and with these: P = 2, 200 M elements 971 -> 897 us; P = 3, 100 M 538 -> 495;
// P = 4, 150 M 836 -> 775; P = 6, 80 M 487 -> 465; P = 8, 200 M 1333 -> 1272, 6 M 42.8 -> 41.0; P = 10, 60 M 440 -> 425; P = 12 to
// 15 as they were; fp32: P = 2, 100 M 566 -> 527; P = 4 687 -> 644; P = 6, 80 M 686 -> 617; P = 8, 20 M 194 -> 183; P = 12, 60
// M 729 -> 707; P = 15, 40 M 559 -> 554; a range of 8 chunks of 7.5 M, P = 8, 405 -> 386.  Not in launches that run in one
// round of waves (P = 8, 1 M: 6.3 -> 7.5).
// A list of few large fp32 tensors whose blocks start on cache lines has look-ups to
// hide as well and wants a few more: 13 waves, 10 from 7 ranks on (Llama-like lists, P = 4, 572 -> 539; P = 6, 2144 -> 2046; P
// = 8, 2725 -> 2610).  Two-byte ones keep the budget (P = 4 2596, 15 waves 2591; P = 3 597, 16 waves 626), and so do blocks
// that share cache lines with their neighbours, which want them close in time, and many small tensors (fp32, ragged, P = 6, 13
// waves 420 -> 391, but P = 7 463 -> 531; Llama-like, P = 7 1901 -> 2032).
// A range of several chunks with two-byte contributions wants that only where its blocks read 81 920 contributions between them, 20 M
// elements: with fewer, the waves of few ranks that were thinned out were too few (three states in turn, by the budget and thinned out: P = 2,
// 2.4 M elements 13.7 and 14.7 us, 4 M 22.9 and 23.2; P = 3, 2.8 M 17.5 and 17.9; P = 4, 3 M with contributions just written 21.6 and 22.7;
// but P = 4, 7 M 41.3 and 40.4, P = 3, 7.8 M 43.1 and 42.6).
enum class Sweep { CHUNK, RANGE, TENSORS_ON_LINES, OTHER_TENSORS };
int fused_waves(int P, bool f32, Sweep over, int64_t blocks) {
    if ((over == Sweep::CHUNK || over == Sweep::RANGE) && runs_at_once(P, f32, over == Sweep::RANGE, blocks)) return 0;
    const int waves = fold_waves(fold_loads(P) + 3, PARO_FUSED_LOADS_PER_CU);
    if (blocks < PARO_FUSED_MIN_BLOCKS || P >= PARO_BATCH || over == Sweep::OTHER_TENSORS) return waves;
    if (over == Sweep::RANGE && !f32 && blocks * P < PARO_FUSED_RANGE_MIN_READS) return waves;
    int most;
    if (over == Sweep::TENSORS_ON_LINES) most = !f32 ? waves : P < 7 ? 13 : 10;
    else most = f32 ? std::max(14 - 5 * P / 6, 8) : P < 8 ? 13 : 12;
    return waves == 0 ? most : std::min(waves, most);
}

// What a launch needs from the device besides the caller's buffers: the LDS size behind the
// occupancy throttle and the scratch array of partial sums (per-block sums of a sweep-1 launch,
// then `level2`, the second-level sums).  Either the plan's own allocation or the library's
// static array.
struct Scratch {
    int lds_per_cu;
    double *partials;
    int64_t n_partials;    // a multiple of 8
    double *level2;
    double *chunk_sums;    // [range_sums()] one sum per chunk, or per group of blocks, of an update range of several chunks
    bool plan_tables;      // the plan's device tables (offset tables, per-tile tables) exist
};

// Room for the second-level sums of n_part partials.
constexpr int64_t level2_sums(int64_t n_part) {
    const int64_t n = (n_part + FINALIZE_CHUNK - 1) / FINALIZE_CHUNK;
    return n < NORM_SLICES ? NORM_SLICES : n;
}

// Room for the sums of a range with n_part partials: of its chunks, or of its groups, cut once more where a
// launch ends (MAX_GRID is a multiple of the group) or the own chunk does.
constexpr int64_t range_sums(int64_t n_part) {
    const int64_t n = n_part / NORM_GROUP + 3;
    return n < PARO_MAX_RANKS ? (int64_t)PARO_MAX_RANKS : n;
}

Scratch plan_scratch(const paro_plan_t *pl) {
    double *level2 = pl->dev.partials + pl->dev.n_partials;
    const int64_t n_level2 = level2_sums(pl->dev.n_partials);
    return Scratch{pl->dev.lds_per_cu, pl->dev.partials, pl->dev.n_partials, level2, level2 + n_level2, true};
}

template <class T>
int upload(T **dst, const T *src, size_t n) {
    PARO_HIP(hipMalloc(reinterpret_cast<void **>(dst), (n ? n : 1) * sizeof(T)));
    if (n) PARO_HIP(hipMemcpy(*dst, src, n * sizeof(T), hipMemcpyHostToDevice));
    return PARO_OK;
}

void free_tables(paro_device_tables &d) {
    // best effort: at process exit the runtime may already be gone
    (void)hipFree(d.nz_off);
    (void)hipFree(d.nz_tensor);
    (void)hipFree(d.nz_dtype);
    (void)hipFree(d.dtype);
    (void)hipFree(d.no_decay);
    for (uint32_t *t : d.decay_tab) (void)hipFree(t);
    for (paro_piece_info *t : d.piece_tab) (void)hipFree(t);
    (void)hipFree(d.partials);
    d = paro_device_tables();
}

int fill_tables(const paro_plan_t *pl, paro_device_tables &d) {
    int rc;
    if ((rc = upload(&d.nz_off, pl->nz_off.data(), pl->nz_off.size()))) return rc;
    if ((rc = upload(&d.nz_tensor, pl->nz_tensor.data(), pl->nz_tensor.size()))) return rc;
    std::vector<uint8_t> nz_dtype(pl->nz_tensor.size());
    for (size_t k = 0; k < nz_dtype.size(); ++k) nz_dtype[k] = pl->dtype[(size_t)pl->nz_tensor[k]];
    if ((rc = upload(&d.nz_dtype, nz_dtype.data(), nz_dtype.size()))) return rc;
    if ((rc = upload(&d.dtype, pl->dtype.data(), pl->dtype.size()))) return rc;
    if ((rc = upload(&d.no_decay, pl->no_decay.data(), pl->no_decay.size()))) return rc;
    d.tiles_per_chunk = (pl->L + TILE - 1) / TILE;
    // a boundary makes one piece more; twice the tiles at most
    d.max_pieces = d.tiles_per_chunk + std::min(d.tiles_per_chunk, (int64_t)pl->nz_tensor.size() + 1);
    d.decay_tab.assign((size_t)pl->P, nullptr);
    d.piece_tab.assign((size_t)pl->P, nullptr);
    d.n_pieces.assign((size_t)pl->P, 0);
    d.on_lines.assign((size_t)pl->P, 0);
    d.f32.assign((size_t)pl->P, 0);
    d.piece_tab_tried.assign((size_t)pl->P, 0);
    d.decay_tab_tried.assign((size_t)pl->P, 0);
    // one partial per block of a sweep-1 launch (which covers a rank's whole update range at most),
    // followed by room for the second-level sums
    int64_t ob, on;
    paro::letter_range(pl, 0, pl->letters[2], &ob, &on);
    // (in the tensor layout one chunk, a wave for each of its pieces)
    int64_t n_part = (std::max(piece_count(on), d.max_pieces) + 7) & ~(int64_t)7;
    if (n_part < PARO_MIN_PARTIALS) n_part = PARO_MIN_PARTIALS;
    d.n_partials = n_part;
    const int64_t n_level2 = level2_sums(n_part);
    PARO_HIP(hipMalloc(reinterpret_cast<void **>(&d.partials), (n_part + n_level2 + range_sums(n_part)) * sizeof(double)));
    return PARO_OK;
}

// Creates the plan's device tables on the current device, once.
int ensure_device(paro_plan_t *pl) {
    std::lock_guard<std::mutex> lock(pl->dev_mutex);
    int dev = -1;
    PARO_HIP(hipGetDevice(&dev));
    if (pl->dev.device >= 0) {
        if (pl->dev.device != dev)
            return fail(PARO_EINVAL, "the plan's device tables live on another device than the current one");
        return PARO_OK;
    }
    paro_device_tables d;
    // LDS per compute unit, for the occupancy throttle; 160 KB on gfx950 if the runtime does not say
    if (hipDeviceGetAttribute(&d.lds_per_cu, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
        d.lds_per_cu < 65536) {
        (void)hipGetLastError();
        d.lds_per_cu = 160 * 1024;
    }
    const int rc = fill_tables(pl, d);
    if (rc != PARO_OK) {
        free_tables(d);                    // nothing half-built stays behind
        return rc;
    }
    d.device = dev;
    pl->dev = d;
    return PARO_OK;
}

// The chunk's pieces, for the tensor layout.  A tile with a boundary inside is cut where the tensors
// meet: taken by one wave, its lanes would each have pointers of their own to fetch, element by element,
// P times over (P = 64, 1.4 M elements of tensors of 1 to 65536 elements: sweep 1 in 195 us, a handful of
// such waves keeping the rest waiting; cut, 85 us).  With few contributions that fetching is short, and in a
// large chunk the cut's partial cache lines of g cost more (P = 2, 59 M elements: whole step 370 us, cut
// 395; P = 4, 4 M elements, though: 22.6 us, cut 20.2).  Nor is a very large chunk of fp32 gradients cut, up to 32
// ranks: few enough waves have slow lanes among their 16-byte loads, and the partial lines weigh as much as ever
// (clipped, cut and whole: 80 M elements, P = 8 938 and 916 us, P = 12 1214 and 1166; 40 M, P = 16 716 and 732, P = 64
// 2273 and 2385; bf16, 80 M, P = 12: 779 and 790).  A tile of more tensors than PARO_SPLIT_MAX stays whole.
void list_pieces(const paro_plan_t *pl, int64_t c, std::vector<paro_piece_info> *tab) {
    const int64_t n_nz = (int64_t)pl->nz_tensor.size(), most = pl->dev.max_pieces;
    int64_t spare = most - pl->dev.tiles_per_chunk;
    const int64_t tiles = pl->dev.tiles_per_chunk;
    const bool f32 = pl->dev.f32[(size_t)c] != 0;
    const bool few = pl->P <= (f32 ? PARO_PAIR_MAX_RANKS : PARO_PAIR_SMALL_MAX_RANKS);
    const bool cut = tiles < PARO_LARGE_TILES || !(few || (f32 && pl->P <= 32 && tiles >= 2 * PARO_LARGE_TILES));
    tab->reserve((size_t)most);
    auto add = [&](int64_t off, int64_t dt, int64_t lo, int64_t hi, int32_t tensor, int64_t i) {
        tab->push_back({off * ((int64_t)1 << 19) + (dt << 17 | hi << 8 | lo), tensor, (uint32_t)i});
    };
    paro::for_each_tile(pl, c, [&](int64_t i, int64_t f0, int64_t f1, int64_t k) {
        if (k == n_nz) return add(0, 0, 0, TILE, -2, i);
        const int32_t t = pl->nz_tensor[(size_t)k];
        if (f1 <= pl->nz_off[(size_t)k + 1]) return add(f0 - pl->nz_off[(size_t)k], pl->dtype[(size_t)t], 0, TILE, t, i);
        int64_t end = k;                                         // one past the tile's last segment
        while (end < n_nz && pl->nz_off[(size_t)end] < f1) ++end;
        const bool pad = f1 > pl->total;
        if (!cut || end - k + pad > PARO_SPLIT_MAX || end - k + pad - 1 > spare) return add(k, 0, 0, TILE, -1, i);
        spare -= end - k + pad - 1;
        for (int64_t q = k; q < end; ++q) {
            const int64_t begin = pl->nz_off[(size_t)q];
            const int32_t u = pl->nz_tensor[(size_t)q];
            add(f0 - begin, pl->dtype[(size_t)u], std::max(begin - f0, (int64_t)0), std::min(pl->nz_off[(size_t)q + 1], f1) - f0, u, i);
        }
        if (pad) add(0, 0, pl->total - f0, f1 - f0, -2, i);
    });
    // a small launch ends sooner when its slow waves start first (step over 10 000 tensors, P = 8, 7.4 M
    // elements: 80.0 -> 75.5 us); a large one is slower for fetching the cache lines around a cut twice
    // (160 000 tensors, single sweep: 925 -> 958 us)
    if (cut && pl->dev.tiles_per_chunk < PARO_LARGE_TILES)
        std::stable_partition(tab->begin(), tab->end(), [](const paro_piece_info &x) { return (x.where & 0x1FFFF) != TILE << 8 || x.tensor == -1; });
}

// Builds, once per chunk, a table of the chunks of a rank's update range.  Too large a one (chunks of more
// than 4 Mi tiles, or what the environment variable PARO_TILE_TABLE_MAX_TILES says) is not built; the
// kernels then search the offset table for every block.
template <class Info, class List>
int ensure_table(paro_plan_t *pl, int rank, std::vector<Info *> &tabs, std::vector<uint8_t> &tried, List list) {
    const paro_device_tables &d = pl->dev;
    int64_t ob, on;
    paro::letter_range(pl, rank, pl->letters[2], &ob, &on);
    int64_t max_tiles = (int64_t)4 << 20;                   // up to 128 MB of pieces, up to 151 MB of weight-decay table
    if (const char *env = std::getenv("PARO_TILE_TABLE_MAX_TILES")) max_tiles = std::atoll(env);
    std::vector<Info> tab;
    for (int64_t c = ob / pl->L; c < (ob + on) / pl->L; ++c) {
        if (tried[(size_t)c]) continue;
        if constexpr (std::is_same_v<Info, paro_piece_info>) {
            pl->dev.on_lines[(size_t)c] = paro::on_cache_lines(pl, c);
            pl->dev.f32[(size_t)c] = paro::mostly_f32(pl, c);
        }
        if (d.tiles_per_chunk > max_tiles) {
            tried[(size_t)c] = 1;                    // decided: this chunk works without a table
            continue;
        }
        tab.clear();
        try {
            list(pl, c, &tab);
        } catch (const std::bad_alloc &) {
            return fail(PARO_ENOMEM, "out of host memory while building the per-tile table");
        }
        Info *dev_tab = nullptr;
        const int rc = upload(&dev_tab, tab.data(), tab.size());
        if (rc != PARO_OK) {                         // the next call tries again (and reports again)
            (void)hipFree(dev_tab);
            return rc;
        }
        tabs[(size_t)c] = dev_tab;
        if constexpr (std::is_same_v<Info, paro_piece_info>) pl->dev.n_pieces[(size_t)c] = (uint32_t)tab.size();
        tried[(size_t)c] = 1;
    }
    return PARO_OK;
}

// The tables that a call needs: the pieces for the tensor layout, the tiles for a weight-decay mask
// applied block by block.
int ensure_tables(paro_plan_t *pl, int rank, bool pieces, bool decays) {
    std::lock_guard<std::mutex> lock(pl->dev_mutex);
    paro_device_tables &d = pl->dev;
    int rc = PARO_OK;
    if (pieces) rc = ensure_table(pl, rank, d.piece_tab, d.piece_tab_tried, list_pieces);
    if (decays && rc == PARO_OK) rc = ensure_table(pl, rank, d.decay_tab, d.decay_tab_tried, paro::list_decays);
    return rc;
}

// The map from elements to tensors for a launch whose element 0 is flat index `begin`.  The
// per-tile tables are per chunk: they serve launches that start on a chunk boundary and stay
// inside that chunk.
TensorMap map_for(const paro_plan_t *pl, const Scratch &sc, int64_t begin, bool one_chunk) {
    TensorMap tm;
    if (!sc.plan_tables) {                  // launches that never look at tensors (chunk layout, no decay mask)
        tm.nz_off = nullptr;
        tm.nz_tensor = nullptr;
        tm.nz_dtype = tm.dtype = tm.no_decay = nullptr;
        tm.n_nz = 0;
        tm.total = pl->total;
        tm.begin = begin;
        tm.decay_tab = nullptr;
        tm.pieces = nullptr;
        tm.n_pieces = 0;
        return tm;
    }
    tm.nz_off = pl->dev.nz_off;
    tm.nz_tensor = pl->dev.nz_tensor;
    tm.nz_dtype = pl->dev.nz_dtype;
    tm.dtype = pl->dev.dtype;
    tm.no_decay = pl->dev.no_decay;
    tm.n_nz = (int)pl->nz_tensor.size();
    tm.total = pl->total;
    tm.begin = begin;
    tm.decay_tab = nullptr;
    tm.pieces = nullptr;
    tm.n_pieces = 0;
    if (one_chunk && begin % pl->L == 0) {
        const size_t c = (size_t)(begin / pl->L);
        tm.decay_tab = pl->dev.decay_tab[c];
        tm.pieces = pl->dev.piece_tab[c];
        tm.n_pieces = pl->dev.n_pieces[c];
    }
    return tm;
}

int check_common(const paro_plan_t *pl, int rank, const char *fn) {
    if (!pl) return fail(PARO_EINVAL, std::string(fn) + ": plan is NULL");
    if (rank < 0 || rank >= pl->P) return fail(PARO_ERANGE, std::string(fn) + ": rank out of range");
    return PARO_OK;
}

int check_contrib(const paro_plan_t *pl, const void *const *contrib, int layout, const char *fn) {
    if (!contrib) return fail(PARO_EINVAL, std::string(fn) + ": contrib is NULL");
    if (layout != PARO_CHUNK && layout != PARO_TENSORS) return fail(PARO_EINVAL, std::string(fn) + ": bad layout");
    if (layout == PARO_CHUNK && !pl->uniform_dtype)
        return fail(PARO_EINVAL, std::string(fn) + ": chunk layout needs one gradient dtype for all tensors");
    for (int q = 0; q < pl->P; ++q) {
        if (!contrib[q]) return fail(PARO_EINVAL, std::string(fn) + ": a contribution pointer is NULL");
        if (layout == PARO_CHUNK && (reinterpret_cast<uintptr_t>(contrib[q]) & 15))
            return fail(PARO_EALIGN, std::string(fn) + ": a contribution is not 16-byte aligned");
        if (layout == PARO_TENSORS && (reinterpret_cast<uintptr_t>(contrib[q]) & 7))
            return fail(PARO_EALIGN, std::string(fn) + ": a pointer table is not 8-byte aligned");
    }
    return PARO_OK;
}

// Elements of a rank's update range: the length of its state arrays and of the reduced gradient.
int64_t update_elems(const paro_plan_t *pl) {
    int64_t ob, on;
    paro::letter_range(pl, 0, pl->letters[2], &ob, &on);
    return on;
}
// Whether the loads of a launch over one chunk of the chunk layout are paced (see load_batch).
bool paces(const paro_plan_t *pl) {
    return piece_count(pl->L) >= (pl->P < 2 * PARO_BATCH ? PARO_PACE_MIN_BLOCKS : PARO_PACE_MIN_BLOCKS / 2);
}
// Whether sweep 1 over one chunk holds its results back for write windows that the whole chip shares.  A trickle of stores among P streams of loads costs the memory
// far more than its bytes: the fold of 16 ranks reads at 7.1 TB/s while nothing is stored and at 6.4 with its 11 % of stores, that of 64 at 6.9 and 6.0 with 3
// %.  So a wave that has its sums waits (asleep, with four registers of results a lane) until the chip's next window, all stores go out within half a microsecond,
// and waves that start then leave the memory to them.  It takes waves to spare: while about half of them wait the others have to keep the memory busy, so they are
// not thinned out - as many as fit of two-byte contributions, 18 per compute unit of fp32 ones - and a window comes after 0.36 us a rank for either type, 16 us at
// most: 0.61 of the time that all their loads take at 7.1 TB/s with two-byte contributions, 0.55 with fp32 ones.  Those that have nobody behind them do not wait.
// Whole clipped steps on the same buffers, without and with windows: P = 64, 100 M elements 2518 -> 2385 us, 35 M 899 -> 869; P = 128, 30 M 1389 -> 1341; P = 100,
// 40 M 1516 -> 1455; P = 48, 60 M 1222 -> 1187; P = 32, 100 M 1495 -> 1440, 12 M 192.1 -> 189.6; P = 24, 60 M 780 -> 755; P = 16, 100 M 1028 -> 1008, 25 M 257.9 ->
// 256.7; P = 12, 100 M 889 -> 876; but P = 16, 17 M 175.9 -> 176.2, 8 M 88.4 -> 88.9; P = 20, 12 M 143 -> 144; P = 64, 15 M 378 -> 383; P = 10, 60 M 495 -> 497; P =
// 8, 100 M 747 -> 759.  fp32: P = 64, 30 M 1341 -> 1309; P = 48, 30 M 1047 -> 1016, 8 M 296 -> 289; P = 32, 40 M 1000 -> 960, 6 M 160 -> 154; P = 24, 10 M 216 ->
// 210; P = 16, 60 M 895 -> 879, 10 M 166 -> 159; P = 12, 10 M 136 -> 133; but P = 16, 17 M 257 -> 262, 30 M 455 -> 457, 2 M 37.0 -> 37.9; P = 10, 60 M 695 ->
// 700.  Between 65 536 and 131 071 blocks fp32 launches of up to 47 ranks, which are paced there and have waves for that, win or lose by the size: on another GPU P
// = 24, 17 M 341 -> 334, 24 M 465 -> 465, 33 M 622 -> 636; P = 40, 17 M 503 -> 504, 30 M 848 -> 871; P = 32, 17 M 417 -> 412, 24 M 590 -> 577, 33 M 778 -> 782; P =
// 20, 30 M 513 -> 506; P = 16, 17 M 255 -> 250, 33 M 479 -> 472.  Sweep 2 and the single sweep of 16 ranks, half and a quarter of whose bytes are stores, are 9 and
// 0 to 3 % slower with windows of any length; a wave that folds 2 to 8 blocks before it waits gains no more than one that folds one.
bool holds_back(const paro_plan_t *pl) {
    const int64_t blocks = piece_count(pl->L);
    if (pl->P < PARO_WINDOW_MIN_RANKS) return false;
    if (pl->dtype[0] == PARO_F32)
        return blocks >= PARO_WINDOW_F32_MIN_BLOCKS &&
               (pl->P >= PARO_WINDOW_MANY_RANKS || blocks < PARO_PACE_MIN_BLOCKS || blocks >= PARO_LARGE_TILES);
    const bool middle = pl->P >= PARO_BATCH * 3 / 2 && pl->P < PARO_WINDOW_MANY_RANKS;
    return blocks >= (middle ? PARO_WINDOW_MIN_BLOCKS / 2 : PARO_WINDOW_MIN_BLOCKS);
}
// ... and over a range of several chunks.  fp32 contributions, whole clipped steps alike: P = 64, 8 x 4 M elements 1495 -> 1400 us, 2 x 15 M 1369 -> 1324; P = 48, 4 x 5 M
// 733 -> 687; P = 32, 4 x 12 M 1232 -> 1164; P = 16, 8 x 10 M 1230 -> 1174, 2 x 30 M 894 -> 867; P = 12, 6 x 3 M 235 -> 224, 4 M in all 57.2 -> 57.2; but P = 16, 3 M 54.1 -> 54.5, P = 64,
// 2.4 M 121.1 -> 124.3.
// Over two-byte ones the loads are not paced, as without windows, and a window comes after 0.24 us a rank, 13 us at most (P = 24, 3 x 20 M with 0.21, 0.29, 0.38 and 0.46 us
// 725, 730, 758, 785; paced, with 0.36, 830 where it is 763 without windows; P = 64, 8 x 4 M with 0.08, 0.14, 0.20 us 779, 766, 761): P = 12, 2 x 20 M 356 -> 346; P = 14, 2 x 20 M
// 389 -> 367; P = 16, 2 x 25 M 495 -> 485, 4 x 6 M 246 -> 239; P = 17, 17 x 0.3 M 63.1 -> 61.4; P = 20, 2 x 2.2 M 58.3 -> 57.7; P = 24, 3 x 20 M 758 -> 713; P = 32, 4 x 12 M 749 -> 681, 2 x
// 2.2 M 75.0 -> 73.5; P = 48, 4 x 10 M 860 -> 776; P = 64, 8 x 4 M 857 -> 761; P = 128, 16 x 2 M 1569 -> 1415; P = 256, 2 x 3 M 550 -> 524; but P = 16, 2 x 4.3 M 92.1 -> 91.8, P = 12,
// 2 x 4.3 M 81.9 -> 82.8, 3 x 4 M 110.4 -> 111.9, P = 10, 2 x 20 M 320.7 -> 320 to 323.
bool range_holds_back(const paro_plan_t *pl) {
    if (pl->P < PARO_WINDOW_MIN_RANKS) return false;
    const bool early = pl->dtype[0] == PARO_F32 || pl->P > PARO_BATCH;
    return piece_count(update_elems(pl)) >= (early ? PARO_RANGE_WINDOW_MIN_BLOCKS : PARO_RANGE_WINDOW_MIN_BLOCKS * 4);
}
int window_waves(const paro_plan_t *pl) { return pl->dtype[0] == PARO_F32 ? PARO_WINDOW_F32_WAVES_PER_CU : 0; }
WriteWindow window_for(int period, int waves, int open, int rest) {
    return WriteWindow{(unsigned)(((uint64_t)1 << 32) / (unsigned)period), (unsigned short)period, (unsigned short)(waves ? waves : MAX_WAVES_PER_CU),
                       (unsigned short)open, (unsigned short)rest};
}
WriteWindow fold_window(const paro_plan_t *pl, bool range = false) {
    const bool soon = range && pl->dtype[0] != PARO_F32;
    const int per_rank = soon ? PARO_RANGE_WINDOW_TICKS_PER_RANK : PARO_WINDOW_TICKS_PER_RANK;
    const int most = soon ? PARO_RANGE_WINDOW_MAX_PERIOD : PARO_WINDOW_MAX_PERIOD;
    return window_for(std::min(per_rank * pl->P, most), window_waves(pl), PARO_WINDOW_TICKS, PARO_WINDOW_REST_TICKS);
}
// ... and whether the single sweep over n elements does (chunk layout), whose waves store their state as well: one comes after 0.26 us for each byte of an element's
// contributions, 28 us at most (fp32 ones: 23), and takes 0.16 of that.  Whole steps on the same buffers, without and with windows: P = 64, 100 M elements 2632 ->
// 2314 us, 30 M 774 -> 690, 8 M 217.5 -> 203.5; P = 128, 20 M 957 -> 894; P = 256, 6 M 586 -> 539; P = 48, 40 M 811 -> 731; P = 40, 60 M 1037 -> 975, 30 M 518 ->
// 499; P = 32, 100 M 1458 -> 1451 and on another GPU 1455 -> 1408, 40 M 572 -> 556, 10 M 149.5 -> 153.2 and 146.3 -> 144.1; a range of 4 x 30 M, P = 32, 1805 ->
// 1741, 8 x 10 M, P = 64, 2176 -> 1948; but P = 28, 60 M 775 -> 772, P = 24, 100 M 1150 -> 1170, P = 16, 200 M 1796 -> 1870; P = 32, 3 M 46.6 -> 49.0, P = 64, 3 M
// 79.1 -> 82.8, P = 128, 2 M 94.8 -> 98.2, P = 256, 2 M 184 -> 187.  fp32: P = 64, 20 M 992 -> 886; P = 32, 15 M 403 -> 371, 4 M 111.0 -> 107.0; P = 24, 50 M 1028 ->
// 961; P = 20, 40 M 686 -> 698 and 725 -> 692; P = 16, 80 M 1204 -> 1170, 15 M 228 -> 222, 8 M 122.6 -> 121.8; but P = 14, 60 M 788 -> 799, P = 16, 5 M 80.0 ->
// 80.6.  Per-tensor gradients of two bytes, whose waves look up their pointers first: P = 32, Llama-like list, 555 -> 618; ragged, 335 -> 366.
// 32 ranks of two bytes, whose waves end with no short last batch, are fastest of all without (14.2 us a million elements, 33 ranks 14.9, 36 16.0) and gain at every
// size only from 26 M elements on: 13 M 190 -> 188, 16 M 228 -> 224, 18 M 255 -> 260, 20 M 283.7 -> 288.5, 22 M 321 -> 315, 25 M 354.7 -> 357.8, 26 M 377 -> 371, 27
// M 387 -> 380, 28 M 408 -> 396, 35 M 498 -> 492, 60 M 870 -> 844; P = 33, 18 M 269 -> 269, 20 M 296 -> 293, 25 M 371 -> 362; P = 34, 14 M 218 -> 207, 20 M 305 ->
// 299; P = 36, 14 M 230 -> 216, 20 M 325 -> 304; fp32, P = 16, 13 M 203 -> 188, 20 M 291 -> 280, 32 M 470 -> 450.
bool fused_holds_back(const paro_plan_t *pl, int64_t n) {
    const bool f32 = pl->dtype[0] == PARO_F32;
    const int bytes = pl->P * (f32 ? 4 : 2);
    if (pl->P == 2 * PARO_BATCH && !f32) return n * bytes >= PARO_FUSED_WINDOW_TWO_BATCHES_BYTES;
    const int64_t least = (int64_t)PARO_FUSED_WINDOW_MIN_BYTES / 64 * std::max(pl->P, 64);
    return bytes >= PARO_FUSED_WINDOW_RANK_BYTES && n * bytes >= (bytes < PARO_FUSED_WINDOW_MANY_BYTES ? least * 3 / 2 : least);
}
// ... over a range of several chunks: two-byte contributions of 28 ranks and more, from 16 384 blocks on or, where a short last batch is a large part of a
// wave's life, from 768 MB.  Up to 96 ranks their loads are not paced, and a window comes after 18 us at most (more beyond 90 ranks).  Whole steps,
// without windows and with: P = 28, 2 x 20 M elements 536 -> 513 us; P = 32, 2 x 2 M 62.3 -> 61.2, 2 x 5 M 148 -> 145; P = 48, 2 x 2 M 87.1 -> 84.6; P = 64, 2 x 2 M 108.1 -> 105.7; P = 128, 2 x 2 M 204.5
// -> 194.6; but P = 36, 3 x 3 M 146.7 -> 148.2, P = 28, 2 x 3 M 83.2 -> 81.7 and 83.5 -> 84.0, 4 x 5 M 258.2 -> 258.9, P = 30, 2 x 5 M 139.6 -> 140.4; P = 24, 2 x 4 M 98.8 -> 98.0, 2 x 2 M 50.0 -> 50.0;
// P = 16, 2 x 6 M 110 -> 118; P = 32, 2 x 1.5 M 45.2 -> 45.7, P = 64 80.6 -> 81.4.  Paced and with a window as above, and so: P = 32, 8 x 3 M 351 -> 342; P = 40, 4 x 10 M 706 -> 686;
// P = 48 803 -> 781; P = 64, 4 x 12 M 1155 -> 1148, 8 x 4 M 762 -> 747 and on another GPU 796 -> 803; P = 96, 4 x 5 M 713 -> 707; but P = 128, 4 x 5 M 867 -> 875.
bool fused_range_holds_back(const paro_plan_t *pl, int64_t n) {
    if (pl->dtype[0] == PARO_F32) return fused_holds_back(pl, n);
    if (pl->P < PARO_FUSED_RANGE_WINDOW_MIN_RANKS) return false;
    if (pl->P % PARO_BATCH == 0 || pl->P > 3 * PARO_BATCH) return piece_count(n) >= PARO_RANGE_WINDOW_MIN_BLOCKS;
    return n * pl->P * 2 >= (int64_t)PARO_FUSED_WINDOW_MIN_BYTES * 3 / 2;
}
bool fused_range_paces(const paro_plan_t *pl) { return pl->dtype[0] == PARO_F32 || pl->P > PARO_FUSED_RANGE_UNPACED_RANKS; }
int fused_window_waves(const paro_plan_t *pl) { return pl->dtype[0] == PARO_F32 ? PARO_FUSED_WINDOW_F32_WAVES_PER_CU : 0; }
WriteWindow fused_window(const paro_plan_t *pl, bool paced = true) {
    const bool f32 = pl->dtype[0] == PARO_F32;
    const int bytes = pl->P * (f32 ? 4 : 2);
    const int most = f32 ? PARO_FUSED_WINDOW_F32_MAX_PERIOD : paced ? PARO_FUSED_WINDOW_MAX_PERIOD : std::max(PARO_FUSED_RANGE_WINDOW_MAX_PERIOD, 10 * bytes);
    const int period = std::min(PARO_FUSED_WINDOW_TICKS_PER_BYTE * bytes, most), open = period * 4 / 25;
    return window_for(period, fused_window_waves(pl), open, open);
}
// Whether the waves of a single sweep over one chunk of n elements pause between the loads of their state and those of the
// contributions.  They start with their arguments in registers, and where the launch reads 21 to 30 MB - all of it runs at once, or
// nearly - with up to 3 ranks they ask for too much at the same moment.  Three states in turn, without preloaded arguments, with
// them, and with this pause as well: P = 1, bf16, 1.57 M elements 7.6, 8.4 and 7.2 us, 1.71 M 8.3, 9.3 and 8.0; P = 2, 1.44 M 7.4, 8.4
// and 7.5, 1.5 M 7.8, 8.9 and 7.7, 1.69 M 10.1, 10.4 and 8.9; P = 3, 1.33 M 7.4, 8.4 and 7.3, 1.5 M 8.9, 9.7 and 8.3; fp32, P = 2,
// 1.2 M 7.3, 8.2 and 6.9.  Contributions just written, P = 2, 1.5 M: 13.9, 12.6 and 11.3; after 512 MB of something else 11.0, 12.6
// and 11.0.  A pause after each contribution's load: 6 % ahead of this one at P = 2, 1.4 M, 8 to 15 % behind it at 1.7 M, nothing for P = 1.
// One fp32 contribution does without (1.4 M 9.0 and 8.3; paused 9.1), and so do 4 ranks.
bool pauses_single(const paro_plan_t *pl, int64_t n) {
    const bool f32 = pl->dtype[0] == PARO_F32;
    const int64_t bytes = n * (12 + pl->P * (f32 ? 4 : 2));
    if (pl->P > PARO_PAUSE_MAX_RANKS || (pl->P == 1 && f32)) return false;
    return bytes >= (pl->P == 1 ? PARO_PAUSE_MIN_BYTES_ONE : PARO_PAUSE_MIN_BYTES) && bytes < PARO_PAUSE_MAX_BYTES;
}
// ... and over an update range of several chunks: up to 8 ranks with two-byte contributions, 4 with fp32 ones, and 19.5 to 31 MB, with 2
// ranks 27.  Measured alike: bf16, P = 2, 1.41 M elements 8.2, 8.6 and 7.9 us; P = 3, 1.33 M 8.1, 8.8 and 7.5; P = 4, 1.13 M 7.3, 8.0 and 6.7,
// 1.3 M 8.2, 9.3 and 7.8; P = 5, 1.27 M 9.0, 10.0 and 8.2; P = 6, 1.25 M 9.2, 9.0 and 8.2; P = 8, 0.8 M 7.3, 7.5 and 7.3; fp32, P = 2, 1.3 M
// 7.9, 8.1 and 7.4, P = 4, 1 M 8.0, 8.3 and 7.9.  Contributions just written, P = 4, 1.3 M: 14.8, 12.2 and 11.6; after 512 MB of something
// else 11.4, 12.4 and 10.9.  With fp32 and 8 ranks a pause costs 3 % below 0.55 M, with P = 2 3 % at 28 MB.
bool pauses_range(const paro_plan_t *pl, int64_t n) {
    const int64_t esize = pl->dtype[0] == PARO_F32 ? 4 : 2, bytes = n * (12 + pl->P * esize);
    return pl->P * esize <= 16 && bytes >= PARO_PAUSE_RANGE_MIN_BYTES &&
           bytes < (pl->P == 2 ? PARO_PAUSE_RANGE_MAX_BYTES_TWO : PARO_PAUSE_RANGE_MAX_BYTES);
}
// Whether sweep 1 stores all of the reduced gradient to stay in the memory-side cache, where sweep 2 finds it.  Contributions of a
// list with both types are counted as two-byte ones.
bool keeps_g(const paro_plan_t *pl, int layout) {
    const int64_t n = update_elems(pl), esize = pl->uniform_dtype && pl->dtype[0] == PARO_F32 ? 4 : 2;
    if (pl->P > PARO_BATCH && n > PARO_KEEP_STATE_ELEMS) return false;
    const int64_t most = layout == PARO_CHUNK && pl->P > PARO_KEEP_G_FEW_RANKS ? PARO_KEEP_G_WIDE_READ_BYTES : PARO_KEEP_G_READ_BYTES;
    return n <= PARO_KEEP_G_ELEMS && n * pl->P * esize <= most;
}
// ... and the block from which on it does (of a range of more than 2^32 blocks none does).
unsigned keeps_g_from(const paro_plan_t *pl, int layout) {
    if (keeps_g(pl, layout)) return 0;
    const int64_t block = std::max(update_elems(pl) - PARO_KEEP_G_TAIL_ELEMS, (int64_t)0) / PIECE;
    return (unsigned)std::min(block, (int64_t)UINT32_MAX);
}

int adam_consts(const paro_adam_t *hp, AdamConsts *a, const char *fn) {
    if (!hp) return fail(PARO_EINVAL, std::string(fn) + ": hp is NULL");
    if (hp->step < 1) return fail(PARO_EINVAL, std::string(fn) + ": step must be >= 1");
    if (!(hp->beta1 >= 0.0f && hp->beta1 < 1.0f && hp->beta2 >= 0.0f && hp->beta2 < 1.0f))
        return fail(PARO_EINVAL, std::string(fn) + ": betas must lie in [0, 1)");
    // element-independent scalars: formed in fp64 from the fp32 hyper-parameters, rounded once
    const double b1 = hp->beta1, b2 = hp->beta2;
    const float bc1 = (float)(1.0 - std::pow(b1, (double)hp->step));
    const float bc2 = (float)(1.0 - std::pow(b2, (double)hp->step));
    a->beta1 = hp->beta1;
    a->beta2 = hp->beta2;
    a->omb1 = (float)(1.0 - b1);
    a->omb2 = (float)(1.0 - b2);
    a->eps = hp->eps;
    a->step_size = (float)((double)hp->lr / (double)bc1);
    a->sqrt_bc2 = (float)std::sqrt((double)bc2);
    a->decay = (float)(1.0 - (double)hp->lr * (double)hp->weight_decay);
    a->wd = hp->weight_decay;
    a->grad_scale = hp->grad_scale;
    a->max_norm = hp->max_norm;
    a->adamw = hp->adamw ? 1 : 0;
    a->skip_nonfinite = hp->skip_nonfinite ? 1 : 0;
    return PARO_OK;
}

// ... and what the plan says.
void plan_consts(const paro_plan_t *pl, AdamConsts *a) {
    a->pack_dtype = pl->pack_dtype;
    a->keep_state = update_elems(pl) <= PARO_KEEP_STATE_ELEMS;
}

// Pointer table of a chunk in fold order.  Chunk layout: pointers advanced to the
// chunk's first element inside the update range.
void src_table(const paro_plan_t *pl, int chunk, const void *const *contrib, int layout, int64_t chunk_off_in_range,
               SrcTable *tab, int *group_len) {
    tab->keep_from = keeps_g_from(pl, layout);
    tab->paced = paces(pl) || holds_back(pl);
    int32_t order[PARO_MAX_RANKS];
    int32_t gl = 0;
    paro::fold_order(pl, chunk, order, &gl);
    const int64_t esize = pl->dtype[0] == PARO_F32 ? 4 : 2;
    for (int k = 0; k < pl->P; ++k) {
        const char *base = static_cast<const char *>(contrib[order[k]]);
        tab->p[k] = layout == PARO_CHUNK ? base + chunk_off_in_range * esize : base;
    }
    for (int k = pl->P; k < PARO_MAX_RANKS; ++k) tab->p[k] = nullptr;
    *group_len = gl;
}

// ... and of a launch over an update range of several chunks: pointers in rank order, the order of
// each chunk's fold follows from the range map.
RangeMap range_map(const paro_plan_t *pl, int64_t ob, int64_t on, int own, const void *const *contrib, SrcTable *tab) {
    tab->keep_from = keeps_g_from(pl, PARO_CHUNK);
    // not with two-byte contributions of 16 ranks and more, where the pauses only delay (paced and not, 90 M elements in
    // all: P = 16, 2 chunks, clipped 969 and 947 us, single sweep 841 and 832; 8 chunks 957 and 930; P = 32, 4 chunks 1533
    // and 1452; P = 64, 8 chunks 2526 and 2493; but P = 8, 8 chunks 687 and 695, fp32 at P = 16 1426 and 1440)
    tab->paced = piece_count(on) >= 2 * PARO_PACE_MIN_BLOCKS && (pl->P < PARO_BATCH || pl->dtype[0] == PARO_F32);
    for (int q = 0; q < pl->P; ++q) tab->p[q] = contrib[q];
    for (int q = pl->P; q < PARO_MAX_RANKS; ++q) tab->p[q] = nullptr;
    const bool ring = pl->sched == PARO_RING;
    const int first = (int)(ob / pl->L);
    return RangeMap{pl->L, 1.0 / (double)pl->L, first, pl->G, pl->g, ring ? pl->P : pl->G, ring ? 1 : pl->g,
                    own < 0 ? -1 : own - first};
}

#define PARO_BY_DTYPE(dt, CALL)            \
    do {                                   \
        if ((dt) == PARO_BF16) {           \
            constexpr int DT = PARO_BF16;  \
            CALL;                          \
        } else if ((dt) == PARO_F16) {     \
            constexpr int DT = PARO_F16;   \
            CALL;                          \
        } else {                           \
            constexpr int DT = PARO_F32;   \
            CALL;                          \
        }                                  \
    } while (0)

SrcTableOf<FEW_SRC> few_sources(const SrcTable &tab) {
    SrcTableOf<FEW_SRC> few;
    std::copy(tab.p, tab.p + FEW_SRC, few.p);
    few.paced = tab.paced;
    few.keep_from = tab.keep_from;
    return few;
}
// ... with the windows of a launch that holds back (window() works them out), which the others neither need nor wait for.
template <bool HELD, int N, class Window>
decltype(auto) with_window(const SrcTableOf<N> &src, Window window) {
    if constexpr (HELD) {
        SrcTableOf<N, true> held;
        static_cast<SrcTableOf<N> &>(held) = src;
        held.window = window();
        return held;
    } else {
        return (src);
    }
}
// CALL with `src`, the pointer table in the size that the kernels for NSRC pointers take.
#define PARO_BY_TABLE(P, tab, CALL)              \
    do {                                         \
        if ((P) <= FEW_SRC) {                    \
            constexpr int NSRC = FEW_SRC;        \
            const auto src = few_sources(tab);   \
            CALL;                                \
        } else {                                 \
            constexpr int NSRC = PARO_MAX_RANKS; \
            const SrcTable &src = tab;           \
            CALL;                                \
        }                                        \
    } while (0)

#define PARO_BY_FLAG(value, FLAG, ...)   \
    do {                                 \
        if (value) {                     \
            constexpr bool FLAG = true;  \
            __VA_ARGS__;                 \
        } else {                         \
            constexpr bool FLAG = false; \
            __VA_ARGS__;                 \
        }                                \
    } while (0)
#define PARO_BY_LINES(on_lines, ...) PARO_BY_FLAG(on_lines, NT, __VA_ARGS__)
// CALL with the constant MASK.
#define PARO_BY_MASK(mask, ...)                                        \
    do {                                                               \
        if ((mask) == MASK_NONE) {                                     \
            constexpr int MASK = MASK_NONE;                            \
            __VA_ARGS__;                                               \
        } else {                                                       \
            PARO_BY_FLAG((mask) == MASK_TABLE, TABLE, {                \
                constexpr int MASK = TABLE ? MASK_TABLE : MASK_TENSORS; \
                __VA_ARGS__;                                           \
            });                                                        \
        }                                                              \
    } while (0)

// Whether chunk c is cut into many small pieces of tensors (fewer than PARO_DENSE_BLOCKS_PER_TENSOR
// blocks per piece on average) rather than a few large ones.
bool many_small_tensors(const paro_plan_t *pl, int64_t c) {
    const int64_t f0 = c * pl->L, f1 = std::min((c + 1) * pl->L, pl->total);
    if (f0 >= f1) return false;                                             // all padding
    const auto first = std::upper_bound(pl->nz_off.begin(), pl->nz_off.end(), f0) - 1;
    const auto last = std::lower_bound(pl->nz_off.begin(), pl->nz_off.end(), f1);
    const int64_t pieces = last - first;
    return (int64_t)piece_grid(pl->L) < pieces * PARO_DENSE_BLOCKS_PER_TENSOR;
}

// Blocks, counted from the start of the update range, that hold elements of the chunk that starts at lo.
int64_t chunk_blocks(const paro_plan_t *pl, int64_t lo) { return piece_count(lo % PIECE + pl->L); }

// Launches sweep 1 over chunk c, which starts at element lo of the update range (and of the arrays that it
// gets); returns the number of per-block partial sums it writes.
template <bool SUMSQ>
int launch_reduce(const paro_plan_t *pl, const Scratch &sc, int layout, const SrcTable &tab, int group_len, int64_t c,
                  int64_t lo, float *g_range, hipStream_t st) {
    const int64_t n = pl->L;
    float *g = g_range + lo;
    double *partials = sc.partials;
    if (layout == PARO_CHUNK) {
        const unsigned grid = (unsigned)((chunk_blocks(pl, lo) + 7) & ~(int64_t)7);       // a multiple of 8: see partial_slot()
        const bool held = holds_back(pl);
        const int waves = held ? window_waves(pl) : fold_waves(fold_loads(pl->P), fold_budget(pl, paces(pl)));
        const unsigned lds = throttle_lds(sc.lds_per_cu, waves);
        PARO_BY_FLAG(held, HELD, PARO_BY_TABLE(pl->P, tab, PARO_BY_DTYPE(pl->dtype[0], {
            hipLaunchKernelGGL((k_reduce4<DT, SUMSQ, NSRC, HELD>), dim3(grid), dim3(WAVE), lds, st, lo, lo + n, pl->P, group_len, g_range,
                               partials, with_window<HELD>(src, [&] { return fold_window(pl); }));
        })));
        return (int)grid;
    }
    const TensorMap tm = map_for(pl, sc, c * pl->L, true);
    const int64_t pieces = tm.pieces ? tm.n_pieces : piece_count(n);
    // Streaming loads where the blocks start on cache lines (see Tensor4Loader).  A wave's kilobyte of an fp32 tensor
    // shares only one line in nine with a neighbour: in a large chunk streaming is better there as well, but with 5 to
    // 8 contributions (ragged tensors, whole clipped step, plain and streaming: 80 M elements, P = 4 677 and 662 us,
    // P = 16 1457 and 1441; 40 M, P = 6 394 and 398, P = 64 2289 and 2162; 10 M, P = 4, which fit the caches, 85 and 92).
    // In the single sweep it is not (P = 8, 80 M: 834 and 872).
    const bool f32_streams = pl->dev.f32[(size_t)c] && piece_count(n) >= PARO_LARGE_TILES && (pl->P <= PARO_PAIR_MAX_RANKS || pl->P > 8);
    const bool on_lines = pl->dev.on_lines[(size_t)c] || f32_streams;
    // The end of a large gradient is kept chunk by chunk, and only beside streaming loads of blocks on cache lines: plain ones fill the cache
    // themselves (whole clipped steps, neither kept nor, and kept: Llama-like lists, P = 8, 28 M elements 371 -> 350 us, P = 4, 57 M 615 -> 600, P = 12, 19 M
    // 291 -> 276; not on lines, P = 16, 14 M 265 -> 267; ragged tensors, P = 8, 66 M 588 -> 600, P = 16, 33 M 430 -> 436).
    const bool keep = keeps_g(pl, layout) || (pl->dev.on_lines[(size_t)c] && lo >= (int64_t)tab.keep_from * PIECE);
    // What decides is the list, see PARO_PAIR_MAX_RANKS.
    const bool small = many_small_tensors(pl, c);
    const bool few = pl->P <= PARO_PAIR_MAX_RANKS;
    int64_t pair_min_blocks = few ? PARO_PAIR_MIN_BLOCKS : PARO_LARGE_TILES;
    if (const char *env = std::getenv("PARO_PAIR_MIN_BLOCKS")) pair_min_blocks = std::atoll(env);     // for tests
    const bool pairs = few || (pl->P <= PARO_PAIR_SMALL_MAX_RANKS && small && !pl->dev.f32[(size_t)c]);
    if (pairs && piece_count(n) >= pair_min_blocks) {
        const unsigned grid = (unsigned)(((pieces + 1) / 2 + 7) & ~(int64_t)7);
        PARO_BY_FLAG(keep, KEEP, PARO_BY_FLAG(on_lines, NT, {
            if (few)
                hipLaunchKernelGGL((k_reduce4t<SUMSQ, 2, PARO_PAIR_MAX_RANKS, NT, FEW_SRC, KEEP>), dim3(grid), dim3(WAVE), 0, st, n,
                                   tm.pieces, tm.n_pieces, pl->P, group_len, g, partials, few_sources(tab), tm);
            else
                hipLaunchKernelGGL((k_reduce4t<SUMSQ, 2, 8, NT, FEW_SRC, KEEP>), dim3(grid), dim3(WAVE), 0, st, n,
                                   tm.pieces, tm.n_pieces, pl->P, group_len, g, partials, few_sources(tab), tm);
        }));
        return (int)grid;
    }
    const unsigned grid = (unsigned)((pieces + 7) & ~(int64_t)7);
    // fp32 gradients in a large chunk want a budget whatever the list (whole clipped steps, before and now: ragged tensors,
    // P = 8, 59 M elements 672 and 634 us, P = 16 652 and 620, P = 32 544 and 526; a Llama-like list, P = 8 2977 and 2942, P = 32 2970 and 2847)
    const bool f32_large = pl->dev.f32[(size_t)c] && piece_count(n) >= PARO_LARGE_TILES;
    const int budget = f32_large ? PARO_FOLD_F32_LIST_LOADS_PER_CU : small ? PARO_FOLD_TM_LOADS_PER_CU : PARO_FOLD_LOADS_PER_CU;
    // Waves that look up 48 pointers and more want company: all that fit (whole clipped steps, by the budget and so: Llama-like lists, P = 64, 20 M elements 622 and 503 us,
    // 8 M 256 and 228, 6 M 179.8 and 177.8; P = 128, 10 M 710 and 584; P = 48, 28 M 668 and 662; fp32, P = 64, 11 M 521 and 516; but P = 40, 33 M 543 and 546; GPT-2's, P = 64, 1.9 M 71.2 and 72.2)
    // A large chunk of fp32 gradients keeps its budget up to 55 ranks and where its tensors are many and small (P = 48, 38 M 1447 and 1473, 56 M 2097 and 2142; P =
    // 50, 43 M 1558 and 1594, P = 52 1819 and 1841; ragged tensors, P = 48 1512 and 1557, P = 64 1925 and 1981; but P = 56, 41 M 1713 and 1561, 64 M 2670 and 2618;
    // P = 64, 39 M 1905 and 1708; P = 80 2490 and 2402; P = 128, 35 M 3288 and 3161).
    const bool all = pl->P >= 3 * PARO_BATCH && piece_count(n) >= PARO_ALL_WAVES_MIN_BLOCKS &&
                     (!f32_large || (!small && pl->P >= PARO_ALL_WAVES_F32_LARGE_RANKS));
    const unsigned lds = throttle_lds(sc.lds_per_cu, all ? 0 : fold_waves(fold_loads(pl->P), budget));
    PARO_BY_FLAG(keep, KEEP, PARO_BY_FLAG(on_lines, NT, {
        if (pl->P <= 8)                                                     // a batch of 8 contributions: fewer registers
            hipLaunchKernelGGL((k_reduce4t<SUMSQ, 1, 8, NT, FEW_SRC, KEEP>), dim3(grid), dim3(WAVE), lds, st, n, tm.pieces,
                               tm.n_pieces, pl->P, group_len, g, partials, few_sources(tab), tm);
        else
            PARO_BY_TABLE(pl->P, tab, hipLaunchKernelGGL((k_reduce4t<SUMSQ, 1, PARO_BATCH, NT, NSRC, KEEP>), dim3(grid), dim3(WAVE), lds,
                                                         st, n, tm.pieces, tm.n_pieces, pl->P, group_len, g, partials, src, tm));
    }));
    return (int)grid;
}

// Whether there are single sweeps with write windows for NSRC pointers: two-byte contributions have none of up to FEW_SRC ranks.
template <int DT, int NSRC>
constexpr bool FUSED_HOLDS = DT == PARO_F32 || NSRC > FEW_SRC;
static_assert(PARO_FUSED_WINDOW_RANK_BYTES > 2 * FEW_SRC && PARO_FUSED_RANGE_WINDOW_MIN_RANKS > FEW_SRC, "see FUSED_HOLDS");

// Launches the single sweep (no clipping) over chunk c.
void launch_fused(const paro_plan_t *pl, const Scratch &sc, int layout, const SrcTable &tab, int group_len, int64_t c,
                  const AdamConsts &a, float *p, float *m, float *v, uint16_t *dst, hipStream_t st) {
    const int64_t n = pl->L;
    const bool small = layout == PARO_TENSORS && many_small_tensors(pl, c), large = piece_count(n) >= PARO_LARGE_TILES;
    const bool f32 = layout == PARO_TENSORS ? pl->dev.f32[(size_t)c] != 0 : pl->dtype[0] == PARO_F32;
    const Sweep over = layout == PARO_CHUNK ? Sweep::CHUNK
                       : !small && pl->dev.on_lines[(size_t)c] ? Sweep::TENSORS_ON_LINES : Sweep::OTHER_TENSORS;
    int waves = small && !large ? fold_waves(fold_loads(pl->P) + 3, PARO_FOLD_TM_LOADS_PER_CU)
                                : fused_waves(pl->P, f32, over, piece_count(n));
    // A large chunk of many small tensors: the budget's 10 waves at P > 8 are too few to hide the look-ups, all that
    // fit too many for DRAM (bf16, budget, 20 waves, all: P = 12, 80 M elements 820, 686, 793 us; P = 16, 115 M 1410,
    // 1197, 1271; P = 64, 80 M 2667, 2408; a quarter fp32, P = 16, 80 M 1021, 935).  fp32 gradients, whose loads are twice
    // as wide and half as many, want the budget (P = 16, 80 M: 1314, 1443).
    if (small && large && pl->P > 8 && !pl->dev.f32[(size_t)c]) waves = PARO_FUSED_TL_WAVES_PER_CU;
    const bool held = layout == PARO_CHUNK && fused_holds_back(pl, n);
    if (held) waves = fused_window_waves(pl);
    const TensorMap tm = map_for(pl, sc, c * pl->L, true);
    const unsigned grid = piece_grid(n), lds = throttle_lds(sc.lds_per_cu, waves);
    const int mask = !pl->any_no_decay ? MASK_NONE : layout == PARO_CHUNK && tm.decay_tab ? MASK_TABLE : MASK_TENSORS;
    if (layout == PARO_TENSORS)
        PARO_BY_TABLE(pl->P, tab, PARO_BY_FLAG(mask != MASK_NONE, MASKED, PARO_BY_LINES(pl->dev.on_lines[(size_t)c] != 0, {
            hipLaunchKernelGGL((k_fused4<true, PARO_BF16, MASKED ? MASK_TENSORS : MASK_NONE, NT, NSRC, 0, false>),
                               dim3(tm.pieces ? tm.n_pieces : grid), dim3(WAVE), lds, st, n, p, m, v, tm.pieces, tm.n_pieces, pl->P,
                               group_len, src, a, dst, tm);
        })));
    else if (pauses_single(pl, n))
        PARO_BY_DTYPE(pl->dtype[0], PARO_BY_MASK(mask, {
            hipLaunchKernelGGL((k_fused4<false, DT, MASK, true, FEW_SRC, PARO_PAUSE_SLEEP, false>), dim3(grid), dim3(WAVE), lds, st, n, p, m, v,
                               tm.pieces, tm.n_pieces, pl->P, group_len, few_sources(tab), a, dst, tm);
        }));
    else
        PARO_BY_FLAG(held, HELD, PARO_BY_TABLE(pl->P, tab, PARO_BY_DTYPE(pl->dtype[0], PARO_BY_MASK(mask, {
            if constexpr (!HELD || FUSED_HOLDS<DT, NSRC>)
                hipLaunchKernelGGL((k_fused4<false, DT, MASK, true, NSRC, 0, HELD>), dim3(grid), dim3(WAVE), lds, st, n, p, m, v, tm.pieces, tm.n_pieces,
                                   pl->P, group_len, with_window<HELD>(src, [&] { return fused_window(pl); }), a, dst, tm);
        }))));
}

// ... over an update range of several chunks (chunk layout, no decay mask).
int launch_fused_range(const paro_plan_t *pl, const Scratch &sc, int64_t ob, int64_t on, const void *const *contrib,
                       const AdamConsts &a, float *p, float *m, float *v, uint16_t *dst, hipStream_t st) {
    SrcTable tab;
    const RangeMap rm = range_map(pl, ob, on, -1, contrib, &tab);
    const bool held = fused_range_holds_back(pl, on), held_paced = fused_range_paces(pl);
    const int waves = held ? fused_window_waves(pl) : fused_waves(pl->P, pl->dtype[0] == PARO_F32, Sweep::RANGE, piece_count(on));
    const unsigned lds = throttle_lds(sc.lds_per_cu, waves);
    if (pauses_range(pl, on)) {                                 // (one grid holds what pauses)
        PARO_BY_DTYPE(pl->dtype[0], hipLaunchKernelGGL((k_fused4r<DT, FEW_SRC, PARO_PAUSE_SLEEP, false>), dim3(piece_grid(on)), dim3(WAVE), lds, st,
                                                       (int64_t)0, on, p, m, v, pl->P, rm, few_sources(tab), a, dst));
        PARO_HIP(hipGetLastError());
        return PARO_OK;
    }
    if (held) tab.paced = held_paced;
    for (int64_t b0 = 0, blocks = piece_count(on); b0 < blocks; b0 += MAX_GRID) {
        const unsigned grid = (unsigned)std::min(MAX_GRID, blocks - b0);
        PARO_BY_FLAG(held, HELD, PARO_BY_TABLE(pl->P, tab, PARO_BY_DTYPE(pl->dtype[0], {
            if constexpr (!HELD || FUSED_HOLDS<DT, NSRC>)
                hipLaunchKernelGGL((k_fused4r<DT, NSRC, 0, HELD>), dim3(grid), dim3(WAVE), lds, st, b0, on, p, m, v, pl->P, rm,
                                   with_window<HELD>(src, [&] { return fused_window(pl, held_paced); }), a, dst);
        })));
        PARO_HIP(hipGetLastError());
    }
    return PARO_OK;
}

// The sum of squares as sweep 1 leaves it for sweep 2: n sums on the device, whose total belongs in *out.
// out null: the one sum is the total, in its place already.
struct NormSums {
    const double *sums;
    int n;
    double *out;
};

// The total of what is left, in its place: for the call that no sweep 2 follows.
int total_of(const NormSums &s, hipStream_t st) {
    PARO_BY_FLAG(s.n > NORM_SLICES, MANY, hipLaunchKernelGGL(k_norm_total<MANY>, dim3(1), dim3(WAVE), 0, st, s.sums, s.n, s.out));
    PARO_HIP(hipGetLastError());
    return PARO_OK;
}

// Adds the n_part partial sums a sweep-1 launch left in the scratch array into *out (device) - or, with
// `rest`, only as far as sweep 2 goes on by itself, and *rest says from where.  Either way the same adds in
// the same order: the fused step clips by the value that paro_reduce_shard leaves, to the last bit.  Every
// kernel more in this chain of short dependent ones costs 2-3 us of a step; what a wave of sweep 2 adds up
// beside its state loads is hidden while it is little.  Whole clipped steps at P = 8, bf16, with the chain of up to two
// small kernels that ended in one scalar, and now:
//   0.5 M elements (1954 partials, added up by every wave)   12.9 -> 10.4 us
//   0.75 M (2930; eight slice sums)                          13.7 -> 13.3; added up by every wave 16.5
//   1.5 M (5860; eight slice sums)                           21.7 -> 19.6
//   16.8 M (65536; eight slice sums)                        135.7 -> 133.7
// Sixteen slice sums fetched one after the other took back all of it at 16 M; eight are one scalar load.
int finalize_partials(const Scratch &sc, const double *partials, int n_part, double *out, hipStream_t st,
                      NormSums *rest = nullptr) {
    if (n_part <= NORM_DIRECT_PARTIALS) {
        const NormSums all{partials, n_part, out};
        return rest ? (*rest = all, PARO_OK) : total_of(all, st);
    }
    const int chunk = (n_part + NORM_SLICES - 1) / NORM_SLICES;
    if (!rest && n_part <= NORM_ONE_BLOCK_PARTIALS) {
        hipLaunchKernelGGL(k_norm_slices_total, dim3(1), dim3(FINALIZE_TPB), 0, st, partials, n_part, chunk, out);
        PARO_HIP(hipGetLastError());
        return PARO_OK;
    }
    if (n_part <= NORM_SLICES_PARTIALS) {
        hipLaunchKernelGGL(k_finalize, dim3(NORM_SLICES), dim3(FINALIZE_TPB), 0, st, partials, n_part, chunk, sc.level2);
        PARO_HIP(hipGetLastError());
        const NormSums slices{sc.level2, NORM_SLICES, out};
        return rest ? (*rest = slices, PARO_OK) : total_of(slices, st);
    }
    // two levels: slices of FINALIZE_CHUNK partials, then their sums
    const int nb = (n_part + FINALIZE_CHUNK - 1) / FINALIZE_CHUNK;
    hipLaunchKernelGGL(k_finalize, dim3(nb), dim3(FINALIZE_TPB), 0, st, partials, n_part, FINALIZE_CHUNK, sc.level2);
    PARO_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(FINALIZE_TPB), 0, st, sc.level2, nb, nb, out);
    PARO_HIP(hipGetLastError());
    if (rest) *rest = NormSums{out, 1, nullptr};
    return PARO_OK;
}

// ... and the sums of several chunks, launches or groups, in sc.chunk_sums.  Up to eight of them are left to
// sweep 2's scalar loads; adding more across the lanes would cost every wave of a large sweep more than one small
// kernel (two sums, 100 M elements: sweep 2 505 us, 470 from one scalar).
int finalize_sums(const Scratch &sc, int n, double *out, hipStream_t st, NormSums *rest) {
    const NormSums all{sc.chunk_sums, n, out};
    if (rest) *rest = n <= NORM_SLICES ? all : NormSums{out, 1, nullptr};
    return rest && n <= NORM_SLICES ? PARO_OK : total_of(all, st);
}

// Sweep 1 over an update range of several chunks, chunk layout: one launch, or, where the norm covers
// the whole range and the scratch array is too small for its partial sums, one for each piece that fits.
// The norm is formed in groups of NORM_GROUP blocks, as many as the static array holds, whose sums are added
// in order: the same value from either scratch array, however many launches it takes.
// own >= 0: the sum of squares of that chunk alone.
int do_reduce_range(const paro_plan_t *pl, const Scratch &sc, int64_t ob, int64_t on, int own, const void *const *contrib,
                    float *grad_out, double *sumsq_out, hipStream_t st, NormSums *rest) {
    int rc;
    SrcTable tab;
    const RangeMap rm = range_map(pl, ob, on, own, contrib, &tab);
    // A small range of two-byte contributions is launched with all waves that fit.  Whole clipped steps, by the budget and so: P = 16, 2 x 0.5 M elements 15.8 -> 14.3
    // us, 2 x 1 M 26.9 -> 25.5, 2 x 1.5 M 37.1 -> 36.6; P = 24, 2 x 0.5 M 18.8 -> 17.0; P = 32, 2 x 0.5 M 22.0 -> 19.7, 2 x 1 M 38.1 -> 37.0; P = 64, 2 x 0.5 M 33.7 -> 30.6, 2 x 1.9 M 107.4 -> 107.0; P = 12, 2 x
    // 1 M 23.8 -> 22.9; P = 10 22.2 -> 21.7; P = 8 21.1 -> 21.0, P = 4 19.3 -> 19.2; fp32, P = 16, 2 x 1 M 36.0 -> 36.2; but P = 12, 2 x 2.2 M 44.7 -> 45.0, 2 x 6 M 107.8 -> 109.2.
    const bool held = range_holds_back(pl), all = pl->dtype[0] != PARO_F32 && pl->P > 8 && piece_count(on) < PARO_RANGE_WINDOW_MIN_BLOCKS;
    const int waves = held ? window_waves(pl) : all ? 0 : fold_waves(fold_loads(pl->P), fold_budget(pl, false));
    if (held) tab.paced = pl->dtype[0] == PARO_F32;
    const auto window = [&] { return fold_window(pl, true); };
    const unsigned lds = throttle_lds(sc.lds_per_cu, waves);
    const int64_t blocks = (piece_count(on) + 7) & ~(int64_t)7;
    const int64_t step = sumsq_out ? std::min(sc.n_partials, MAX_GRID) : MAX_GRID;
    int n_sums = 0;
    bool one_sum = false;
    for (int64_t b0 = 0; b0 < blocks; b0 += step) {
        const int64_t grid = std::min(step, blocks - b0);
        int64_t first = b0, last = b0 + grid;                     // the blocks whose squares count
        if (own >= 0) {
            const int64_t lo = own * pl->L - ob;
            first = std::max((lo / PIECE) & ~(int64_t)7, first);
            last = std::min((piece_count(lo + pl->L) + 7) & ~(int64_t)7, last);
        }
        if (sumsq_out && first < last) {
            PARO_BY_FLAG(held, HELD, PARO_BY_TABLE(pl->P, tab, PARO_BY_DTYPE(pl->dtype[0], {
                hipLaunchKernelGGL((k_reduce4r<DT, true, NSRC, HELD>), dim3((unsigned)grid), dim3(WAVE), lds, st, b0, on,
                                   pl->P, (unsigned)(first - b0), (unsigned)(last - first), grad_out, sc.partials, rm,
                                   with_window<HELD>(src, window));
            })));
            PARO_HIP(hipGetLastError());
            // the next launch reuses the scratch array: this one's partials are added up first
            one_sum = step >= blocks && last - first <= NORM_GROUP;
            for (int64_t k = 0; k < last - first; k += NORM_GROUP) {
                const int n_part = (int)std::min(last - first - k, (int64_t)NORM_GROUP);
                if (one_sum)
                    rc = finalize_partials(sc, sc.partials, n_part, sumsq_out, st, rest);
                else
                    rc = finalize_partials(sc, sc.partials + k, n_part, sc.chunk_sums + n_sums++, st);
                if (rc) return rc;
            }
        } else {
            PARO_BY_FLAG(held, HELD, PARO_BY_TABLE(pl->P, tab, PARO_BY_DTYPE(pl->dtype[0], {
                hipLaunchKernelGGL((k_reduce4r<DT, false, NSRC, HELD>), dim3((unsigned)grid), dim3(WAVE), lds, st, b0, on,
                                   pl->P, 0u, 0u, grad_out, sc.partials, rm, with_window<HELD>(src, window));
            })));
            PARO_HIP(hipGetLastError());
        }
    }
    return sumsq_out && !one_sum ? finalize_sums(sc, n_sums, sumsq_out, st, rest) : PARO_OK;
}

// Whether sweep 1 over an update range of several chunks in the chunk layout goes chunk by chunk.  A wave of the
// one launch over the range works out its chunk and the order of its ranks before its first load; with few
// contributions of two bytes that is as much work as the fold (P = 2, two chunks of 50 M: 200 us against 2 x 66), and
// large chunks repay a launch each; with many, only launches over one chunk are paced to advantage.  Whole clipped steps, one
// launch and one per chunk, from how many blocks on:
//   up to 4 ranks, two bytes, 65 536    P = 2, 2 x 24 M 310 and 294 us, 2 x 120 M 1517 and 1400; P = 4, 2 x 50 M 664 and 643; but 4 x 12 M
//                                       321 and 331, fp32 2 x 60 M 906 and 918
//   two bytes, 12 to 99 ranks, 131 072  where the one launch has write windows, P = 16, 2 x 40 M 793 and 788; P = 48, 2 x 40 M 1528 and 1514; P = 24, 2 x 50 M 1252 and 1199;
//                                       but P = 32, 2 x 18 M 511 and 521, P = 64, 4 x 14 M 1362 and 1380, 8 x 9 M 1717 and 1785; P = 12, 2 x 40 M 700 and 705,
//                                       on another GPU 702 and 701, 2 x 60 M 1051 and 1040, P = 16, 2 x 35 M 692 and 689, 2 x 60 M 1186 and 1167; P = 32,
//                                       2 x 32 M 913 and 922; P = 100, 2 x 20 M 1415 and 1452; P = 128, 2 x 20 M 1760 and 1800; P = 8 (no windows),
//                                       2 x 60 M 920 and 919, 8 x 17 M 1029 and 1083
//   fp32, 8 to 11 ranks, 131 072        P = 8, 2 x 40 M 826 and 812; but 8 x 15 M 1232 and 1277; with 12 and more, where the one launch has write
//                                       windows, P = 24, 3 x 20 M 1172 and 1202, P = 16, 2 x 60 M 1785 and 1787
bool chunk_by_chunk(const paro_plan_t *pl) {
    const int P = pl->P;
    int64_t from;
    if (pl->dtype[0] == PARO_F32) from = P < 8 || P >= PARO_WINDOW_MIN_RANKS ? 0 : PARO_RANGE_MAX_BLOCKS * 2;
    else from = P <= PARO_PAIR_MAX_RANKS ? PARO_RANGE_MAX_BLOCKS : P < 12 || P >= PARO_RANGE_ALWAYS_RANKS ? 0 : PARO_RANGE_MAX_BLOCKS * 2;
    if (!from) return false;
    const int64_t blocks = (chunk_blocks(pl, PIECE - 1) + 7) & ~(int64_t)7;       // at most
    // (no more than a group of the norm, so that the scratch array does not matter)
    return blocks >= from && blocks <= (pl->L > PARO_STATIC_MAX_CHUNK ? MAX_GRID : (int64_t)NORM_GROUP);
}

// Sweep 1 over the whole update range, chunk by chunk.  The sum of squares covers the rank's own
// chunk only (so that the ranks' values add up to the model's) - or, with norm_over_range, every
// chunk of the update range, in a fixed order.  rest: sweep 2 finishes the norm.
int do_reduce(const paro_plan_t *pl, const Scratch &sc, int rank, const void *const *contrib, int layout, float *grad_out,
              double *sumsq_out, bool norm_over_range, hipStream_t st, NormSums *rest = nullptr) {
    int rc;
    int64_t ob, on;
    paro::letter_range(pl, rank, pl->letters[2], &ob, &on);
    const int own = paro::chunk_of_rank(pl, rank);
    const int64_t c0 = ob / pl->L, c1 = (ob + on) / pl->L;
    if (layout == PARO_CHUNK && c1 - c0 > 1 && !chunk_by_chunk(pl))
        return do_reduce_range(pl, sc, ob, on, norm_over_range ? -1 : own, contrib, grad_out, sumsq_out, st, rest);
    const bool per_chunk = sumsq_out && norm_over_range && c1 - c0 > 1;
    for (int64_t c = c0; c < c1; ++c) {
        SrcTable tab;
        int gl;
        const int64_t lo = c * pl->L - ob;
        src_table(pl, (int)c, contrib, layout, 0, &tab, &gl);
        if (sumsq_out && (per_chunk || c == own)) {
            const int n_part = launch_reduce<true>(pl, sc, layout, tab, gl, c, lo, grad_out, st);
            PARO_HIP(hipGetLastError());
            // the next launch reuses the scratch array: this chunk's partials are added up first
            rc = per_chunk ? finalize_partials(sc, sc.partials, n_part, sc.chunk_sums + (c - c0), st)
                           : finalize_partials(sc, sc.partials, n_part, sumsq_out, st, rest);
            if (rc) return rc;
        } else {
            launch_reduce<false>(pl, sc, layout, tab, gl, c, lo, grad_out, st);
            PARO_HIP(hipGetLastError());
        }
    }
    return per_chunk ? finalize_sums(sc, (int)(c1 - c0), sumsq_out, st, rest) : PARO_OK;
}

template <bool PACK, bool KEPT>
int launch_adam(const paro_plan_t *pl, const Scratch &sc, int rank, const AdamConsts &a, const float *grad,
                const NormSums &norm, float *p, float *m, float *v, uint16_t *dst, hipStream_t st) {
    int64_t ob, on;
    paro::letter_range(pl, rank, pl->letters[2], &ob, &on);
    const bool many = norm.n > NORM_SLICES;
    if (!pl->any_no_decay) {
        const int waves = on <= PARO_ADAM_SMALL_ELEMS ? PARO_ADAM_MASK_WAVES_PER_CU
                          : piece_count(on) < PARO_LARGE_TILES ? PARO_ADAM_WAVES_PER_CU : PARO_ADAM_LARGE_WAVES_PER_CU;
        const unsigned lds = throttle_lds(sc.lds_per_cu, waves);
        PARO_BY_FLAG(many, MANY, {
            hipLaunchKernelGGL((k_adam4<PACK, MASK_NONE, KEPT, MANY>), dim3(piece_grid(on)), dim3(WAVE), lds, st, on, grad, p, m, v,
                               norm.sums, norm.n, a, dst, norm.out, map_for(pl, sc, ob, false));
        });
        PARO_HIP(hipGetLastError());
        return PARO_OK;
    }
    for (int64_t c = ob / pl->L; c < (ob + on) / pl->L; ++c) {      // chunk by chunk: each has its own weight-decay table
        const int64_t lo = c * pl->L - ob;
        const unsigned lds = throttle_lds(sc.lds_per_cu, PARO_ADAM_MASK_WAVES_PER_CU), grid = piece_grid(pl->L);
        const TensorMap tm = map_for(pl, sc, c * pl->L, true);
        uint16_t *dst_c = dst ? dst + lo : nullptr;
        PARO_BY_FLAG(many, MANY, PARO_BY_FLAG(tm.decay_tab != nullptr, TABLE, {
            hipLaunchKernelGGL((k_adam4<PACK, TABLE ? MASK_TABLE : MASK_TENSORS, TABLE && KEPT, MANY>), dim3(grid), dim3(WAVE), lds, st,
                               pl->L, grad + lo, p + lo, m + lo, v + lo, norm.sums, norm.n, a, dst_c, norm.out, tm);
        }));
        PARO_HIP(hipGetLastError());
    }
    return PARO_OK;
}

// Sweep 2 behind sweep 1, whose gradient may be in the memory-side cache (kept), or with a gradient that another call, or another program's kernel, left anywhere:
// that is read with streaming loads, the last block first unless there is a mask (paro_adam_shard alone, from the start and from the end, P = 8: gradient just
// copied in, 6 M elements 32.8 and 32.8 us, 30 M 137.5 and 136.9, 50 M 220.6 and 218.4, 120 M 535 and 533, 400 M 1775 and 1776; after 512 MB of something else, 12 M
// 58.9 and 58.9, 50 M 225.0 and 222.1, 120 M 536 and 533).  Plain loads of a gradient that is no longer in the cache drive out of it what other kernels wrote there
// (paro_adam_shard after 512 MB of something else, P = 8, streaming and plain: 4 M elements 25.0 and 27.6 us, 12 M 58.4 and 65.7; of one just written 24.3 and 23.3,
// 55.8 and 54.4).
int do_adam(const paro_plan_t *pl, const Scratch &sc, int rank, const AdamConsts &a, const float *grad, bool kept,
            const NormSums &norm, float *p, float *m, float *v, uint16_t *dst /* nullable: no pack */, hipStream_t st) {
    return !dst ? launch_adam<false, false>(pl, sc, rank, a, grad, norm, p, m, v, dst, st)
           : kept ? launch_adam<true, true>(pl, sc, rank, a, grad, norm, p, m, v, dst, st)
                  : launch_adam<true, false>(pl, sc, rank, a, grad, norm, p, m, v, dst, st);
}

// The launches of the fused step, arguments already checked: two sweeps when the update waits for
// the norm (clipping, skip on overflow), else one.
int launch_step(const paro_plan_t *pl, const Scratch &sc, int rank, const void *const *contrib, int layout,
                const AdamConsts &a, float *grad_scratch, double *sumsq_scratch, float *p, float *m, float *v,
                uint16_t *dst_base, hipStream_t st) {
    int rc;
    int64_t dl, so, sl, ob, on;
    paro_pack_slot(pl, rank, &dl, &so, &sl);
    uint16_t *dst = dst_base + so;
    if (a.max_norm > 0.0f || a.skip_nonfinite) {
        // the norm this rank can form on its own: over everything it updates (its update range)
        NormSums norm{nullptr, 0, nullptr};
        if ((rc = do_reduce(pl, sc, rank, contrib, layout, grad_scratch, sumsq_scratch, true, st, &norm))) return rc;
        return do_adam(pl, sc, rank, a, grad_scratch, keeps_g(pl, layout), norm, p, m, v, dst, st);
    }
    paro::letter_range(pl, rank, pl->letters[2], &ob, &on);
    if (layout == PARO_CHUNK && !pl->any_no_decay && on > pl->L) return launch_fused_range(pl, sc, ob, on, contrib, a, p, m, v, dst, st);
    for (int64_t c = ob / pl->L; c < (ob + on) / pl->L; ++c) {
        SrcTable tab;
        int gl;
        const int64_t lo = c * pl->L - ob;
        src_table(pl, (int)c, contrib, layout, lo, &tab, &gl);
        tab.paced = paces(pl) || fused_holds_back(pl, pl->L);
        launch_fused(pl, sc, layout, tab, gl, c, a, p + lo, m + lo, v + lo, dst + lo, st);
        PARO_HIP(hipGetLastError());
    }
    return PARO_OK;
}

// ---- the library's own scratch, for the entry point that allocates nothing --------------------
// Partial sums of squares of one sweep-1 launch over a chunk of at most PARO_STATIC_MAX_CHUNK
// elements (one per block of 256), followed by the second-level sums.  Every device the library
// runs on holds its own copy of this array, at its own address, until the process ends.
constexpr int64_t STATIC_PARTIALS = PARO_STATIC_MAX_CHUNK / PIECE;
constexpr int64_t STATIC_LEVEL2 = level2_sums(STATIC_PARTIALS);
static_assert(STATIC_PARTIALS == NORM_GROUP, "a launch on the static array is one group of the norm");
static __device__ __align__(256) double scratch[STATIC_PARTIALS + STATIC_LEVEL2 + PARO_MAX_RANKS];

constexpr int MAX_DEVICES = 64;
struct StaticScratch {
    std::mutex mutex;
    double *ptr[MAX_DEVICES] = {};       // device address of `scratch` on each device, once asked for
    int lds_per_cu[MAX_DEVICES] = {};
};
StaticScratch g_static;

// The current device's copy of `scratch`.  In host code the array's name is only a handle for the
// runtime: its device address comes from hipGetSymbolAddress, once per device with that device
// current, and that address is what kernels, copies and fills get.  Allocates nothing.
int static_scratch(Scratch *out) {
    int dev = -1;
    PARO_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(PARO_EINVAL, "paro_step_fused_static: device index out of range");
    std::lock_guard<std::mutex> lock(g_static.mutex);
    if (!g_static.ptr[dev]) {
        double *ptr = nullptr;
        PARO_HIP(hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)));
        if (!ptr) return fail(PARO_EHIP, "hipGetSymbolAddress gave no address for the static scratch array");
        int lds = 0;
        if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess ||
            lds < 65536) {
            (void)hipGetLastError();
            lds = 160 * 1024;
        }
        g_static.lds_per_cu[dev] = lds;
        g_static.ptr[dev] = ptr;
    }
    *out = Scratch{g_static.lds_per_cu[dev], g_static.ptr[dev], STATIC_PARTIALS, g_static.ptr[dev] + STATIC_PARTIALS,
                   g_static.ptr[dev] + STATIC_PARTIALS + STATIC_LEVEL2, false};
    return PARO_OK;
}

}  // namespace

extern "C" {

void paro_plan_destroy(paro_plan_t *pl) {
    if (!pl) return;
    if (pl->dev.device >= 0) free_tables(pl->dev);
    delete pl;
}

int paro_reduce_shard(paro_plan_t *pl, int rank, const void *const *contrib, int layout, float *grad_out,
                      double *sumsq_out, void *stream) {
    int rc;
    if ((rc = check_common(pl, rank, "paro_reduce_shard"))) return rc;
    if ((rc = check_contrib(pl, contrib, layout, "paro_reduce_shard"))) return rc;
    if ((rc = check_ptr(grad_out, "paro_reduce_shard: grad_out"))) return rc;
    if (sumsq_out && (reinterpret_cast<uintptr_t>(sumsq_out) & 7))
        return fail(PARO_EALIGN, "paro_reduce_shard: sumsq_out is not 8-byte aligned");
    if ((rc = ensure_device(pl))) return rc;
    if (layout == PARO_TENSORS && (rc = ensure_tables(pl, rank, true, false))) return rc;
    return do_reduce(pl, plan_scratch(pl), rank, contrib, layout, grad_out, sumsq_out, false, static_cast<hipStream_t>(stream));
}

int paro_adam_shard(paro_plan_t *pl, int rank, const paro_adam_t *hp, const float *grad, const double *total_sumsq,
                    float *p, float *m, float *v, uint16_t *dst_base, void *stream) {
    int rc;
    AdamConsts a;
    if ((rc = check_common(pl, rank, "paro_adam_shard"))) return rc;
    if ((rc = adam_consts(hp, &a, "paro_adam_shard"))) return rc;
    if ((rc = check_ptr(grad, "paro_adam_shard: grad"))) return rc;
    if ((rc = check_ptr(p, "paro_adam_shard: p"))) return rc;
    if ((rc = check_ptr(m, "paro_adam_shard: m"))) return rc;
    if ((rc = check_ptr(v, "paro_adam_shard: v"))) return rc;
    if ((a.max_norm > 0.0f || a.skip_nonfinite) && !total_sumsq)
        return fail(PARO_EINVAL, "paro_adam_shard: clipping and skip_nonfinite need total_sumsq");
    plan_consts(pl, &a);
    if (dst_base && (reinterpret_cast<uintptr_t>(dst_base) & 15))
        return fail(PARO_EALIGN, "paro_adam_shard: dst_base is not 16-byte aligned");
    if ((rc = ensure_device(pl))) return rc;
    if (pl->any_no_decay && (rc = ensure_tables(pl, rank, false, true))) return rc;
    uint16_t *dst = nullptr;
    if (dst_base) {
        int64_t dl, so, sl;
        paro_pack_slot(pl, rank, &dl, &so, &sl);
        dst = dst_base + so;
    }
    const bool needs_norm = a.max_norm > 0.0f || a.skip_nonfinite;
    return do_adam(pl, plan_scratch(pl), rank, a, grad, false, NormSums{total_sumsq, needs_norm ? 1 : 0, nullptr}, p, m, v, dst,
                   static_cast<hipStream_t>(stream));
}

int paro_pack_params(paro_plan_t *pl, int rank, const float *p, uint16_t *dst_base, void *stream) {
    int rc;
    if ((rc = check_common(pl, rank, "paro_pack_params"))) return rc;
    if ((rc = check_ptr(p, "paro_pack_params: p"))) return rc;
    if ((rc = check_ptr(dst_base, "paro_pack_params: dst_base"))) return rc;
    if ((rc = ensure_device(pl))) return rc;
    int64_t dl, so, sl;
    paro_pack_slot(pl, rank, &dl, &so, &sl);
    hipLaunchKernelGGL(k_pack, dim3(piece_grid(sl)), dim3(WAVE), throttle_lds(pl->dev.lds_per_cu, PARO_COPY_WAVES_PER_CU),
                       static_cast<hipStream_t>(stream), p, dst_base + so, sl, pl->pack_dtype);
    PARO_HIP(hipGetLastError());
    return PARO_OK;
}

int paro_step_fused(paro_plan_t *pl, int rank, const void *const *contrib, int layout, const paro_adam_t *hp,
                    float *grad_scratch, double *sumsq_scratch, float *p, float *m, float *v, uint16_t *dst_base,
                    void *stream) {
    int rc;
    AdamConsts a;
    if ((rc = check_common(pl, rank, "paro_step_fused"))) return rc;
    if ((rc = check_contrib(pl, contrib, layout, "paro_step_fused"))) return rc;
    if ((rc = adam_consts(hp, &a, "paro_step_fused"))) return rc;
    if ((rc = check_ptr(p, "paro_step_fused: p"))) return rc;
    if ((rc = check_ptr(m, "paro_step_fused: m"))) return rc;
    if ((rc = check_ptr(v, "paro_step_fused: v"))) return rc;
    if ((rc = check_ptr(dst_base, "paro_step_fused: dst_base"))) return rc;
    plan_consts(pl, &a);
    const bool clip = a.max_norm > 0.0f || a.skip_nonfinite;       // both need the norm before the update
    if (clip) {
        if ((rc = check_ptr(grad_scratch, "paro_step_fused: grad_scratch"))) return rc;
        if (!sumsq_scratch || (reinterpret_cast<uintptr_t>(sumsq_scratch) & 7))
            return fail(sumsq_scratch ? PARO_EALIGN : PARO_EINVAL, "paro_step_fused: clipping and skip_nonfinite need sumsq_scratch");
    }
    if ((rc = ensure_device(pl))) return rc;
    const bool tensors = layout == PARO_TENSORS;          // its single sweep has the mask from the pieces
    if ((rc = ensure_tables(pl, rank, tensors, pl->any_no_decay && (clip || !tensors)))) return rc;
    return launch_step(pl, plan_scratch(pl), rank, contrib, layout, a, grad_scratch, sumsq_scratch, p, m, v, dst_base,
                       static_cast<hipStream_t>(stream));
}

int paro_step_fused_static(const paro_plan_t *pl, int rank, const void *const *contrib, const paro_adam_t *hp,
                           float *grad_scratch, double *sumsq_scratch, float *p, float *m, float *v,
                           uint16_t *dst_base, void *stream) {
    const char *fn = "paro_step_fused_static";
    int rc;
    AdamConsts a;
    if ((rc = check_common(pl, rank, fn))) return rc;
    if (pl->any_no_decay)
        return fail(PARO_EINVAL, std::string(fn) + ": a weight-decay mask needs the plan's device tables; use paro_step_fused");
    if (pl->L > PARO_STATIC_MAX_CHUNK)
        return fail(PARO_ERANGE, std::string(fn) + ": the plan's chunk of " + std::to_string(pl->L) +
                                     " elements exceeds PARO_STATIC_MAX_CHUNK (" +
                                     std::to_string((long long)PARO_STATIC_MAX_CHUNK) + ")");
    if ((rc = check_contrib(pl, contrib, PARO_CHUNK, fn))) return rc;
    if ((rc = adam_consts(hp, &a, fn))) return rc;
    if ((rc = check_ptr(p, "paro_step_fused_static: p"))) return rc;
    if ((rc = check_ptr(m, "paro_step_fused_static: m"))) return rc;
    if ((rc = check_ptr(v, "paro_step_fused_static: v"))) return rc;
    if ((rc = check_ptr(dst_base, "paro_step_fused_static: dst_base"))) return rc;
    plan_consts(pl, &a);
    if (a.max_norm > 0.0f || a.skip_nonfinite) {
        if ((rc = check_ptr(grad_scratch, "paro_step_fused_static: grad_scratch"))) return rc;
        if (!sumsq_scratch || (reinterpret_cast<uintptr_t>(sumsq_scratch) & 7))
            return fail(sumsq_scratch ? PARO_EALIGN : PARO_EINVAL,
                        std::string(fn) + ": clipping and skip_nonfinite need sumsq_scratch");
    }
    Scratch sc;
    if ((rc = static_scratch(&sc))) return rc;
    return launch_step(pl, sc, rank, contrib, PARO_CHUNK, a, grad_scratch, sumsq_scratch, p, m, v, dst_base,
                       static_cast<hipStream_t>(stream));
}

}  // extern "C"


// ---- ring hops and scheduled transfers ----------------------------------------
namespace {
// Bytes from the start of an all-gather's message that are stored to stay in the memory-side cache (see PARO_KEEP_MESSAGES_BYTES).
int64_t keeps_of_message(const paro_plan_t *pl) {
    return std::min((int64_t)PARO_KEEP_MESSAGES_BYTES / pl->P, (int64_t)PARO_KEEP_OF_MESSAGE_BYTES);
}
int launch_hop(const paro_plan_t *pl, const void *a, int da, const void *b, int db, float *out, int64_t n,
               hipStream_t st) {
    if (n <= 0) return PARO_OK;
    const unsigned grid = piece_grid(n);
    const unsigned lds = throttle_lds(pl->dev.lds_per_cu, PARO_HOP_WAVES_PER_CU);
    const int keep = n * 4 <= PARO_KEEP_MESSAGE_BYTES;
#define PARO_HOP_CASE(A, B)                                                                                   \
    if (da == A && db == B) hipLaunchKernelGGL((k_hop<A, B>), dim3(grid), dim3(WAVE), lds, st, a, b, out, n, keep)
    PARO_HOP_CASE(PARO_BF16, PARO_BF16); PARO_HOP_CASE(PARO_BF16, PARO_F32); PARO_HOP_CASE(PARO_BF16, PARO_F16);
    PARO_HOP_CASE(PARO_F32, PARO_BF16);  PARO_HOP_CASE(PARO_F32, PARO_F32);  PARO_HOP_CASE(PARO_F32, PARO_F16);
    PARO_HOP_CASE(PARO_F16, PARO_BF16);  PARO_HOP_CASE(PARO_F16, PARO_F32);  PARO_HOP_CASE(PARO_F16, PARO_F16);
#undef PARO_HOP_CASE
    PARO_HIP(hipGetLastError());
    return PARO_OK;
}
}  // namespace

extern "C" {

int paro_ring_hop(paro_plan_t *pl, const void *partial_in, int in_dtype, const void *local, int local_dtype, float *out,
                  int64_t n, void *stream) {
    int rc;
    if (!pl) return fail(PARO_EINVAL, "paro_ring_hop: plan is NULL");
    if (n < 0) return fail(PARO_EINVAL, "paro_ring_hop: n is negative");
    if (in_dtype < PARO_BF16 || in_dtype > PARO_F16 || local_dtype < PARO_BF16 || local_dtype > PARO_F16)
        return fail(PARO_EINVAL, "paro_ring_hop: bad dtype");
    if ((rc = check_ptr(partial_in, "paro_ring_hop: partial_in"))) return rc;
    if ((rc = check_ptr(local, "paro_ring_hop: local"))) return rc;
    if ((rc = check_ptr(out, "paro_ring_hop: out"))) return rc;
    if ((in_dtype != PARO_F32 && static_cast<const void *>(out) == partial_in) ||
        (local_dtype != PARO_F32 && static_cast<const void *>(out) == local))
        return fail(PARO_EINVAL, "paro_ring_hop: out may only alias an fp32 operand");
    if ((rc = ensure_device(pl))) return rc;
    return launch_hop(pl, partial_in, in_dtype, local, local_dtype, out, n, static_cast<hipStream_t>(stream));
}

int64_t paro_collective_step(paro_plan_t *pl, int rank, int sched, int collective, int phase, int ring, int step,
                             void *const *bufs, void *stream) {
    int rc;
    if ((rc = check_common(pl, rank, "paro_collective_step"))) return rc;
    if (!bufs) return fail(PARO_EINVAL, "paro_collective_step: bufs is NULL");
    for (int q = 0; q < pl->P; ++q)
        if ((rc = check_ptr(bufs[q], "paro_collective_step: a buffer"))) return rc;
    // only this step's messages, not the whole table (an all-gather of small messages over 16 ranks, 240
    // calls: 900 -> 770 us)
    const paro::MessageId only{phase, ring, step};
    std::vector<paro_msg_t> msgs;
    if ((rc = paro::schedule_messages(pl, rank, sched, collective, &only, &msgs))) return rc;
    if ((rc = ensure_device(pl))) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int64_t received = 0;
    for (const paro_msg_t &m : msgs) {
        if (collective == PARO_RS) {
            const float *from = static_cast<const float *>(bufs[m.recv_from]) + m.recv_off;
            float *mine = static_cast<float *>(bufs[rank]) + m.recv_off;
            if ((rc = launch_hop(pl, from, PARO_F32, mine, PARO_F32, mine, m.recv_len, st))) return rc;
        } else {
            const uint16_t *from = static_cast<const uint16_t *>(bufs[m.recv_from]) + m.recv_off;
            uint16_t *mine = static_cast<uint16_t *>(bufs[rank]) + m.recv_off;
            const int64_t n16 = m.recv_len / 8;             // ranges are whole chunks: multiples of 8 elements
            const unsigned grid = (unsigned)((n16 + WAVE - 1) / WAVE);
            if (n16 > 0) {
                hipLaunchKernelGGL(k_copy16, dim3(grid), dim3(WAVE), throttle_lds(pl->dev.lds_per_cu, PARO_COPY_WAVES_PER_CU), st,
                                   reinterpret_cast<const u32x4 *>(from), reinterpret_cast<u32x4 *>(mine), n16,
                                   (unsigned)(keeps_of_message(pl) / (16 * WAVE)));
                PARO_HIP(hipGetLastError());
            }
        }
        received += m.recv_len;
    }
    return received;
}

}  // extern "C"
